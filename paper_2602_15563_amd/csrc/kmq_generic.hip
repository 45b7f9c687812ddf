// Shape-agnostic kernels: products of the canonical layout, any K >= 1, any bit-width, batch 1..16 -- for few rows of 8 bits
// and for few long rows, split over K; the rest has faster kernels -- and the
// bit-exact dequantiser of both layouts.  Operation: paper App. E, "Kernel implementations"
// (lookup, then multiply-accumulate), per-row codebooks, fp32 accumulation.
#include <mutex>

#include "kmq_device.h"
#include "kmq_launch.h"

// Scratch of kmq_gemm_smallbatch_noalloc: the split-K partial sums of callers that cannot allocate.
// Every GPU the library runs on holds its own copy at its own address until the process ends.  In host
// code this name is a stand-in, not a device address: the address comes from hipGetSymbolAddress below.
static __device__ __align__(256) unsigned char scratch[KMQ_NOALLOC_SCRATCH_BYTES];

namespace kmq {

// Device address of this GPU's scratch array (looked up once per device, with that device current).
hipError_t noalloc_scratch(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* per_device[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        per_device[dev] = p;
    }
    *ptr = per_device[dev];
    return hipSuccess;
}

// b-bit field `e` (0..31) of a 32-element group held in BITS consecutive words.
template <int BITS>
__device__ __forceinline__ uint32_t group_field(const uint32_t (&w)[BITS], int e) {
    constexpr uint32_t mask = (1u << BITS) - 1u;
    const int p = e * BITS;               // bit position inside the group
    const int wi = p >> 5, sh = p & 31;
    uint32_t v = w[wi] >> sh;
    if constexpr (BITS == 3) {
        if (sh > 29) v |= w[wi + 1] << (32 - sh);   // field straddles two words
    }
    return v & mask;
}

// One wave per output row, four rows per workgroup.  Each lane walks over
// 32-element groups (BITS words each, so groups start on a word boundary for
// every bit-width), looks weights up in the row's codebook (fp32 copy in LDS)
// and accumulates MT batch columns.
//
// Split-K (few rows, long rows: too few workgroups to fill the CUs otherwise): blockIdx.y
// selects one of gridDim.y slices of K (whole 32-element groups); the slice's fp32 partial
// sums go to partial[slice][m][n] and splitk_reduce_kernel adds the slices in index order, so
// the result does not depend on which workgroup finishes first.  partial == nullptr: one
// slice, bf16 output written directly.
template <int BITS, int MT>
__global__ __launch_bounds__(256) void gemm_generic_kernel(
    const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook,
    const uint16_t* __restrict__ X, uint16_t* __restrict__ Y,
    int64_t N, int64_t K, int M, float* __restrict__ partial) {
    constexpr int C = 1 << BITS;
    __shared__ float lut[4][C];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t n = static_cast<int64_t>(blockIdx.x) * 4 + wave;
    const bool live = n < N;
    if (live)
        for (int e = lane; e < C; e += kWave) lut[wave][e] = bf16_to_f32(codebook[n * C + e]);
    __syncthreads();
    if (!live) return;

    const int64_t wpr = words_per_row(BITS, K);
    const int64_t ngroups = (K + 31) >> 5;
    const bool vec_x = (K & 7) == 0;      // rows of X start 16-byte aligned
    float acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = 0.f;

    const int64_t gps = (ngroups + gridDim.y - 1) / gridDim.y;     // groups per slice
    const int64_t g_begin = blockIdx.y * gps, g_end = g_begin + gps < ngroups ? g_begin + gps : ngroups;
    for (int64_t g = g_begin + lane; g < g_end; g += kWave) {
        const int64_t k0 = g << 5;
        const bool full = k0 + 32 <= K;
        float wt[32];
        uint32_t w[BITS];
#pragma unroll
        for (int j = 0; j < BITS; ++j) {
            const int64_t wi = g * BITS + j;
            w[j] = wi < wpr ? W[n * wpr + wi] : 0u;
        }
#pragma unroll
        for (int e = 0; e < 32; ++e) wt[e] = lut[wave][group_field<BITS>(w, e)];
        if (full && vec_x) {
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if (m < M) {
                    const u32x4_t* xp = reinterpret_cast<const u32x4_t*>(X + m * K + k0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const u32x4_t xv = xp[q];
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            acc[m] = fmaf(wt[q * 8 + t * 2], __uint_as_float(xv[t] << 16), acc[m]);
                            acc[m] = fmaf(wt[q * 8 + t * 2 + 1], __uint_as_float(xv[t] & 0xFFFF0000u), acc[m]);
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                if (k0 + e < K) {
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        if (m < M) acc[m] = fmaf(wt[e], bf16_to_f32(X[m * K + k0 + e]), acc[m]);
                }
            }
        }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const float s = group_sum<64>(acc[m]);
        if (lane == 63 && m < M) {
            if (partial) partial[(static_cast<int64_t>(blockIdx.y) * M + m) * N + n] = s;
            else Y[static_cast<int64_t>(m) * N + n] = f32_to_bf16(s);
        }
    }
}

// Second pass of split-K: Y[m][n] = bf16( partial[0][m][n] + partial[1][m][n] + ... ), slices in order.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, uint16_t* __restrict__ Y,
                                                            int64_t MN, int slices) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= MN) return;
    float s = 0.f;
    for (int k = 0; k < slices; ++k) s += partial[static_cast<int64_t>(k) * MN + i];
    Y[i] = f32_to_bf16(s);
}

// One thread per (row, 32-element group): Wdense[n][k] = codebook[n][idx[n][k]].
template <int BITS>
__global__ __launch_bounds__(256) void dequant_kernel(
    const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook,
    uint16_t* __restrict__ Wd, int64_t N, int64_t K, int layout) {
    constexpr int C = 1 << BITS;
    const int64_t wpr = words_per_row(BITS, K);
    const int64_t ngroups = (K + 31) >> 5;
    const int64_t total = N * ngroups;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t n = i / ngroups, g = i % ngroups;
        uint32_t w[BITS];
#pragma unroll
        for (int j = 0; j < BITS; ++j) {
            const int64_t wi = g * BITS + j;
            w[j] = (layout == KMQ_LAYOUT_CANONICAL && wi < wpr) ? W[n * wpr + wi] : 0u;
        }
        [[maybe_unused]] uint16_t c[BITS <= 4 ? C : 1];
        if constexpr (BITS <= 4) {
#pragma unroll
            for (int j = 0; j < C; ++j) c[j] = codebook[n * C + j];
        }
        const int64_t k0 = g << 5;
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const uint32_t f = layout == KMQ_LAYOUT_CANONICAL ? group_field<BITS>(w, e)
                                                              : tiled_fetch_index(W, BITS, K, n, k0 + e);
            uint16_t v;
            if constexpr (BITS <= 4) {
                v = c[0];
#pragma unroll
                for (int j = 1; j < C; ++j) v = f == static_cast<uint32_t>(j) ? c[j] : v;
            } else {
                v = codebook[n * C + f];     // 256 entries: read through the caches instead of held in registers
            }
            if (k0 + e < K) Wd[n * K + k0 + e] = v;
        }
    }
}

// The canonical layout, bits 1..4, rows of at least kDequantWaveK columns of any length.  Bound by the store of the dense matrix.
// A wave takes 64 * U chunks of eight columns of ONE row, so that the row's centroids become a table in the wave's own piece of
// LDS (1 bit: four weights per entry, 2 and 3 bits: pairs, 4 bits: one; entries of one dword lie in different banks) and no thread
// divides.  Chunks are cut at the 16-byte boundaries of Wd, not at the row's start: all but the row's first and last are whole
// 16-byte stores whatever K and the address of Wd, 1 KB per wave and instruction, past the caches.
// Measured (us), one thread per chunk and centroids through the caches (odd K: per 32 columns, 2-byte stores) / this kernel / a
// fill of Wd: 8192 x 8192, 1 bit 23.9 / 22.2 / 20.4, 4 bits 41.3 / 25.0 / 20.4; 5001 x 4101, 3 bits 98.0 / 9.9 / 7.7.  From 512
// columns on because a wave's segment is 1024: 100000 x 512 still gains (4 bits 31.7 / 18.9), shorter rows leave most lanes idle.
constexpr int64_t kDequantWaveK = 512;
template <int BITS, int U>
__global__ __launch_bounds__(256) void dequant_wave_kernel(const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook,
                                                           uint16_t* __restrict__ Wd, uint32_t N, int K, uint32_t segs) {
    static_assert(BITS <= 4, "eight fields in one word");
    constexpr int C = 1 << BITS;
    __shared__ u32x2_t tab2[4][BITS == 1 ? 16 : 1];
    __shared__ uint32_t tab[4][BITS == 3 ? 64 : 16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t id = blockIdx.x * 4u + wave, n = id / segs, seg = id % segs;
    if (n >= N) return;                                  // (the waves of a workgroup share nothing)
    const uint16_t* c = codebook + static_cast<int64_t>(n) * C;
    const int wpr = static_cast<int>(words_per_row(BITS, K));
    const uint32_t* row = W + static_cast<int64_t>(n) * wpr;
    uint16_t* out = Wd + static_cast<int64_t>(n) * K;
    const int head = static_cast<int>((0u - static_cast<uint32_t>(reinterpret_cast<uintptr_t>(out))) & 15u) >> 1;   // columns ahead of a 16-byte boundary
    const int k0 = (head ? head - 8 : 0) + 8 * (static_cast<int>(seg) * (64 * U) + lane);

    uint32_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = k0 + u * 512;
        const int bit = (k > 0 ? k : 0) * BITS, wi = bit >> 5;
        const uint32_t lo = row[wi < wpr ? wi : wpr - 1];
        uint32_t hi = 0;
        if (BITS == 3 || head) hi = row[wi + 1 < wpr ? wi + 1 : wpr - 1];
        v[u] = __builtin_amdgcn_alignbit(hi, lo, bit & 31);
        if (k < 0) v[u] <<= -k * BITS;                    // field e is column k + e
    }
    if constexpr (BITS == 1) {
        if (lane < 16) {
            const uint32_t a = c[0], b = c[1];
            tab2[wave][lane] = u32x2_t{(lane & 1 ? b : a) | ((lane & 2 ? b : a) << 16), (lane & 4 ? b : a) | ((lane & 8 ? b : a) << 16)};
        }
    } else if constexpr (BITS == 4) {
        if (lane < 16) tab[wave][lane] = c[lane];
    } else {
        if (lane < C * C) tab[wave][lane] = c[lane % C] | (static_cast<uint32_t>(c[lane / C]) << 16);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = k0 + u * 512;
        if (k >= K) break;
        u32x4_t o;
        if constexpr (BITS == 1) {
            const u32x2_t a = tab2[wave][v[u] & 15u], b = tab2[wave][(v[u] >> 4) & 15u];
            o = u32x4_t{a[0], a[1], b[0], b[1]};
        } else if constexpr (BITS == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = tab[wave][(v[u] >> (8 * e)) & 15u] | (tab[wave][(v[u] >> (8 * e + 4)) & 15u] << 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = tab[wave][(v[u] >> (2 * BITS * e)) & (C * C - 1u)];
        }
        if (k >= 0 && k + 8 <= K) {
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4_t*>(out + k));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (k + e >= 0 && k + e < K) out[k + e] = static_cast<uint16_t>(o[e >> 1] >> (16 * (e & 1)));
        }
    }
}

template <int BITS, int U>
static void launch_dequant_wave(const uint32_t* W, const uint16_t* codebook, uint16_t* Wd, int64_t N, int64_t K, uint32_t segs, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>((N * segs + 3) / 4)), block(256);
    hipLaunchKernelGGL((dequant_wave_kernel<BITS, U>), grid, block, 0, s, W, codebook, Wd, static_cast<uint32_t>(N), static_cast<int>(K), segs);
}

// The canonical layout with K % 8 == 0, short rows and 8 bits: one thread per 8 consecutive elements, one 16-byte
// store per thread (a wave writes 1 KB of consecutive bytes, past the caches: the matrix is read by a later
// kernel).  The row's centroids are read through the caches.
template <int BITS>
__global__ __launch_bounds__(256) void dequant_rows8_kernel(const uint32_t* __restrict__ W,
                                                            const uint16_t* __restrict__ codebook,
                                                            uint16_t* __restrict__ Wd, int64_t N, int64_t K) {
    constexpr int C = 1 << BITS;
    constexpr uint32_t mask = C - 1;
    const int64_t cpr = K >> 3;                                   // chunks per row
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= N * cpr) return;
    const int64_t n = i / cpr, c8 = i % cpr;
    const int64_t wpr = words_per_row(BITS, K);
    const int64_t bit0 = c8 * (8 * BITS);
    const int64_t wi = bit0 >> 5;
    const int sh = static_cast<int>(bit0 & 31);
    const uint32_t* row = W + n * wpr;
    const uint64_t lo = row[wi], hi = wi + 1 < wpr ? row[wi + 1] : 0u;
    const uint64_t v = (lo | (hi << 32)) >> sh;
    const uint16_t* c = codebook + n * C;
    uint32_t out[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const uint32_t a = c[static_cast<uint32_t>(v >> (e * BITS)) & mask];
        const uint32_t b = c[static_cast<uint32_t>(v >> ((e + 1) * BITS)) & mask];
        out[e >> 1] = a | (b << 16);
    }
    __builtin_nontemporal_store(u32x4_t{out[0], out[1], out[2], out[3]}, reinterpret_cast<u32x4_t*>(Wd + n * K + (c8 << 3)));
}

template <int BITS>
static hipError_t launch_generic_bits(const GemmArgs& a, int slices, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>((a.N + 3) / 4), static_cast<unsigned>(slices)), block(256);
    float* partial = slices > 1 ? static_cast<float*>(a.workspace) : nullptr;
#define KMQ_GEN_LAUNCH(MT) \
    hipLaunchKernelGGL((gemm_generic_kernel<BITS, MT>), grid, block, 0, s, a.W, a.codebook, a.X, a.Y, a.N, a.K, a.M, partial)
    if (a.M == 1) KMQ_GEN_LAUNCH(1);
    else if (a.M <= 4) KMQ_GEN_LAUNCH(4);
    else if (a.M <= 8) KMQ_GEN_LAUNCH(8);
    else KMQ_GEN_LAUNCH(16);
#undef KMQ_GEN_LAUNCH
    if (slices > 1) {
        const int64_t mn = static_cast<int64_t>(a.M) * a.N;
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(static_cast<unsigned>((mn + 255) / 256)), dim3(256), 0, s,
                           partial, a.Y, mn, slices);
    }
    return hipGetLastError();
}

// Slices of K for the shape-agnostic kernel: 1 unless its one-wave-per-row grid would leave more
// than half of the 256 CUs idle on a product with long rows; then enough slices to fill them, each
// at least 4096 elements long.
int generic_splitk_slices(int64_t N, int64_t K, int layout) {
    if (layout != KMQ_LAYOUT_CANONICAL) return 1;
    const int64_t wgs = (N + 3) / 4;
    if (wgs * 2 > 256 || K < 16384) return 1;   // measured: at K = 8192 the second launch costs more than the split saves
    int64_t s = 256 / wgs;
    if (s > K / 4096) s = K / 4096;
    if (s > 64) s = 64;
    return s < 2 ? 1 : static_cast<int>(s);
}

hipError_t launch_generic(const GemmArgs& a, hipStream_t s) {
    const int slices = (a.workspace && a.workspace_bytes > 0) ? generic_splitk_slices(a.N, a.K, a.layout) : 1;
    switch (a.bits) {
        case 1: return launch_generic_bits<1>(a, slices, s);
        case 2: return launch_generic_bits<2>(a, slices, s);
        case 3: return launch_generic_bits<3>(a, slices, s);
        case 8: return launch_generic_bits<8>(a, slices, s);
        default: return launch_generic_bits<4>(a, slices, s);
    }
}

hipError_t launch_dequant(const uint32_t* W, const uint16_t* codebook, uint16_t* Wd, int64_t N,
                          int64_t K, int bits, int layout, hipStream_t s) {
    if (layout == KMQ_LAYOUT_CANONICAL && bits <= 4 && K >= kDequantWaveK) {
        constexpr int U = 2;
        const bool even = (K & 7) == 0 && (reinterpret_cast<uintptr_t>(Wd) & 15) == 0;
        const int64_t chunks = even ? K >> 3 : (K + 14) >> 3;      // a first chunk of 1..8 columns, whole ones, a last one
        const int64_t segs = (chunks + 64 * U - 1) / (64 * U);
        if (N * segs < (int64_t(1) << 31)) {
            const uint32_t sg = static_cast<uint32_t>(segs);
            switch (bits) {
                case 1: launch_dequant_wave<1, U>(W, codebook, Wd, N, K, sg, s); break;
                case 2: launch_dequant_wave<2, U>(W, codebook, Wd, N, K, sg, s); break;
                case 3: launch_dequant_wave<3, U>(W, codebook, Wd, N, K, sg, s); break;
                default: launch_dequant_wave<4, U>(W, codebook, Wd, N, K, sg, s); break;
            }
            return hipGetLastError();
        }
    }
    if (layout == KMQ_LAYOUT_CANONICAL && (K & 7) == 0 && (reinterpret_cast<uintptr_t>(Wd) & 15) == 0 &&
        N * (K >> 3) <= (int64_t(1) << 38)) {                  // one workgroup per 256 chunks must fit the grid
        const int64_t chunks = N * (K >> 3);
        const dim3 grid8(static_cast<unsigned>((chunks + 255) / 256)), block8(256);
        switch (bits) {
            case 1: hipLaunchKernelGGL(dequant_rows8_kernel<1>, grid8, block8, 0, s, W, codebook, Wd, N, K); break;
            case 2: hipLaunchKernelGGL(dequant_rows8_kernel<2>, grid8, block8, 0, s, W, codebook, Wd, N, K); break;
            case 3: hipLaunchKernelGGL(dequant_rows8_kernel<3>, grid8, block8, 0, s, W, codebook, Wd, N, K); break;
            case 8: hipLaunchKernelGGL(dequant_rows8_kernel<8>, grid8, block8, 0, s, W, codebook, Wd, N, K); break;
            default: hipLaunchKernelGGL(dequant_rows8_kernel<4>, grid8, block8, 0, s, W, codebook, Wd, N, K); break;
        }
        return hipGetLastError();
    }
    const int64_t total = N * ((K + 31) >> 5);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    const dim3 grid(static_cast<unsigned>(blocks)), block(256);
    switch (bits) {
        case 1: hipLaunchKernelGGL(dequant_kernel<1>, grid, block, 0, s, W, codebook, Wd, N, K, layout); break;
        case 2: hipLaunchKernelGGL(dequant_kernel<2>, grid, block, 0, s, W, codebook, Wd, N, K, layout); break;
        case 3: hipLaunchKernelGGL(dequant_kernel<3>, grid, block, 0, s, W, codebook, Wd, N, K, layout); break;
        case 8: hipLaunchKernelGGL(dequant_kernel<8>, grid, block, 0, s, W, codebook, Wd, N, K, layout); break;
        default: hipLaunchKernelGGL(dequant_kernel<4>, grid, block, 0, s, W, codebook, Wd, N, K, layout); break;
    }
    return hipGetLastError();
}

}  // namespace kmq
