// The quantiser that produces the k-means weight formats from dense bf16 weights
// (paper Sec. 2.1 "Rounding to nearest centroids": f_c(x) = argmin_{c_i} |x - c_i| with
// the centroids from 1-D k-means clustering; "Block formats"; Sec. 2.2 "Nonlinear
// k-means quantization": per tensor, on weights normalised by a 16-bit scale per block
// of 64 elements).  The paper names Lloyd's algorithm and leaves its details open; the
// rules fixed here (kmq.h states them for callers):
//
//   * fp64 throughout; centroids stay sorted; a value is assigned to the cluster whose
//     index is the number of boundaries (c_i + c_{i+1}) / 2 below it (a value on a boundary
//     goes down); an empty cluster keeps its centroid; exactly `iters` rounds;
//   * start: 2^b points evenly spaced over the data's range (row min..max, or [-1, 1]
//     for normalised weights);
//   * the stored codebook is the centroids rounded to bf16 (nearest even) and the indices
//     are nearest STORED centroids.
//
// Sums of a cluster's members are formed per lane, then over a wave's lanes, then over
// waves (and workgroups) in a fixed order: deterministic, and exact whenever the members'
// exponents span fewer than 53 - log2(count) bits (always so for rows of bf16 weights of
// one layer), in which case the result does not depend on the order at all.
//
// Compiled with floating-point contraction off: the arithmetic is specified operation by
// operation.
#include "kmq_device.h"
#include "kmq_launch.h"

#pragma clang fp contract(off)

namespace kmq {

__device__ __forceinline__ double bf16_to_f64(uint32_t h) { return static_cast<double>(__uint_as_float(h << 16)); }

// Nearest-even rounding of a finite double to bf16, decided on the double's own bits.
// Magnitudes below bf16's normal range give zero.
__device__ __forceinline__ uint16_t f64_to_bf16(double c) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(c));
    const uint32_t sign = static_cast<uint32_t>(u >> 63) << 15;
    const int e32 = static_cast<int>((u >> 52) & 0x7FF) - 1023 + 127;
    if (e32 <= 0) return static_cast<uint16_t>(sign);
    const uint64_t mant = u & ((1ull << 52) - 1);
    uint32_t m7 = static_cast<uint32_t>(mant >> 45);
    const uint64_t rem = mant & ((1ull << 45) - 1), half = 1ull << 44;
    if (rem > half || (rem == half && (m7 & 1u))) ++m7;
    return static_cast<uint16_t>(sign | ((static_cast<uint32_t>(e32) << 7) + m7));   // m7 == 128 carries into the exponent
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ long long wave_sum(long long v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int C>
struct Clusters {
    double b[C > 1 ? C - 1 : 1];   // boundaries
    double s[C];
    int n[C];                      // per lane: at most a few thousand members, widened when lanes are added up
    __device__ __forceinline__ void begin(const double* c) {
#pragma unroll
        for (int i = 0; i + 1 < C; ++i) b[i] = 0.5 * (c[i] + c[i + 1]);
#pragma unroll
        for (int j = 0; j < C; ++j) { s[j] = 0.0; n[j] = 0; }
    }
    __device__ __forceinline__ int assign(double v) const {
        int a = 0;
#pragma unroll
        for (int i = 0; i + 1 < C; ++i) a += v > b[i] ? 1 : 0;
        return a;
    }
    __device__ __forceinline__ void add(double v) {
        const int a = assign(v);
#pragma unroll
        for (int j = 0; j < C; ++j) {       // compile-time j: the sums stay in registers
            s[j] += a == j ? v : 0.0;
            n[j] += a == j ? 1 : 0;
        }
    }
};

// 32 consecutive indices -> BITS words of the canonical stream (LSB first, 3-bit fields may straddle).
template <int BITS>
struct GroupPacker {
    uint32_t w[BITS];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int j = 0; j < BITS; ++j) w[j] = 0;
    }
    template <int E>
    __device__ __forceinline__ void put(uint32_t a) {
        constexpr int p = E * BITS, wi = p >> 5, sh = p & 31;
        w[wi] |= a << sh;
        if constexpr (sh + BITS > 32) w[wi + 1] |= a >> (32 - sh);
    }
};

template <int BITS, int E = 0, typename F>
__device__ __forceinline__ void pack_group(GroupPacker<BITS>& g, F&& index_of) {
    if constexpr (E < 32) {
        g.template put<E>(index_of(E));
        pack_group<BITS, E + 1>(g, index_of);
    }
}

// ---- one codebook per row: sorted histogram ---------------------------------------------------------
// A bf16 row has few distinct values, and a Lloyd round needs of them only how many members lie below each
// boundary and what they sum to.  So the row is read once, into a histogram over its values (32 octaves below the
// row's largest magnitude, 128 mantissas: 4096 dwords, positive members counted in the low half and negative ones
// in the high half, zeros in a dword of their own), prefix sums are taken in ascending order of the values over
// buckets of 32, and a round is one bucket look-up per boundary plus the partial sum of that bucket, done by one wave.
// Sums are kept as 64-bit integers in units of the window's smallest unit, so they are exact; so are the fp64 sums of
// quantize_rows_kernel on every row this kernel accepts (exponent span + 8 + log2 K <= 53), and the results are the
// same bits.  A row outside that (or with non-finite or subnormal-sized data) is marked in its codebook and left to
// quantize_rows_kernel, in a second launch.
//
// What bounds it: vector issue.  25 rounds at 14336 x 4096, 1 / 2 / 3 / 4 bits: 107 / 132 / 150 / 169 us (61 - 68 without
// the rounds; every element against every boundary in fp64, each round, took 1033 / 1864 / 3767 / 8470 us); 4096 x 14336:
// 65 / 74 / 77 / 82.  One row per workgroup and 20 KB of LDS put eight rows on a CU; a round is about 110 instructions and
// a chain of 600 clocks (boundary -> LDS -> sum over lanes -> fp64 division), which eight rows a CU hide only in part.
constexpr int kHistMags = 4096, kHistBucket = 32, kHistBuckets = 2 * kHistMags / kHistBucket;
constexpr int kHistOctaves = 32;
constexpr int64_t kHistMaxK = 65535;       // 16-bit counters
constexpr uint16_t kRowMark = 0x7FFF;      // a NaN: no codebook entry of a row with finite weights

// Number of values <= b in the window's ascending order (0..2 * kHistMags; zeros not counted): negative values by
// falling magnitude, then positive ones by rising magnitude.
__device__ __forceinline__ int hist_below(double b, int base) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(b));
    const uint32_t top = static_cast<uint32_t>(u >> 45);                                  // sign, exponent, seven mantissa bits
    const int mag = static_cast<int>(top & 0x3FFFFu) - ((1023 - 127) << 7);               // bf16 magnitude, towards zero (below the normal range: negative)
    if (b < 0.0) {
        const int mi = mag + ((u & ((1ull << 45) - 1)) != 0 ? 1 : 0) - base;              // smallest magnitude not above b
        return kHistMags - (mi < 0 ? 0 : mi > kHistMags ? kHistMags : mi);
    }
    const int mi = mag - base + 1;
    return kHistMags + (mi < 0 ? 0 : mi > kHistMags ? kHistMags : mi);
}

typedef u32x4_t __attribute__((aligned(2))) u32x4_a2_t;
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
typedef __attribute__((ext_vector_type(2))) short i16x2_t;

__device__ __forceinline__ uint32_t udot2(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b), c, false);
}

// Sum over groups of LANES (4, 8, 16) consecutive lanes, in every lane of the group.
template <int LANES>
__device__ __forceinline__ uint32_t lanes_sum(uint32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);                        // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);                        // quad_perm [2,3,0,1]
    if (LANES >= 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);       // row_half_mirror
    if (LANES >= 16) v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true);      // row_mirror
    return v;
}

// Minimum (or maximum) over the wave, in lane 63; inclusive sums over the wave's lanes.  DPP: shifts inside rows of 16
// lanes, then the last lane of a row into the next ones.
template <bool MAX>
__device__ __forceinline__ int wave_extreme(int v) {
    auto step = [&](int o) { v = MAX ? (o > v ? o : v) : (o < v ? o : v); };
    step(__builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false));       // row_shr 1, 2, 4, 8 (outside a row: the lane's own value)
    step(__builtin_amdgcn_update_dpp(v, v, 0x112, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x118, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x142, 0xA, 0xF, false));       // row_bcast15 into rows 1 and 3
    step(__builtin_amdgcn_update_dpp(v, v, 0x143, 0xC, 0xF, false));       // row_bcast31 into rows 2 and 3
    return v;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_step(long long& s, uint32_t& c) {
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(s), CTRL, ROWS, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(static_cast<uint64_t>(s) >> 32), CTRL, ROWS, 0xF, false);
    c += __builtin_amdgcn_update_dpp(0, c, CTRL, ROWS, 0xF, false);
    s += static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo);
}
__device__ __forceinline__ void wave_scan(long long& s, uint32_t& c) {
    scan_step<0x111, 0xF>(s, c);
    scan_step<0x112, 0xF>(s, c);
    scan_step<0x114, 0xF>(s, c);
    scan_step<0x118, 0xF>(s, c);
    scan_step<0x142, 0xA>(s, c);
    scan_step<0x143, 0xC>(s, c);
}

// 16 consecutive elements from row element k0 on; those beyond the row repeat the piece's first (k0 < K).
__device__ __forceinline__ void load16(const uint16_t* w, int k0, int K, uint32_t (&v)[8]) {
    if (k0 + 16 <= K) {
        const u32x4_t a = *reinterpret_cast<const u32x4_a2_t*>(w + k0), b = *reinterpret_cast<const u32x4_a2_t*>(w + k0 + 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t lo = w[k0 + 2 * i < K ? k0 + 2 * i : k0], hi = w[k0 + 2 * i + 1 < K ? k0 + 2 * i + 1 : k0];
            v[i] = lo | (hi << 16);
        }
    }
}

// NI > 0: the row is at most NI * 4096 elements and a thread keeps its NI pieces of 16 in registers; 0: re-read.
template <int BITS, int NI>
__global__ __launch_bounds__(256, NI == 4 ? 6 : 8) void quantize_rows_hist_kernel(const uint16_t* __restrict__ W, int64_t rowlen, int iters,
                                                                                 uint32_t* __restrict__ packed,
                                                                                 uint16_t* __restrict__ codebook) {
    constexpr int C = 1 << BITS;
    constexpr int LG = C <= 4 ? 16 : 64 / C;                // lanes per boundary in the clustering wave
    constexpr int DW = kHistBucket / LG;                    // histogram dwords (of a bucket's 32) per lane
    constexpr int H = kHistMags;
    struct alignas(16) Smem {
        uint32_t cells[4 + H];                              // the histogram from cell 4 on; cell 3 counts the zeros
        long long psum[kHistBuckets + 1];                   // sum of the members below bucket i, in units
        uint32_t pcnt[kHistBuckets + 1];                    // ... and their number
        long long wsum[4];
        uint32_t wcnt[4];
        int wlo[4], whi[4], wmin[4];
        int thr[16];                                        // values at or below each boundary of the stored codebook
        int zero_cluster;
    };
    __shared__ Smem sm;
    uint32_t* const hist = sm.cells + 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t n = blockIdx.x;
    const uint16_t* w = W + n * rowlen;
    const int K = static_cast<int>(rowlen), pieces = (K + 15) >> 4;

    // ---- 1. the row, its range and its smallest non-zero magnitude, two elements at a time
    uint32_t reg[NI > 0 ? NI : 1][8];
    i16x2_t lo2 = {0x7FFF, 0x7FFF}, hi2 = {-0x7FFF - 1, -0x7FFF - 1};        // of the order-preserving keys
    u16x2_t mn2 = {0xFFFF, 0xFFFF};                                          // magnitude - 1 (zero: 65535)
    auto range_of = [&](const uint32_t (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const i16x2_t h = __builtin_bit_cast(i16x2_t, v[i]);
            const u16x2_t mag = __builtin_bit_cast(u16x2_t, v[i] & 0x7FFF7FFFu);
            mn2 = __builtin_elementwise_min(mn2, static_cast<u16x2_t>(mag - u16x2_t{1, 1}));
            const i16x2_t sg = h >> i16x2_t{15, 15};
            const i16x2_t key = __builtin_bit_cast(i16x2_t, v[i] ^ (__builtin_bit_cast(uint32_t, sg) & 0x7FFF7FFFu));
            lo2 = __builtin_elementwise_min(lo2, key);
            hi2 = __builtin_elementwise_max(hi2, key);
        }
    };
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid + i * 256 < pieces) load16(w, (tid + i * 256) << 4, K, reg[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) reinterpret_cast<u32x4_t*>(hist)[tid + i * 256] = u32x4_t{0, 0, 0, 0};
    if (tid == 0) hist[-1] = 0;
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid + i * 256 < pieces) range_of(reg[i]);
    } else {
        for (int p = tid; p < pieces; p += 256) {
            load16(w, p << 4, K, reg[0]);
            range_of(reg[0]);
        }
    }
    // keys back to signed magnitudes: a negative key k stands for -(k ^ 0x7FFF)
    int lo = lo2[0] < lo2[1] ? lo2[0] : lo2[1], hi = hi2[0] > hi2[1] ? hi2[0] : hi2[1];
    int mn = mn2[0] < mn2[1] ? mn2[0] : mn2[1];
    lo = wave_extreme<false>(lo);
    hi = wave_extreme<true>(hi);
    mn = wave_extreme<false>(mn);
    if (lane == 63) { sm.wlo[wave] = lo; sm.whi[wave] = hi; sm.wmin[wave] = mn; }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        lo = sm.wlo[q] < lo ? sm.wlo[q] : lo;
        hi = sm.whi[q] > hi ? sm.whi[q] : hi;
        mn = sm.wmin[q] < mn ? sm.wmin[q] : mn;
    }
    const uint32_t lo_h = static_cast<uint32_t>(lo < 0 ? (lo ^ 0x7FFF) : lo) & 0xFFFFu;       // the bf16 patterns again
    const uint32_t hi_h = static_cast<uint32_t>(hi < 0 ? (hi ^ 0x7FFF) : hi) & 0xFFFFu;
    const int lo_m = static_cast<int>(lo_h & 0x7FFFu), hi_m = static_cast<int>(hi_h & 0x7FFFu), maxmag = lo_m > hi_m ? lo_m : hi_m;
    const bool all_zero = maxmag == 0;
    const int emax = all_zero ? 127 : maxmag >> 7, emin = all_zero ? 127 : ((mn + 1) >> 7 > 0 ? (mn + 1) >> 7 : 1);
    const int log2k = 32 - __clz(K - 1);                    // K <= 2^log2k (K = 1: 0)
    if (maxmag >= 0x7F80 || emax <= kHistOctaves || emax - emin >= kHistOctaves || emax - emin + 8 + log2k > 53) {
        if (tid == 0) codebook[n * C] = kRowMark;           // the same for every thread: the whole workgroup leaves
        return;
    }
    const int base = __builtin_amdgcn_readfirstlane((emax - (kHistOctaves - 1)) << 7);

    // ---- 2. histogram: dword `magnitude - base`, low half for positive values, high half for negative ones.  From here on
    // an element is 2 * (magnitude - base) + sign, a signed half-word; a zero is -2 or -1 (the dword in front).
    const uint32_t floor2 = static_cast<uint32_t>(base - 1) * 0x00010001u, base2 = static_cast<uint32_t>(base) * 0x00010001u;
    auto place = [&](uint32_t (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const u16x2_t h = __builtin_bit_cast(u16x2_t, v[i]);
            const u16x2_t mag = __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, v[i] & 0x7FFF7FFFu), __builtin_bit_cast(u16x2_t, floor2));
            const u16x2_t mi = mag - __builtin_bit_cast(u16x2_t, base2);
            v[i] = __builtin_bit_cast(uint32_t, static_cast<u16x2_t>(mi * u16x2_t{2, 2} + (h >> u16x2_t{15, 15})));
        }
    };
    auto count = [&](const uint32_t (&v)[8], int piece) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t d = v[e >> 1];
            const int mi = e & 1 ? static_cast<int>(d) >> 17 : static_cast<int>(d << 16) >> 17;
            atomicAdd(&hist[mi], (e & 1 ? (d >> 16) & 1u : d & 1u) * 0xFFFFu + 1u);
        }
        const int extra = (piece << 4) + 16 - K;            // repeats of the first element in the row's last piece
        if (extra > 0) atomicSub(&hist[static_cast<int16_t>(v[0]) >> 1], static_cast<uint32_t>(extra) << (v[0] & 1u ? 16 : 0));
    };
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid + i * 256 < pieces) { place(reg[i]); count(reg[i], tid + i * 256); }
    } else {
        for (int p = tid; p < pieces; p += 256) {
            load16(w, p << 4, K, reg[0]);
            place(reg[0]);
            count(reg[0], p);
        }
    }
    __syncthreads();

    // ---- 3. buckets of 32 magnitudes (two lanes read one), then prefix sums over them in ascending order of the values
    // mantissa sum of a bucket: (128 + first mantissa) * members + sum of members times their place in the bucket
    {
        uint32_t both = 0, sp = 0, sn = 0;                  // members (both halves), place sums of positive / negative ones
        const int bucket = tid >> 1, half = tid & 1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x4_t d = reinterpret_cast<const u32x4_t*>(hist)[tid * 4 + q];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                both += d[j];
                sp = udot2(d[j], static_cast<uint32_t>(q * 4 + j), sp);
                sn = udot2(d[j], static_cast<uint32_t>(q * 4 + j) << 16, sn);
            }
        }
        sp += half * 16 * (both & 0xFFFFu);
        sn += half * 16 * (both >> 16);
        both += __builtin_amdgcn_update_dpp(0, both, 0xB1, 0xF, 0xF, true);                  // the pair's other lane
        sp += __builtin_amdgcn_update_dpp(0, sp, 0xB1, 0xF, 0xF, true);
        sn += __builtin_amdgcn_update_dpp(0, sn, 0xB1, 0xF, 0xF, true);
        // the even lane writes the bucket of positive values, the odd one that of the negative values
        const uint32_t m0 = 128u + static_cast<uint32_t>((bucket * kHistBucket) & 127);
        const uint32_t c = half ? both >> 16 : both & 0xFFFFu, si = m0 * c + (half ? sn : sp);
        const int at = half ? kHistBuckets / 2 - 1 - bucket : kHistBuckets / 2 + bucket;
        const long long v = static_cast<long long>(static_cast<uint64_t>(si) << (bucket >> 2));
        sm.psum[at] = half ? -v : v;
        sm.pcnt[at] = c;
    }
    __syncthreads();
    {
        long long incl_s = sm.psum[tid];
        uint32_t incl_c = sm.pcnt[tid];
        wave_scan(incl_s, incl_c);
        if (lane == 63) { sm.wsum[wave] = incl_s; sm.wcnt[wave] = incl_c; }
        __syncthreads();
        for (int q = 0; q < wave; ++q) { incl_s += sm.wsum[q]; incl_c += sm.wcnt[q]; }
        sm.psum[tid + 1] = incl_s;
        sm.pcnt[tid + 1] = incl_c;
        if (tid == 0) { sm.psum[0] = 0; sm.pcnt[0] = 0; }
    }
    __syncthreads();

    // ---- 4. the rounds, one wave: LG lanes per cluster and for the boundary above it
    if (wave == 0) {
        const int G = lane / LG, p = lane % LG;
        const uint32_t nzero = (hist[-1] & 0xFFFFu) + (hist[-1] >> 16);
        const double l = bf16_to_f64(lo_h), h = bf16_to_f64(hi_h);
        const double unit = __longlong_as_double(static_cast<long long>(emax - (kHistOctaves - 1) - 127 - 7 + 1023) << 52);
        const bool top = G >= C - 1;                        // no boundary above the last cluster: everything is below
        double c = l + (G + 0.5) * (h - l) / C;
        int seen = -1;
        for (int t = 0; t < iters; ++t) {
            const double b = 0.5 * (c + __shfl_down(c, LG, 64));
            const int below = top ? 2 * H : hist_below(b, base);
            const bool with_zeros = top || !(b < 0.0);
            // the members of every cluster as in the round before: a fixed point
            const int now = below * 2 + (with_zeros ? 1 : 0);
            if (__all(now == seen)) break;
            seen = now;
            const int bucket = below >> 5, part = below & 31;
            const bool pos = bucket >= kHistBuckets / 2;
            const int mb = pos ? (bucket - kHistBuckets / 2) & (kHistBuckets / 2 - 1) : kHistBuckets / 2 - 1 - bucket;   // bucket of magnitudes
            uint32_t cnt = 0, si = 0;
            // which of the bucket's magnitudes are below, bit i: positive, the first `part`; negative, the last `part`
            const uint32_t first = (1u << part) - 1u;
            const uint32_t inside = (pos ? first : __builtin_bitreverse32(first)) >> (p * DW);
            const uint32_t one = pos ? 1u : 0x10000u;       // picks the half
#pragma unroll
            for (int j = 0; j < DW; ++j) {
                const uint32_t d = hist[mb * kHistBucket + p * DW + j] & static_cast<uint32_t>(static_cast<int>(inside << (31 - j)) >> 31);
                cnt = udot2(d, one, cnt);
                si = udot2(d, one * j, si);
            }
            si += cnt * static_cast<uint32_t>(p * DW);
            const long long S1 = sm.psum[bucket];
            const uint32_t M1 = sm.pcnt[bucket] + (with_zeros ? nzero : 0u);
            cnt = lanes_sum<LG>(cnt);
            si = lanes_sum<LG>(si);
            const uint32_t m0 = 128u + static_cast<uint32_t>((mb * kHistBucket) & 127);
            const long long ds = static_cast<long long>(static_cast<uint64_t>(m0 * cnt + si) << (mb >> 2));
            long long S = S1 + (pos ? ds : -ds);
            uint32_t M = M1 + cnt;
            const long long S0 = __shfl_up(S, LG, 64);
            const uint32_t M0 = __shfl_up(M, LG, 64);
            if (G > 0) { S -= S0; M -= M0; }
            if (M > 0) c = static_cast<double>(S) * unit / static_cast<double>(M);
        }
        const uint16_t hc = f64_to_bf16(c);
        if (p == 0 && G < C) codebook[n * C + G] = hc;
        c = bf16_to_f64(hc);
        const double b = 0.5 * (c + __shfl_down(c, LG, 64));
        if (p == 0 && G < C - 1) sm.thr[G] = hist_below(b, base);
        const uint64_t neg = __ballot(p == 0 && G < C - 1 && b < 0.0);
        if (lane == 0) sm.zero_cluster = __popcll(neg);
    }
    __syncthreads();

    // ---- 5. cluster of every value, over the histogram: two bytes per magnitude, positive and negative
    uint8_t* const table = reinterpret_cast<uint8_t*>(hist);
    {
        const int m = tid * 16;                             // this thread's magnitudes m..m + 15
        int p0 = 0, n1 = 0;                                 // clusters of +m and -m
#pragma unroll
        for (int i = 0; i < C - 1; ++i) {
            const int th = sm.thr[i];
            p0 += th <= H + m ? 1 : 0;
            n1 += th <= H - 1 - m ? 1 : 0;
        }
        // ... and of +-(m + 16), the next thread's (lane 63: the widest range; the loops below then find nothing)
        int p1 = __shfl_down(p0, 1, 64), n0 = __shfl_down(n1, 1, 64);
        if (lane == 63) { p1 = C - 1; n0 = 0; }
        const uint32_t f = static_cast<uint32_t>(p0 | (n1 << 8)) * 0x00010001u;
        reinterpret_cast<u32x4_t*>(table)[tid * 2] = u32x4_t{f, f, f, f};
        reinterpret_cast<u32x4_t*>(table)[tid * 2 + 1] = u32x4_t{f, f, f, f};
        for (int i = p0; i < p1; ++i)                       // boundaries among them, ascending values
            for (int q = sm.thr[i] - H; q < m + 16; ++q) table[2 * q] = static_cast<uint8_t>(i + 1);
        for (int i = n1 - 1; i >= n0; --i)                  // ... and among the negative ones, from the smallest magnitude on
            for (int q = H - sm.thr[i]; q < m + 16; ++q) table[2 * q + 1] = static_cast<uint8_t>(i);
        if (tid < 2) table[-1 - tid] = static_cast<uint8_t>(sm.zero_cluster);   // of either sign
    }
    __syncthreads();

    // ---- 6. indices, 16 elements (BITS half-words of the stream) per thread and piece
    const int wpr = static_cast<int>(words_per_row(BITS, K));
    uint16_t* out = reinterpret_cast<uint16_t*>(packed + n * wpr);
    auto emit = [&](const uint32_t (&v)[8], int piece) {
        uint32_t half[2] = {0, 0};                          // eight elements each: 8 * BITS bits
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int at = e & 1 ? static_cast<int>(v[e >> 1]) >> 16 : static_cast<int16_t>(v[e >> 1]);
            half[e >> 3] |= static_cast<uint32_t>(table[at]) << ((e & 7) * BITS);
        }
        uint64_t bits = static_cast<uint64_t>(half[1]) << (8 * BITS) | half[0];
        const int live = K - (piece << 4);
        if (live < 16) bits &= (uint64_t(1) << (live * BITS)) - 1;
        if constexpr (BITS == 2 || BITS == 4) {
            uint32_t* o32 = reinterpret_cast<uint32_t*>(out);
#pragma unroll
            for (int j = 0; j < BITS / 2; ++j)
                if (piece * (BITS / 2) + j < wpr) o32[piece * (BITS / 2) + j] = static_cast<uint32_t>(bits >> (32 * j));
        } else {
#pragma unroll
            for (int j = 0; j < BITS; ++j)
                if (piece * BITS + j < 2 * wpr) out[piece * BITS + j] = static_cast<uint16_t>(bits >> (16 * j));
        }
    };
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid + i * 256 < pieces) emit(reg[i], tid + i * 256);
    } else {
        for (int p = tid; p < pieces; p += 256) {
            load16(w, p << 4, K, reg[0]);
            place(reg[0]);
            emit(reg[0], p);
        }
    }
    // the half-words behind the last piece that the row's last word still has (16 * BITS bits per piece)
    if (tid == 0)
        for (int i = pieces * BITS; i < 2 * wpr; ++i) out[i] = 0;
}

// ---- one codebook per row: any data ----------------------------------------------------------------
// One workgroup of four waves per row; the row is re-read from the caches each round.  MARKED: only the rows that
// quantize_rows_hist_kernel left (their codebook starts with kRowMark), kMarkedRows rows looked at per workgroup.
constexpr int kMarkedRows = 4;
template <int BITS>
struct RowShared {
    double cs[1 << BITS];
    double ps[4][1 << BITS];
    long long pn[4][1 << BITS];
    double plo[4], phi[4];
};

template <int BITS>
__device__ __forceinline__ void quantize_row(RowShared<BITS>& sh, const uint16_t* W, int64_t n, int64_t K, int iters,
                                             uint32_t* packed, uint16_t* codebook) {
    constexpr int C = 1 << BITS;
    auto& cs = sh.cs;
    auto& ps = sh.ps;
    auto& pn = sh.pn;
    auto &plo = sh.plo, &phi = sh.phi;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint16_t* w = W + n * K;

    double lo = __builtin_huge_val(), hi = -__builtin_huge_val();
    for (int64_t k = tid; k < K; k += 256) {
        const double v = bf16_to_f64(w[k]);
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double l2 = __shfl_xor(lo, off, 64), h2 = __shfl_xor(hi, off, 64);
        lo = l2 < lo ? l2 : lo;
        hi = h2 > hi ? h2 : hi;
    }
    if (lane == 0) { plo[wave] = lo; phi[wave] = hi; }
    __syncthreads();
    if (tid < C) {
        double l = plo[0], h = phi[0];
#pragma unroll
        for (int q = 1; q < 4; ++q) { l = plo[q] < l ? plo[q] : l; h = phi[q] > h ? phi[q] : h; }
        cs[tid] = l + (tid + 0.5) * (h - l) / C;
    }
    __syncthreads();

    Clusters<C> cl;
    double c[C];
    for (int t = 0; t < iters; ++t) {
#pragma unroll
        for (int j = 0; j < C; ++j) c[j] = cs[j];
        cl.begin(c);
        for (int64_t k = tid; k < K; k += 256) cl.add(bf16_to_f64(w[k]));
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const double s = wave_sum(cl.s[j]);
            const long long m = wave_sum(static_cast<long long>(cl.n[j]));
            if (lane == 0) { ps[wave][j] = s; pn[wave][j] = m; }
        }
        __syncthreads();
        if (tid < C) {
            const double s = ((ps[0][tid] + ps[1][tid]) + ps[2][tid]) + ps[3][tid];
            const long long m = pn[0][tid] + pn[1][tid] + pn[2][tid] + pn[3][tid];
            if (m > 0) cs[tid] = s / static_cast<double>(m);
        }
        __syncthreads();
    }

    if (tid < C) {
        const uint16_t h = f64_to_bf16(cs[tid]);
        codebook[n * C + tid] = h;
        cs[tid] = bf16_to_f64(h);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C; ++j) c[j] = cs[j];
    cl.begin(c);
    const int64_t wpr = words_per_row(BITS, K), ngroups = (K + 31) >> 5;
    for (int64_t g = tid; g < ngroups; g += 256) {
        GroupPacker<BITS> gp;
        gp.clear();
        const int64_t k0 = g << 5;
        pack_group<BITS>(gp, [&](int e) -> uint32_t {
            return k0 + e < K ? static_cast<uint32_t>(cl.assign(bf16_to_f64(w[k0 + e]))) : 0u;
        });
#pragma unroll
        for (int j = 0; j < BITS; ++j)
            if (g * BITS + j < wpr) packed[n * wpr + g * BITS + j] = gp.w[j];
    }
}

template <int BITS, bool MARKED>
__global__ __launch_bounds__(256) void quantize_rows_kernel(const uint16_t* __restrict__ W, int64_t N, int64_t K, int iters,
                                                            uint32_t* __restrict__ packed, uint16_t* codebook) {
    constexpr int C = 1 << BITS;
    __shared__ RowShared<BITS> sh;
    if constexpr (!MARKED) {
        quantize_row<BITS>(sh, W, blockIdx.x, K, iters, packed, codebook);
    } else {
        const int64_t n0 = static_cast<int64_t>(blockIdx.x) * kMarkedRows;
        uint32_t marks = 0;                                 // bit i: row n0 + i is to be done (the same in every thread)
#pragma unroll
        for (int i = 0; i < kMarkedRows; ++i)
            marks |= n0 + i < N && codebook[(n0 + i) * C] == kRowMark ? 1u << i : 0u;
        if (marks == 0) return;
        for (int i = 0; i < kMarkedRows; ++i) {
            __syncthreads();                                // marks read by all before the first is overwritten; shared arrays free
            if (marks >> i & 1u) quantize_row<BITS>(sh, W, n0 + i, K, iters, packed, codebook);
        }
    }
}

// ---- the paper's format: scale per 64-element block, one codebook per tensor -------------------------
constexpr int kQuantPartials = 1024;   // workgroups of a clustering pass = partial sums per cluster

struct QuantScratch {                  // layout of the caller's workspace
    double cent[16];
    double psum[kQuantPartials][16];
    long long pcnt[kQuantPartials][16];
};

// scale = largest magnitude of the block (bf16 magnitudes order like their bit patterns); wave per block
__global__ __launch_bounds__(256) void bs_scales_kernel(const uint16_t* __restrict__ W, int64_t nblocks,
                                                        uint16_t* __restrict__ scales, QuantScratch* q, int C) {
    const int lane = threadIdx.x & 63;
    const int64_t blk = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x < C) q->cent[threadIdx.x] = -1.0 + (2 * static_cast<int>(threadIdx.x) + 1) / static_cast<double>(C);
    if (blk >= nblocks) return;
    int mag = W[blk * KMQ_BLOCK + lane] & 0x7FFF;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const int o = __shfl_xor(mag, off, 64);
        mag = o > mag ? o : mag;
    }
    if (lane == 0) scales[blk] = static_cast<uint16_t>(mag);
}

__device__ __forceinline__ double normalised(uint32_t w, uint32_t scale) {
    const double s = bf16_to_f64(scale);
    return s > 0.0 ? bf16_to_f64(w) / s : 0.0;
}

// one clustering round, first half: every workgroup sums the members of each cluster over its blocks
template <int BITS>
__global__ __launch_bounds__(256) void bs_lloyd_pass_kernel(const uint16_t* __restrict__ W,
                                                            const uint16_t* __restrict__ scales, int64_t nblocks,
                                                            QuantScratch* q) {
    constexpr int C = 1 << BITS;
    __shared__ double ps[4][C];
    __shared__ long long pn[4][C];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double c[C];
#pragma unroll
    for (int j = 0; j < C; ++j) c[j] = q->cent[j];
    Clusters<C> cl;
    cl.begin(c);
    // a lane takes 8 consecutive elements (one 16-byte load; eight lanes share a block's scale), a wave 8 blocks
    const int64_t nchunks = nblocks * (KMQ_BLOCK / 8);
    for (int64_t c = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * kWave + lane; c < nchunks;
         c += static_cast<int64_t>(gridDim.x) * 4 * kWave) {
        const u32x4_t w8 = *reinterpret_cast<const u32x4_t*>(W + c * 8);
        const uint32_t scale = scales[c >> 3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            cl.add(normalised(w8[e] & 0xFFFFu, scale));
            cl.add(normalised(w8[e] >> 16, scale));
        }
    }
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const double s = wave_sum(cl.s[j]);
        const long long m = wave_sum(static_cast<long long>(cl.n[j]));
        if (lane == 0) { ps[wave][j] = s; pn[wave][j] = m; }
    }
    __syncthreads();
    if (tid < C) {
        q->psum[blockIdx.x][tid] = ((ps[0][tid] + ps[1][tid]) + ps[2][tid]) + ps[3][tid];
        q->pcnt[blockIdx.x][tid] = pn[0][tid] + pn[1][tid] + pn[2][tid] + pn[3][tid];
    }
}

// second half: partial sums added in workgroup order, centroids updated; on the last round the
// codebook is written as well
__global__ __launch_bounds__(64) void bs_lloyd_update_kernel(QuantScratch* q, int C, int partials, bool update,
                                                             uint16_t* __restrict__ codebook) {
    const int j = threadIdx.x;
    if (j >= C) return;
    if (update) {
        double s = 0.0;
        long long m = 0;
        for (int p = 0; p < partials; ++p) { s += q->psum[p][j]; m += q->pcnt[p][j]; }
        if (m > 0) q->cent[j] = s / static_cast<double>(m);
    }
    if (codebook) codebook[j] = f64_to_bf16(q->cent[j]);
}

// nearest stored centroid for every element, packed; one thread per 32 elements
template <int BITS>
__global__ __launch_bounds__(256) void bs_assign_pack_kernel(const uint16_t* __restrict__ W,
                                                             const uint16_t* __restrict__ scales,
                                                             const uint16_t* __restrict__ codebook, int64_t ngroups,
                                                             uint32_t* __restrict__ packed) {
    constexpr int C = 1 << BITS;
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (g >= ngroups) return;
    double c[C];
#pragma unroll
    for (int j = 0; j < C; ++j) c[j] = bf16_to_f64(codebook[j]);
    Clusters<C> cl;
    cl.begin(c);
    const uint32_t scale = scales[g >> 1];
    const uint16_t* w = W + (g << 5);
    GroupPacker<BITS> gp;
    gp.clear();
    pack_group<BITS>(gp, [&](int e) -> uint32_t { return static_cast<uint32_t>(cl.assign(normalised(w[e], scale))); });
#pragma unroll
    for (int j = 0; j < BITS; ++j) packed[g * BITS + j] = gp.w[j];
}

size_t quantize_blockscaled_workspace_bytes() { return sizeof(QuantScratch); }

template <int BITS>
static hipError_t quantize_rows_bits(const uint16_t* W, int64_t N, int64_t K, int iters, uint32_t* packed,
                                     uint16_t* codebook, hipStream_t s) {
    const dim3 rows(static_cast<unsigned>(N)), block(256);
    if (K > kHistMaxK) {
        hipLaunchKernelGGL((quantize_rows_kernel<BITS, false>), rows, block, 0, s, W, N, K, iters, packed, codebook);
        return hipGetLastError();
    }
#define KMQ_HIST(NI) hipLaunchKernelGGL((quantize_rows_hist_kernel<BITS, NI>), rows, block, 0, s, W, K, iters, packed, codebook)
    if (K <= 4096) KMQ_HIST(1);
    else if (K <= 8192) KMQ_HIST(2);
    else if (K <= 16384) KMQ_HIST(4);
    else KMQ_HIST(0);
#undef KMQ_HIST
    hipLaunchKernelGGL((quantize_rows_kernel<BITS, true>), dim3(static_cast<unsigned>((N + kMarkedRows - 1) / kMarkedRows)), block, 0, s,
                       W, N, K, iters, packed, codebook);
    return hipGetLastError();
}

hipError_t launch_quantize_rows(const uint16_t* W, int64_t N, int64_t K, int bits, int iters, uint32_t* packed,
                                uint16_t* codebook, hipStream_t s) {
    switch (bits) {
        case 1: return quantize_rows_bits<1>(W, N, K, iters, packed, codebook, s);
        case 2: return quantize_rows_bits<2>(W, N, K, iters, packed, codebook, s);
        case 3: return quantize_rows_bits<3>(W, N, K, iters, packed, codebook, s);
        default: return quantize_rows_bits<4>(W, N, K, iters, packed, codebook, s);
    }
}

template <int BITS>
static hipError_t quantize_blockscaled_bits(const uint16_t* W, int64_t N, int64_t K, int iters, uint32_t* packed,
                                            uint16_t* codebook, uint16_t* scales, QuantScratch* q, hipStream_t s) {
    constexpr int C = 1 << BITS;
    const int64_t nblocks = N * (K / KMQ_BLOCK), ngroups = nblocks * 2;
    const int64_t want = (nblocks + 31) / 32;          // a wave takes 8 blocks at a time
    const int partials = static_cast<int>(want < kQuantPartials ? want : kQuantPartials);
    hipLaunchKernelGGL(bs_scales_kernel, dim3(static_cast<unsigned>((nblocks + 3) / 4)), dim3(256), 0, s, W, nblocks, scales, q, C);
    for (int t = 0; t < iters; ++t) {
        hipLaunchKernelGGL((bs_lloyd_pass_kernel<BITS>), dim3(partials), dim3(256), 0, s, W, scales, nblocks, q);
        hipLaunchKernelGGL(bs_lloyd_update_kernel, dim3(1), dim3(64), 0, s, q, C, partials, true,
                           t + 1 == iters ? codebook : static_cast<uint16_t*>(nullptr));
    }
    if (iters == 0)
        hipLaunchKernelGGL(bs_lloyd_update_kernel, dim3(1), dim3(64), 0, s, q, C, 0, false, codebook);
    hipLaunchKernelGGL((bs_assign_pack_kernel<BITS>), dim3(static_cast<unsigned>((ngroups + 255) / 256)), dim3(256), 0, s, W,
                       scales, codebook, ngroups, packed);
    return hipGetLastError();
}

hipError_t launch_quantize_blockscaled(const uint16_t* W, int64_t N, int64_t K, int bits, int iters, uint32_t* packed,
                                       uint16_t* codebook, uint16_t* scales, void* workspace, hipStream_t s) {
    QuantScratch* q = static_cast<QuantScratch*>(workspace);
    switch (bits) {
        case 1: return quantize_blockscaled_bits<1>(W, N, K, iters, packed, codebook, scales, q, s);
        case 2: return quantize_blockscaled_bits<2>(W, N, K, iters, packed, codebook, scales, q, s);
        case 3: return quantize_blockscaled_bits<3>(W, N, K, iters, packed, codebook, scales, q, s);
        default: return quantize_blockscaled_bits<4>(W, N, K, iters, packed, codebook, scales, q, s);
    }
}

}  // namespace kmq
