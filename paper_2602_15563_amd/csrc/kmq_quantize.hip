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
// Both quantisers replace "every element against every boundary, each round" by counts over the few distinct values
// there are, taken once (the comments at the kernels).  Sums of members are deterministic.  A row's are exact whenever its
// exponents span fewer than 53 - log2(count) bits (always so for rows of bf16 weights of one layer); a tensor's are exact per
// scale mantissa, and rounded to 64 bits where those are scaled and added up.
//
// Compiled with floating-point contraction off: the arithmetic is specified operation by
// operation.
#include <cstddef>
#include <type_traits>

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
    int n[C];                      // per lane: at most 2^16 members (K <= 2^24), widened when lanes are added up
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
// For few rows, long ones, and what the kernel of four rows a workgroup (below) leaves.
// What bounds it: vector issue.  25 rounds at 14336 x 4096, 1 / 2 / 3 / 4 bits: 107 / 132 / 150 / 169 us (61 - 68 without
// the rounds; every element against every boundary in fp64, each round, took 1033 / 1864 / 3767 / 8470 us); 4096 x 14336:
// 65 / 74 / 77 / 82.  One row per workgroup and 20 KB of LDS put eight rows on a CU; a round is about 110 instructions and
// a chain of 600 clocks (boundary -> LDS -> sum over lanes -> fp64 division), which eight rows a CU hide only in part.
constexpr int kHistMags = 4096, kHistBucket = 32, kHistBuckets = 2 * kHistMags / kHistBucket;
constexpr int kHistOctaves = 32;
constexpr int64_t kHistMaxK = 65535;       // 16-bit counters
constexpr uint16_t kRowMark = 0x7FFF;      // a NaN: no codebook entry of a row with finite weights

// Number of values <= b in the ascending order of a window of MAGS magnitudes (0..2 * MAGS; zeros not counted): negative values by
// falling magnitude, then positive ones by rising magnitude.
template <int MAGS = kHistMags>
__device__ __forceinline__ int hist_below(double b, int base) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(b));
    if constexpr (MAGS == kHistMags) {                                                        // (a wave's boundaries of one row: the branch is the faster one)
        const uint32_t top = static_cast<uint32_t>(u >> 45);                                  // sign, exponent, seven mantissa bits
        const int mag = static_cast<int>(top & 0x3FFFFu) - ((1023 - 127) << 7);               // bf16 magnitude, towards zero (below the normal range: negative)
        if (b < 0.0) {
            const int mi = mag + ((u & ((1ull << 45) - 1)) != 0 ? 1 : 0) - base;              // smallest magnitude not above b
            return MAGS - (mi < 0 ? 0 : mi > MAGS ? MAGS : mi);
        }
        const int mi = mag - base + 1;
        return MAGS + (mi < 0 ? 0 : mi > MAGS ? MAGS : mi);
    } else {                                                                                  // (boundaries of four rows in a wave)
        const uint32_t hi = static_cast<uint32_t>(u >> 32);
        const int mag = static_cast<int>((hi & 0x7FFFFFFFu) >> 13) - ((1023 - 127) << 7) - base;
        const bool neg = b < 0.0, more = (static_cast<uint32_t>(u) | (hi & 0x1FFFu)) != 0;
        const int mi = mag + ((neg ? more : true) ? 1 : 0);
        const int in = mi < 0 ? 0 : mi > MAGS ? MAGS : mi;
        return neg ? MAGS - in : MAGS + in;
    }
}

typedef u32x4_t __attribute__((aligned(2))) u32x4_a2_t;
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
typedef __attribute__((ext_vector_type(2))) short i16x2_t;

// all ones in the halves that are negative (as assembly: the compiler takes vector shifts by 15 apart into compares)
__device__ __forceinline__ uint32_t sign_masks(uint32_t v) {
    uint32_t r;
    asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(r) : "v"(v));
    return r;
}

__device__ __forceinline__ uint32_t udot2(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b), c, false);
}

__device__ __forceinline__ uint32_t udot4(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_udot4(a, b, c, false); }

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

// NI > 0: the row is at most NI * 4096 elements and a thread keeps its NI pieces of 16 in registers; 0: re-read.  MARKED: only the rows that the kernel of four rows a workgroup left.
template <int BITS, int NI, bool MARKED>
__global__ __launch_bounds__(256, NI == 4 ? 6 : 8) void quantize_rows_hist_kernel(const uint16_t* __restrict__ W, int64_t rowlen, int iters,
                                                                                 uint32_t* __restrict__ packed,
                                                                                 uint16_t* codebook) {
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
    if constexpr (MARKED) {
        if (codebook[n * C] != kRowMark) return;          // (the same for every thread; overwritten behind the first barrier only)
    }
    const uint16_t* w = W + n * rowlen;
    const int K = static_cast<int>(rowlen), pieces = (K + 15) >> 4;

    // ---- 1. the row, its range and its smallest non-zero magnitude, two elements at a time
    uint32_t reg[NI > 0 ? NI : 1][8];
    i16x2_t lo2 = {0x7FFF, 0x7FFF}, hi2 = {-0x7FFF - 1, -0x7FFF - 1};        // of the order-preserving keys
    u16x2_t mn2 = {0xFFFF, 0xFFFF};                                          // magnitude - 1 (zero: 65535)
    auto range_of = [&](const uint32_t (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const u16x2_t mag = __builtin_bit_cast(u16x2_t, v[i] & 0x7FFF7FFFu);
            mn2 = __builtin_elementwise_min(mn2, static_cast<u16x2_t>(mag - u16x2_t{1, 1}));
            const i16x2_t key = __builtin_bit_cast(i16x2_t, v[i] ^ (sign_masks(v[i]) & 0x7FFF7FFFu));
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

// ---- one codebook per row: four rows a workgroup --------------------------------------------------
// The same rounds for many rows.  What bounds them is the instructions of the rounds (a wave for one row's
// few boundaries: 25 rounds are two thirds of all instructions at 4096 elements), so here one wave runs the rounds of four rows
// at once, 16 lanes a row, and everything else is done by the row's own wave.  A round is a chain of
// 1400 clocks that only other rows hide, so a row has to be small in LDS: counters of a byte over a window of 15 octaves below the
// row's largest magnitude, prefix sums over buckets of 16 with number and sum in one 64-bit integer; 24 rows a CU.  A few elements
// below the window ("tiny": one row in three of 4096 normal weights has one) are kept in a list and met one by one where a boundary
// lies among them; rows with more, or with more than 255 of one value other than zero, are left to the kernel above.
// The sums are the same integers, exact in fp64, so the results are the same bits.
// 25 rounds, 14336 x 4096, 1 / 2 / 4 bits, a workgroup a row / this (us): 104 / 132 / 170 -> 78 / 89 / 109;
// 100000 x 64, 2 bits, 10 rounds: 401 -> 160.  Vector issue is 63 % of the busy time at 2 bits, LDS 37 % (61 % of that conflicts of the atomics).
// Where every row is left over, the look at it comes on top: rows of more than 1024 elements are left once a part of their first 1024 has
// shown it.  25 rounds, 2 / 4 bits, a workgroup a row / a look at the whole row / this (us): 4096 x 4096, elements spread evenly over 22
// octaves 42 / 69 / 51 and 59 / 86 / 68; a grid of 15 values (4-bit integers times a scale) 48 / 80 / 61 and 50 / 82 / 63; 14336 x 4096, that
// grid 150 / 245 / 180 and 156 / 251 / 187.  (The look costs ordinary rows 0 to 0.6 %.)
constexpr int kWinOctaves = 15, kWinMags = kWinOctaves * 128, kWinBucket = 16, kWinBuckets = 2 * kWinMags / kWinBucket;
constexpr int kWinRows = 4, kWinTiny = 16, kWinCountBits = 17;
// Cells of a byte, a plane of 2048 for either sign: the window's magnitudes from 16 on, tiny elements at 15, zeros at 1940 (alone in their
// four bytes: a count of 32 bits)
constexpr int kWinPlane = 2048, kWinFirst = 16, kWinTinyKey = 15, kWinZeroKey = 1940;
static_assert(kWinFirst + kWinMags <= kWinZeroKey && kWinZeroKey % 4 == 0, "planes");

typedef uint32_t WinCells[2 * kWinPlane / 4];               // (a power of two: a row's base can be or-ed into an address)
typedef __attribute__((address_space(3))) uint32_t lds_u32_t;
typedef __attribute__((address_space(3))) uint8_t lds_u8_t;
struct alignas(16) WinRow {
    long long below[kWinBuckets + 2];                       // below bucket i: sum in units << 17, plus number
    double lo, hi;
    int base, valid, ntiny, exact;
    uint32_t nzero;
    uint16_t tiny[kWinTiny];
    int thr[16];
    double bound[16];                                       // boundaries of the stored codebook
};

__device__ __forceinline__ uint32_t pk_max_u(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b))); }
__device__ __forceinline__ uint32_t pk_min_u(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b))); }
__device__ __forceinline__ uint32_t pk_max_i(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2_t, a), __builtin_bit_cast(i16x2_t, b))); }

// a value of the lane N below (SHR) or above in the same row of 16 (0 outside)
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(v), CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(v >> 32), CTRL, 0xF, 0xF, true);
    return static_cast<uint64_t>(hi) << 32 | lo;
}
template <int CTRL>
__device__ __forceinline__ double dpp_row_f64(double v) {
    return __longlong_as_double(static_cast<long long>(dpp_u64<CTRL>(static_cast<uint64_t>(__double_as_longlong(v)))));
}

template <int BITS>
__global__ __launch_bounds__(kWinRows * 64, BITS == 4 ? 5 : 6) void quantize_rows_window_kernel(const uint16_t* __restrict__ W, int64_t N, int K, int iters,
                                                                                  uint32_t* __restrict__ packed, uint16_t* __restrict__ codebook) {
    constexpr int C = 1 << BITS, NI = 4, H = kWinMags;
    __shared__ alignas(sizeof(WinCells)) WinCells all_cells[kWinRows];
    __shared__ WinRow rows[kWinRows];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    WinRow& sm = rows[wave];
    uint32_t* const cells = all_cells[wave];
    uint32_t cells_at = static_cast<uint32_t>(reinterpret_cast<size_t>((lds_u32_t*)cells));
    asm volatile("" : "+v"(cells_at));                      // (in a vector register: v_and_or_b32 takes one scalar, the mask)
    const int64_t n = static_cast<int64_t>(blockIdx.x) * kWinRows + wave;
    const bool there = n < N;                               // (uniform over the wave)
    const uint16_t* const w = W + (there ? n : 0) * K;
    const int pieces = there ? (K + 15) >> 4 : 0;
    auto row_sync = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };      // a lone wave's LDS instructions run in order

    // ---- 1. the row and its range.  As patterns: the largest unsigned one is the most negative value, if there is a negative one, the
    // largest signed one the largest value, if there is a positive one; else the smallest unsigned one is that
    uint32_t reg[NI][8];
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if (lane + i * 64 < pieces) load16(w, (lane + i * 64) << 4, K, reg[i]);
    for (int i = lane; i < 2 * kWinPlane / 16; i += 64) reinterpret_cast<u32x4_t*>(cells)[i] = u32x4_t{0, 0, 0, 0};
    uint32_t umax = 0, umin = 0xFFFFFFFFu, smax = 0x80008000u;
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if (lane + i * 64 < pieces) {
#pragma unroll
            for (int j = 0; j < 8; ++j) { umax = pk_max_u(umax, reg[i][j]); umin = pk_min_u(umin, reg[i][j]); smax = pk_max_i(smax, reg[i][j]); }
        }
    const auto halves = [](uint32_t v, bool is_signed, int h) { return is_signed ? static_cast<int>(static_cast<int16_t>(h ? v >> 16 : v)) : static_cast<int>(h ? v >> 16 : v & 0xFFFFu); };
    const auto of_wave = [](int v) { return __builtin_amdgcn_readlane(v, 63); };
    int um = max(halves(umax, false, 0), halves(umax, false, 1)), un = min(halves(umin, false, 0), halves(umin, false, 1)), sx = max(halves(smax, true, 0), halves(smax, true, 1));
    um = of_wave(wave_extreme<true>(um));
    un = of_wave(wave_extreme<false>(un));
    sx = of_wave(wave_extreme<true>(sx));
    const uint32_t lo_h = static_cast<uint32_t>(um >= 0x8000 ? um : un), hi_h = static_cast<uint32_t>(sx >= 0 ? sx : un);
    const int maxmag = max(static_cast<int>(lo_h & 0x7FFFu), static_cast<int>(hi_h & 0x7FFFu));
    const int emax = maxmag == 0 ? 127 : maxmag >> 7;
    bool valid = there && maxmag < 0x7F80 && emax > kWinOctaves;
    const int base = (emax - (kWinOctaves - 1)) << 7;
    row_sync();                                             // cells cleared

    // ---- 2. histogram.  From here on an element is the number of its cell (place in the plane, bit 11 the sign) times 8: the low
    // five bits are the shift that puts a one into the cell's byte
    const auto code_of = [](const uint32_t (&v)[8], int e) { return e & 1 ? v[e >> 1] >> 16 : v[e >> 1] & 0xFFFFu; };
    const uint32_t floor2 = static_cast<uint32_t>(base - 2) * 0x00010001u, base2 = static_cast<uint32_t>(base - 2 - kWinTinyKey) * 0x00010001u;
    const auto to_cells = [&](uint32_t (&v)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t d = v[j];
            const u16x2_t less = __builtin_bit_cast(u16x2_t, d & 0x7FFF7FFFu) - u16x2_t{1, 1};      // (zeros: 65535)
            const u16x2_t k = __builtin_bit_cast(u16x2_t, pk_max_u(__builtin_bit_cast(uint32_t, less), floor2)) - __builtin_bit_cast(u16x2_t, base2);
            const uint32_t key = pk_min_u(__builtin_bit_cast(uint32_t, k), kWinZeroKey * 0x00010001u);
            v[j] = (key << 3) | ((d >> 1) & 0x40004000u);
        }
    };
    const auto count = [&](const uint32_t (&v)[8], auto first) {     // elements first .. first + 7 of a piece
#pragma unroll
        for (int e = decltype(first)::value; e < decltype(first)::value + 8; ++e) {
            const uint32_t d = code_of(v, e);
            lds_u32_t* const cell = reinterpret_cast<lds_u32_t*>(static_cast<size_t>(((d >> 3) & (2 * kWinPlane - 4)) | cells_at));
            __hip_atomic_fetch_add(cell, 1u << (d & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    using std::integral_constant;
    if (valid) {
        if (lane < pieces) {
            to_cells(reg[0]);
            count(reg[0], integral_constant<int, 0>{});
        }
        // A row that will be left over shows it in half of its first pieces: a lane's first element lies below the window and too many
        // others do, or it is one of more equal ones than the share that 255 of the row are.  (A row of one piece a lane has little to leave.)
        if (pieces > 64) {
            row_sync();
            const uint32_t place = code_of(reg[0], 0) >> 3, key = place & (kWinPlane - 1);
            const int alike = *reinterpret_cast<const lds_u8_t*>(static_cast<size_t>(place | cells_at));
            count(reg[0], integral_constant<int, 8>{});              // (while it is on its way)
            const int most = key == kWinTinyKey ? kWinTiny * K : key == kWinZeroKey ? 255 * K : 255 * 8 * 64;
            valid = !__any(alike * K > most);
        }
    }
    if (valid) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (lane + i * 64 < pieces) {
                if (i > 0) {
                    to_cells(reg[i]);
                    count(reg[i], integral_constant<int, 0>{});
                }
                if (i > 0 || pieces <= 64) count(reg[i], integral_constant<int, 8>{});
                const int extra = ((lane + i * 64) << 4) + 16 - K;   // repeats of the first element in the row's last piece
                if (extra > 0) atomicSub(&cells[code_of(reg[i], 0) >> 5], static_cast<uint32_t>(extra) << (reg[i][0] & 31u));
            }
    }
    row_sync();
    const int ntiny = __builtin_amdgcn_readfirstlane(static_cast<int>((cells[kWinTinyKey / 4] >> 24) + (cells[(kWinPlane + kWinTinyKey) / 4] >> 24)));
    if (ntiny > kWinTiny) valid = false;
    if (valid && ntiny > 0 && lane == 0) sm.ntiny = 0;
    row_sync();
    if (valid && ntiny > 0) {                               // the tiny elements themselves
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (lane + i * 64 < pieces) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int k = ((lane + i * 64) << 4) + e;
                    if (((code_of(reg[i], e) >> 3) & (kWinPlane - 1)) == kWinTinyKey && k < K) {
                        const int slot = atomicAdd(&sm.ntiny, 1);
                        if (slot < kWinTiny) sm.tiny[slot] = w[k];
                    }
                }
            }
    }
    row_sync();
    // (the sums have to fit 53 bits down to the smallest element's unit; a counter of more than 255 has lost them)
    if (valid && ntiny > 0) {
        const int log2k = 32 - __clz(K - 1);
        int emin = emax;
        for (int i = 0; i < ntiny; ++i) emin = min(emin, max((sm.tiny[i] & 0x7FFF) >> 7, 1));
        if (emax - emin + 8 + log2k > 53 || sm.ntiny != ntiny) valid = false;
        valid = __builtin_amdgcn_readfirstlane(valid);
    }

    // ---- 3. buckets of 16 magnitudes (a thread each), then prefix sums over them in ascending order of the values
    if (valid) {
        for (int bucket = lane; bucket < kWinBuckets / 2; bucket += 64) {
            uint32_t cp = 0, cn = 0, sp = 0, sn = 0;        // members and place sums of positive / negative ones
            const u32x4_t dp = reinterpret_cast<const u32x4_t*>(cells)[kWinFirst / 16 + bucket], dn = reinterpret_cast<const u32x4_t*>(cells)[(kWinPlane + kWinFirst) / 16 + bucket];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t places = 0x03020100u + j * 0x04040404u;
                cp = udot4(dp[j], 0x01010101u, cp);
                sp = udot4(dp[j], places, sp);
                cn = udot4(dn[j], 0x01010101u, cn);
                sn = udot4(dn[j], places, sn);
            }
            const uint32_t m0 = 128u + static_cast<uint32_t>((bucket * kWinBucket) & 127);
            const long long vp = static_cast<long long>(static_cast<uint64_t>(m0 * cp + sp) << (bucket >> 3));
            const long long vn = static_cast<long long>(static_cast<uint64_t>(m0 * cn + sn) << (bucket >> 3));
            sm.below[kWinBuckets / 2 + bucket + 1] = (vp << kWinCountBits) + cp;
            sm.below[kWinBuckets / 2 - 1 - bucket + 1] = cn - (vn << kWinCountBits);
        }
    }
    row_sync();
    if (valid) {
        constexpr int PER = 4;
        static_assert(kWinBuckets <= PER * 64, "buckets per lane");
        long long v[PER];
        long long mine = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            v[i] = lane * PER + i < kWinBuckets ? sm.below[lane * PER + i + 1] : 0;
            mine += v[i];
        }
        long long run = mine;
        uint32_t unused = 0;
        wave_scan(run, unused);
        run -= mine;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            run += v[i];
            if (lane * PER + i < kWinBuckets) sm.below[lane * PER + i + 1] = run;
        }
        const uint32_t counted = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(run), 63)) & ((1u << kWinCountBits) - 1);
        const uint32_t nzero = cells[kWinZeroKey / 4] + cells[(kWinPlane + kWinZeroKey) / 4];
        if (__builtin_amdgcn_readfirstlane(counted + nzero) + ntiny != static_cast<uint32_t>(K)) valid = false;      // a counter ran over
        if (lane == 0) {
            sm.below[0] = 0;
            sm.lo = bf16_to_f64(lo_h);
            sm.hi = bf16_to_f64(hi_h);
            sm.base = base;
            sm.ntiny = ntiny;
            sm.nzero = nzero;
        }
    }
    valid = __builtin_amdgcn_readfirstlane(valid) != 0;     // (the same in every lane; for the scalar unit)
    if (lane == 0) sm.valid = valid ? 1 : 0;
    __syncthreads();

    // ---- 4. the rounds, one wave: 16 lanes a row, LG of them per cluster and for the boundary above it.  Waves of one number
    // share a SIMD: neighbouring workgroups of a CU take different ones
    if (wave == static_cast<int>((blockIdx.x >> 8) & 3)) {
        constexpr int LG = 16 / C, DPL = LG < 4 ? 4 / LG : 1;   // dwords of a bucket's 16 cells per lane (1 bit: half of the lanes have none)
        WinRow& r = rows[lane >> 4];
        const uint32_t* const rcells = all_cells[lane >> 4];
        const int G = (lane & 15) / LG, p = lane % LG;
        const bool live = r.valid != 0;
        const int rbase = live ? r.base : 128;
        const uint32_t nzero = live ? r.nzero : 0u;
        const int rtiny = live ? r.ntiny : 0;
        const bool any_tiny = __any(rtiny > 0);
        const double l = live ? r.lo : 0.0, h = live ? r.hi : 0.0;
        const double unit = __longlong_as_double(static_cast<long long>((rbase >> 7) - 127 - 7 + 1023) << 52);
        const double floor_mag = __longlong_as_double(static_cast<long long>((rbase >> 7) - 127 + 1023) << 52);   // the window's smallest magnitude
        double tiny_sum = 0.0;
        for (int i = 0; i < rtiny; ++i) tiny_sum += bf16_to_f64(r.tiny[i]);
        const bool top = G >= C - 1;                        // no boundary above the last cluster: everything is below
        double c = l + (G + 0.5) * (h - l) / C;
        int seen = -1;
        for (int t = 0; t < iters; ++t) {
            const double b = 0.5 * (c + dpp_row_f64<0x100 + LG>(c));
            const int below = top ? 2 * H : hist_below<H>(b, rbase);
            const bool middle = top || !(b < 0.0);          // zeros are below
            const bool among = rtiny > 0 && !top && b != 0.0 && fabs(b) < floor_mag;
            const int now = below * 2 + (middle ? 1 : 0);
            if (__all((now == seen && !among) || !live)) break;   // the members of every cluster as in the round before: a fixed point
            seen = among ? -1 : now;
            const int bucket = below >> 4, rest = below & 15;
            const bool pos = bucket >= kWinBuckets / 2;
            const int mb0 = pos ? bucket - kWinBuckets / 2 : kWinBuckets / 2 - 1 - bucket;   // bucket of magnitudes
            const int mb = mb0 < kWinBuckets / 2 ? mb0 : kWinBuckets / 2 - 1;                 // (all below: none of the last one's cells, rest = 0)
            // the bucket's magnitudes below: positive, the first `rest`; negative, all but the first 16 - rest
            const int head = pos ? rest : kWinBucket - rest, plane = pos ? 0 : kWinPlane;
            const uint32_t* const cell = rcells + (plane + kWinFirst + mb * kWinBucket) / 4;
            uint32_t cnt = 0, si = 0;
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const int q = p * DPL + j, bytes = head - 4 * q;
                const uint32_t first = bytes <= 0 ? 0u : 0xFFFFFFFFu >> (bytes < 4 ? 32 - 8 * bytes : 0);
                uint32_t d = cell[LG > 4 ? q & 3 : q] & (pos ? first : ~first);
                if (LG > 4) d = q < 4 ? d : 0u;
                cnt = udot4(d, 0x01010101u, cnt);
                si = udot4(d, 0x03020100u + j * 0x04040404u, si);
            }
            if constexpr (LG > 1) {
                si += cnt * static_cast<uint32_t>(p * DPL * 4);
                auto lanes = [](uint32_t v) {
                    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);
                    if (LG >= 4) v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);
                    if (LG >= 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);
                    return v;
                };
                cnt = lanes(cnt);
                si = lanes(si);
            }
            const uint32_t m0 = 128u + static_cast<uint32_t>((mb * kWinBucket) & 127);
            const long long ds = static_cast<long long>(static_cast<uint64_t>(m0 * cnt + si) << ((mb >> 3) + kWinCountBits));
            long long P = r.below[bucket] + (pos ? ds : -ds) + cnt + (middle ? nzero : 0u);
            double Tt = 0.0;
            if (any_tiny) {
                uint32_t tc = 0;
                if (__any(among)) {
                    for (int i = 0; i < kWinTiny; ++i) {
                        if (__all(i >= rtiny)) break;
                        const double v = bf16_to_f64(r.tiny[i < rtiny ? i : 0]);
                        if (i < rtiny && (top || v <= b)) { Tt += v; ++tc; }
                    }
                } else {                                    // (b = 0: the negative ones; among them only if there is no other case)
                    const bool zero = b == 0.0 && !top;
                    if (__any(zero)) {
                        for (int i = 0; i < rtiny; ++i) {
                            const double v = bf16_to_f64(r.tiny[i]);
                            if (top || v <= b) { Tt += v; ++tc; }
                        }
                    } else if (top || b > 0.0) {
                        Tt = tiny_sum;
                        tc = static_cast<uint32_t>(rtiny);
                    }
                }
                P += tc;
            }
            const long long P0 = static_cast<long long>(dpp_u64<0x110 + LG>(static_cast<uint64_t>(P)));      // (the first cluster's: 0)
            const long long D = P - P0;
            const uint32_t M = static_cast<uint32_t>(D) & ((1u << kWinCountBits) - 1);
            double S = static_cast<double>(D >> kWinCountBits) * unit;
            if (any_tiny) S += Tt - dpp_row_f64<0x110 + LG>(Tt);
            if (M > 0) c = S / static_cast<double>(M);
        }
        const uint16_t hc = f64_to_bf16(c);
        const int64_t rn = static_cast<int64_t>(blockIdx.x) * kWinRows + (lane >> 4);
        if (p == 0 && G < C && rn < N) {
            if (live) codebook[rn * C + G] = hc;
            else if (G == 0) codebook[rn * C] = kRowMark;
        }
        c = bf16_to_f64(hc);
        const double b = 0.5 * (c + dpp_row_f64<0x100 + LG>(c));
        if (p == 0 && G < C - 1) { r.thr[G] = hist_below<H>(b, rbase); r.bound[G] = b; }
        // a boundary among the tiny elements: such a row's elements are compared one by one
        const uint64_t odd = __ballot(G < C - 1 && rtiny > 0 && b != 0.0 && fabs(b) < floor_mag);
        if ((lane & 15) == 0) r.exact = ((odd >> (lane & 48)) & 0xFFFFu) != 0 ? 1 : 0;
    }
    __syncthreads();

    // ---- 5. cluster of every value, over the histogram
    const int wpr = static_cast<int>(words_per_row(BITS, K));
    uint8_t* const table = reinterpret_cast<uint8_t*>(cells);
    if (valid) {
        for (int g = lane; g < H / 16; g += 64) {
            const int m = g * 16;                           // this thread's magnitudes m..m + 15, all like the first of them (of +m and -(m + 15) ...
            int p0 = 0, n1 = 0;                             // ... upwards, that is)
#pragma unroll
            for (int i = 0; i < C - 1; ++i) {
                const int th = sm.thr[i];
                p0 += th <= H + m ? 1 : 0;
                n1 += th <= H - 1 - (m + 15) ? 1 : 0;
            }
            const uint32_t fp = static_cast<uint32_t>(p0) * 0x01010101u, fn = static_cast<uint32_t>(n1) * 0x01010101u;
            reinterpret_cast<u32x4_t*>(table + kWinFirst)[g] = u32x4_t{fp, fp, fp, fp};
            reinterpret_cast<u32x4_t*>(table + kWinPlane + kWinFirst)[g] = u32x4_t{fn, fn, fn, fn};
        }
    }
    row_sync();
    if (valid) {
        for (int task = lane; task < (C - 1) * 16; task += 64) {   // ... and one by one where a boundary lies among them
            const int th = sm.thr[task >> 4], e = task & 15;    // values in ascending order, 0..2H - 1: the 16 around the boundary
            const int v = (th & ~15) + e;
            int z = 0;
#pragma unroll
            for (int i = 0; i < C - 1; ++i) z += sm.thr[i] <= v ? 1 : 0;
            if (v < 2 * H) table[v >= H ? kWinFirst + (v - H) : kWinPlane + kWinFirst + (H - 1 - v)] = static_cast<uint8_t>(z);
        }
        if (lane < 4) {                                       // tiny elements and zeros of either sign: no boundary lies among them (or `exact`)
            int z = 0;
#pragma unroll
            for (int i = 0; i < C - 1; ++i) z += sm.bound[i] < 0.0 || (sm.bound[i] == 0.0 && lane == 0) ? 1 : 0;
            table[(lane & 1 ? kWinPlane : 0) + (lane < 2 ? kWinTinyKey : kWinZeroKey)] = static_cast<uint8_t>(z);
        }
    }
    row_sync();

    // ---- 6. indices, 16 elements (BITS half-words of the stream) per thread and piece
    if (!valid) return;
    uint16_t* const out = reinterpret_cast<uint16_t*>(packed + n * wpr);
    const bool exact = __builtin_amdgcn_readfirstlane(sm.exact) != 0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int piece = lane + i * 64;
        if (piece >= pieces) continue;
        uint32_t half[2] = {0, 0};                          // eight elements each: 8 * BITS bits
        if (exact) {
#pragma unroll 1
            for (int e = 0; e < 16; ++e) {
                const int k = (piece << 4) + e;
                const double v = bf16_to_f64(w[k < K ? k : K - 1]);
                uint32_t a = 0;
                for (int j = 0; j < C - 1; ++j) a += v > sm.bound[j] ? 1u : 0u;
                half[e >> 3] |= a << ((e & 7) * BITS);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t two = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2_t, reg[i][e >> 1]) >> u16x2_t{3, 3});
                const lds_u8_t* const entry = reinterpret_cast<const lds_u8_t*>(static_cast<size_t>((e & 1 ? two >> 16 : two & 0xFFFFu) + cells_at));   // (the halves picked by the addition itself)
                half[e >> 3] |= static_cast<uint32_t>(*entry) << ((e & 7) * BITS);
            }
        }
        uint64_t bits = static_cast<uint64_t>(half[1]) << (8 * BITS) | half[0];
        const int last = K - (piece << 4);
        if (last < 16) bits &= (uint64_t(1) << (last * BITS)) - 1;
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
    }
    if (lane == 0)
        for (int i = pieces * BITS; i < 2 * wpr; ++i) out[i] = 0;
}

// ---- one codebook per row: any data ----------------------------------------------------------------
// One workgroup of four waves per row; the row is re-read from the caches each round.  Where all rows are left by the histogram, 8 rounds, 1 bit / 4 bits: 256 x 4096
// 30 / 112 us, 4096 x 4096 118 / 834 (without the histogram kernel in front 32 / 104 and 116 / 818; with four rows one after the other
// per workgroup, of which none are left as a rule, 114 / 398 and 190 / 1003; the look at the marks costs 1 us at 14336 rows).
template <int BITS, typename F>
__device__ __forceinline__ void row_elements(const uint16_t* w, int64_t K, F&& f) {      // a thread's elements, ascending
    int64_t k = threadIdx.x;
    if constexpr (BITS == 1) {                            // eight in flight (wider: the registers of the clusters' sums are needed)
        for (; k + 7 * 256 < K; k += 8 * 256) {
            uint16_t h[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) h[i] = w[k + i * 256];
#pragma unroll
            for (int i = 0; i < 8; ++i) f(bf16_to_f64(h[i]));
        }
    }
    for (; k < K; k += 256) f(bf16_to_f64(w[k]));
}
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
    row_elements<BITS>(w, K, [&](double v) {
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
    });
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
        row_elements<BITS>(w, K, [&](double v) { cl.add(v); });
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
__global__ __launch_bounds__(256) void quantize_rows_kernel(const uint16_t* __restrict__ W, int64_t K, int iters,
                                                            uint32_t* __restrict__ packed, uint16_t* codebook) {
    constexpr int C = 1 << BITS;
    __shared__ RowShared<BITS> sh;
    const int64_t n = blockIdx.x;
    if constexpr (MARKED) {
        if (codebook[n * C] != kRowMark) return;          // (the same for every thread; overwritten behind the first barrier only)
    }
    quantize_row<BITS>(sh, W, n, K, iters, packed, codebook);
}

// ---- the paper's format: scale per 64-element block, one codebook per tensor -------------------------
// A normalised weight is w / scale, and the quotient of two bf16 values depends only on the scale's mantissa (128 of
// them), the weight's mantissa, the distance of the exponents and the sign.  So the tensor's N*K quotients are counted
// once, per scale mantissa, over the 32 octaves below the scale, in ascending order: 128 x 8192 counters, which carry
// everything a Lloyd round asks for.  The steps:
//   scales   largest magnitude of every block; blocks counted per scale mantissa
//   group    block numbers sorted by scale mantissa (kept in the output's index words until those are written)
//   count    a workgroup takes a run of that list, counts its elements in LDS and adds the counts to the tensor's
//   sort     the counters into the ascending order of their quotients, which is the same for every tensor; number and sum of the
//            members below every sixteenth
//   rounds   one workgroup, all rounds: per boundary its place in that order, and one look-up there
//   assign   every element against its scale mantissa's boundaries, as 16-bit integers
// Quotients are added up as integers (a counter times its quotient's 57 leading bits), so that a cluster's sum, the difference of
// what lies below two boundaries, does not depend on what else lies below.  A boundary b stands for the exact test fl(w / scale) > b: where b * scale comes
// within a few units in the last place of a weight, the division itself decides.
// Infinities and NaNs count as the magnitudes that their patterns continue (in range everywhere); the codebook says NaN then.
// Elements more than 31 octaves below their scale ("far", next to none in most trained tensors) are counted apart per sign, and
// their sums taken from the tensor (below).
//
// 8192 x 8192, 25 rounds, 1 / 2 / 3 / 4 bits, a new tensor each time: 136 / 146 / 154 / 168 us (142 / 154 / 171 / 206 with a look-up per boundary and scale
// mantissa in every round; 8519 / 9344 / 10727 / 13475 with every element divided by its scale and compared with every boundary in fp64, each round);
// 1024 x 1024, 4 bits: 81 (120; 3570).  At 8192 x 8192 and 4 bits: clear 3, scales 22 (6.1 TB/s), group 13, count 30 (blocks gathered 128 bytes at a time,
// LDS atomics, 14 for the adding up), sort 10, rounds 44 (1.5 us each, a chain of latencies of one wave a SIMD; 78 before), assign 45 us (vector issue).
constexpr int kQuantMants = 128;
constexpr double kFar = 4.656612873077393e-10;           // 2^-31: no far element reaches it

// The order of the quotients.  A weight's mantissa a and the scale's s (both 128..255) give a quotient f = a / s where a >= s, else 2a / s,
// times a power of two: every octave of quotients holds each of the 16384 pairs once, in an order that f alone decides (two
// different fractions are far more than an fp64 rounding apart; equal ones follow each other by s).  A place in it is
// octave * 16384 + rank; pairs that the window does not hold (a >= s in octave 0, a < s in the last one) are counters that
// stay zero.  One order per sign, from small magnitudes to large ones.
constexpr int kOctaves = kHistOctaves + 1, kPairs = kQuantMants * 128, kPlaces = kOctaves * kPairs, kRun = 16, kParts = 4096;
constexpr int kLook = 2;                                 // runs that a boundary's row looks at together
constexpr int kSortThreads = 256, kStretch = kSortThreads * kRun, kStretches = kPlaces / kStretch;      // places of a workgroup of the sorting step
// Sums are integers in units of 2^-56 of the octave's lowest quotient: 57 bits of quotient, at most 2^38 members.
struct Below {                                           // members of a stretch below a run of kRun places (or of a whole stretch): number and sum
    unsigned long long n, lo, hi;
};
typedef __int128 int128_t;
typedef unsigned __int128 uint128_t;
__device__ __forceinline__ double sum_to_f64(int128_t v) {
    const uint128_t m = v < 0 ? -static_cast<uint128_t>(v) : static_cast<uint128_t>(v);
    const double d = static_cast<double>(static_cast<unsigned long long>(m >> 64)) * 18446744073709551616.0 + static_cast<double>(static_cast<unsigned long long>(m));
    return v < 0 ? -d : d;
}
// 2^63 / s, and from that the 57 bits of a pair's quotient
__device__ __forceinline__ unsigned long long reciprocal(uint32_t s) { return ((1ull << 63) + s / 2) / s; }
__device__ __forceinline__ unsigned long long quotient_bits(uint32_t a, uint32_t s, unsigned long long recip) { return ((a < s ? 2 * a : a) * recip) >> 7; }
constexpr int kFarChunks = 512, kBlockCounters = 16;
struct FarPart {
    double sum;
    long long num;
};
struct FarScratch {                                      // starts as zeros
    unsigned long long next;                             // search number << 32 | pieces claimed
    unsigned long long done;                             // pieces done, over all searches
    uint32_t arrived, finished, unused[2];
    double bounds[16];                                   // of the present search: changed only when all its pieces are done
};
struct QuantScratch {                                    // layout of the caller's workspace; everything down to `members` starts as zeros
    // (narrow: to its first half)
    FarScratch far;
    unsigned long long cursor[kQuantMants];              // blocks of a scale mantissa placed so far
    unsigned long long zeros, far_neg, far_pos;
    uint32_t exact_assign;                               // a stored boundary lies among the far elements
    uint32_t nonfinite;                                  // a weight is an infinity or a NaN
    union {                                              // (until the rounds begin, when nobody asks for the blocks any more)
        FarPart far_part[kFarChunks][16];
        // blocks per scale mantissa, starting as zeros: a workgroup adds to one of sixteen (all to one: 33 us instead of 20 at 8192 x 8192)
        unsigned long long blocks[kBlockCounters][kQuantMants];
    };
    // per sign, scale mantissa and window position; narrow: both signs in one, the positive ones in the low half
    unsigned long long members[2][kQuantMants][kHistMags];
    Below total[2][kStretches];                          // per sign and stretch
    Below base[2][kPlaces / kRun];
    unsigned long long sorted[2][kPlaces];               // members per place; narrow: 32 bits each
    uint16_t order[kPairs];                              // rank -> scale's mantissa << 7 | weight's mantissa
    uint16_t part_start[kParts];                         // first rank of every part of an octave: of 1 + part / kParts or above (behind `order`: copied together)
    uint32_t above[kQuantMants][16];                     // per stored boundary: largest element key at or below it, in both halves
};

constexpr size_t kClearAll = (offsetof(QuantScratch, members) + sizeof(QuantScratch::members)) / 16, kClearNarrow = (offsetof(QuantScratch, members) + sizeof(QuantScratch::members) / 2) / 16,
                 kClearSmall = offsetof(QuantScratch, far_part) / 16;
// Tensors below this size are "narrow": a counter holds both signs, places are 32 bits wide, and sums of a look's members, times the halves of a
// quotient, 64.  (The copies of
// a 4096 x 4096 tensor that make 2^28 elements take the wide path; 8192 x 8192, 4 bits, narrow instead of wide: count 36 -> 32 us.)
constexpr int64_t kNarrowElements = int64_t(1) << 28;
__global__ __launch_bounds__(256) void bs_clear_kernel(QuantScratch* q, size_t n16) {
    typedef u32x4_t __attribute__((aligned(8))) u32x4_a8_t;
    static_assert(alignof(QuantScratch) == 8 && offsetof(QuantScratch, far_part) % 16 == 0 && offsetof(QuantScratch, members) % 16 == 0, "cleared in 16-byte pieces");
    for (size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x; i < n16; i += static_cast<size_t>(gridDim.x) * 256)
        reinterpret_cast<u32x4_a8_t*>(q)[i] = u32x4_t{0, 0, 0, 0};
}

// The order of the quotients, eight lanes a pair, and the parts' first ranks, eight lanes a part: pairs whose quotient lies below p / q
// (1 <= p / q < 2; of equal ones those of a scale mantissa below s), for sixteen scale mantissas t from `first` on, from p * t / q, which is
// carried from t to t + 1.
__device__ __forceinline__ uint32_t pairs_before(uint32_t p, uint32_t q, int s, int first) {
    int quo = static_cast<int>(p * first / q), rem = static_cast<int>(p * first % q), before = 0;
#pragma unroll 4
    for (int t = first; t < first + 16; ++t) {
        const bool whole = rem == 0, even = (quo & 1) == 0;
        const int below1 = quo - (whole ? 1 : 0), below2 = (quo >> 1) - (whole && even ? 1 : 0);      // largest a with a / t, with 2a / t under p / q
        const int n1 = (below1 < 255 ? below1 : 255) - t + 1, n2 = (below2 < t - 1 ? below2 : t - 1) - 127;
        before += (n1 > 0 ? n1 : 0) + (n2 > 0 ? n2 : 0);
        if (t < s && whole) before += (quo >= t && quo <= 255 ? 1 : 0) + (even && quo >= 256 && quo < 2 * t ? 1 : 0);
        ++quo;
        rem += static_cast<int>(p - q);
        if (rem >= static_cast<int>(q)) { rem -= static_cast<int>(q); ++quo; }
    }
    return lanes_sum<8>(static_cast<uint32_t>(before));
}
constexpr int kOrderGroups = (kPairs + kParts) * 8 / 256;      // workgroups of 256 lanes
__device__ __forceinline__ void bs_order(QuantScratch* q, int group) {
    const int i = (group * 256 + static_cast<int>(threadIdx.x)) >> 3, first = 128 + 16 * (threadIdx.x & 7);
    if (i < kPairs) {                                     // (whole workgroups)
        const int a = 128 + (i & 127), s = 128 + (i >> 7);
        const uint32_t rank = pairs_before(a >= s ? a : 2 * a, s, s, first);
        if ((threadIdx.x & 7) == 0) q->order[rank] = static_cast<uint16_t>(i);
    } else {
        const int part = i - kPairs;
        const uint32_t rank = pairs_before(kParts + part, kParts, 0, first);
        if ((threadIdx.x & 7) == 0) q->part_start[part] = static_cast<uint16_t>(rank < kPairs ? rank : kPairs - 1);      // (none at or above the last parts)
    }
}

// Scales below 2^-95 put part of the window into bf16's subnormal range, where patterns are not spaced by exponents:
// scale and weights are multiplied by 2^64 first (exact; the quotients stay the same).
constexpr uint32_t kSmallScale = 32u << 7;
__device__ __forceinline__ uint32_t lifted(uint32_t h) { return __float_as_uint(__uint_as_float(h << 16) * 1.8446744073709552e19f) >> 16; }
__device__ __forceinline__ uint32_t scale_pattern(uint32_t scale) { return scale < kSmallScale ? lifted(scale) : scale; }
__device__ __forceinline__ void lift_pairs(u32x4_t& v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = lifted(v[i] & 0xFFFFu) | (lifted(v[i] >> 16) << 16);
}

// Magnitude keys of two elements against the block's scale: 0 zero, 1 far, 2 + window position.
__device__ __forceinline__ u16x2_t magnitude_keys(uint32_t pair, uint32_t scale_pat) {
    const uint32_t base = (scale_pat & 0x7F80u) - ((kHistOctaves - 1) << 7);
    const u16x2_t mag = __builtin_bit_cast(u16x2_t, pair & 0x7FFF7FFFu);
    const u16x2_t k = __builtin_elementwise_max(mag, __builtin_bit_cast(u16x2_t, (base - 1) * 0x00010001u)) - __builtin_bit_cast(u16x2_t, (base - 2) * 0x00010001u);
    return __builtin_elementwise_min(k, mag);
}

// largest magnitude of the block that eight neighbouring lanes hold (16 bytes each), in each of them
__device__ __forceinline__ uint32_t block_scale(const u32x4_t& v) {
    const auto mags = [](uint32_t d) { return __builtin_bit_cast(u16x2_t, d & 0x7FFF7FFFu); };
    const u16x2_t m = __builtin_elementwise_max(__builtin_elementwise_max(mags(v[0]), mags(v[1])), __builtin_elementwise_max(mags(v[2]), mags(v[3])));
    uint32_t s = m[0] > m[1] ? m[0] : m[1];
    auto step = [&](uint32_t o) { s = o > s ? o : s; };
    step(__builtin_amdgcn_update_dpp(0, s, 0xB1, 0xF, 0xF, true));         // quad_perm [1,0,3,2]
    step(__builtin_amdgcn_update_dpp(0, s, 0x4E, 0xF, 0xF, true));         // quad_perm [2,3,0,1]
    step(__builtin_amdgcn_update_dpp(0, s, 0x141, 0xF, 0xF, true));        // row_half_mirror
    return s;
}

constexpr int kScaleTurn = 128;                          // blocks per workgroup and turn
__global__ __launch_bounds__(256) void bs_scales_kernel(const uint16_t* __restrict__ W, int64_t nblocks,
                                                        uint16_t* __restrict__ scales, int orders, QuantScratch* q) {
    // (the last workgroups make the order of the quotients: the others wait for memory meanwhile)
    const int group = blockIdx.x, groups = gridDim.x - orders;
    if (group >= groups) {
        bs_order(q, group - groups);
        return;
    }
    __shared__ uint32_t cnt[kQuantMants];
    if (threadIdx.x < kQuantMants) cnt[threadIdx.x] = 0;
    __syncthreads();
    // eight lanes per block, kScaleTurn / 32 blocks in flight per lane
    constexpr int U = kScaleTurn / 32;
    const int64_t step = static_cast<int64_t>(groups) * kScaleTurn;
    for (int64_t b0 = static_cast<int64_t>(group) * kScaleTurn + (threadIdx.x >> 3); b0 < nblocks; b0 += step) {
        u32x4_t v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int64_t blk = b0 + i * 32 < nblocks ? b0 + i * 32 : nblocks - 1;
            v[i] = *reinterpret_cast<const u32x4_t*>(W + blk * KMQ_BLOCK + (threadIdx.x & 7) * 8);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint32_t s = block_scale(v[i]);
            if ((threadIdx.x & 7) == 0 && b0 + i * 32 < nblocks) {
                scales[b0 + i * 32] = static_cast<uint16_t>(s);
                atomicAdd(&cnt[scale_pattern(s) & 127u], 1u);
                if (s >= 0x7F80u) q->nonfinite = 1;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < kQuantMants && cnt[threadIdx.x]) atomicAdd(&q->blocks[group % kBlockCounters][threadIdx.x], static_cast<unsigned long long>(cnt[threadIdx.x]));
}

// First list position of every scale mantissa's blocks (start[128]: their number); by the workgroup's first wave,
// valid behind the next barrier.
__device__ __forceinline__ void list_starts(const QuantScratch* q, long long* start) {
    if (threadIdx.x < 64) {
        const int t = threadIdx.x;
        long long a = 0, b = 0;
#pragma unroll
        for (int i = 0; i < kBlockCounters; ++i) {
            a += static_cast<long long>(q->blocks[i][2 * t]);
            b += static_cast<long long>(q->blocks[i][2 * t + 1]);
        }
        long long incl = a + b;
        uint32_t unused = 0;
        wave_scan(incl, unused);
        start[2 * t] = incl - a - b;
        start[2 * t + 1] = incl - b;
        if (t == 63) start[kQuantMants] = incl;
    }
}

// EACH blocks a thread: at most 128 workgroups where eight suffice for that (every one adds to 128 shared cursors; 8192 x 8192, 1 bit: 135.6 us in all
// with eight, 136.7 with four, 139.0 with sixteen), of as few blocks as that leaves (1024 x 1024, 4 bits: 86.3 us with eight, 81.4 with one).
constexpr int kGroupThreads = 1024;
template <int EACH>
__global__ __launch_bounds__(kGroupThreads) void bs_group_kernel(const uint16_t* __restrict__ scales, int64_t nblocks, QuantScratch* q,
                                                       uint32_t* __restrict__ list) {
    __shared__ long long start[kQuantMants + 1];
    __shared__ uint32_t cnt[kQuantMants];
    __shared__ long long at[kQuantMants];
    list_starts(q, start);
    if (threadIdx.x < kQuantMants) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b0 = static_cast<int64_t>(blockIdx.x) * (kGroupThreads * EACH) + threadIdx.x;
    uint32_t mant[EACH], rank[EACH];
#pragma unroll
    for (int i = 0; i < EACH; ++i)
        if (b0 + i * kGroupThreads < nblocks) {
            mant[i] = scale_pattern(scales[b0 + i * kGroupThreads]) & 127u;
            rank[i] = atomicAdd(&cnt[mant[i]], 1u);
        }
    __syncthreads();
    if (threadIdx.x < kQuantMants && cnt[threadIdx.x])
        at[threadIdx.x] = start[threadIdx.x] + static_cast<long long>(atomicAdd(&q->cursor[threadIdx.x], static_cast<unsigned long long>(cnt[threadIdx.x])));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EACH; ++i)
        if (b0 + i * kGroupThreads < nblocks) list[at[mant[i]] + rank[i]] = static_cast<uint32_t>(b0 + i * kGroupThreads);
}

// Every workgroup counts the elements of its run of the block list, in LDS: cell 2 * magnitude key + sign.
constexpr int kCountThreads = 1024, kCountCells = 2 * (kHistMags + 2);
__global__ __launch_bounds__(kCountThreads) void bs_count_kernel(const uint16_t* __restrict__ W, const uint32_t* __restrict__ list,
                                                                 int64_t nblocks, int64_t run, bool narrow, QuantScratch* q) {
    __shared__ long long start[kQuantMants + 1];
    __shared__ alignas(8) uint32_t cell[kCountCells];
    const int tid = threadIdx.x;
    list_starts(q, start);
    for (int i = tid; i < kCountCells; i += kCountThreads) cell[i] = 0;
    __syncthreads();
    int64_t p = static_cast<int64_t>(blockIdx.x) * run;
    const int64_t end = p + run < nblocks ? p + run : nblocks;
    int mant = 0;
    while (p < end) {
        while (start[mant + 1] <= p) ++mant;              // (uniform; start[128] = nblocks > p)
        const int64_t stop = start[mant + 1] < end ? start[mant + 1] : end;
        // eight lanes per block, two blocks of 64 per turn; the next turn's are requested ahead of the present one's counting
        constexpr int kTurn = kCountThreads / 8 * 2;
        auto request = [&](int64_t t0, u32x4_t (&v)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int64_t t = t0 + i * (kCountThreads / 8);
                v[i] = *reinterpret_cast<const u32x4_t*>(W + static_cast<int64_t>(list[t < stop ? t : stop - 1]) * KMQ_BLOCK + (tid & 7) * 8);
            }
        };
        u32x4_t ahead[2];
        request(p + (tid >> 3), ahead);
        for (int64_t t0 = p + (tid >> 3); t0 < stop; t0 += kTurn) {
            u32x4_t v[2] = {ahead[0], ahead[1]};
            request(t0 + kTurn, ahead);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t s = block_scale(v[i]);
                if (t0 + i * (kCountThreads / 8) >= stop) continue;
                if (s < kSmallScale) { s = lifted(s); lift_pairs(v[i]); }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t d = v[i][j];           // (a vector element itself must not go into a bit cast: it reads element 0)
                    const u16x2_t c = magnitude_keys(d, s) * u16x2_t{2, 2} + (__builtin_bit_cast(u16x2_t, d) >> u16x2_t{15, 15});
                    atomicAdd(&cell[c[0]], 1u);
                    atomicAdd(&cell[c[1]], 1u);
                }
            }
        }
        __syncthreads();
        for (int key = tid; key < kCountCells / 2; key += kCountThreads) {
            u32x2_t* const at = reinterpret_cast<u32x2_t*>(cell) + key;      // positive ones, negative ones
            const u32x2_t c = *at;
            if ((c[0] | c[1]) == 0) continue;
            *at = u32x2_t{0, 0};
            const unsigned long long pos = c[0], neg = c[1];
            if (key < 2) {
                if (key == 0) {
                    atomicAdd(&q->zeros, pos + neg);
                } else {
                    if (pos) atomicAdd(&q->far_pos, pos);
                    if (neg) atomicAdd(&q->far_neg, neg);
                }
            } else if (narrow) {                          // one addition for both signs: 32 us instead of 36
                atomicAdd(&q->members[0][mant][key - 2], neg << 32 | pos);
            } else {
                if (pos) atomicAdd(&q->members[0][mant][key - 2], pos);
                if (neg) atomicAdd(&q->members[1][mant][key - 2], neg);
            }
        }
        __syncthreads();
        p = stop;
    }
}

// Counters -> the order of the quotients, and what lies below every run of a stretch: a run a thread.  Bound by latency: counters are picked
// one by one from the caches, by one workgroup a CU (vector issue 16 %, LDS 6 % of the busy time).  8192 x 8192: 13.5 us with a workgroup per octave and sign, the
// octave's counters in LDS, 9.5 as here.
template <bool NARROW>
__global__ __launch_bounds__(kSortThreads) void bs_sort_kernel(QuantScratch* q) {
    using Count = std::conditional_t<NARROW, uint32_t, unsigned long long>;
    constexpr int WAVES = kSortThreads / 64;
    __shared__ Count turned[kStretch];
    __shared__ unsigned long long recip[kQuantMants];
    __shared__ unsigned long long wn[WAVES];
    __shared__ uint128_t ws[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sign = blockIdx.x / kStretches, stretch = blockIdx.x % kStretches, oct = stretch * kStretch / kPairs;      // quotients from 2^(oct - 32) on; sign 1: negative
    const uint16_t* const order = q->order + stretch * kStretch % kPairs + tid * kRun;
    typedef u32x4_t __attribute__((aligned(8))) u32x4_a8_t;      // (as the workspace)
    const u32x4_t pairs[2] = {reinterpret_cast<const u32x4_a8_t*>(order)[0], reinterpret_cast<const u32x4_a8_t*>(order)[1]};
    auto pair_of = [&](int k) { return (pairs[k >> 3][(k >> 1) & 3] >> (16 * (k & 1))) & 0xFFFFu; };
    if (tid < kQuantMants) recip[tid] = reciprocal(128 + tid);
    Count got[kRun], any = 0;
#pragma unroll
    for (int k = 0; k < kRun; ++k) {
        const uint32_t pair = pair_of(k), m = pair >> 7, a = pair & 127;
        const int o = a >= m ? oct - 1 : oct, in = o < 0 ? 0 : o >= kHistOctaves ? kHistOctaves - 1 : o;      // the weight's octave
        if constexpr (NARROW) {
            const uint32_t c = reinterpret_cast<const uint32_t*>(&q->members[0][m][(in << 7) + a])[sign];
            got[k] = in != o ? 0 : c;
        } else {
            const unsigned long long c = q->members[sign][m][(in << 7) + a];
            got[k] = in != o ? 0 : c;
        }
    }
#pragma unroll
    for (int k = 0; k < kRun; ++k) any |= got[k];
    Count* const sorted = reinterpret_cast<Count*>(q->sorted[0]) + sign * kPlaces + stretch * kStretch;
    Below* const base = q->base[sign] + stretch * kSortThreads;
    if (!__syncthreads_or(any != 0)) {                     // (most octaves of most tensors)
#pragma unroll
        for (int i = 0; i < kRun; ++i) sorted[i * kSortThreads + tid] = 0;
        base[tid] = Below{0, 0, 0};
        if (tid == 0) q->total[sign][stretch] = Below{0, 0, 0};
        return;
    }
    unsigned long long tn = 0, t0 = 0, t1 = 0;
    uint128_t ts = 0;
#pragma unroll
    for (int k = 0; k < kRun; ++k) {
        const uint32_t pair = pair_of(k), m = pair >> 7;
        const unsigned long long f = quotient_bits(128 + (pair & 127), 128 + m, recip[m]);
        tn += got[k];
        if constexpr (NARROW) {                            // (members below 2^28: sums of their halves of a quotient in 64 bits)
            t0 += static_cast<unsigned long long>(got[k]) * (static_cast<uint32_t>(f) & 0x0FFFFFFFu);
            t1 += static_cast<unsigned long long>(got[k]) * static_cast<uint32_t>(f >> 28);
        } else {
            ts += static_cast<uint128_t>(got[k]) * f;
        }
        // a thread's run through LDS, one place turned per thread, so that a wave writes whole lines
        turned[tid * kRun + ((k + tid) & (kRun - 1))] = got[k];
    }
    if constexpr (NARROW) ts = (static_cast<uint128_t>(t1) << 28) + t0;
    unsigned long long in = tn;
    uint128_t is = ts;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long pn = __shfl_up(in, off, 64);
        const unsigned long long lo = __shfl_up(static_cast<unsigned long long>(is), off, 64);
        const unsigned long long hi = __shfl_up(static_cast<unsigned long long>(is >> 64), off, 64);
        if (lane >= off) { in += pn; is += static_cast<uint128_t>(hi) << 64 | lo; }
    }
    if (lane == 63) { wn[wave] = in; ws[wave] = is; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES - 1; ++w)
        if (w < wave) { in += wn[w]; is += ws[w]; }
    auto below = [](unsigned long long n, uint128_t v) { return Below{n, static_cast<unsigned long long>(v), static_cast<unsigned long long>(v >> 64)}; };
    if (tid == kSortThreads - 1) q->total[sign][stretch] = below(in, is);
    base[tid] = below(in - tn, is - ts);
#pragma unroll
    for (int i = 0; i < kRun; ++i) {
        const int at = i * kSortThreads + tid, of = at / kRun;
        sorted[at] = turned[of * kRun + ((at + of) & (kRun - 1))];
    }
}

// Window magnitudes g = mantissa * 2^octave (units of 2^-31 / (128 + scale mantissa)) with fl(g / scale) <= a (STRICT: < a).
template <bool STRICT>
__device__ __forceinline__ int magnitudes_within(double a, double scale) {
    const double x = a * scale;                           // within one unit in the last place of the exact product
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(x));
    int mi = static_cast<int>(static_cast<uint32_t>(u >> 32) >> 13) - ((1023 + 7) << 7);   // largest magnitude <= x (below 0: none)
    const uint64_t r = u + 8;
    if ((static_cast<uint32_t>(r >> 32) & 0x1FFFu) == 0 && static_cast<uint32_t>(r) < 16) {
        mi = static_cast<int>(static_cast<uint32_t>(r >> 32) >> 13) - ((1023 + 7) << 7);   // the magnitude that x is next to
        if (mi >= 0 && mi < kHistMags) {
            const double quot = static_cast<double>(static_cast<uint64_t>(128 + (mi & 127)) << (mi >> 7)) / scale;
            if (!(STRICT ? quot < a : quot <= a)) --mi;
        }
    }
    return mi < -1 ? 0 : mi >= kHistMags ? kHistMags : mi + 1;
}

// Sum over the wave, in every lane: DPP adds within and across rows of 16, then lane 63's value.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(u), CTRL, ROWS, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(u >> 32), CTRL, ROWS, 0xF, false);
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}
__device__ __forceinline__ double wave_total(double v) {
    v += dpp_f64<0x111, 0xF>(v);
    v += dpp_f64<0x112, 0xF>(v);
    v += dpp_f64<0x114, 0xF>(v);
    v += dpp_f64<0x118, 0xF>(v);
    v += dpp_f64<0x142, 0xA>(v);
    v += dpp_f64<0x143, 0xC>(v);
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(u), 63), hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(u >> 32), 63);
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}
// a value that is the same in every lane, for the scalar unit
__device__ __forceinline__ double uniform(double v) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u)), hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32));
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}

// ---- the far elements of the rounds
// Their sums are not in the counters: they are taken from the tensor, once per sign, and again in every round that has a
// boundary among them.  The whole grid does that: the first workgroup to arrive leads (it runs the rounds), the others wait
// for work.  A search cuts the tensor into nchunks pieces; leader and helpers claim them from one counter until none is left,
// and the leader then waits for the claimed ones to be done.  Whoever is waited for is running: nothing depends on how many
// workgroups are resident or in which order they start, and the helpers end when the leader says so.  A piece's sums are
// added in a fixed order, and the pieces' sums in theirs.
// 8192 x 8192, 4 bits, 8 / 25 rounds: 153 / 172 us without far elements, 227 / 254 with 0.01 % of them (one search), 2.7 / 8.0 ms where all but the
// scales are far (a search every round, 0.3 ms each; before the grid helped the rounds' workgroup, 25 rounds took 133 ms with 0.01 %).
template <int C>
struct FarShared {
    double bounds[C];
    double sum[C][C];                                    // per wave and cluster
    int num[C][C];
    uint32_t chunk;
};
constexpr uint32_t kNoChunk = ~0u, kFarEnd = ~0u - 1;

// A piece of the present search for this workgroup, or kNoChunk.
template <int C>
__device__ __forceinline__ uint32_t far_claim(FarShared<C>& sh, FarScratch* f, uint32_t nchunks, bool helper) {
    __syncthreads();                                      // (sh.chunk read by all)
    if (threadIdx.x == 0) {
        uint32_t c = kNoChunk;
        const unsigned long long seen = __hip_atomic_load(&f->next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (seen >> 32 != 0 && static_cast<uint32_t>(seen) < nchunks) {         // (search 0: none has begun)
            const uint32_t got = static_cast<uint32_t>(__hip_atomic_fetch_add(&f->next, 1ull, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT));
            if (got < nchunks) c = got;
        } else if (helper) {
            // (no ordering asked for: an acquire would empty the caches that the leader's rounds live from, at every look)
            if (__hip_atomic_load(&f->finished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) c = kFarEnd;
            else __builtin_amdgcn_s_sleep(32);
        }
        sh.chunk = c;
    }
    __syncthreads();
    return sh.chunk;
}

template <int C>
__device__ __forceinline__ void far_chunk(FarShared<C>& sh, QuantScratch* q, uint32_t chunk, uint32_t nchunks, const uint16_t* W,
                                          const uint16_t* scales, int64_t nblocks) {
    constexpr int T = C * 64, U = 4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < C) sh.bounds[threadIdx.x] = q->far.bounds[threadIdx.x];
    if (lane < C) { sh.sum[wave][lane] = 0.0; sh.num[wave][lane] = 0; }
    __syncthreads();
    const int64_t per = (nblocks + nchunks - 1) / nchunks, first = chunk * per, end = first + per < nblocks ? first + per : nblocks;
    for (int64_t base = first + wave * 8; base < end; base += T / 8 * U) {      // (the whole wave together: eight lanes per block)
        u32x4_t v[U];
        uint32_t sc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = base + u * (T / 8) + (lane >> 3), blk = at < end ? at : end - 1;
            v[u] = *reinterpret_cast<const u32x4_t*>(W + blk * KMQ_BLOCK + (lane & 7) * 8);
            sc[u] = scales[blk];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = base + u * (T / 8) + (lane >> 3) < end;
            const uint32_t sp = scale_pattern(sc[u]);
            u32x4_t l = v[u];
            if (sc[u] < kSmallScale) lift_pairs(l);
            for (int j = 0; j < 4; ++j) {
                const uint32_t d = l[j], raw = v[u][j];
                const u16x2_t k = magnitude_keys(d, sp);
                for (int h = 0; h < 2; ++h) {
                    const bool far = live && k[h] == 1;
                    uint64_t left = __ballot(far);
                    if (left == 0) continue;
                    const double quot = bf16_to_f64(h ? raw >> 16 : raw & 0xFFFFu) / bf16_to_f64(sc[u]);
                    int a = 0;
                    for (int e = 0; e + 1 < C; ++e) a += quot > sh.bounds[e] ? 1 : 0;
                    do {                                  // one cluster after the other
                        const int e = __builtin_amdgcn_readlane(a, __ffsll(static_cast<unsigned long long>(left)) - 1);
                        const bool in = far && a == e;
                        const uint64_t members = __ballot(in);
                        const double t = wave_total(in ? quot : 0.0);
                        if (lane == 0) { sh.sum[wave][e] += t; sh.num[wave][e] += __popcll(members); }
                        left &= ~members;
                    } while (left);
                }
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < C) {
        FarPart p{0.0, 0};
        for (int w = 0; w < C; ++w) { p.sum += sh.sum[w][threadIdx.x]; p.num += sh.num[w][threadIdx.x]; }
        q->far_part[chunk][threadIdx.x] = p;
    }
    __syncthreads();                                      // the workgroup's stores ahead of the leader's sight of them
    if (threadIdx.x == 0) __hip_atomic_fetch_add(&q->far.done, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// All rounds, in one workgroup: a row of sixteen lanes per boundary (four a wave), which finds the boundary's place in the order of the
// quotients and what lies below it; then a lane per cluster, in each of those waves, for the means.  (A wave per
// cluster there is for searches; those without a boundary of their own only meet the barriers of a round.)  Numbers of members are kept as doubles where a
// search adds to them (exact: at most 2^38).
template <int BITS, bool NARROW>
__global__ __launch_bounds__((1 << BITS) * 64) void bs_rounds_kernel(QuantScratch* q, const uint16_t* __restrict__ W,
                                                                  const uint16_t* __restrict__ scales, int64_t nblocks, uint32_t nchunks,
                                                                  int iters, uint16_t* __restrict__ codebook) {
    constexpr int C = 1 << BITS, T = C * 64, ACTIVE = (C + 3) / 4;      // waves with boundaries
    struct Side { unsigned long long n; int128_t s; };    // number and sum, in units of 2^-88
    __shared__ double cs[C];
    __shared__ Side bb[2][16];                            // what lies below boundary i (i = C - 1: all), of this round and the next
    __shared__ Side stretch[2][kStretches], all[2];       // per sign: members of the stretches below; of all
    __shared__ unsigned long long recip[kQuantMants];
    __shared__ alignas(8) uint16_t order[kPairs + kParts];
    const uint16_t* const part_start = order + kPairs;
    __shared__ double fsum_of[C], fnum_of[C];
    __shared__ FarShared<C> fs;
    __shared__ int moved[2], search[2];                   // the round (from 1), of even and odd ones, if a boundary passed a member in it, or lay among the far ones
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, row = tid >> 4, e = tid & 15;
    const double far_neg = static_cast<double>(q->far_neg), far_pos = static_cast<double>(q->far_pos), zeros = static_cast<double>(q->zeros);
    const bool any_far = far_neg + far_pos > 0.0;
    FarScratch* const f = &q->far;
    if (!any_far) {
        if (blockIdx.x != 0) return;
    } else {
        if (tid == 0) fs.chunk = __hip_atomic_fetch_add(&f->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (fs.chunk != 0) {
            for (;;) {
                const uint32_t c = far_claim<C>(fs, f, nchunks, true);
                if (c == kFarEnd) return;
                if (c != kNoChunk) far_chunk<C>(fs, q, c, nchunks, W, scales, nblocks);
            }
        }
    }
    unsigned long long searches = 0;
    // sums and numbers of every cluster's far members, for the boundaries in f->bounds (written by the caller's threads): fsum_of, fnum_of
    auto far_search = [&] {
        ++searches;
        __syncthreads();
        if (tid == 0) __hip_atomic_store(&f->next, searches << 32, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        for (;;) {
            const uint32_t c = far_claim<C>(fs, f, nchunks, false);
            if (c == kNoChunk) break;
            far_chunk<C>(fs, q, c, nchunks, W, scales, nblocks);
        }
        if (tid == 0) {
            while (__hip_atomic_load(&f->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < searches * nchunks) __builtin_amdgcn_s_sleep(2);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        {
            const int i = wave;
            double s = 0.0, n = 0.0;
            for (uint32_t c = lane; c < nchunks; c += 64) { s += q->far_part[c][i].sum; n += static_cast<double>(q->far_part[c][i].num); }
            s = wave_total(s);
            n = wave_total(n);
            if (lane == 0) { fsum_of[i] = s; fnum_of[i] = n; }
        }
        __syncthreads();
    };
    if (iters > 0) {
        if (tid < kQuantMants) recip[tid] = reciprocal(128 + tid);      // (T >= kQuantMants)
        // (part_start lies behind order, in LDS as in the workspace)
        constexpr int kCopies = (kPairs + kParts) / 4 / T;
        unsigned long long v[kCopies];
#pragma unroll
        for (int i = 0; i < kCopies; ++i) v[i] = reinterpret_cast<const unsigned long long*>(q->order)[i * T + tid];
#pragma unroll
        for (int i = 0; i < kCopies; ++i) reinterpret_cast<unsigned long long*>(order)[i * T + tid] = v[i];
        if (wave < 2) {                                   // wave 0: positive, wave 1: negative quotients
            constexpr int EACH = (kStretches + 63) / 64;  // stretches a lane
            Below t[EACH];
#pragma unroll
            for (int k = 0; k < EACH; ++k) t[k] = q->total[wave][lane * EACH + k < kStretches ? lane * EACH + k : 0];
            unsigned long long n = 0, n_of[EACH];
            uint128_t sum = 0, sum_of[EACH];
#pragma unroll
            for (int k = 0; k < EACH; ++k) {
                const int at = lane * EACH + k;
                const bool is = at < kStretches;
                n_of[k] = n;
                sum_of[k] = sum;
                n += is ? t[k].n : 0;
                sum += is ? (static_cast<uint128_t>(t[k].hi) << 64 | t[k].lo) << (at * kStretch / kPairs) : 0;
            }
            const unsigned long long n0 = n;
            const uint128_t sum0 = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const unsigned long long pn = __shfl_up(n, off, 64);
                const unsigned long long lo = __shfl_up(static_cast<unsigned long long>(sum), off, 64);
                const unsigned long long hi = __shfl_up(static_cast<unsigned long long>(sum >> 64), off, 64);
                if (lane >= off) { n += pn; sum += static_cast<uint128_t>(hi) << 64 | lo; }
            }
#pragma unroll
            for (int k = 0; k < EACH; ++k)
                if (lane * EACH + k < kStretches) stretch[wave][lane * EACH + k] = Side{n - n0 + n_of[k], static_cast<int128_t>(sum - sum0 + sum_of[k])};
            if (lane == 63) all[wave] = Side{n, static_cast<int128_t>(sum)};
        }
    }
    if (tid < C) cs[tid] = -1.0 + (2 * tid + 1) / static_cast<double>(C);
    if (tid < 2) moved[tid] = search[tid] = 0;
    double neg_sum = 0.0, pos_sum = 0.0;
    if (any_far && iters > 0) {                           // per sign: all boundaries 0, so the first cluster and the last
        if (tid < C) f->bounds[tid] = 0.0;
        far_search();
        neg_sum = fsum_of[0];
        pos_sum = fsum_of[C - 1];
    }
    __syncthreads();
    // what lies below b of something with a negative and a positive part (b not among the far elements)
    auto far_below = [&](double b, double neg, double pos) { return b >= kFar ? neg + pos : b >= 0.0 ? neg : 0.0; };
    auto zeros_below = [&](double b) { return b >= 0.0 ? zeros : 0.0; };
    auto among_far = [&](double b) { return any_far && b != 0.0 && fabs(b) < kFar; };
    auto row_sum = [](unsigned long long v) {             // in every lane of the row
        auto step = [&](auto ctrl) {
            constexpr int CTRL = decltype(ctrl)::value;
            const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(v), CTRL, 0xF, 0xF, true);
            const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(v >> 32), CTRL, 0xF, 0xF, true);
            v += static_cast<unsigned long long>(hi) << 32 | lo;
        };
        step(std::integral_constant<int, 0xB1>{});        // quad_perm [1,0,3,2]
        step(std::integral_constant<int, 0x4E>{});        // quad_perm [2,3,0,1]
        step(std::integral_constant<int, 0x141>{});       // row_half_mirror
        step(std::integral_constant<int, 0x140>{});       // row_mirror
        return v;
    };
    const bool bounded = row < C - 1;                     // the row has a boundary
    double centroid = cs[e < C ? e : 0];                  // of cluster e, in every row
    unsigned long long seen = ~0ull;
    auto lane_f64 = [&](int from) {
        const uint64_t u = static_cast<uint64_t>(__double_as_longlong(centroid));
        const uint32_t lo = __builtin_amdgcn_ds_bpermute(from * 4, static_cast<uint32_t>(u)), hi = __builtin_amdgcn_ds_bpermute(from * 4, static_cast<uint32_t>(u >> 32));
        return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
    };
    for (int t = 0; t < iters; ++t) {
      if (wave < ACTIVE) {
        // the row's boundary, from its lanes `row` and `row + 1`
        const double b = 0.5 * (lane_f64(bounded ? row : 0) + lane_f64(bounded ? row + 1 : 0));
        const bool neg = b < 0.0;
        const int sign = neg ? 1 : 0;
        // Its place: the octave and the part by its leading bits; from that part's run on all quotients up to the first one above b.
        // An equal quotient lies below a positive boundary and (by falling magnitude) above a negative one.
        const uint64_t u = static_cast<uint64_t>(__double_as_longlong(b)) & 0x7FFFFFFFFFFFFFFFull;
        const int oct = static_cast<int>(u >> 52) - (1023 - kHistOctaves);      // quotients of 2^(oct - 32) and more
        const uint32_t o = oct < 0 ? 0 : oct >= kOctaves ? kOctaves - 1 : oct;
        const unsigned long long bits = oct < 0 ? 0 : oct >= kOctaves ? ~0ull : (1ull << 56) | (u & ((1ull << 52) - 1)) << 4;
        uint32_t first = oct < 0 ? 0 : part_start[static_cast<int>(u >> 40) & (kParts - 1)] & ~(kRun - 1u);      // in the octave
        const Side below = stretch[sign][(o * kPairs + first) / kStretch];
        // (atomic loads, so that they are issued here and not behind the search)
        const unsigned long long* const base = reinterpret_cast<const unsigned long long*>(&q->base[sign][(o * kPairs + first) / kRun]);
        auto now = [](const auto* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
        const unsigned long long base_n = now(base), base_lo = now(base + 1), base_hi = now(base + 2);
        unsigned long long num = 0, s0 = 0, s1 = 0, s2 = 0;
        for (;;) {
            unsigned long long c[kLook], fq[kLook];
#pragma unroll
            for (int k = 0; k < kLook; ++k) {
                const uint32_t at = sign * kPlaces + o * kPairs + first + k * kRun + e;
                const uint32_t* const p = reinterpret_cast<const uint32_t*>(q->sorted[0]) + (NARROW ? at : 2 * at);
                c[k] = now(p);
                if constexpr (!NARROW) c[k] |= static_cast<unsigned long long>(now(p + 1)) << 32;
            }
            bool near = false, in[kLook];
#pragma unroll
            for (int k = 0; k < kLook; ++k) {
                const uint32_t rank = first + k * kRun + e, pair = order[rank & (kPairs - 1)], m = pair >> 7;
                fq[k] = quotient_bits(128 + (pair & 127), 128 + m, recip[m]);
                in[k] = fq[k] < bits && rank < kPairs;
                near |= fq[k] - bits + 64 < 128;
            }
            if (__any(near)) {                            // quotients next to their boundary: the division itself decides
#pragma unroll
                for (int k = 0; k < kLook; ++k) {
                    const uint32_t rank = first + k * kRun + e, pair = order[rank & (kPairs - 1)], a = 128 + (pair & 127), s = 128 + (pair >> 7);
                    const double quot = static_cast<double>(a < s ? 2 * a : a) / static_cast<double>(s), mid = __longlong_as_double(static_cast<long long>(1023ull << 52 | (u & ((1ull << 52) - 1))));
                    if (fq[k] - bits + 64 < 128) in[k] = (neg ? quot < mid : quot <= mid) && rank < kPairs;
                }
            }
#pragma unroll
            for (int k = 0; k < kLook; ++k) {
                c[k] = in[k] ? c[k] : 0;
                num += c[k];
                if constexpr (NARROW) {
                    s0 += static_cast<unsigned long long>(static_cast<uint32_t>(c[k])) * (static_cast<uint32_t>(fq[k]) & 0x0FFFFFFFu);
                    s1 += static_cast<unsigned long long>(static_cast<uint32_t>(c[k])) * static_cast<uint32_t>(fq[k] >> 28);
                } else {                                  // (at most 2^38 members, 19 bits of quotient at a time)
                    s0 += c[k] * (static_cast<uint32_t>(fq[k]) & 0x7FFFFu);
                    s1 += c[k] * (static_cast<uint32_t>(fq[k] >> 19) & 0x7FFFFu);
                    s2 += c[k] * static_cast<uint32_t>(fq[k] >> 38);
                }
            }
            // rows whose last quotient lies below go on (the others' further looks would find nothing: their quotients are above)
            if (__ballot(in[kLook - 1] && bounded && e == kRun - 1) == 0) break;
            first += kLook * kRun;
        }
        uint128_t sum = static_cast<uint128_t>(base_hi) << 64 | base_lo;
        sum += row_sum(s0);
        if constexpr (NARROW) {
            num = lanes_sum<16>(static_cast<uint32_t>(num));
            sum += static_cast<uint128_t>(row_sum(s1)) << 28;
        } else {
            num = row_sum(num);
            sum += static_cast<uint128_t>(row_sum(s1)) << 19;
            sum += static_cast<uint128_t>(row_sum(s2)) << 38;
        }
        if (e == 0 && bounded) {
            num += below.n + base_n;
            const int128_t vs = below.s + static_cast<int128_t>(sum << o);
            bb[t & 1][row] = neg ? Side{all[1].n - num, vs - all[1].s} : Side{all[1].n + num, vs - all[1].s};
            num = num * 4 + (neg ? 0 : 1) + (fabs(b) < kFar ? 0 : 2);      // (b passes zeros and far members, too)
            if (num != seen) moved[t & 1] = t + 1;
            seen = among_far(b) ? ~0ull : num;            // (on its way to 0 it passes far members that are counted nowhere)
        }
        if (e == 0 && row == C - 1) bb[t & 1][row] = Side{all[0].n + all[1].n, all[0].s - all[1].s};
        if (any_far && e == 0 && bounded) {
            f->bounds[row] = b;
            if (among_far(b)) moved[t & 1] = search[t & 1] = t + 1;
        }
      }
        __syncthreads();
        if (moved[t & 1] != t + 1) break;                        // every boundary where it was: a fixed point
        const bool searched = any_far && search[t & 1] == t + 1;
        if (searched) far_search();
        if (wave >= ACTIVE) continue;
        const int i = e < C ? e : 0;
        const Side hi = bb[t & 1][i], lo = i > 0 ? bb[t & 1][i - 1] : Side{0, 0};
        double n = static_cast<double>(hi.n - lo.n), s = sum_to_f64(hi.s - lo.s) * 3.2311742677852644e-27;      // 2^-88
        // boundaries of cluster e
        const double above = lane_f64(i + 1 < C ? i + 1 : i), under = lane_f64(i > 0 ? i - 1 : 0);
        const double bh = i + 1 < C ? 0.5 * (centroid + above) : 2.0, bl = i > 0 ? 0.5 * (under + centroid) : -2.0;
        n += zeros_below(bh) - zeros_below(bl);
        if (any_far) {
            s += searched ? fsum_of[i] : far_below(bh, neg_sum, pos_sum) - far_below(bl, neg_sum, pos_sum);
            n += searched ? fnum_of[i] : far_below(bh, far_neg, far_pos) - far_below(bl, far_neg, far_pos);
        }
        const double mean = s / n;
        centroid = n > 0.0 ? mean : centroid;
    }
    __syncthreads();
    if (any_far && tid == 0) __hip_atomic_store(&f->finished, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    if (tid < C) {
        const uint16_t hc = f64_to_bf16(centroid);
        codebook[tid] = q->nonfinite ? 0x7FC0 : hc;
        cs[tid] = bf16_to_f64(hc);
    }
    __syncthreads();
    if (wave < C - 1) {
        const int i = wave;
        const double b = uniform(0.5 * (cs[i] + cs[i + 1]));
        if (lane == 0 && among_far(b)) q->exact_assign = 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double scale = static_cast<double>(static_cast<uint64_t>(128 + lane + 64 * h) << (kHistOctaves - 1));      // in the window's unit
            // largest key (sign * magnitude key) at or below b: zero 0, far 1, window position + 2
            const int below = b < 0.0 ? kHistMags - magnitudes_within<true>(-b, scale) : kHistMags + magnitudes_within<false>(b, scale);
            const int key = b < 0.0 ? -(kHistMags - below) - 2 : b == 0.0 ? 0 : below - kHistMags + 1;
            q->above[lane + 64 * h][i] = (static_cast<uint32_t>(key) & 0xFFFFu) * 0x00010001u;
        }
    }
}

// Nearest stored centroid for every element, packed: a lane takes 16 elements (BITS half-words of the stream).
// Two elements at a time, as 16-bit keys: a binary search over the boundaries with the sign masks of differences.
template <int BITS>
__global__ __launch_bounds__(256) void bs_assign_pack_kernel(const uint16_t* __restrict__ W,
                                                             const uint16_t* __restrict__ scales,
                                                             const uint16_t* __restrict__ codebook, int64_t npieces,
                                                             const QuantScratch* __restrict__ q, uint32_t* __restrict__ packed) {
    constexpr int C = 1 << BITS;
    // rows of 4 dwords more than they hold: the 16 rows that a wave's lanes read start in different bank groups
    __shared__ alignas(16) uint32_t above[kQuantMants][C < 4 ? 4 : C == 4 ? 4 : C + 4];
    for (int i = threadIdx.x; i < kQuantMants * C; i += 256) above[i / C][i % C] = q->above[i / C][i % C];
    const bool exact = q->exact_assign != 0;
    __syncthreads();
    for (int64_t piece = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; piece < npieces; piece += static_cast<int64_t>(gridDim.x) * 256) {
        u32x4_t v[2];
        v[0] = *reinterpret_cast<const u32x4_t*>(W + piece * 16);
        v[1] = *reinterpret_cast<const u32x4_t*>(W + piece * 16 + 8);
        const uint32_t scale = scales[piece >> 2];
        uint64_t bits = 0;
        if (exact) {                                      // boundaries among the far elements: in fp64
            const double s = bf16_to_f64(scale);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t d = v[e >> 3][(e >> 1) & 3];
                const double x = s > 0.0 ? bf16_to_f64(e & 1 ? d >> 16 : d & 0xFFFFu) / s : 0.0;
                uint32_t a = 0;
                for (int j = 0; j + 1 < C; ++j) a += x > 0.5 * (bf16_to_f64(codebook[j]) + bf16_to_f64(codebook[j + 1])) ? 1 : 0;
                bits |= static_cast<uint64_t>(a) << (e * BITS);
            }
        } else {
            uint32_t sp = scale;
            if (scale < kSmallScale) { sp = lifted(scale); lift_pairs(v[0]); lift_pairs(v[1]); }
            const uint32_t* row = above[sp & 127u];
            uint32_t th[C < 4 ? 4 : C];
#pragma unroll
            for (int j = 0; j < (C < 4 ? 4 : C); j += 4) {
                const u32x4_t r = *reinterpret_cast<const u32x4_t*>(row + j);
                th[j] = r[0]; th[j + 1] = r[1]; th[j + 2] = r[2]; th[j + 3] = r[3];
            }
            uint32_t half[2] = {0, 0};
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const uint32_t d = v[e >> 3][(e >> 1) & 3];
                const uint32_t sg = sign_masks(d);
                const i16x2_t key = __builtin_bit_cast(i16x2_t, __builtin_bit_cast(uint32_t, magnitude_keys(d, sp)) ^ sg) - __builtin_bit_cast(i16x2_t, sg);
                auto greater = [&](uint32_t t) {          // all ones where the key lies above boundary key t
                    return sign_masks(__builtin_bit_cast(uint32_t, static_cast<i16x2_t>(__builtin_bit_cast(i16x2_t, t) - key)));
                };
                auto pick = [](uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); };
                uint32_t idx;                             // the two indices, in the two halves
                const uint32_t m0 = greater(th[C / 2 - 1]);
                idx = m0 & (0x00010001u << (BITS - 1));
                if constexpr (BITS >= 2) {
                    const uint32_t m1 = greater(pick(m0, th[C / 2 + C / 4 - 1], th[C / 4 - 1]));
                    idx |= m1 & (0x00010001u << (BITS - 2));
                    if constexpr (BITS >= 3) {
                        const uint32_t m2 = greater(pick(m0, pick(m1, th[7 * C / 8 - 1], th[5 * C / 8 - 1]), pick(m1, th[3 * C / 8 - 1], th[C / 8 - 1])));
                        idx |= m2 & (0x00010001u << (BITS - 3));
                        if constexpr (BITS >= 4) {
                            const uint32_t hi = pick(m1, pick(m2, th[14], th[12]), pick(m2, th[10], th[8]));
                            const uint32_t lo = pick(m1, pick(m2, th[6], th[4]), pick(m2, th[2], th[0]));
                            idx |= greater(pick(m0, hi, lo)) & 0x00010001u;
                        }
                    }
                }
                const uint32_t two = (idx | (idx >> (16 - BITS))) & ((1u << (2 * BITS)) - 1);
                half[e >> 3] |= two << ((e & 7) * BITS);
            }
            bits = static_cast<uint64_t>(half[1]) << (8 * BITS) | half[0];
        }
        if constexpr (BITS == 2) {
            packed[piece] = static_cast<uint32_t>(bits);
        } else if constexpr (BITS == 4) {
            typedef u32x2_t __attribute__((aligned(4))) u32x2_a4_t;
            *reinterpret_cast<u32x2_a4_t*>(packed + piece * 2) = u32x2_t{static_cast<uint32_t>(bits), static_cast<uint32_t>(bits >> 32)};
        } else {
            uint16_t* out = reinterpret_cast<uint16_t*>(packed);
#pragma unroll
            for (int j = 0; j < BITS; ++j) out[piece * BITS + j] = static_cast<uint16_t>(bits >> (16 * j));
        }
    }
}

// All of it in one workgroup, every element against every boundary: a few rounds on a small tensor, which the counters' fixed
// cost of about 40 us outweighs.  64 x 64, 1 round, 1 / 4 bits: 17 / 19 us (counts: 42 / 46); 4 rounds: 17 / 45 (46 / 56).
constexpr int kSmallChunks = 4;                          // of eight elements per thread
constexpr int64_t kSmallBlocks = 256 * kSmallChunks / 8;
constexpr int kSmallRounds = 4;
template <int BITS>
__global__ __launch_bounds__(256) void bs_small_kernel(const uint16_t* __restrict__ W, int nblocks, int iters, uint32_t* __restrict__ packed,
                                                       uint16_t* __restrict__ codebook, uint16_t* __restrict__ scales) {
    constexpr int C = 1 << BITS, U = kSmallChunks;
    __shared__ double cs[C];
    __shared__ double ps[4][C];
    __shared__ int pn[4][C];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nchunks = nblocks * 8;
    double v[U][8];
    bool nonfinite = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {                         // eight lanes per block
        const int c = tid + u * 256;
        const u32x4_t w = *reinterpret_cast<const u32x4_t*>(W + (c < nchunks ? c : nchunks - 8 + (tid & 7)) * 8);
        const uint32_t s = block_scale(w);
        if ((tid & 7) == 0 && c < nchunks) scales[c >> 3] = static_cast<uint16_t>(s);
        nonfinite |= s >= 0x7F80u;
        const double scale = bf16_to_f64(s);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t d = w[e >> 1];
            v[u][e] = s != 0 ? bf16_to_f64(e & 1 ? d >> 16 : d & 0xFFFFu) / scale : 0.0;
        }
    }
    if (tid < C) cs[tid] = -1.0 + (2 * tid + 1) / static_cast<double>(C);
    nonfinite = __syncthreads_or(nonfinite ? 1 : 0) != 0;
    Clusters<C> cl;
    double c[C];
    for (int t = 0; t < iters; ++t) {
#pragma unroll
        for (int j = 0; j < C; ++j) c[j] = cs[j];
        cl.begin(c);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (tid + u * 256 < nchunks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) cl.add(v[u][e]);
            }
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const double s = wave_sum(cl.s[j]);
            const int m = static_cast<int>(wave_sum(static_cast<long long>(cl.n[j])));
            if (lane == 0) { ps[wave][j] = s; pn[wave][j] = m; }
        }
        __syncthreads();
        if (tid < C) {
            const double s = ((ps[0][tid] + ps[1][tid]) + ps[2][tid]) + ps[3][tid];
            const int m = pn[0][tid] + pn[1][tid] + pn[2][tid] + pn[3][tid];
            if (m > 0) cs[tid] = s / static_cast<double>(m);
        }
        __syncthreads();
    }
    if (tid < C) {
        const uint16_t h = f64_to_bf16(cs[tid]);
        codebook[tid] = nonfinite ? 0x7FC0 : h;
        cs[tid] = bf16_to_f64(h);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C; ++j) c[j] = cs[j];
    cl.begin(c);
    uint8_t* const out = reinterpret_cast<uint8_t*>(packed);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (tid + u * 256 >= nchunks) break;
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) bits |= static_cast<uint32_t>(cl.assign(v[u][e])) << (e * BITS);
#pragma unroll
        for (int i = 0; i < BITS; ++i) out[(tid + u * 256) * BITS + i] = static_cast<uint8_t>(bits >> (8 * i));
    }
}

// Four rows a workgroup need many rows, and more of them where rows are long and rounds few: what it saves is the rounds.  Measured (us), a
// workgroup a row / four rows, 1 / 2 / 3 / 4 bits:
//   2560 x 2048, no round 13.3 / 13.4, 13.7 / 13.6, 14.3 / 14.4, 15.8 / 15.9; one 14.2 / 14.1, 14.7 / 14.2, 15.3 / 15.1, 17.2 / 16.6; three
//     15.9 / 15.0, 16.5 / 15.1, 17.3 / 16.3, 19.3 / 17.9
//   3000 x 4096, no round 16.8 / 18.0, 17.4 / 18.3, 18.4 / 19.3, 20.1 / 20.8; one 17.8 / 19.0, 18.4 / 19.2, 19.4 / 20.2, 21.6 / 21.8; three
//     19.6 / 19.9, 20.2 / 20.1, 21.5 / 21.4, 23.6 / 23.0; four 20.6 / 20.5, 21.0 / 20.6, 22.5 / 22.0, 24.7 / 23.6; 25 31.6 / 30.1,
//     38.2 / 31.6, 41.4 / 34.6, 46.1 / 36.3 (2560 x 4096, 2 bits, 8 rounds: 21.8 / 23.0)
//   7000 x 4096, no round 31.5 / 33.2, 32.7 / 33.6, 34.6 / 35.5, 37.8 / 38.8; 10240 x 4096 42.7 / 40.8, 44.4 / 41.4, 46.6 / 43.4, 51.1 / 47.2
constexpr int64_t kWinMostK = 4096;
static int64_t window_least_rows(int64_t K, int iters) { return K <= 2048 ? 2560 : iters >= 4 ? 3000 : 9216; }

size_t quantize_blockscaled_workspace_bytes() { return sizeof(QuantScratch); }

template <int BITS>
static hipError_t quantize_rows_bits(const uint16_t* W, int64_t N, int64_t K, int iters, uint32_t* packed,
                                     uint16_t* codebook, hipStream_t s) {
    const dim3 rows(static_cast<unsigned>(N)), block(256);
    // without rounds a short row does not repay its histogram (100000 x 64, 1 / 2 / 3 / 4 bits: 258 / 276 / 303 / 339 us with it,
    // 148 / 158 / 237 / 413 without)
    if (K > kHistMaxK || (iters == 0 && K <= 512 && BITS <= 3)) {
        hipLaunchKernelGGL((quantize_rows_kernel<BITS, false>), rows, block, 0, s, W, K, iters, packed, codebook);
        return hipGetLastError();
    }
    if (K <= kWinMostK && N >= window_least_rows(K, iters)) {
        hipLaunchKernelGGL((quantize_rows_window_kernel<BITS>), dim3(static_cast<unsigned>((N + kWinRows - 1) / kWinRows)), dim3(kWinRows * 64), 0, s,
                           W, N, static_cast<int>(K), iters, packed, codebook);
        hipLaunchKernelGGL((quantize_rows_hist_kernel<BITS, 1, true>), rows, block, 0, s, W, K, iters, packed, codebook);
        hipLaunchKernelGGL((quantize_rows_kernel<BITS, true>), rows, block, 0, s, W, K, iters, packed, codebook);
        return hipGetLastError();
    }
#define KMQ_HIST(NI) hipLaunchKernelGGL((quantize_rows_hist_kernel<BITS, NI, false>), rows, block, 0, s, W, K, iters, packed, codebook)
    if (K <= 4096) KMQ_HIST(1);
    else if (K <= 8192) KMQ_HIST(2);
    else if (K <= 16384) KMQ_HIST(4);
    else KMQ_HIST(0);
#undef KMQ_HIST
    hipLaunchKernelGGL((quantize_rows_kernel<BITS, true>), rows, block, 0, s, W, K, iters, packed, codebook);
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
    const int64_t nblocks = N * (K / KMQ_BLOCK), npieces = nblocks * 4;
    auto grid = [](int64_t items, int64_t each, int64_t most) {
        const int64_t g = (items + each - 1) / each;
        return dim3(static_cast<unsigned>(g < most ? g : most));
    };
    if (nblocks <= kSmallBlocks && iters <= kSmallRounds) {
        hipLaunchKernelGGL((bs_small_kernel<BITS>), dim3(1), dim3(256), 0, s, W, static_cast<int>(nblocks), iters, packed, codebook, scales);
        return hipGetLastError();
    }
    const bool narrow = N * K < kNarrowElements;
    const size_t clear = iters == 0 ? kClearSmall : narrow ? kClearNarrow : kClearAll;
    const int orders = iters ? kOrderGroups : 0;
    hipLaunchKernelGGL(bs_clear_kernel, grid(static_cast<int64_t>(clear), 256, 2048), dim3(256), 0, s, q, clear);
    hipLaunchKernelGGL(bs_scales_kernel, dim3(grid(nblocks, kScaleTurn, 1024).x + orders), dim3(256), 0, s, W, nblocks, scales, orders, q);
    if (iters) {                                          // (without rounds nothing is counted)
        auto group = [&](auto each) {
            constexpr int EACH = decltype(each)::value;
            hipLaunchKernelGGL(bs_group_kernel<EACH>, dim3(static_cast<unsigned>((nblocks + kGroupThreads * EACH - 1) / (kGroupThreads * EACH))), dim3(kGroupThreads), 0, s,
                               scales, nblocks, q, packed);
        };
        if (nblocks <= 128 * kGroupThreads) group(std::integral_constant<int, 1>{});
        else if (nblocks <= 256 * kGroupThreads) group(std::integral_constant<int, 2>{});
        else if (nblocks <= 512 * kGroupThreads) group(std::integral_constant<int, 4>{});
        else group(std::integral_constant<int, 8>{});
        // Two workgroups of 16 waves a CU, of at least 64 blocks each to spread the clearing and flushing of 8196 counters (1024 x 1024: 6 us more
        // with 16; 8192 x 8192: 44 us in all with four workgroups of eight waves, 34 with two), but at least one workgroup a CU: it flushes once per scale mantissa among its blocks (64 x 64: 171 us in one
        // workgroup, 49 with a block each; 25 rounds, 1 bit).
        const int64_t least = nblocks < 64 * 256 ? (nblocks + 255) / 256 : 64, run = (nblocks + 511) / 512 < least ? least : (nblocks + 511) / 512;
        hipLaunchKernelGGL(bs_count_kernel, dim3(static_cast<unsigned>((nblocks + run - 1) / run)), dim3(kCountThreads), 0, s, W, packed, nblocks, run, narrow, q);
        if (narrow) hipLaunchKernelGGL(bs_sort_kernel<true>, dim3(2 * kStretches), dim3(kSortThreads), 0, s, q);
        else hipLaunchKernelGGL(bs_sort_kernel<false>, dim3(2 * kStretches), dim3(kSortThreads), 0, s, q);
    }
    // one workgroup runs the rounds; the others, a few a CU, end at once unless there are far elements
    const uint32_t nchunks = static_cast<uint32_t>(nblocks < 256 * kFarChunks ? (nblocks + 255) / 256 : kFarChunks);
    const dim3 round_grid(iters == 0 ? 1 : BITS <= 2 ? 512 : 256), round_block((1 << BITS) * 64);
    if (narrow) hipLaunchKernelGGL((bs_rounds_kernel<BITS, true>), round_grid, round_block, 0, s, q, W, scales, nblocks, nchunks, iters, codebook);
    else hipLaunchKernelGGL((bs_rounds_kernel<BITS, false>), round_grid, round_block, 0, s, q, W, scales, nblocks, nchunks, iters, codebook);
    hipLaunchKernelGGL((bs_assign_pack_kernel<BITS>), grid(npieces, 256, 4096), dim3(256), 0, s, W, scales, codebook, npieces, q, packed);
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
