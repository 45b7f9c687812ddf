// Products with the matrix cores for any row length: any N and K, batch 1..16, canonical or tiled layout, one codebook per row or
// the block-scaled format (paper App. D/E: up to a batch of a few tens the product is bound by the transfer of W, provided
// each weight is dequantised once for the whole batch).  Instances of one bit-width per file: kmq_mfma_any_b1.hip .. b4.hip.
//
// Split.  K is cut into tiles of 256 columns (1-bit tiled: 512, a super-block of that layout).  A workgroup owns RB blocks of 16
// rows; its NW waves take the tiles in turn (wave w: tiles w, w + NW, ...), so that at any time they read neighbouring pieces of
// the same rows.  For a tile a wave stages its columns of X through a wave-private piece of LDS (global loads in runs of at least
// 64 bytes, read back as matrix operands), keeps those operands in registers and goes through the RB row blocks: lane (n, q) =
// (lane & 15, lane >> 4) holds a quarter of the tile's columns of row n -- canonical: columns 64q..64q+63, 2 * BITS consecutive
// words; tiled: the layout's granules, every eighth column 32j + 8q -- decodes eight weights at a time into the second operand
// of v_mfma_f32_16x16x32_bf16 (k = the lanes' eight columns, X first), and requests the words of its next tile as soon as the
// present ones are decoded.  D holds batch columns 4q..4q+3 of row n, so what belongs to a row (scales, centroids) is needed by
// the lane that loads it.  The partial tiles of the waves (of a wave's two chains) are added through LDS, pairwise.  A last tile that K does not fill is one
// wave's; columns past K are zeros in both operands, so that an infinite centroid meets no zero.
//
// Decode.  The columns of a matrix step may be any eight, as long as both operands agree:
//   1-bit  nibble -> four 16-bit masks from a table in LDS; the mask chooses between the row's two centroids;
//   2-bit  (w >> 2c) & 0x03030303 are four indices in four bytes (canonical: columns c, c+4, c+8, c+12 of a word, tiled: four
//          neighbours): a v_perm_b32 selector into the low and high bytes of the row's four centroids; canonical X is staged in
//          that order;
//   3-bit  canonical: 24 bits of eight columns are spread to four bytes of two fields; even and odd fields are the selectors, X is
//          staged as columns 0, 2, 4, 6, 1, 3, 5, 7; tiled: the granule holds selectors;
//   4-bit  a table [centroid][lane] in LDS (a lane reads its own bank).
//
// Block scales.  A scale may only be applied to a sum over its own 64 columns, and a matrix step adds over the four lane
// groups q.  On the tiled layout two steps are a block.  On the canonical one the groups exchange words (a 4 x 4 transpose with
// half-row swaps, four instructions per four registers) so that a step's 32 columns lie in one block; two steps give the
// block's sum, which is added to the result times the scale.
#ifndef KMQ_MFMA_ANY_H
#define KMQ_MFMA_ANY_H

#include <type_traits>

#include "kmq_device.h"
#include "kmq_launch.h"

namespace kmq {

constexpr int kCanonTile = 256;

typedef u32x4_t __attribute__((aligned(2))) cu32x4_a2_t;
typedef u32x2_t __attribute__((aligned(2))) cu32x2_a2_t;
typedef __attribute__((address_space(3))) const uint32_t clds_cu32_t;

// Words w[0..WPL-1] of a lane, 4-byte aligned.  Not non-temporal, and neither are scales: one instruction takes 32 to 64 bytes from each of
// 16 rows, and other instructions and waves take the rest of those 128-byte lines a little later; with the hint they were asked for from the L2 again (requests of
// the first-level caches, non-temporal / as here: 3-bit 5001 x 4101, batch 3 328000 / 120000; 1-bit scaled 8192 x 8192, batch 8 786000 / 352000; misses of the L2 the
// same).  us, 16 and 8 matrices in turn: 8.1 / 7.2 and 10.0 / 8.4; 90 drawn canonical and tiled products 9 % less on the average, none more than 1 % slower.  Tiled granules come in whole lines and stay non-temporal.
template <int WPL>
__device__ __forceinline__ void canon_words(const uint32_t* p, uint32_t (&w)[WPL]) {
    typedef u32x4_t __attribute__((aligned(4))) u32x4_a4_t;
    typedef u32x2_t __attribute__((aligned(4))) u32x2_a4_t;
#pragma unroll
    for (int i = 0; i + 4 <= WPL; i += 4) {
        const u32x4_t v = *reinterpret_cast<const u32x4_a4_t*>(p + i);
        w[i] = v[0]; w[i + 1] = v[1]; w[i + 2] = v[2]; w[i + 3] = v[3];
    }
    if constexpr (WPL % 4 == 2) {
        const u32x2_t v = *reinterpret_cast<const u32x2_a4_t*>(p + WPL - 2);
        w[WPL - 2] = v[0]; w[WPL - 1] = v[1];
    }
}

// 4 x 4 transpose across the lane groups q: register j of group q becomes register q of group j
__device__ __forceinline__ void canon_transpose(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
    auto swap32 = [](uint32_t& x, uint32_t& y) {          // upper half of x <-> lower half of y
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = r[0]; y = r[1];
    };
    auto swap16 = [](uint32_t& x, uint32_t& y) {          // odd rows of x <-> even rows of y
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0]; y = r[1];
    };
    swap32(a, c);
    swap32(b, d);
    swap16(a, b);
    swap16(c, d);
}

template <int BYTE>
__device__ __forceinline__ void canon_index_to_byte1(uint32_t& a, uint32_t src, uint32_t mask) {
    if constexpr (BYTE == 0)
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_0 src1_sel:DWORD" : "+v"(a) : "v"(src), "v"(mask));
    else if constexpr (BYTE == 1)
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1 src1_sel:DWORD" : "+v"(a) : "v"(src), "v"(mask));
    else if constexpr (BYTE == 2)
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_2 src1_sel:DWORD" : "+v"(a) : "v"(src), "v"(mask));
    else
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:DWORD" : "+v"(a) : "v"(src), "v"(mask));
}

// Waves a SIMD that the registers have to leave room for: what an instance keeps without spilling (sixteen waves a workgroup: four in any case).  Left alone the compiler spends
// up to a third more of them, and a SIMD loses a wave or two (1-bit 18624 x 2843, batch 1: 10.3 us against 7.4).
template <int BITS, bool SC, bool TILED, int MR, int RB>
constexpr int canon_waves() {
    if (BITS == 1 && TILED) return RB == 1 && MR <= 2 ? 4 : MR == 1 ? 3 : 2;             // (tiles of 512 columns)
    if (RB == 2) return MR == 1 ? 4 : MR == 2 ? (BITS == 4 && SC ? 3 : 4) : 3;
    if (BITS == 4) return MR == 1 ? 5 : MR == 2 ? 4 : SC ? 3 : 4;
    return MR <= 2 ? 5 : 4;
}

// TILED: the matrix-core layout instead of the canonical one.  MR: groups of four batch rows that are staged (M <= 4 * MR).
// CHAINS: sums a wave has, which take its tiles in turn.  With two of them a result is, bit for bit, that of twice the waves with one.
template <int BITS, bool SC, bool TILED, int MR, int RB, int NW, int CHAINS>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(canon_waves<BITS, SC, TILED, MR, RB>()))) void gemm_canon_kernel(const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook,
                                                             const uint16_t* __restrict__ X, uint16_t* __restrict__ Y,
                                                             int64_t N, int64_t K, int M, const uint16_t* __restrict__ scales) {
    constexpr int C = 1 << BITS, R = 4 * MR;
    constexpr int TC = TILED && BITS == 1 ? 512 : 256;    // columns of a tile
    constexpr int PAIRS = TC / 256, HALVES = TC / 128;
    constexpr int WPL = TC * BITS / 128;                  // words per lane and tile
    constexpr int GW = BITS == 3 ? 3 : 4, GT = WPL / GW;  // tiled: words per granule, granules per tile
    constexpr int SVW = TC / 128;                         // words of scales per row and tile
    constexpr bool SPREAD = SC || TILED;                  // a step's columns lie in one 64-column block
    constexpr int TAB = BITS == 4 ? (SC ? 1 : RB) : 0;
    // 1-bit canonical rows of whole words: sums of x as they are (nearly exact: no products), over the row's ones and over all
    // columns, and the centroids in the epilogue, c0 * sum + (c1 - c0) * sum over the ones, as the table kernels do at batch 1.
    // Rows with a non-finite centroid, and all rows where K is no multiple of 32, multiply by the centroids themselves.
    constexpr bool SUMS = BITS == 1 && !SC && !TILED;
    static_assert(RB * CHAINS <= 4 && CHAINS <= 2, "partial tiles reuse the staging memory");
    struct alignas(256) Smem {
        uint32_t ptab[TAB ? TAB : 1][TAB ? 16 : 1][64];   // 4-bit: centroid (in both halves) per entry and lane
        u32x2_t masks[16];                                // 1-bit: nibble -> four 16-bit masks
        u32x4_t xs[NW][R * 17];                           // per wave: R batch rows x 16 pieces of eight columns (+ 1 pad)
        uint32_t cc[SUMS ? RB * 16 : 1];                  // the rows' centroids
        float sx[SUMS ? NW * CHAINS : 1][16];             // per chain: sum of its columns of X, per batch column
    };
    __shared__ Smem sm;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 15, q = lane >> 4;
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * (RB * 16);
    const int64_t wpr = words_per_row(BITS, K), nblk = K / KMQ_BLOCK;
    [[maybe_unused]] const int64_t nsb = K / tiled_superblock_elems(BITS);
    const int full = static_cast<int>(K / TC), rest = static_cast<int>(K % TC);
    [[maybe_unused]] const bool sums = SUMS && (K & 31) == 0;
    auto finite = [](uint32_t cc) { return (cc & 0x7F80u) != 0x7F80u && (cc & 0x7F800000u) != 0x7F800000u; };

    // ---- what belongs to the lane's rows
    const uint32_t* wp[RB];
    [[maybe_unused]] const uint16_t* sp[RB];
    [[maybe_unused]] uint32_t lo0[RB], lo1[RB], hi0[RB], hi1[RB];      // 2- and 3-bit: bytes of the centroids
    [[maybe_unused]] uint32_t c0[RB], c1[RB];                           // 1-bit: each centroid in both halves
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        int64_t row = row0 + r * 16 + n;
        row = row < N ? row : N - 1;
        if constexpr (TILED) {
            int64_t rb = static_cast<int64_t>(blockIdx.x) * RB + r;
            const int64_t nrb = (N + 15) >> 4;
            rb = rb < nrb ? rb : nrb - 1;
            wp[r] = W + (rb * nsb * 64 + lane) * GW;
        } else {
            wp[r] = W + row * wpr + q * WPL;
        }
        if constexpr (SC) sp[r] = scales + row * nblk;
        const uint32_t* cw = reinterpret_cast<const uint32_t*>(codebook + (SC ? 0 : row * C));
        if constexpr (BITS == 1) {
            const uint32_t cc = cw[0];
            c0[r] = __builtin_amdgcn_perm(cc, cc, 0x01000100u);
            c1[r] = __builtin_amdgcn_perm(cc, cc, 0x03020302u);
            if (sums && finite(cc)) { c0[r] = 0u; c1[r] = 0x3F803F80u; }
            if (SUMS && wave == 0 && q == 0) sm.cc[r * 16 + n] = cc;
        } else if constexpr (BITS == 2 || BITS == 3) {
            lo0[r] = __builtin_amdgcn_perm(cw[1], cw[0], 0x06040200u);
            hi0[r] = __builtin_amdgcn_perm(cw[1], cw[0], 0x07050301u);
            if constexpr (BITS == 3) {
                lo1[r] = __builtin_amdgcn_perm(cw[3], cw[2], 0x06040200u);
                hi1[r] = __builtin_amdgcn_perm(cw[3], cw[2], 0x07050301u);
            } else {
                lo1[r] = lo0[r];
                hi1[r] = hi0[r];
            }
        }
    }

    // ---- X: piece n of half hh of a tile, batch rows 4i + q; where the half's pieces lie in the tile depends on which
    // columns the lanes hold
    auto piece_col = [&](int hh, int p) {                 // first column (in the tile) of staged piece p
        if constexpr (SPREAD) return 128 * hh + 8 * p;    // the half's two blocks, in order
        else return 64 * (p >> 2) + 32 * hh + 8 * (p & 3);   // columns 32hh..32hh+31 of every lane group's 64
    };
    uint32_t xoff[MR];
#pragma unroll
    for (int i = 0; i < MR; ++i) {
        const int m = 4 * i + q < M ? 4 * i + q : M - 1;
        xoff[i] = (static_cast<uint32_t>(m) * static_cast<uint32_t>(K) + static_cast<uint32_t>(piece_col(0, n))) * 2u;
    }
    constexpr uint32_t kHalf = SPREAD ? 256u : 64u;       // bytes from half 0 to half 1
    u32x4_t xr[HALVES][MR];
    auto load_x = [&](int tile) {
        const char* base = reinterpret_cast<const char*>(X) + static_cast<int64_t>(tile) * (TC * 2);
#pragma unroll
        for (int hh = 0; hh < HALVES; ++hh)
#pragma unroll
            for (int i = 0; i < MR; ++i) xr[hh][i] = *reinterpret_cast<const cu32x4_a2_t*>(base + (xoff[i] + hh * kHalf));
    };
    // the tile that K does not fill: X (or, with `marks`, all ones) where there is a column, else zeros.  A piece that the row ends in is
    // fetched as the row's last eight columns and shifted down (column by column, 3000 x 2060, 4 bits, batch 16: 8.7 us against 8.0; 4-bit 10496 x 2496, batch 9: 15.1 and 12.0; such a
    // piece is rare on the tiled layout, whose rows end with a super-block)
    auto load_x_tail = [&](int tile, bool marks) {
#pragma unroll
        for (int hh = 0; hh < HALVES; ++hh) {
            const int64_t k0 = static_cast<int64_t>(tile) * TC + piece_col(hh, n);
            const int live = static_cast<int>(K - k0);    // columns of this piece
#pragma unroll
            for (int i = 0; i < MR; ++i) {
                const int m = 4 * i + q < M ? 4 * i + q : M - 1;
                const uint16_t* x = X + static_cast<int64_t>(m) * K;
                if (!TILED && !marks && K >= 8) {
                    const u32x4_t v = *reinterpret_cast<const cu32x4_a2_t*>(x + (live > 8 ? k0 : K - 8));
                    const int drop = live >= 8 ? 0 : live <= 0 ? 8 : 8 - live;      // columns before the piece
                    const uint64_t lo = static_cast<uint64_t>(v[1]) << 32 | v[0], hi = static_cast<uint64_t>(v[3]) << 32 | v[2];
                    const uint64_t lo1 = drop & 4 ? hi : lo, hi1 = drop & 4 ? 0 : hi;
                    const int sh = 16 * (drop & 3);
                    const uint64_t lo2 = sh ? lo1 >> sh | hi1 << (64 - sh) : lo1, hi2 = hi1 >> sh;
                    const bool none = drop == 8;
                    xr[hh][i] = u32x4_t{none ? 0u : static_cast<uint32_t>(lo2), none ? 0u : static_cast<uint32_t>(lo2 >> 32),
                                        none ? 0u : static_cast<uint32_t>(hi2), none ? 0u : static_cast<uint32_t>(hi2 >> 32)};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t a, b;
                        if (marks) {
                            a = 2 * e < live ? 0xFFFFu : 0u;
                            b = 2 * e + 1 < live ? 0xFFFFu : 0u;
                        } else {
                            a = 2 * e < live ? x[k0 + 2 * e] : 0u;
                            b = 2 * e + 1 < live ? x[k0 + 2 * e + 1] : 0u;
                        }
                        xr[hh][i][e] = a | (b << 16);
                    }
                }
            }
        }
    };
    // words (and scales) of a tile
    uint32_t w[RB][WPL];
    [[maybe_unused]] uint32_t sv[RB][SVW];
    auto load_w = [&](int r, int tile) {
        if constexpr (TILED) {
#pragma unroll
            for (int g = 0; g < GT; ++g) {
                const uint32_t* p = wp[r] + (static_cast<int64_t>(tile) * GT + g) * (64 * GW);
                if constexpr (GW == 3) {
                    typedef u32x3_t __attribute__((aligned(4))) u32x3_a4_t;
                    const u32x3_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x3_a4_t*>(p));
#pragma unroll
                    for (int j = 0; j < 3; ++j) w[r][g * GW + j] = v[j];
                } else {
                    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[r][g * GW + j] = v[j];
                }
            }
        } else {
            canon_words<WPL>(wp[r] + static_cast<int64_t>(tile) * (8 * BITS), w[r]);
        }
        if constexpr (SC) {
            const uint16_t* s = sp[r] + static_cast<int64_t>(tile) * (TC / KMQ_BLOCK);
            if constexpr (SVW == 4) {
                const u32x4_t v = *reinterpret_cast<const cu32x4_a2_t*>(s);
#pragma unroll
                for (int j = 0; j < 4; ++j) sv[r][j] = v[j];
            } else {
                const u32x2_t v = *reinterpret_cast<const cu32x2_a2_t*>(s);
                sv[r][0] = v[0];
                sv[r][1] = v[1];
            }
        }
    };
    auto load_w_tail = [&](int r, int tile) {             // words past the row's end: any of the row's (their weights are cleared)
        if constexpr (TILED) {
#pragma unroll
            for (int g = 0; g < GT; ++g) {
                int64_t sb = static_cast<int64_t>(tile) * GT + g;
                sb = sb < nsb ? sb : nsb - 1;
#pragma unroll
                for (int j = 0; j < GW; ++j) w[r][g * GW + j] = wp[r][sb * (64 * GW) + j];
            }
        } else {
            const int64_t first = static_cast<int64_t>(tile) * (8 * BITS);
#pragma unroll
            for (int j = 0; j < WPL; ++j) {
                const int64_t at = first + q * WPL + j;
                w[r][j] = wp[r][(at < wpr ? at : wpr - 1) - q * WPL];
            }
        }
        if constexpr (SC) {
#pragma unroll
            for (int b = 0; b < 2 * SVW; ++b) {
                const int64_t at = static_cast<int64_t>(tile) * (TC / KMQ_BLOCK) + b;
                const uint32_t s = at < nblk ? sp[r][at] : 0u;      // (an infinity times a missing block's zero would be a NaN)
                if (b & 1) sv[r][b >> 1] |= s << 16;
                else sv[r][b >> 1] = s;
            }
        }
    };

    int tile = wave;
    if (tile < full) {
        load_x(tile);
#pragma unroll
        for (int r = 0; r < RB; ++r) load_w(r, tile);
    }

    // ---- tables
    if constexpr (BITS == 1) {
        if (threadIdx.x < 16) {
            const uint32_t e = threadIdx.x;
            u32x2_t m;
            m[0] = ((e & 1u) ? 0xFFFFu : 0u) | ((e & 2u) ? 0xFFFF0000u : 0u);
            m[1] = ((e & 4u) ? 0xFFFFu : 0u) | ((e & 8u) ? 0xFFFF0000u : 0u);
            sm.masks[e] = m;
        }
    }
    if constexpr (BITS == 4) {
#pragma unroll
        for (int r = 0; r < TAB; ++r) {
            int64_t row = row0 + r * 16 + n;
            row = row < N ? row : N - 1;
            if constexpr (SC) row = 0;
            const uint32_t* cw = reinterpret_cast<const uint32_t*>(codebook + row * C);
            for (int e2 = wave; e2 < C / 2; e2 += NW) {   // the waves share the entries; every lane fills its own column
                const uint32_t dw = cw[e2];
                sm.ptab[r][2 * e2][lane] = __builtin_amdgcn_perm(dw, dw, 0x01000100u);
                sm.ptab[r][2 * e2 + 1][lane] = __builtin_amdgcn_perm(dw, dw, 0x03020302u);
            }
        }
    }
    if constexpr (BITS == 1 || BITS == 4) __syncthreads();

    f32x4_t acc[CHAINS][RB];                              // [0]: the chain whose turn it is
    [[maybe_unused]] float accx[CHAINS][MR] = {};         // sums of X, batch rows 4i + q
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int r = 0; r < RB; ++r) acc[c][r] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    int turn = 0;                                         // which chain [0] is
    auto next_chain = [&] {
        if constexpr (CHAINS == 2) {
            turn ^= 1;
#pragma unroll
            for (int r = 0; r < RB; ++r) { const f32x4_t t = acc[0][r]; acc[0][r] = acc[1][r]; acc[1][r] = t; }
#pragma unroll
            for (int i = 0; i < MR; ++i) { const float t = accx[0][i]; accx[0][i] = accx[1][i]; accx[1][i] = t; }
        }
    };
    [[maybe_unused]] uint32_t areg[8];                    // 4-bit: look-up addresses, byte 0 = lane * 4, byte 1 = index
#pragma unroll
    for (int e = 0; e < 8; ++e) areg[e] = static_cast<uint32_t>(lane) * 4u;
    u32x4_t* const xs = sm.xs[wave];

    // staged X of a half into LDS, in the order the decoder produces weights
    auto stage = [&](int hh) {
#pragma unroll
        for (int i = 0; i < MR; ++i) {
            const u32x4_t v = xr[hh][i];
            u32x4_t* const at = xs + (4 * i + q) * 17;
            if constexpr (BITS == 2 && !TILED) {
                // pieces 2g, 2g+1 are 16 columns: staged as (0,4) (8,12) (1,5) (9,13) | (2,6) (10,14) (3,7) (11,15)
                uint32_t* const dst = reinterpret_cast<uint32_t*>(at + (n & ~1)) + (n & 1);
                dst[0] = __builtin_amdgcn_perm(v[2], v[0], 0x05040100u);
                dst[2] = __builtin_amdgcn_perm(v[2], v[0], 0x07060302u);
                dst[4] = __builtin_amdgcn_perm(v[3], v[1], 0x05040100u);
                dst[6] = __builtin_amdgcn_perm(v[3], v[1], 0x07060302u);
            } else if constexpr (BITS == 3 && !TILED) {
                at[n] = u32x4_t{__builtin_amdgcn_perm(v[1], v[0], 0x05040100u), __builtin_amdgcn_perm(v[3], v[2], 0x05040100u),
                                __builtin_amdgcn_perm(v[1], v[0], 0x07060302u), __builtin_amdgcn_perm(v[3], v[2], 0x07060302u)};
            } else {
                at[n] = v;
            }
        }
    };
    // operand of step t (0..7) of 256 columns
    auto fragment_piece = [&](int t) {
        if constexpr (TILED) return 4 * (t & 3) + q;                    // columns 32t + 8q
        else if constexpr (!SPREAD) return 4 * q + (t & 3);             // columns 64q + 8t
        else if constexpr (BITS <= 2) return 8 * ((t >> 1) & 1) + 2 * q + (t & 1);   // block t / 2, columns 16q + 8 (t % 2)
        else return 8 * ((t >> 1) & 1) + 4 * (t & 1) + q;                // block t / 2, columns 8 (4 (t % 2) + q)
    };
    // eight weights (2- and 3-bit: from selectors of four)
    auto gather4 = [&](int r, uint32_t sel, uint32_t& d0, uint32_t& d1) {
        const uint32_t lo = __builtin_amdgcn_perm(lo1[r], lo0[r], sel), hi = __builtin_amdgcn_perm(hi1[r], hi0[r], sel);
        d0 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
        d1 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
    };
    constexpr int NU = BITS == 1 ? 2 : BITS == 2 ? 4 : BITS == 3 && TILED ? 6 : 8;
    auto decode = [&](int r, const uint32_t (&u)[NU], int t) -> u32x4_t {
        u32x4_t a;
        uint32_t d0, d1, d2, d3;
        if constexpr (BITS == 1) {
            // byte t of 64 consecutive columns, or byte t % 2 of the 16 columns a word's half holds of block t / 2
            uint32_t b;
            if constexpr (SC && !TILED) b = u[(t >> 1) & 1] >> (16 * (t >> 2) + 8 * (t & 1));
            else b = u[t >> 2] >> (8 * (t & 3));
            const u32x2_t l = sm.masks[b & 15u], h = sm.masks[(b >> 4) & 15u];
            auto choose = [&](uint32_t m) { return (m & c1[r]) | (~m & c0[r]); };
            a = u32x4_t{choose(l[0]), choose(l[1]), choose(h[0]), choose(h[1])};
        } else if constexpr (BITS == 2) {
            const uint32_t x = u[t >> 1];
            gather4(r, (x >> (4 * (t & 1))) & 0x03030303u, d0, d1);
            gather4(r, (x >> (4 * (t & 1) + 2)) & 0x03030303u, d2, d3);
            a = u32x4_t{d0, d1, d2, d3};
        } else if constexpr (BITS == 3 && TILED) {
            const uint32_t A = u[3 * (t >> 2)], B = u[3 * (t >> 2) + 1], E = u[3 * (t >> 2) + 2];
            uint32_t s0, s1;
            if ((t & 3) < 3) {
                const uint32_t x = u[3 * (t >> 2) + (t & 3)];
                s0 = x & 0x07070707u;
                s1 = (x >> 3) & 0x07070707u;
            } else {
                s0 = ((A >> 6) & 0x03030303u) | ((B >> 4) & 0x04040404u);
                s1 = ((B >> 7) & 0x01010101u) | ((E >> 5) & 0x06060606u);
            }
            gather4(r, s0, d0, d1);
            gather4(r, s1, d2, d3);
            a = u32x4_t{d0, d1, d2, d3};
        } else if constexpr (BITS == 3) {
            // 24 bits -> 12 + 12 in the halves -> 6 + 6 in the bytes
            const uint32_t x = (u[t] & 0xFFFu) | ((u[t] << 4) & 0x0FFF0000u);
            const uint32_t y = (x & 0x003F003Fu) | ((x << 2) & 0x3F003F00u);
            gather4(r, y & 0x07070707u, d0, d1);
            gather4(r, (y >> 3) & 0x07070707u, d2, d3);
            a = u32x4_t{d0, d1, d2, d3};
        } else {
            const uint32_t x = u[t], y = x >> 4;
            const uint32_t toff = static_cast<uint32_t>(reinterpret_cast<size_t>((clds_cu32_t*)(&sm.ptab[SC ? 0 : r][0][0])));
            uint32_t wv[8];
            auto look = [&](auto bc) {
                constexpr int b = decltype(bc)::value;
                canon_index_to_byte1<b>(areg[2 * b], x, 0x0Fu);
                wv[2 * b] = *reinterpret_cast<clds_cu32_t*>(static_cast<size_t>(areg[2 * b] + toff));
                canon_index_to_byte1<b>(areg[2 * b + 1], y, 0x0Fu);
                wv[2 * b + 1] = *reinterpret_cast<clds_cu32_t*>(static_cast<size_t>(areg[2 * b + 1] + toff));
            };
            look(std::integral_constant<int, 0>{});
            look(std::integral_constant<int, 1>{});
            look(std::integral_constant<int, 2>{});
            look(std::integral_constant<int, 3>{});
            a = u32x4_t{__builtin_amdgcn_perm(wv[1], wv[0], 0x07060100u), __builtin_amdgcn_perm(wv[3], wv[2], 0x07060100u),
                        __builtin_amdgcn_perm(wv[5], wv[4], 0x07060100u), __builtin_amdgcn_perm(wv[7], wv[6], 0x07060100u)};
        }
        return a;
    };
    auto mfma = [](u32x4_t x, u32x4_t b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    };

    u32x4_t xf[8];
    [[maybe_unused]] u32x4_t xm[8];                       // last tile: all ones where there is a column
    auto fragments = [&](u32x4_t (&f)[8], int hh) {       // of a pair's first or second half
#pragma unroll
        for (int t = 4 * hh; t < 4 * hh + 4; ++t) f[t] = xs[(n & (R - 1)) * 17 + fragment_piece(t)];
    };
    auto multiply = [&](auto tail, int r, int pair) {      // 256 columns
        // eight-column units (3, 4 bits), 16-column words (2 bits) or 32-column words (1 bit) in step order
        uint32_t u[NU];
        if constexpr (BITS == 3 && !TILED) {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const uint32_t a = w[r][3 * g], b = w[r][3 * g + 1], c = w[r][3 * g + 2];
                u[4 * g] = a;
                u[4 * g + 1] = __builtin_amdgcn_alignbit(b, a, 24);
                u[4 * g + 2] = __builtin_amdgcn_alignbit(c, b, 16);
                u[4 * g + 3] = c >> 8;
            }
        } else {
#pragma unroll
            for (int j = 0; j < NU; ++j) u[j] = w[r][pair * NU + j];
        }
        if constexpr (SC && !TILED && BITS == 1) {
            // 16-column units: word 0 / 1 of lane group b hold units 0, 1 / 2, 3 of block b; wanted: unit q of every block
            const auto s = __builtin_amdgcn_permlane32_swap(u[0], u[1], false, false);
            const auto v = __builtin_amdgcn_permlane16_swap(__builtin_amdgcn_perm(s[1], s[0], 0x05040100u),
                                                            __builtin_amdgcn_perm(s[1], s[0], 0x07060302u), false, false);
            u[0] = v[0];                                  // blocks 0, 2
            u[1] = v[1];                                  // blocks 1, 3
        } else if constexpr (SC && !TILED) {
            canon_transpose(u[0], u[1], u[2], u[3]);
            if constexpr (BITS >= 3) {
                canon_transpose(u[4], u[5], u[6], u[7]);
                // unit 4i + j of lane group b is now register 4i + b of group j: block b's units 4i + q
                uint32_t v[8];
#pragma unroll
                for (int b = 0; b < 4; ++b) { v[2 * b] = u[b]; v[2 * b + 1] = u[4 + b]; }
#pragma unroll
                for (int j = 0; j < 8; ++j) u[j] = v[j];
            }
        }
        auto weights = [&](int t) {
            u32x4_t a = decode(r, u, t);
            if constexpr (decltype(tail)::value) {        // no column, no weight: a centroid there may be an infinity
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] &= xm[t][e];
            }
            return a;
        };
        // A tile's 256 columns are summed from zero in four chains, and their sums added to the running one: a chain over all of
        // a wave's columns gathers more rounding than the short sums of 64 lanes do.  Results that are not the correctly rounded
        // exact ones, of 4.7 million, one chain a wave / this / the vector kernels: 3-bit K = 4101 738 / 505 / 529, 2-bit 11008
        // 823 / 497 / 500; batch 16.  Level in time (3-bit 5001 x 4101, batch 16: 11.6 / 11.7 us),
        // 1-bit rows with the sums of X aside (4096 x 11008, batch 4: 6.2 / 6.5).
        f32x4_t tile_sum;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            f32x4_t t = mfma(xf[2 * b], weights(2 * b), f32x4_t{0.f, 0.f, 0.f, 0.f});
            t = mfma(xf[2 * b + 1], weights(2 * b + 1), t);
            if constexpr (SC) {
                const uint32_t s2 = sv[r][2 * pair + (b >> 1)];
                const float s = b & 1 ? __uint_as_float(s2 & 0xFFFF0000u) : __uint_as_float(s2 << 16);
#pragma unroll
                for (int i = 0; i < 4; ++i) tile_sum[i] = b ? fmaf(s, t[i], tile_sum[i]) : s * t[i];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) tile_sum[i] = b ? tile_sum[i] + t[i] : t[i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][r][i] += tile_sum[i];
    };
    auto sum_x = [&] {                                    // this lane's pieces of a tile
#pragma unroll
        for (int i = 0; i < MR; ++i)
#pragma unroll
            for (int hh = 0; hh < HALVES; ++hh)
#pragma unroll
                for (int j = 0; j < 4; ++j) accx[0][i] = dot2_bf16(0x3F803F80u, xr[hh][i][j], accx[0][i]);
    };

    // The pieces pass between lanes of one wave, whose LDS instructions run in order: the compiler has to keep that order.
    auto in_wave = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    auto exchange = [&](u32x4_t (&f)[8], int hh, int piece) {
        in_wave();
        stage(piece);
        in_wave();
        fragments(f, hh);
    };
    // one tile; `more`: another one follows, its operands are requested as their registers become free
    auto step = [&](auto more, auto tail) {
        const int next = tile + NW;
#pragma unroll
        for (int pair = 0; pair < PAIRS; ++pair) {
            if constexpr (decltype(tail)::value) {
                load_x_tail(full, true);
                exchange(xm, 0, 2 * pair);
                exchange(xm, 1, 2 * pair + 1);
                load_x_tail(full, false);
            }
            if constexpr (SUMS) {
                if (sums) sum_x();
            }
            exchange(xf, 0, 2 * pair);
            exchange(xf, 1, 2 * pair + 1);
            if constexpr (decltype(more)::value) {
                if (pair == PAIRS - 1) load_x(next);
                __builtin_amdgcn_sched_barrier(0x100);    // (the scheduler would put these loads behind the decoding; LDS reads may move)
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                multiply(tail, r, pair);
                if constexpr (decltype(more)::value) {
                    if (pair == PAIRS - 1) load_w(r, next);
                }
            }
        }
    };
    // the last tile is a copy of the code of its own: a branch around the loads would make every wait assume the fewest of them
    for (; tile + NW < full; tile += NW) {
        step(std::true_type{}, std::false_type{});
        next_chain();
    }
    if (tile < full) {
        step(std::false_type{}, std::false_type{});
        next_chain();
    }
    if (rest && wave == full % NW) {
#pragma unroll
        for (int r = 0; r < RB; ++r) load_w_tail(r, full);
        step(std::false_type{}, std::true_type{});
        next_chain();
    }

    // ---- the chains' partial tiles: [chain, row block, batch column][row, padded to 17], added pairwise
    float* const part = reinterpret_cast<float*>(xs);
#pragma unroll
    for (int c = 0; c < CHAINS; ++c) {
        const int chain = c ^ turn;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            if (q < MR) {
#pragma unroll
                for (int j = 0; j < 4; ++j) part[((chain * RB + r) * R + 4 * q + j) * 17 + n] = acc[c][r][j];
            }
        }
        if constexpr (SUMS) {
#pragma unroll
            for (int i = 0; i < MR; ++i) {
                const float t = group_sum<16>(accx[c][i]);
                if (n == 15) sm.sx[chain * NW + wave][4 * i + q] = t;
            }
        }
    }
    __syncthreads();
    auto over_chains = [](auto&& of) {                    // chain c of wave w as wave c * NW + w of more of them
        constexpr int PARTS = NW * CHAINS;
        float v[PARTS];
#pragma unroll
        for (int k = 0; k < PARTS; ++k) v[k] = of(k);
#pragma unroll
        for (int w = 1; w < PARTS; w *= 2)
#pragma unroll
            for (int k = 0; k < PARTS; k += 2 * w) v[k] += v[k + w];
        return v[0];
    };
    for (int o = threadIdx.x; o < RB * R * 16; o += NW * 64) {
        const int m = o / (RB * 16), nl = o % (RB * 16);  // consecutive threads: consecutive rows
        const int64_t row = row0 + nl;
        if (m < M && row < N) {
            float s = over_chains([&](int k) { return reinterpret_cast<const float*>(sm.xs[k % NW])[((k / NW * RB + (nl >> 4)) * R + m) * 17 + (nl & 15)]; });
            if constexpr (SUMS) {
                const uint32_t cc = sm.cc[nl];
                if (sums && finite(cc)) {
                    const float c0f = bf16_to_f32(cc & 0xFFFFu), d = bf16_to_f32(cc >> 16) - c0f;
                    s = fmaf(d, s, c0f * over_chains([&](int k) { return sm.sx[k][m]; }));
                }
            }
            Y[static_cast<int64_t>(m) * N + row] = f32_to_bf16(s);
        }
    }
}

// ---- launch ------------------------------------------------------------------------------------

template <int BITS, bool SC, bool TILED, int MR, int RB, int NW, int CHAINS = 1>
static void canon_launch(const GemmArgs& a, hipStream_t s) {
    const int64_t nrb = (a.N + 15) / 16;
    hipLaunchKernelGGL((gemm_canon_kernel<BITS, SC, TILED, MR, RB, NW, CHAINS>), dim3(static_cast<unsigned>((nrb + RB - 1) / RB)), dim3(NW * 64), 0, s,
                       a.W, a.codebook, a.X, a.Y, a.N, a.K, a.M, a.scales);
}

// Largest odd share of row blocks at which one a workgroup is no slower than two, by the mean of its shapes (time of one / of two at shares 3, 5,
// 7 to 9, 11 to 15, above 31): any at batches up to 4 (per row, 2 bits .91 .94 .96 .99 1.02; block-scaled, 4 bits .96 .88 .97 .96 .99) and
// where two blocks are short of registers (block-scaled, 4 bits, batch 5 to 8 .73 .78 .80 .79 .70; batch 9 to 16 .75 .78 .82 .80 .85).  Between: per row, 2
// bits, batch 5 to 8 .97 1.00 1.05 1.07 1.24, 3 bits .91 .95 .97 1.05 1.06, 1 bit 1.03 1.03 1.07 1.11 1.13.
// Rows of more than 40 tiles: 7 at most (47 of 700 shapes of 8192 to 16384 columns more than 3 % slower than with two blocks otherwise, 15 so).
template <int BITS, bool SC, bool TILED, int MR>
static int64_t most_one_block(int64_t K) {
    const int64_t any = K > 10240 ? 7 : int64_t(1) << 40;
    if (MR == 1 || (SC && (MR == 4 || BITS == 4))) return any;
    int64_t most;
    if (SC) most = BITS == 1 ? 31 : 5;
    else if (MR == 2) most = BITS == 1 ? 0 : BITS == 3 ? 7 : 3;
    else if (BITS == 1) most = K % 32 == 0 ? 31 : 0;      // (rows of whole words have no products)
    else most = BITS == 2 ? (TILED ? 0 : 3) : BITS == 3 ? 9 : any;
    return most < any ? most : any;
}

// Launch shape, measured (us) over both layouts and formats at batch 1..16, drawn shapes, each with every shape of launch that is named:
//   few row blocks (at most one a CU): eight waves, sixteen for long rows (2-bit 2773 x 14592 tiled, batch 1: 6.7 with sixteen, 7.5
//     with eight, 8.0 with four), at batches up to 4 and at 4 bits already from 14 tiles on (17 at batches above 8; 3-bit 2419 x 6016, batch 3: 5.4 with
//     eight, 4.8 with sixteen; 4-bit 4032 x 4224, batch 10: 9.6 and 8.6; but 1-bit 2368 x 7104, batch 15: 7.9 and 8.9); four for rows of at most
//     four tiles.  500 shapes of 1300 columns and more: 1.5 % over the fastest on the average; the 106 that sixteen waves take from 14 tiles on 6 % less
//     time, four of them 2 to 5 % more.  Sixteen waves leave 128 registers, which 1-bit and 4-bit block-scaled tiled instances of batch 9 to 16 do not fit in: eight with two
//     chains each, the same sums (84 shapes: 1-bit per row 6 % less time, block-scaled 24 and 5 %; 1-bit block-scaled 3680 x 13824, batch 13: 16.0 -> 11.1);
//   one to two a CU: the same, and from batch 5 on two row blocks a workgroup, so that X is read half as often and no CU has
//     twice the work of another (3-bit scaled 7424 x 8064, batch 11: 13.4 against 15.6; 7650 x 14336, batch 6: 15.4 against
//     18.4; at batch 6 short rows keep one: 6976 x 3136 9.3 against 10.5);
//   more, rows of up to 16 tiles, which eight waves do not share evenly: one block and four (4-bit 10496 x 2496, batch 9: 14.9 against 23.5);
//   more, longer rows: two row blocks and eight waves (3-bit scaled 15616 x 10880, batch 1: 21.2 against 21.7), but one block a workgroup where the
//     busiest CU's share of them is odd, so that two would give it one more (4-bit scaled 8256 x 4480, batch 6, three instead of four: 12.5 against
//     18.4).  Against that one block reads X twice as often, which counts for more the larger the share and the batch and the fewer the bits:
//     most_one_block().  One block has four waves with two chains each, so that a sum is of eight as it is with eight waves (one
//     chain each: 2 % less time, 5 to 18 % more rounding in the 32-bit sums); at a share of three and batches up to 4 eight waves where they are
//     faster (`eight`: 283 shapes, 7 % less time than with four; 125 of the other instances: 4 % more).
//     1957 drawn shapes of odd shares from 3 to 73: 9 % less time than with two blocks everywhere (12 % at 3 and 5, 4 % from 11 on), 45 of
//     them 3 to 10 % more; 1.7 % over the fastest of the three shapes of launch on the average.
// Neither pipe binds: vector issue is 37 % and LDS 9 % of the busy time at 3-bit 5001 x 4101, batch 3, and 47 % and 33 % at 1-bit scaled 8192 x 8192,
// batch 8 (two waves a SIMD); the waves wait for memory.  Two or four tiles in flight per wave instead of one were no faster anywhere all the
// same (1 to 10 % slower at batch 1, 10 to 20 % above; with the loads past the end clamped instead of branched around 10 to 40 %).  Not among the shapes measured: a wave count fitted to the tiles (17 tiles on eight waves
// are three for one and two for the others).  Sixteen waves for two row blocks: 18 % slower on the average.  The last piece taken first, its operands asked for
// at the start, or with the last whole tile's: 3 to 4 % slower at 3-bit 5001 x 4101, batch 3 (words one by one, ahead of everybody else's first tile).  Words through LDS,
// so that four neighbouring lanes load 64 bytes of a row: 3 to 12 % slower.
template <int BITS, bool SC, bool TILED, int MR>
static void canon_shape(const GemmArgs& a, hipStream_t s) {
    const int64_t tiles = (a.K + kCanonTile - 1) / kCanonTile, nrb = (a.N + 15) / 16;
    const int64_t share = (nrb + 255) / 256;              // row blocks of the busiest CU
    constexpr bool spills = TILED && MR == 4 && (BITS == 1 || (BITS == 4 && SC));      // with sixteen waves
    constexpr bool one = SC || !((MR == 2 && BITS == 1) || (MR == 4 && BITS == 2 && TILED));      // where most_one_block() is not 0 throughout
    constexpr bool eight = TILED ? !SC && (BITS == 2 || BITS == 3) : !SC || BITS <= 2;
    if (nrb <= 256) {
        if (tiles >= 40 || (tiles >= 14 && MR == 1) || (BITS == 4 && tiles >= (MR == 4 ? 17 : 14))) {
            if constexpr (spills) canon_launch<BITS, SC, TILED, MR, 1, 8, 2>(a, s);
            else canon_launch<BITS, SC, TILED, MR, 1, 16>(a, s);
        }
        else if (tiles > 4) canon_launch<BITS, SC, TILED, MR, 1, 8>(a, s);
        else canon_launch<BITS, SC, TILED, MR, 1, 4>(a, s);
    } else if (nrb <= 512) {
        if (MR == 4 || (MR == 2 && tiles > 16)) canon_launch<BITS, SC, TILED, MR, 2, 8>(a, s);
        else if (tiles > 4) canon_launch<BITS, SC, TILED, MR, 1, 8>(a, s);
        else canon_launch<BITS, SC, TILED, MR, 1, 4>(a, s);
    } else {
        if (tiles <= 16) canon_launch<BITS, SC, TILED, MR, 1, 4>(a, s);
        else if (share % 2 == 0 || share > most_one_block<BITS, SC, TILED, MR>(a.K)) canon_launch<BITS, SC, TILED, MR, 2, 8>(a, s);
        else if (MR == 1 && share == 3 && eight) canon_launch<BITS, SC, TILED, MR, 1, 8>(a, s);
        else if constexpr (one) canon_launch<BITS, SC, TILED, MR, 1, 4, 2>(a, s);
    }
}

template <int BITS, bool SC, bool TILED>
static void canon_batch(const GemmArgs& a, hipStream_t s) {
    if (a.M <= 4) canon_shape<BITS, SC, TILED, 1>(a, s);
    else if (a.M <= 8) canon_shape<BITS, SC, TILED, 2>(a, s);
    else canon_shape<BITS, SC, TILED, 4>(a, s);
}

template <int BITS>
static hipError_t canon_dispatch(const GemmArgs& a, hipStream_t s) {
    const bool tiled = a.layout == KMQ_LAYOUT_TILED;
    if (a.scales) {
        if (tiled) canon_batch<BITS, true, true>(a, s);
        else canon_batch<BITS, true, false>(a, s);
    } else {
        if (tiled) canon_batch<BITS, false, true>(a, s);
        else canon_batch<BITS, false, false>(a, s);
    }
    return hipGetLastError();
}

}  // namespace kmq

#endif
