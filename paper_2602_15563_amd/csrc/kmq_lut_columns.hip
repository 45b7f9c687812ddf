// Batches on the canonical layout with the table kernels' sums: two to four columns of a batch per workgroup, each of them the
// batch-1 result bit for bit (kmq_lut.hip, whose split of a row over lanes and waves, tables and lookup blocks are used here).
//
// What the columns share is everything but their multiply-accumulates: index words, addresses, lookups, tables.  At batch 1 a
// lane keeps its slice of x in registers and goes through it row by row; with four columns that is 128 registers and two waves
// a SIMD.  Here the slice stays in LDS and the loops are the other way round: a lane fetches the activations of one unit (eight
// registers a column), uses them for all its RS rows and replaces them, column by column, behind the last row's dots.  The two
// chains of a (row, column) live through the whole slice, so that its sum is taken in the order of batch 1.
//
// Bound by vector issue: 8 * MC dots (4 clocks each) for 8 lookups, whose LDS time (2.9 clocks each and a CU) and the reads of x
// (2 * MC of 16 bytes per unit and RS rows) lie behind them.  2-bit 14336 x 4096, batch 16: 41.7 -> 27.4 us (two columns with their
// slices in registers -> this), vector issue 85 % of the busy time, LDS 43 %; 4096 x 14336, batch 4: 14.1 -> 12.1, vector issue 49 %: half of that
// time the one workgroup a CU waits for x and its words; 4-bit 8192 x 6144, batch 16: 105.7 -> 45.3.
#include <cstdlib>

#include "kmq_device.h"
#include "kmq_launch.h"
#include "kmq_lut_blocks.h"
#include "kmq_lut_shapes.h"

namespace kmq {

// NWR1: row waves of the batch-1 kernel of the same shape (1-bit: its sum of x is taken in that kernel's order).
template <int BITS, int G, int LPR, int NWK, int NWR1, bool SC, int MC, int RSX>
struct LutColumns {
    static constexpr int EL = G * 32 / BITS, K = NWK * LPR * EL, RPL = kWave / LPR;
    static constexpr int RS = RSX / (LPR == 16 ? 2 : 1);                     // rows per lane group
    static constexpr int C16 = EL * 2 / 16, XSTR = C16 | 1;                 // 16-byte pieces of x per lane slice, and their stride in LDS
    static constexpr int XCHUNKS = K / 8;
    static constexpr int ENT = BITS == 3 ? 64 : 16;
    // x of a workgroup takes half a CU's LDS or more at long rows: its waves are then as many as the registers allow
    static constexpr int BYTES8 = MC * XCHUNKS / C16 * XSTR * 16 + (BITS == 1 ? 0 : 8 * RPL * RS * ENT * 4);
    static constexpr int WAVES = BYTES8 >= 80 * 1024 ? 16 : BYTES8 >= 40 * 1024 ? 8 : 4;
    // (three waves along K fill four SIMDs evenly by fours; their short rows keep the smallest row groups, which spread best)
    static constexpr int NWR0 = NWK == 3 ? (LPR == 64 ? 4 : 1) : WAVES / NWK > 1 ? WAVES / NWK : 1, NWR = BITS == 1 && NWR0 < NWR1 ? NWR1 : NWR0;
    static constexpr int THREADS = NWK * NWR * 64, ROWS_WAVE = RPL * RS, ROWS_WG = NWR * ROWS_WAVE;
    static constexpr int XPT = (XCHUNKS + THREADS - 1) / THREADS, XSLOTS = XPT * THREADS;
    static constexpr int LUT_PASSES = BITS == 1 ? 0 : (ROWS_WAVE * ENT + 63) / 64;
    static constexpr int TBL = (RS * ENT + 63) / 64 * 64;                   // dwords per row group: bases are 256-byte aligned
    struct alignas(256) Smem {
        uint32_t lut[BITS == 1 ? 1 : NWK * NWR * RPL][TBL];
        u32x4_t xs[MC][(XSLOTS + C16 - 1) / C16 * XSTR];
        float part[MC][NWK][ROWS_WG];
        float sxp[MC][NWK * NWR1];
    };
    static constexpr int kLds = 160 * 1024;
    // (1-bit with scales keeps two more sums per row and column than registers hold; of twelve waves with three or four columns
    // a CU holds one workgroup: 4-bit 8192 x 6144, batch 16: 64 and 52 us, two columns 47)
    static constexpr bool fits = sizeof(Smem) <= kLds && THREADS <= 1024 && !(BITS == 1 && SC) && !(NWK == 3 && LPR == 64 && MC > 2);
    // waves a SIMD that registers have to leave room for: what LDS lets in, up to what the columns need without spilling
    static constexpr int BY_LDS = static_cast<int>(kLds / sizeof(Smem)) * (THREADS / 64) / 4;
    static constexpr int WPE = BY_LDS < 1 ? 1 : BY_LDS < (MC == 2 ? 5 : 4) ? BY_LDS : (MC == 2 ? 5 : 4);
};

// Sums of V values over groups of LPR lanes, value v in lane v of its group: the tree of group_sum, but every level that adds
// neighbouring lanes halves the number of registers (a lane keeps one of two values and adds the other lane's part of it).
// 16 values: 49 instructions and one store, group_sum 96 and a store each.
template <int CTRL>
__device__ __forceinline__ float add_moved(float v) { return v + dpp_move<CTRL>(v); }
__device__ __forceinline__ float from_4_away(float low, float high) {      // lanes 0-3, 8-11: `low` from four lanes up; the others `high` from four down
    int t = __builtin_amdgcn_update_dpp(0, __float_as_int(low), 0x104, 0xF, 0x5, true);
    t = __builtin_amdgcn_update_dpp(t, __float_as_int(high), 0x114, 0xF, 0xA, false);
    return __int_as_float(t);
}
template <int V, int LPR>
__device__ __forceinline__ float spread_sums(float (&r)[V], int lane) {
    constexpr int V1 = (V + 1) / 2, V2 = (V1 + 1) / 2, V3 = (V2 + 1) / 2;
    static_assert((V3 + 1) / 2 == 1, "at most 16 values");
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
#pragma unroll
    for (int i = 0; i < V1; ++i) {
        const float a = add_moved<0xB1>(r[2 * i]);
        if (2 * i + 1 < V) { const float b = add_moved<0xB1>(r[2 * i + 1]); r[i] = b0 ? b : a; }
        else r[i] = a;
    }
#pragma unroll
    for (int i = 0; i < V2; ++i) {
        const float a = add_moved<0x4E>(r[2 * i]);
        if (2 * i + 1 < V1) { const float b = add_moved<0x4E>(r[2 * i + 1]); r[i] = b1 ? b : a; }
        else r[i] = a;
    }
#pragma unroll
    for (int i = 0; i < V3; ++i) {
        if (2 * i + 1 < V2) r[i] = (b2 ? r[2 * i + 1] : r[2 * i]) + from_4_away(r[2 * i], r[2 * i + 1]);
        else r[i] = r[2 * i] + from_4_away(r[2 * i], r[2 * i]);
    }
    float s = add_moved<0x128>(r[0]);                        // row_ror:8
    if constexpr (V3 > 1) { const float b = add_moved<0x128>(r[1]); s = b3 ? b : s; }
    if constexpr (LPR >= 32) {
        const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
        s = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    if constexpr (LPR >= 64) {
        const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
        s = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    return s;
}

template <int BITS, int G, int LPR, int NWK, int NWR1, bool SC, int MC, int RSX>
__global__ __launch_bounds__((LutColumns<BITS, G, LPR, NWK, NWR1, SC, MC, RSX>::THREADS)) __attribute__((amdgpu_waves_per_eu(LutColumns<BITS, G, LPR, NWK, NWR1, SC, MC, RSX>::WPE)))
void gemm_lut_columns_kernel(const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook, const uint16_t* __restrict__ X,
                             uint16_t* __restrict__ Y, int Nr, const uint16_t* __restrict__ scales, int mcols) {
    using S = LutColumns<BITS, G, LPR, NWK, NWR1, SC, MC, RSX>;
    constexpr int C = 1 << BITS, EL = S::EL, K = S::K, WPR = K * BITS / 32, RPL = S::RPL, RS = S::RS, ROWS_WAVE = S::ROWS_WAVE, ROWS_WG = S::ROWS_WG;
    constexpr int THREADS = S::THREADS, XPT = S::XPT, C16 = S::C16, XSTR = S::XSTR, ENT = S::ENT, LUT_PASSES = S::LUT_PASSES;
    constexpr int U = BITS == 1 ? 2 * G : BITS == 3 ? 2 * G / 3 : G;       // units (eight lookups, 1-bit: four) per row slice
    constexpr int XC = C16 / U;                                             // 16-byte pieces of x per unit
    static_assert(XC * U == C16 && XC == (BITS == 4 ? 1 : 2), "pieces per unit");
    static_assert(!SC || KMQ_BLOCK % EL == 0, "a lane slice lies in one block");
    __shared__ typename S::Smem sm;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wk = wave % NWK, wr = wave / NWK, sub = lane / LPR, pos = lane % LPR;
    // as in the batch-1 kernel: the workgroups that read the same rows of W sit on one XCD, one after the other
    const int t8 = blockIdx.x >> 3, cgroups = (mcols + MC - 1) / MC;
    const int col = t8 % cgroups * MC, wg = (t8 / cgroups) * 8 + (blockIdx.x & 7);
    if (wg * ROWS_WG >= Nr) return;                          // the grid is padded to a multiple of 8 row groups
    const int live = mcols - col < MC ? mcols - col : MC;    // columns past the batch repeat the last one
    X += static_cast<int64_t>(col) * K;
    Y += static_cast<int64_t>(col) * Nr;
    const int wg_row0 = wg * ROWS_WG, wave_row0 = wg_row0 + wr * ROWS_WAVE;

    // ---- x, then the codebook rows, then every index word (the order is pinned, see kmq_lut.hip)
    u32x4_t xt[MC][XPT];
#pragma unroll
    for (int m = 0; m < MC; ++m)
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            int c = threadIdx.x + i * THREADS;
            c = c < S::XCHUNKS ? c : S::XCHUNKS - 1;
            xt[m][i] = *reinterpret_cast<const u32x4_t*>(X + static_cast<int64_t>(m < live ? m : live - 1) * K + c * 8);
        }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    uint32_t cbv[LUT_PASSES > 0 ? LUT_PASSES : 1][BITS == 4 ? 1 : BITS == 3 ? 4 : 2];
#pragma unroll
    for (int p = 0; p < LUT_PASSES; ++p) {
        const int rw = (lane + p * 64) / ENT;                // row inside the wave: t * RPL + sub
        int row = wave_row0 + (rw < ROWS_WAVE ? rw : ROWS_WAVE - 1);
        row = SC ? 0 : row < Nr ? row : Nr - 1;
        const uint16_t* const cb = codebook + static_cast<int64_t>(row) * C;
        if constexpr (BITS == 2) {
            typedef u32x2_t __attribute__((aligned(4))) u32x2_a4_t;
            const u32x2_t c = *reinterpret_cast<const u32x2_a4_t*>(cb);
            cbv[p][0] = c[0];
            cbv[p][1] = c[1];
        } else if constexpr (BITS == 3) {
            typedef u32x4_t __attribute__((aligned(4))) u32x4_a4_t;
            const u32x4_t c = *reinterpret_cast<const u32x4_a4_t*>(cb);
#pragma unroll
            for (int j = 0; j < 4; ++j) cbv[p][j] = c[j];
        } else {
            cbv[p][0] = cb[lane & 15];
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    uint32_t w[RS][G];
#pragma unroll
    for (int t = 0; t < RS; ++t) {
        int row = wave_row0 + t * RPL + sub;
        row = row < Nr ? row : Nr - 1;
        load_words<G>(W + static_cast<int64_t>(row) * WPR + (wk * LPR + pos) * G, w[t]);
    }
    [[maybe_unused]] uint16_t sv[RS];
    if constexpr (SC) {
        const int blk0 = ((wk * LPR + pos) * EL) / KMQ_BLOCK;
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            int row = wave_row0 + t * RPL + sub;
            row = row < Nr ? row : Nr - 1;
            sv[t] = __builtin_nontemporal_load(&scales[static_cast<int64_t>(row) * (K / KMQ_BLOCK) + blk0]);
        }
    }
    const int xbase = (wk * LPR + pos) * XSTR;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // ---- x into LDS
#pragma unroll
    for (int m = 0; m < MC; ++m)
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = threadIdx.x + i * THREADS;
            sm.xs[m][c / C16 * XSTR + c % C16] = xt[m][i];
        }
    if constexpr (BITS == 1) {
        if (threadIdx.x < 16) {
            const uint32_t e = threadIdx.x;
            u32x2_t m;
            m[0] = ((e & 1u) ? 0x3F80u : 0u) | ((e & 2u) ? 0x3F800000u : 0u);
            m[1] = ((e & 4u) ? 0x3F80u : 0u) | ((e & 8u) ? 0x3F800000u : 0u);
            reinterpret_cast<u32x2_t*>(&sm.lut[0][0])[e] = m;
        }
    }
    __syncthreads();
    if constexpr (BITS == 1 && !SC) {
        // sum of x for the two-centroid closed form, over the pieces that each thread of the batch-1 kernel stages
        constexpr int T1 = NWK * NWR1 * 64, XPT1 = (S::XCHUNKS + T1 - 1) / T1;
        if (wave < NWK * NWR1) {
            const int c0 = static_cast<int>(threadIdx.x) * XPT1;
#pragma unroll
            for (int m = 0; m < MC; ++m) {
                float sx = 0.f;
#pragma unroll
                for (int h = 0; h < XPT1; ++h) {
                    const int c = c0 < S::XCHUNKS ? c0 + h : 0;
                    const u32x4_t v = sm.xs[m][c / C16 * XSTR + c % C16];
#pragma unroll
                    for (int j = 0; j < 4; ++j) sx = dot2_bf16(0x3F803F80u, v[j], sx);
                }
                sx = c0 < S::XCHUNKS ? sx : 0.f;
                sx = group_sum<64>(sx);
                if (lane == 63) sm.sxp[m][wave] = sx;
            }
        }
    }

    // ---- this wave's tables (it reads back only what it wrote itself)
    if constexpr (BITS != 1) {
#pragma unroll
        for (int p = 0; p < LUT_PASSES; ++p) {
            const int rw = (lane + p * 64) / ENT, e = lane % ENT;
            uint32_t entry;
            if constexpr (BITS == 2) {
                const uint64_t c64 = static_cast<uint64_t>(cbv[p][0]) | (static_cast<uint64_t>(cbv[p][1]) << 32);
                entry = (static_cast<uint32_t>(c64 >> (16 * (e & 3))) & 0xFFFFu) | ((static_cast<uint32_t>(c64 >> (16 * (e >> 2))) & 0xFFFFu) << 16);
            } else if constexpr (BITS == 3) {
                auto pick = [&](int i) -> uint32_t {
                    const uint32_t lo2 = (i & 2) ? cbv[p][1] : cbv[p][0], hi2 = (i & 2) ? cbv[p][3] : cbv[p][2];
                    const uint32_t d = (i & 4) ? hi2 : lo2;
                    return (i & 1) ? d >> 16 : d & 0xFFFFu;
                };
                entry = pick(e & 7) | (pick(e >> 3) << 16);
            } else {
                entry = cbv[p][0] << 16;
            }
            if (ROWS_WAVE * ENT % 64 == 0 || rw < ROWS_WAVE) sm.lut[wave * RPL + rw % RPL][rw / RPL * ENT + e] = entry;
        }
    }

    // ---- lookups and dots, one row slice ahead; x of the next unit replaces a column's registers behind its last dots
    const uint32_t lut_base = static_cast<uint32_t>(reinterpret_cast<size_t>((lds_cu32_t*)(&sm.lut[BITS == 1 ? 0 : wave * RPL + sub][0])));
    uint32_t ar[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ar[i] = lut_base;
    const uint32_t mask = BITS == 1 ? 0x78u : BITS == 3 ? 0xFCu : 0x3Cu;
    float a0[MC][RS], a1[MC][RS];
#pragma unroll
    for (int m = 0; m < MC; ++m) {
#pragma unroll
        for (int t = 0; t < RS; ++t) a0[m][t] = a1[m][t] = 0.f;
    }
    uint32_t xu[MC][8];
    auto load_x = [&](auto uc, int m) {
        constexpr int u = decltype(uc)::value;
#pragma unroll
        for (int q = 0; q < XC; ++q) {
            const u32x4_t v = sm.xs[m][xbase + u * XC + q];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (BITS == 4) {
                    xu[m][2 * j] = v[j] << 16;
                    xu[m][2 * j + 1] = v[j] & 0xFFFF0000u;
                } else {
                    xu[m][q * 4 + j] = v[j];
                }
            }
        }
    };
    using std::integral_constant;
#pragma unroll
    for (int m = 0; m < MC; ++m) load_x(integral_constant<int, 0>{}, m);
    // the compiler's own scalar loads must have landed: they share the counter of the hand-counted reads and return out of
    // order with them (its LDS reads return in order: waits of either side only become longer by the other's).  The first unit's
    // x, too (up to eight reads, tied to the wait): with the twelve lookups ahead of the first counted wait they were up to 20 in
    // flight, more than the counter's four bits tell apart; later reads of x come between lookups, at most 15 in all
#pragma unroll
    for (int m = 0; m < MC; ++m)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xu[m][0]), "+v"(xu[m][1]), "+v"(xu[m][2]), "+v"(xu[m][3]),
                                              "+v"(xu[m][4]), "+v"(xu[m][5]), "+v"(xu[m][6]), "+v"(xu[m][7]) : : "memory");
    constexpr int NS = U * RS;                               // steps: unit by unit, the rows of each
    if constexpr (BITS == 1) {
        u32x2_t vv[2][4];
        uint32_t re[RS], ro[RS];                             // a word's two halves are units of their own
        issue4_b64<0>(w[0][0], re[0], ro[0], ar, vv[0], mask);
        static_for<0, NS>([&](auto ic) {
            constexpr int n = decltype(ic)::value, t = n % RS, u1 = (n + 1) / RS, t1 = (n + 1) % RS;
            constexpr bool more = n + 1 < NS;
            if constexpr (more) issue4_b64<u1 % 2>(w[t1][u1 / 2], re[t1], ro[t1], ar, vv[(n + 1) & 1], mask);
#pragma unroll
            for (int m = 0; m < MC; ++m) {
                consume4_b64<more ? 4 : 0>(vv[n & 1], xu[m], a0[m][t], a1[m][t]);
                if constexpr (more && t == RS - 1) load_x(integral_constant<int, u1>{}, m);
            }
        });
    } else {
        uint32_t v[2][8];
        uint32_t re = 0, ro = 0;
        auto issue_half = [&](auto tc, auto uc, auto hc, uint32_t (&vd)[8]) {
            constexpr int tt = decltype(tc)::value, uu = decltype(uc)::value, hh = decltype(hc)::value;
            if constexpr (BITS == 3) {
                constexpr int g3 = 3 * (uu / 2);
                issue4_p6<tt * ENT * 4, 2 * (uu % 2) + hh>(w[tt][g3], w[tt][g3 + 1], w[tt][g3 + 2], ar, &vd[4 * hh], mask);
            } else {
                issue4_b32<tt * ENT * 4, hh>(w[tt][uu], re, ro, ar, vd, mask);
            }
        };
        auto consume = [&](auto pc, int m, int t, const uint32_t (&vd)[8]) {
            if constexpr (BITS != 4) consume8_dot2<decltype(pc)::value>(vd, xu[m], a0[m][t], a1[m][t]);
            else consume8_fma<decltype(pc)::value>(vd, xu[m], a0[m][t], a1[m][t]);
        };
        constexpr int MF = MC / 2;                           // columns between the two halves of the next slice's lookups
        issue_half(integral_constant<int, 0>{}, integral_constant<int, 0>{}, integral_constant<int, 0>{}, v[0]);
        issue_half(integral_constant<int, 0>{}, integral_constant<int, 0>{}, integral_constant<int, 1>{}, v[0]);
        static_for<0, NS>([&](auto ic) {
            constexpr int n = decltype(ic)::value, u1 = (n + 1) / RS, t = n % RS, t1 = (n + 1) % RS;
            constexpr bool more = n + 1 < NS, fetch = more && t == RS - 1;
            if constexpr (more) issue_half(integral_constant<int, t1>{}, integral_constant<int, u1>{}, integral_constant<int, 0>{}, v[(n + 1) & 1]);
#pragma unroll
            for (int m = 0; m < MF; ++m) {
                consume(integral_constant<int, more ? 4 : 0>{}, m, t, v[n & 1]);
                if constexpr (fetch) load_x(integral_constant<int, u1>{}, m);
            }
            if constexpr (more) issue_half(integral_constant<int, t1>{}, integral_constant<int, u1>{}, integral_constant<int, 1>{}, v[(n + 1) & 1]);
#pragma unroll
            for (int m = MF; m < MC; ++m) {
                consume(integral_constant<int, more ? 8 : 0>{}, m, t, v[n & 1]);
                if constexpr (fetch) load_x(integral_constant<int, u1>{}, m);
            }
        });
    }

    // ---- K-reduction: lanes of the group, then slices through LDS
    __builtin_amdgcn_sched_barrier(0);
    // (with scales the first level of the sum is a fused multiply-add, whose rounding differs between its two lanes: the batch-1
    // kernel's own sum, lane for lane)
    float sums[MC * RS];
#pragma unroll
    for (int m = 0; m < MC; ++m) {
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            settle_dot(a0[m][t], a1[m][t]);
            sums[m * RS + t] = a0[m][t] + a1[m][t];
            if constexpr (SC) {
                const float s = group_sum_scaled<LPR>(sums[m * RS + t], bf16_to_f32(sv[t]));
                if (pos == LPR - 1) sm.part[m][wk][wr * ROWS_WAVE + t * RPL + sub] = s;
            }
        }
    }
    if constexpr (!SC) {
        const float total = spread_sums<MC * RS, LPR>(sums, lane);
        if (pos < MC * RS) sm.part[pos / RS][wk][wr * ROWS_WAVE + pos % RS * RPL + sub] = total;
    }
    __syncthreads();

    // ---- epilogue: a thread per row and column
    for (int o = threadIdx.x; o < MC * ROWS_WG; o += THREADS) {
        const int m = o / ROWS_WG, rl = o % ROWS_WG, row = wg_row0 + rl;
        if (m >= live || row >= Nr) continue;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NWK; ++k) s += sm.part[m][k][rl];
        if constexpr (BITS == 1 && !SC) {
            float sx = 0.f;
#pragma unroll
            for (int k = 0; k < NWK * NWR1; ++k) sx += sm.sxp[m][k];
            const uint32_t cc = *reinterpret_cast<const uint32_t*>(codebook + static_cast<int64_t>(row) * C);
            const float c0 = bf16_to_f32(cc & 0xFFFFu), c1 = bf16_to_f32(cc >> 16);
            s = fmaf(c1 - c0, s, c0 * sx);
        }
        Y[static_cast<int64_t>(m) * Nr + row] = f32_to_bf16(s);
    }
}

template <int BITS, int G, int LPR, int NWK, int NWR1, bool SC, int MC, int RSX>
static bool launch_columns_of(const GemmArgs& a, int least_waves, hipStream_t s) {
    using S = LutColumns<BITS, G, LPR, NWK, NWR1, SC, MC, RSX>;
    if constexpr (S::fits) {
        const int64_t groups = (a.N + S::ROWS_WG - 1) / S::ROWS_WG, cgroups = (a.M + MC - 1) / MC;
        if (groups * cgroups < 192 || groups * cgroups * (S::THREADS / 64) < least_waves * 256) return false;
        const dim3 grid(static_cast<unsigned>((groups + 7) / 8 * 8 * cgroups));
        hipLaunchKernelGGL((gemm_lut_columns_kernel<BITS, G, LPR, NWK, NWR1, SC, MC, RSX>), grid, dim3(S::THREADS), 0, s,
                           a.W, a.codebook, a.X, a.Y, static_cast<int>(a.N), a.scales, a.M);
        return true;
    }
    return false;
}

// The most columns and rows a wave that still give the chip its work: at least 192 workgroups, and for four columns and four rows a
// wave eight waves a CU (a lone group of three columns: four), else two columns and four rows with eight, else two and two with six
// (1 bit: eight, and no group with a column that the batch does not have), else one column.  Measured (us), one column a workgroup / two
// and two / two and four / four and four:
//   2-bit 14336 x 4096, batch 4: 14.3 / 11.3 / 11.2 / 10.4, batch 16: 49.0 / 38.1 / 33.4 / 27.8; 4096 x 14336, batch 4: 20.4 / 18.6 /
//   13.5 / 12.2; 2048 x 6144 (four waves a CU with four columns): 6.7 / 5.3 / 4.7 / 5.9; 2048 x 2048, batch 8: 4.0 / 3.7 / 4.1 / 4.8;
//   3-bit 4096 x 14336, batch 4: 25.0 / 27.7 / 20.7 / 17.0; 4-bit 4096 x 4096: 9.0 / 7.8 / 7.0 / 6.6; 1-bit 8192 x 8192: 13.8 / 11.2 /
//   10.4 / 9.2, 3072 x 8192, batch 2: 4.6 / 5.1 / 5.1 / -.
template <int BITS, int G, int LPR, int NWK, int NWR1, bool SC>
static bool launch_columns(const GemmArgs& a, hipStream_t s) {
#ifdef KMQ_TUNING
    if (const char* const v = std::getenv("KMQ_LUT_MC")) {
        switch (v[0]) {
            case '2': return launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 2, 2>(a, 0, s);
            case '5': return launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 2, 4>(a, 0, s);
            case '3': return launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 3, 4>(a, 0, s);
            case '4': return launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 4, 4>(a, 0, s);
            case '1': return false;
        }
    }
#endif
    if (a.N * a.K * a.M <= (int64_t(24) << 20)) return false;
    const int cgroups = (a.M + 3) / 4, mc = (a.M + cgroups - 1) / cgroups;
    if (mc == 4 && launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 4, 4>(a, 8, s)) return true;
    if (mc == 3 && launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 3, 4>(a, a.M == 3 && BITS > 1 ? 4 : 8, s)) return true;
    if (BITS == 1 && a.M % 2) return false;
    return launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 2, 4>(a, 8, s) || launch_columns_of<BITS, G, LPR, NWK, NWR1, SC, 2, 2>(a, BITS == 1 ? 8 : 6, s);
}

static bool (*const kLutColumns[])(const GemmArgs&, hipStream_t) = {
#define KMQ_ROW(BITS, G, LPR, NWK, NWR, RS, WPE) &launch_columns<BITS, G, LPR, NWK, NWR, false>,
#define KMQ_SC(BITS, G, LPR, NWK, NWR, RS, WPE) &launch_columns<BITS, G, LPR, NWK, NWR, true>,
    KMQ_LUT_SHAPES(KMQ_ROW, KMQ_SC)
#undef KMQ_ROW
#undef KMQ_SC
};

bool launch_lut_columns(int table_index, const GemmArgs& a, hipStream_t s) { return kLutColumns[table_index](a, s); }

}  // namespace kmq
