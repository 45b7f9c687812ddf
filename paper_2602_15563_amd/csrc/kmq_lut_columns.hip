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
    static constexpr int COLUMNS = MC;
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

// Which batches take several columns a workgroup, and how many.  The time of a call is a line in the number of workgroups on the busiest CU, whatever
// the batch: so many us for the first of them, and for every further one.  The rows a wave and the columns make few large workgroups or many small
// ones, so that a shape pays for a last workgroup that one CU in eight has (2-bit 1536 x 14336, batch 10: 288 workgroups of four columns 20.6, 960 of
// two 12.6) or for columns that the batch does not have; the least of the five lines is taken.  Lines fitted to 10717 shapes (both formats, batch 2
// to 16, 64..20480 rows; rms 2 to 6 % of a line's shapes).  Of the 8071 above the size asked for below, the pick is 0.3 % slower than the best of the five
// on average and more than 10 % in 13.  Against the kernels of at most two columns that came before: 2525 other shapes, drawn, 18 % less time on
// average, 12 of them more than 5 % slower, none more than 10 %.  (The most columns that give eight waves a CU, by preference: 3.9 % over the best
// of the five on average, more than 10 % in 1157 of the 8071, and up to 59 % slower than at most two columns.)
struct ColumnTimes {
    int bits, G, LPR, NWK, NWR, RS;                          // the batch-1 shape
    struct { float first, further; } us[5];                  // one column, two (two rows a wave), two, three, four (four rows a wave); zeros: never the least
};
constexpr ColumnTimes kColumnTimes[] = {
    {1, 3, 16, 1, 4, 1, {{2.55f, 0.37f}, {3.06f, 0.38f}, {3.25f, 0.60f}, {3.21f, 0.86f}, {3.37f, 1.09f}}},   // 1 bit, K = 1536
    {1, 4, 16, 1, 4, 1, {{2.54f, 0.44f}, {3.12f, 0.47f}, {3.50f, 0.73f}, {3.40f, 1.05f}, {3.56f, 1.33f}}},   // 1 bit, K = 2048
    {1, 4, 16, 1, 2, 1, {{2.80f, 0.22f}, {3.23f, 0.45f}, {3.46f, 0.74f}, {3.43f, 1.05f}, {3.62f, 1.31f}}},   // 1 bit, K = 2048
    {1, 3, 32, 1, 4, 2, {{2.88f, 0.53f}, {3.40f, 0.67f}, {3.71f, 1.12f}, {3.92f, 1.59f}, {3.90f, 2.16f}}},   // 1 bit, K = 3072
    {1, 3, 32, 1, 3, 3, {{2.92f, 0.60f}, {3.32f, 0.66f}, {3.59f, 1.10f}, {3.77f, 1.59f}, {3.85f, 2.14f}}},   // 1 bit, K = 3072
    {1, 3, 32, 1, 3, 2, {{2.90f, 0.41f}, {3.32f, 0.66f}, {3.59f, 1.10f}, {3.77f, 1.59f}, {3.85f, 2.14f}}},   // 1 bit, K = 3072
    {1, 4, 32, 1, 4, 2, {{2.88f, 0.61f}, {3.48f, 0.81f}, {3.82f, 1.41f}, {3.85f, 2.04f}, {4.01f, 2.69f}}},   // 1 bit, K = 4096
    {1, 3, 64, 1, 6, 2, {{2.30f, 1.24f}, {3.34f, 1.18f}, {3.87f, 2.01f}, {4.05f, 3.17f}, {4.08f, 4.34f}}},   // 1 bit, K = 6144
    {1, 4, 64, 1, 4, 2, {{3.04f, 0.67f}, {3.48f, 1.01f}, {3.85f, 1.58f}, {4.06f, 4.04f}, {4.25f, 5.20f}}},   // 1 bit, K = 8192
    {1, 4, 64, 1, 4, 3, {{3.33f, 0.85f}, {3.49f, 1.01f}, {4.10f, 1.48f}, {4.19f, 3.88f}, {4.19f, 5.13f}}},   // 1 bit, K = 8192
    {2, 3, 32, 1, 4, 2, {{2.76f, 0.34f}, {2.95f, 0.43f}, {3.29f, 0.73f}, {3.37f, 1.00f}, {3.58f, 1.26f}}},   // 2 bits, K = 1536
    {2, 4, 32, 1, 4, 2, {{2.87f, 0.40f}, {3.12f, 0.51f}, {3.53f, 0.92f}, {3.59f, 1.23f}, {3.83f, 1.55f}}},   // 2 bits, K = 2048
    {2, 3, 64, 1, 4, 2, {{2.85f, 0.36f}, {3.14f, 0.48f}, {3.36f, 0.75f}, {3.50f, 1.01f}, {3.60f, 1.32f}}},   // 2 bits, K = 3072
    {2, 4, 64, 1, 4, 2, {{3.00f, 0.40f}, {3.31f, 0.56f}, {3.72f, 0.92f}, {3.89f, 1.23f}, {4.09f, 1.58f}}},   // 2 bits, K = 4096
    {2, 3, 64, 2, 3, 2, {{2.57f, 0.75f}, {3.18f, 0.61f}, {3.40f, 0.84f}, {3.35f, 2.29f}, {3.57f, 2.87f}}},   // 2 bits, K = 6144
    {2, 4, 64, 2, 2, 4, {{3.41f, 0.82f}, {3.49f, 0.76f}, {3.80f, 1.05f}, {4.08f, 2.64f}, {4.27f, 3.28f}}},   // 2 bits, K = 8192
    {2, 4, 64, 2, 2, 2, {{3.29f, 0.43f}, {3.21f, 0.77f}, {3.73f, 1.05f}, {4.06f, 2.61f}, {4.30f, 3.23f}}},   // 2 bits, K = 8192
    {2, 4, 32, 7, 1, 4, {{3.03f, 1.92f}, {2.94f, 1.72f}, {3.22f, 2.49f}, {2.42f, 7.80f}, {2.24f, 9.54f}}},   // 2 bits, K = 14336
    {2, 2, 64, 7, 1, 4, {{3.12f, 1.06f}, {2.37f, 1.48f}, {2.88f, 1.76f}, {2.37f, 5.39f}, {2.42f, 6.58f}}},   // 2 bits, K = 14336
    {3, 3, 16, 3, 1, 2, {{3.03f, 0.34f}, {}, {3.20f, 0.38f}, {3.17f, 0.47f}, {3.23f, 0.54f}}},   // 3 bits, K = 1536
    {3, 6, 32, 1, 4, 2, {{2.97f, 0.55f}, {3.22f, 0.66f}, {3.77f, 1.19f}, {3.85f, 1.49f}, {4.00f, 1.82f}}},   // 3 bits, K = 2048
    {3, 3, 32, 3, 1, 4, {{3.35f, 0.46f}, {3.20f, 0.35f}, {3.40f, 0.60f}, {3.49f, 0.79f}, {3.60f, 1.02f}}},   // 3 bits, K = 3072
    {3, 6, 64, 1, 4, 2, {{3.03f, 0.57f}, {3.31f, 0.68f}, {3.94f, 1.18f}, {4.07f, 1.48f}, {4.52f, 3.62f}}},   // 3 bits, K = 4096
    {3, 3, 64, 3, 2, 4, {{2.89f, 1.12f}, {2.73f, 1.47f}, {3.34f, 2.20f}, {}, {}}},   // 3 bits, K = 6144
    {3, 6, 64, 2, 2, 4, {{3.75f, 1.09f}, {3.75f, 1.38f}, {4.31f, 2.56f}, {4.52f, 3.12f}, {2.35f, 11.04f}}},   // 3 bits, K = 8192
    {3, 6, 64, 2, 2, 2, {{3.23f, 0.60f}, {3.63f, 1.39f}, {4.16f, 2.56f}, {4.51f, 3.07f}, {2.67f, 10.67f}}},   // 3 bits, K = 8192
    {3, 3, 64, 7, 1, 4, {{3.07f, 1.33f}, {2.52f, 1.49f}, {2.73f, 2.00f}, {2.13f, 5.79f}, {2.03f, 7.03f}}},   // 3 bits, K = 14336
    {4, 3, 64, 1, 4, 2, {{2.74f, 0.32f}, {3.07f, 0.43f}, {3.36f, 0.62f}, {3.42f, 0.85f}, {3.67f, 1.07f}}},   // 4 bits, K = 1536
    {4, 4, 64, 1, 4, 2, {{2.87f, 0.38f}, {3.28f, 0.51f}, {3.82f, 0.76f}, {3.91f, 1.02f}, {4.22f, 1.30f}}},   // 4 bits, K = 2048
    {4, 3, 64, 2, 2, 2, {{2.88f, 0.34f}, {3.29f, 0.44f}, {3.47f, 0.65f}, {3.57f, 0.90f}, {3.72f, 1.17f}}},   // 4 bits, K = 3072
    {4, 4, 64, 2, 2, 2, {{2.98f, 0.40f}, {3.47f, 0.54f}, {3.91f, 0.81f}, {4.03f, 1.10f}, {3.96f, 2.88f}}},   // 4 bits, K = 4096
    {4, 4, 64, 3, 2, 2, {{2.57f, 0.84f}, {3.18f, 1.82f}, {3.67f, 2.60f}, {}, {}}},   // 4 bits, K = 6144
    {4, 4, 64, 4, 1, 4, {{3.45f, 0.78f}, {3.69f, 1.18f}, {3.99f, 1.74f}, {3.83f, 2.51f}, {2.04f, 8.28f}}},   // 4 bits, K = 8192
    {4, 4, 64, 4, 1, 2, {{3.19f, 0.42f}, {3.41f, 1.22f}, {3.99f, 1.68f}, {4.04f, 2.37f}, {2.46f, 7.83f}}},   // 4 bits, K = 8192
    {4, 4, 64, 7, 1, 4, {{3.24f, 1.79f}, {3.52f, 1.80f}, {3.36f, 2.34f}, {2.58f, 7.03f}, {2.52f, 8.39f}}},   // 4 bits, K = 14336
    {4, 4, 64, 7, 1, 2, {{2.73f, 1.03f}, {2.68f, 1.83f}, {3.33f, 2.29f}, {2.44f, 6.97f}, {2.45f, 8.30f}}},   // 4 bits, K = 14336
    {3, 6, 32, 7, 1, 4, {{3.26f, 2.55f}, {2.96f, 2.01f}, {4.00f, 2.94f}, {1.87f, 10.54f}, {1.10f, 12.90f}}},   // 3 bits, K = 14336
    {4, 4, 64, 4, 2, 4, {{2.82f, 1.85f}, {3.44f, 1.47f}, {3.90f, 2.16f}, {3.86f, 2.97f}, {1.21f, 10.07f}}},   // 4 bits, K = 8192
};
template <int BITS, int G, int LPR, int NWK, int NWR, int RS>
constexpr int column_times() {
    int i = 0;
    for (const ColumnTimes& t : kColumnTimes) {
        if (t.bits == BITS && t.G == G && t.LPR == LPR && t.NWK == NWK && t.NWR == NWR && t.RS == RS) return i;
        ++i;
    }
    return -1;
}

template <int BITS, int G, int LPR, int NWK, int NWR1, int RS1, bool SC>
static bool launch_columns(const GemmArgs& a, hipStream_t s) {
    constexpr int T = column_times<BITS, G, LPR, NWK, NWR1, RS1>();
    static_assert(T >= 0 || (BITS == 1 && SC), "no times for this shape");
    if constexpr (T >= 0 && !(BITS == 1 && SC)) {
        // (below that the batch is one column a workgroup's: the lines are those of launches that fill the chip)
        if (a.N * a.K * a.M <= (int64_t(24) << 20)) return false;
        // (the grid's row groups are padded to the eight XCDs, whose 32 CUs share theirs)
        auto grid = [&](int rows, int columns) { return ((a.N + rows - 1) / rows + 7) / 8 * 8 * ((a.M + columns - 1) / columns); };
        auto us = [&](int i, int64_t workgroups) { return kColumnTimes[T].us[i].first + kColumnTimes[T].us[i].further * static_cast<float>((workgroups + 255) / 256); };
        float least = us(0, grid(NWR1 * (kWave / LPR) * RS1, 1));
        int pick = 0;
        auto offer = [&](auto mc, auto rsx, auto index) {
            using S = LutColumns<BITS, G, LPR, NWK, NWR1, SC, decltype(mc)::value, decltype(rsx)::value>;
            constexpr int i = decltype(index)::value;
            if constexpr (S::fits && kColumnTimes[T].us[i].first > 0.f) {
                const int64_t workgroups = grid(S::ROWS_WG, S::COLUMNS);
                if (workgroups >= 192 && us(i, workgroups) < least) {
                    least = us(i, workgroups);
                    pick = i;
                }
            }
        };
        bool launched = false;
        auto launch = [&](auto mc, auto rsx, auto index) {
            using S = LutColumns<BITS, G, LPR, NWK, NWR1, SC, decltype(mc)::value, decltype(rsx)::value>;
            if constexpr (S::fits && kColumnTimes[T].us[decltype(index)::value].first > 0.f) {
                hipLaunchKernelGGL((gemm_lut_columns_kernel<BITS, G, LPR, NWK, NWR1, SC, decltype(mc)::value, decltype(rsx)::value>),
                                   dim3(static_cast<unsigned>(grid(S::ROWS_WG, S::COLUMNS))), dim3(S::THREADS), 0, s,
                                   a.W, a.codebook, a.X, a.Y, static_cast<int>(a.N), a.scales, a.M);
                launched = true;
            }
        };
        using std::integral_constant;
        auto each = [&](auto&& f, int only) {
            if (only < 0 || only == 1) f(integral_constant<int, 2>{}, integral_constant<int, 2>{}, integral_constant<int, 1>{});
            if (only < 0 || only == 2) f(integral_constant<int, 2>{}, integral_constant<int, 4>{}, integral_constant<int, 2>{});
            if (only < 0 || only == 3) f(integral_constant<int, 3>{}, integral_constant<int, 4>{}, integral_constant<int, 3>{});
            if (only < 0 || only == 4) f(integral_constant<int, 4>{}, integral_constant<int, 4>{}, integral_constant<int, 4>{});
        };
        each(offer, -1);
#ifdef KMQ_TUNING
        if (const char* const v = std::getenv("KMQ_LUT_MC")) pick = v[0] - '0';      // 0..4, an index of us[]
#endif
        if (pick > 0) each(launch, pick);
        return launched;
    }
    return false;
}

static bool (*const kLutColumns[])(const GemmArgs&, hipStream_t) = {
#define KMQ_ROW(BITS, G, LPR, NWK, NWR, RS, WPE) &launch_columns<BITS, G, LPR, NWK, NWR, RS, false>,
#define KMQ_SC(BITS, G, LPR, NWK, NWR, RS, WPE) &launch_columns<BITS, G, LPR, NWK, NWR, RS, true>,
    KMQ_LUT_SHAPES(KMQ_ROW, KMQ_SC)
#undef KMQ_ROW
#undef KMQ_SC
};

bool launch_lut_columns(int table_index, const GemmArgs& a, hipStream_t s) { return kLutColumns[table_index](a, s); }

}  // namespace kmq
