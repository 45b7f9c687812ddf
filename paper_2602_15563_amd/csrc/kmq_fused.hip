// Shape-agnostic kernel for the decoder-layer fusions at batch 1 (paper App. E "Model
// benchmarks": token generation runs the projections of a decoder layer back to back, and
// at low bit-widths the elementwise work between them -- RMSNorm, the activation function,
// the residual sums -- is a visible share of the time).  One launch computes
//
//     xn[k] = bf16( x[k] * g[k] )                       RMSNorm in front (optional; xn = x for unit gains)
//     r     = 1 / sqrt( mean_k x[k]^2 + eps )           (1 without the norm)
//     p[n]  = r * sum_k w[n][k] * xn[k]                 the product of kmq_gemv
//     y[n]  = bf16( residual[n] + p[n] )                residual behind (optional), or
//     y[n]  = bf16( silu(p_gate[n]) * p_up[n] )         for a pair of matrices (gate, up)
//
// The scalar r commutes with the sum, so the normalised activations enter the product as
// bf16(x * g) and r is applied once per row.  Canonical layout, any N and K; the
// shape-specialised kernels (kmq_lut.hip) carry the same fusions for their shapes.
#include "kmq_device.h"
#include "kmq_launch.h"

namespace kmq {

template <int BITS>
__device__ __forceinline__ uint32_t stream_field(const uint32_t* row, int64_t k) {
    constexpr uint32_t mask = (1u << BITS) - 1u;
    const int64_t p = k * BITS;
    const int64_t wi = p >> 5;
    const int sh = static_cast<int>(p & 31);
    uint32_t v = row[wi] >> sh;
    if (sh + BITS > 32) v |= row[wi + 1] << (32 - sh);
    return v & mask;
}

typedef __attribute__((ext_vector_type(2))) float f32x2_t;

// A workgroup computes four rows of one matrix (or two of a pair); its threads take the row's chunks of eight columns in turn.
// Bound by its vector instructions and look-ups, not by memory, so both are spent once for as much as possible: x is read 16
// bytes at a time, normalised and rounded once for the four rows; a chunk's indices are one word (8 bits: two); the tables in LDS
// hold four weights per entry at 1 bit and two at 2 and 3.  The waves' sums are added in wave order.  The four launches of a decoder
// layer (us), one row a wave and one column a lane and step / this kernel: hidden 2560, MLP 6912, 1 / 2 / 3 / 4 bits 64.3 / 75.5 / 101 /
// 80.6 -> 26.9 / 27.6 / 33.1 / 32.4; 5120, 13824: 201 / 237 / 452 / 343 -> 54.6 / 57.5 / 80.6 / 77.5.  Eight rows a
// workgroup were no faster but at 3 bits (5120, 13824: 56.6 / 57.0 / 69.1 / 78.2).
// Rows of at most 512 columns are one wave's (NW = 1), as a second one would have no chunk: 20000 x 72 with gains and residual, 1 / 2 /
// 3 / 4 / 8 bits 8.5 / 8.1 / 10.1 / 9.2 / 15.0 -> 5.4 / 5.3 / 5.4 / 5.4 / 10.0 us.  The tables of 8 bits want all four waves to fill them where
// there are few workgroups (300 x 512: 4.0 against 5.0).
template <int BITS, bool PAIR, int NW>
__global__ __launch_bounds__(NW * 64) void gemv_fused_generic_kernel(
    const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook,
    const uint32_t* __restrict__ W2, const uint16_t* __restrict__ codebook2,
    const uint16_t* __restrict__ x, bool norm, const uint16_t* __restrict__ norm_w, float eps,
    const uint16_t* residual, uint16_t* y, int64_t N, int64_t K) {   // (may be one buffer: no __restrict__)
    constexpr int C = 1 << BITS, ROWS = 4, OUT = PAIR ? 2 : 4;
    constexpr int WE = BITS == 1 ? 4 : BITS <= 3 ? 2 : 1;             // weights per table entry
    constexpr int T = WE == 1 ? C : BITS == 1 ? 16 : C * C;
    constexpr int EW = BITS == 1 ? 2 : 1;                             // words per entry
    __shared__ alignas(8) uint32_t tab[ROWS][T * EW];
    __shared__ float red[NW][ROWS + 1];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t n0 = static_cast<int64_t>(blockIdx.x) * OUT;
    const int64_t wpr = words_per_row(BITS, K);
    const uint32_t* row[ROWS];
    const uint16_t* cb[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        int64_t n = n0 + (PAIR ? r >> 1 : r);
        n = n < N ? n : N - 1;
        row[r] = (PAIR && (r & 1) ? W2 : W) + n * wpr;
        cb[r] = (PAIR && (r & 1) ? codebook2 : codebook) + n * C;
#pragma unroll
        for (int e = tid; e < T; e += NW * 64) {
            if constexpr (BITS == 1) {
                const uint32_t a = cb[r][0], b = cb[r][1];
                tab[r][2 * e] = (e & 1 ? b : a) | ((e & 2 ? b : a) << 16);
                tab[r][2 * e + 1] = (e & 4 ? b : a) | ((e & 8 ? b : a) << 16);
            } else if constexpr (WE == 2) {
                tab[r][e] = cb[r][e % C] | (static_cast<uint32_t>(cb[r][e / C]) << 16);
            } else {
                tab[r][e] = static_cast<uint32_t>(cb[r][e]) << 16;    // as a float
            }
        }
    }
    __syncthreads();

    float acc[ROWS] = {0.f, 0.f, 0.f, 0.f}, ss = 0.f;
    auto pair_fma = [](uint32_t w, float x0, float x1, float a) {
        return fmaf(__uint_as_float(w & 0xFFFF0000u), x1, fmaf(__uint_as_float(w << 16), x0, a));
    };
    const int chunks = static_cast<int>(K >> 3);
#pragma unroll 2
    for (int c = tid; c < chunks; c += NW * 64) {
        uint32_t v[ROWS];
        [[maybe_unused]] uint32_t vh[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int bit = c * (8 * BITS), wi = bit >> 5;
            const uint32_t lo = row[r][wi];
            if constexpr (BITS == 3) v[r] = __builtin_amdgcn_alignbit(row[r][wi + 1 < wpr ? wi + 1 : wi], lo, bit & 31);
            else v[r] = lo >> (bit & 31);
            if constexpr (BITS == 8) vh[r] = row[r][wi + 1];
        }
        const u32x4_t xw = reinterpret_cast<const u32x4_t*>(x)[c];
        float xv[8];
#pragma unroll
        for (int t = 0; t < 4; ++t) { xv[2 * t] = __uint_as_float(xw[t] << 16); xv[2 * t + 1] = __uint_as_float(xw[t] & 0xFFFF0000u); }
        if (norm) {
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf(xv[e], xv[e], ss);
            if (norm_w) {
                const u32x4_t gw = reinterpret_cast<const u32x4_t*>(norm_w)[c];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const f32x2_t p{xv[2 * t] * __uint_as_float(gw[t] << 16), xv[2 * t + 1] * __uint_as_float(gw[t] & 0xFFFF0000u)};
                    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf16x2_t));
                    xv[2 * t] = __uint_as_float(h << 16);
                    xv[2 * t + 1] = __uint_as_float(h & 0xFFFF0000u);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if constexpr (BITS == 1) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const u32x2_t w = *reinterpret_cast<const u32x2_t*>(&tab[r][2 * ((v[r] >> (4 * t)) & 15u)]);
                    acc[r] = pair_fma(w[0], xv[4 * t], xv[4 * t + 1], acc[r]);
                    acc[r] = pair_fma(w[1], xv[4 * t + 2], xv[4 * t + 3], acc[r]);
                }
            } else if constexpr (WE == 2) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[r] = pair_fma(tab[r][(v[r] >> (2 * BITS * t)) & (T - 1u)], xv[2 * t], xv[2 * t + 1], acc[r]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    uint32_t f;
                    if constexpr (BITS == 8) f = ((e < 4 ? v[r] : vh[r]) >> (8 * (e & 3))) & 255u;
                    else f = (v[r] >> (4 * e)) & 15u;
                    acc[r] = fmaf(__uint_as_float(tab[r][f]), xv[e], acc[r]);
                }
            }
        }
    }
    if (tid < static_cast<int>(K & 7)) {                  // the columns past the last whole chunk, one per thread
        const int64_t k = (K & ~int64_t(7)) + tid;
        float xv = bf16_to_f32(x[k]);
        if (norm) {
            ss = fmaf(xv, xv, ss);
            if (norm_w) xv = bf16_to_f32(f32_to_bf16(xv * bf16_to_f32(norm_w[k])));
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] = fmaf(bf16_to_f32(cb[r][stream_field<BITS>(row[r], k)]), xv, acc[r]);
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        acc[r] = group_sum<64>(acc[r]);
        if (lane == 63) red[wave][r] = acc[r];
    }
    ss = group_sum<64>(ss);
    if (lane == 63) red[wave][ROWS] = ss;
    __syncthreads();
    const int64_t n = n0 + tid;
    if (tid >= OUT || n >= N) return;
    auto total = [&](int r) {
        float t = red[0][r];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += red[w][r];
        return t;
    };
    const float s = norm ? 1.f / sqrtf(total(ROWS) * (1.f / static_cast<float>(K)) + eps) : 1.f;
    float out = total(PAIR ? 2 * tid : tid) * s;
    if constexpr (PAIR) {
        out = out / (1.f + __expf(-out)) * (total(2 * tid + 1) * s);
    } else {
        if (residual) out += bf16_to_f32(residual[n]);
    }
    y[n] = f32_to_bf16(out);
}

template <int BITS, int NW>
static void launch_fused_waves(const GemmArgs& a, hipStream_t s) {
    const dim3 block(NW * 64);
    if (a.W2)
        hipLaunchKernelGGL((gemv_fused_generic_kernel<BITS, true, NW>), dim3(static_cast<unsigned>((a.N + 1) / 2)), block, 0, s, a.W, a.codebook, a.W2, a.codebook2, a.X,
                           a.norm, a.norm_w, a.eps, static_cast<const uint16_t*>(nullptr), a.Y, a.N, a.K);
    else
        hipLaunchKernelGGL((gemv_fused_generic_kernel<BITS, false, NW>), dim3(static_cast<unsigned>((a.N + 3) / 4)), block, 0, s, a.W, a.codebook,
                           static_cast<const uint32_t*>(nullptr), static_cast<const uint16_t*>(nullptr), a.X, a.norm, a.norm_w, a.eps,
                           a.residual, a.Y, a.N, a.K);
}

template <int BITS>
static hipError_t launch_fused_bits(const GemmArgs& a, hipStream_t s) {
    if (a.K <= 512 && (BITS <= 4 || a.N >= 4096)) launch_fused_waves<BITS, 1>(a, s);
    else launch_fused_waves<BITS, 4>(a, s);
    return hipGetLastError();
}

hipError_t launch_fused_generic(const GemmArgs& a, hipStream_t s) {
    switch (a.bits) {
        case 1: return launch_fused_bits<1>(a, s);
        case 2: return launch_fused_bits<2>(a, s);
        case 3: return launch_fused_bits<3>(a, s);
        case 8: return launch_fused_bits<8>(a, s);
        default: return launch_fused_bits<4>(a, s);
    }
}

}  // namespace kmq
