// Products of 8-bit weights on the canonical layout, batch 1..16, any K, on the matrix cores.
//
// A workgroup is 16 rows, whose 256 centroids each it keeps in LDS (8 KB), and NW waves that split K in tiles of 256 columns.  Lane
// (n, q) reads 16 indices of row n at a time (columns 16q.. of 64), looks them up and has the row operands of two steps of
// v_mfma_f32_16x16x32_bf16; the other operand is the same 16 columns of batch column n, straight from memory (X is small and
// stays in the caches), so that a weight is looked up once for the whole batch.  64 columns are summed from zero and added to the
// wave's tile in fp32; the waves' tiles are added in their order.
//
// Bound by the look-ups: a 2-byte LDS read a weight, whose 64 lanes meet on banks at random (about 6 clocks a wave and CU), then by X
// from the L2s (every workgroup reads all of it: 14336 x 4096, batch 1 / 16: 21.8 / 28.6).  The indices of the next tile are on their way
// meanwhile; X of the next tile too gave nothing at batch 1 and lost at batch 16 (34), as did six waves a SIMD (28 / 36).
// A wave per row, every column's activations fetched per row / this (us): 14336 x 4096, batch 1 / 4 / 16: 39.3 / 55.4 / 140 -> 21.8 /
// 22.3 / 28.6; 4096 x 14336: 37.0 / 54.9 / 129 -> 19.5 / 20.2 / 25.2; 20480 x 1999: 98 / 311 / 1181 -> 22.9 / 31.9 / 46.4; 2049 x 4101,
// batch 16: 263 -> 15.7.  Results that are not the correctly rounded exact ones: 207 -> 179 over 28 shapes.
#include "kmq_device.h"
#include "kmq_launch.h"

namespace kmq {

template <int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void gemm_mfma_b8_kernel(const uint32_t* __restrict__ W, const uint16_t* __restrict__ codebook,
                                                               const uint16_t* __restrict__ X, uint16_t* __restrict__ Y, int64_t N, int K, int M) {
    typedef u32x4_t __attribute__((aligned(4))) u32x4_a4_t;
    typedef u32x4_t __attribute__((aligned(2))) u32x4_a2_t;
    constexpr int C = 256, TC = 256, H = TC / 64;
    __shared__ alignas(16) uint16_t tab[16][C + 8];          // (rows four banks apart: equal indices of different rows don't collide)
    __shared__ alignas(16) float part[NW][16][20];           // a wave's tile: [batch column][row], a column 16-byte aligned
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * 16;
    // rows past N and columns past M repeat the last one and are not stored
    const int64_t row = row0 + n < N ? row0 + n : N - 1;
    const int wpr = (K + 3) >> 2;
    const uint32_t* const w = W + row * wpr;
    const uint16_t* const x = X + static_cast<int64_t>(n < M ? n : M - 1) * K;
    const int whole = K / TC;

    u32x4_t wn[H];
    auto request = [&](int t) {
#pragma unroll
        for (int h = 0; h < H; ++h) wn[h] = *reinterpret_cast<const u32x4_a4_t*>(w + t * (TC / 4) + h * 16 + q * 4);
    };
    if (wave < whole) request(wave);
    for (int i = threadIdx.x; i < 16 * C / 8; i += NW * 64) {
        const int r = i >> 5;
        const int64_t rr = row0 + r < N ? row0 + r : N - 1;
        *reinterpret_cast<u32x4_t*>(&tab[r][(i & 31) * 8]) = *reinterpret_cast<const u32x4_a4_t*>(codebook + rr * C + (i & 31) * 8);
    }
    __syncthreads();

    // the eight weights of two words of indices
    const uint16_t* const lut = tab[row - row0];             // (copies of the last row read one table: with one each, from the same banks, the last workgroup took twice the others' time)
    auto weights = [&](uint32_t a, uint32_t b) {
        u32x4_t o;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t d = i ? b : a;
            o[2 * i] = lut[d & 0xFFu] | static_cast<uint32_t>(lut[(d >> 8) & 0xFFu]) << 16;
            o[2 * i + 1] = lut[(d >> 16) & 0xFFu] | static_cast<uint32_t>(lut[d >> 24]) << 16;
        }
        return o;
    };
    auto step = [](u32x4_t a, u32x4_t b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    };
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    f32x4_t acc = zero;
    for (int t = wave; t < whole; t += NW) {
        u32x4_t xv[H][2], wv[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            wv[h] = wn[h];
#pragma unroll
            for (int s = 0; s < 2; ++s) xv[h][s] = *reinterpret_cast<const u32x4_a2_t*>(x + t * TC + h * 64 + q * 16 + s * 8);
        }
        if (t + NW < whole) request(t + NW);
        f32x4_t part4[H];
#pragma unroll
        for (int h = 0; h < H; ++h) part4[h] = step(weights(wv[h][2], wv[h][3]), xv[h][1], step(weights(wv[h][0], wv[h][1]), xv[h][0], zero));
        acc += (part4[0] + part4[1]) + (part4[2] + part4[3]);
    }
    // the tile that K does not fill: 16 columns a lane, of which `live` are there; zeros on both sides for the others
    if (K % TC != 0 && wave == whole % NW) {
#pragma unroll 1
        for (int h = 0; h < H; ++h) {
            if (whole * TC + h * 64 >= K) break;             // (the same for every lane; looking up zeros up to column 256 all the same: 2048 x 64, batch 1: 5.0 us, now 3.2; 1030 x 320: 5.0, 3.4)
            const int k0 = whole * TC + h * 64 + q * 16, live = K - k0;
            u32x4_t wv = {0, 0, 0, 0}, xv[2] = {wv, wv};
            if (live >= 16) {
                wv = *reinterpret_cast<const u32x4_a4_t*>(w + (k0 >> 2));
                xv[0] = *reinterpret_cast<const u32x4_a2_t*>(x + k0);
                xv[1] = *reinterpret_cast<const u32x4_a2_t*>(x + k0 + 8);
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    if (e < live) {
                        if (e % 4 == 0) wv[e / 4] = w[(k0 + e) >> 2];
                        xv[e / 8][e / 2 % 4] |= static_cast<uint32_t>(x[k0 + e]) << (16 * (e & 1));
                    }
                }
            }
            u32x4_t wt[2] = {weights(wv[0], wv[1]), weights(wv[2], wv[3])};
#pragma unroll
            for (int p = 0; p < 8; ++p) wt[p / 4][p % 4] &= (2 * p < live ? 0xFFFFu : 0u) | (2 * p + 1 < live ? 0xFFFF0000u : 0u);
            acc += step(wt[1], xv[1], step(wt[0], xv[0], zero));
        }
    }
    *reinterpret_cast<f32x4_t*>(&part[wave][n][4 * q]) = acc;
    __syncthreads();
    for (int o = threadIdx.x; o < 16 * M; o += NW * 64) {
        const int m = o >> 4, r = o & 15;
        float s = part[0][m][r];
#pragma unroll
        for (int i = 1; i < NW; ++i) s += part[i][m][r];
        if (row0 + r < N) Y[static_cast<int64_t>(m) * N + row0 + r] = f32_to_bf16(s);
    }
}

// Where 16 rows a workgroup are the faster ones.  With few rows its workgroups leave CUs idle that a wave per row fills: a lone column
// pays until there are more than 1024 of them (us, a wave per row / this: 256 x 4096 5.7 / 6.9, 512 x 8192 9.7 / 10.4, 1024 x 4096 6.9 / 7.1, 1500 x
// 4096 8.5 / 7.2), two until 512 (256 x 4096 6.4 / 6.9; 512 x 8192 11.5 / 10.3); three on and rows that no 16-byte load divides never
// (256 x 4096, batch 4: 7.8 / 6.9; 256 x 1025, batch 1: 6.3 / 4.2).  Fewer than 256 rows, too little to matter, stay where they were.
bool mfma_b8_takes(int64_t N, int64_t K, int M) {
    return N >= 256 && (M >= 3 || K % 8 != 0 || (M == 2 ? N >= 512 : N > 1024));
}

hipError_t launch_mfma_b8(const GemmArgs& a, hipStream_t s) {
    const int64_t groups = (a.N + 15) / 16, tiles = (a.K + 255) / 256;
    const dim3 grid(static_cast<unsigned>(groups));
#define KMQ_B8(NW) hipLaunchKernelGGL((gemm_mfma_b8_kernel<NW>), grid, dim3(NW * 64), 0, s, a.W, a.codebook, a.X, a.Y, a.N, static_cast<int>(a.K), a.M)
    // Eight waves a workgroup, four where rows are many and short (20480 x 1024, batch 1: 12.0 and 11.1 us; 14336 x 4096 the same; 4096 x
    // 14336: 18.8 and 22.4; sixteen: 256 x 4096, batch 16: 8.0 for 8.7, but 14336 x 4096 28.8 for 21.6)
    if (tiles <= 8 && groups >= 1024) KMQ_B8(4);
    else KMQ_B8(8);
#undef KMQ_B8
    return hipGetLastError();
}

}  // namespace kmq
