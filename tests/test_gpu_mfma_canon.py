"""The matrix-core kernel of the canonical layout at its edges, against the oracle through the C ABI: row lengths around its
256-column tiles (a lone element, a partly filled tile alone and behind whole ones, tile counts below, at and above the
waves of a workgroup), row counts around its blocks of 16, every group of batch rows it stages, both weight formats."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


PER_ROW = [(1, 1, 1), (3, 31, 2), (16, 255, 4), (17, 257, 5), (33, 515, 8), (15, 1023, 9), (250, 1025, 16), (40, 2047, 3),
           (31, 2305, 1), (19, 4097, 16), (300, 4111, 6), (4100, 333, 2), (8209, 777, 7), (600, 5001, 1),
           (1000, 2560, 4), (47, 12007, 16), (513, 24590, 1), (9000, 1056, 12)]


@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("N,K,M", PER_ROW)
def test_per_row_vs_oracle(gpu, bits, N, K, M):
    assert kmq.workspace_bytes(N, K, bits, M) == 0      # (few long rows would be split over K)
    seed = 7 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits, symmetric=(bits == 1))
    X = synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    Yg = gpu.run_gemm(gpu.dev(p), gpu.dev(cb), X, N, K, bits)
    gpu.check_against_oracle(Yg, p, cb, X, K, bits, gpu.sample_ranges(N, seed), label=f"b{bits} {N}x{K} M{M}")


SCALED = [(1, 64, 2), (16, 192, 4), (17, 256, 1), (33, 320, 5), (15, 1024 + 64, 16), (250, 2560, 1), (300, 2304, 9),
          (40, 6400, 3), (4100, 640, 8), (8193, 384, 2), (520, 16448, 16), (4096, 4096, 3), (1100, 8192, 16)]


@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("N,K,M", SCALED)
def test_blockscaled_vs_oracle(gpu, bits, N, K, M):
    seed = 5 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_shared_codebook(seed, 0, bits)
    sc, X = synth.make_scales(seed, 0, N, K), synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    Yg = gpu.run_gemm_blockscaled(gpu.dev(p), gpu.dev(cb), gpu.dev(sc), X, N, K, bits)
    gpu.check_blockscaled_against_oracle(Yg, p, cb, sc, X, K, bits, row_ranges=gpu.sample_ranges(N, seed), label=f"b{bits} {N}x{K} M{M}")


@pytest.mark.parametrize("bits", (2, 3, 4))
def test_one_hot_columns_are_bit_exact(gpu, bits):
    """Row m of X is e_k: a sum with one non-zero term is the weight itself, so every column of every tile position has to
    meet its own weight (the operands' column order, the transposes, the tile behind the last whole one)."""
    N, K = 35, 2 * 2048 + 77
    seed = 40 + bits
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits)
    p = oracle.pack(idx, bits)
    Wd = oracle.dequant(p, cb, K, bits)
    pd, cd = gpu.dev(p), gpu.dev(cb)
    for k0 in list(range(0, 256, 16)) + [2040, 2048, 4080, 4096, K - 16]:
        X = np.zeros((16, K), dtype=np.uint16)
        X[np.arange(16), k0 + np.arange(16)] = 0x3F80
        assert np.array_equal(gpu.run_gemm(pd, cd, X, N, K, bits), Wd[:, k0:k0 + 16].T), f"k0={k0}"


@pytest.mark.parametrize("K", (2500, 3333))
@pytest.mark.parametrize("bits", (1, 2, 3, 4))
def test_columns_do_not_depend_on_the_batch(gpu, bits, K):
    """A column's sums run in the same order whatever the batch, as long as the waves split K the same way: 10 tiles on eight waves at every batch; 14 on
    sixteen (two of them idle) at batches up to 4 and, with 4 bits, up to 8, else on eight."""
    N = 100
    idx, cb, X = synth.make_indices(60, 0, N, K, bits), synth.make_codebook(60, 0, N, bits), synth.make_x(60, 0, 16, K)
    half = K // 2                                          # taken back in the second half: the sums' roundings are the result
    idx[:, half:2 * half], X[:, half:2 * half] = idx[:, :half], X[:, :half] ^ 0x8000
    p = oracle.pack(idx, bits)
    pd, cd = gpu.dev(p), gpu.dev(cb)
    full = gpu.run_gemm(pd, cd, X, N, K, bits)
    assert np.array_equal(full, gpu.run_gemm(pd, cd, X, N, K, bits))
    for M in (3, 5, 9):
        got = gpu.run_gemm(pd, cd, X[:M], N, K, bits)
        gpu.check_against_oracle(got, p, cb, X[:M], K, bits, label=f"b{bits} K{K} M{M}", strict=False)
        if K == 2500 or M == 9 or (M == 5 and bits < 4):
            assert np.array_equal(full[:M], got)


@pytest.mark.parametrize("bits,K", [(1, 5002), (2, 5002), (2, 11008), (3, 13824), (4, 5002), (4, 11008), (1, 6912)])
def test_rounding_of_long_sums(gpu, bits, K):
    """Rows whose second half takes back the first (the same centroids, x negated) have the exact result 0, so what comes out
    is the rounding of the 32-bit sums.  It is no larger than that of a wave per row with a lane per 32 consecutive columns
    -- the order of the vector kernels -- where one chain per wave gathers 1.4 to 2 times as much.  1.15: four standard
    errors of the ratio of two root mean squares over 1536 results."""
    N, M, half = 96, 16, K // 2
    idx, cb = synth.make_indices(80 + bits, 0, N, K, bits), synth.make_codebook(80 + bits, 0, N, bits, symmetric=(bits == 1))
    X = synth.make_x(80 + bits, 0, M, K)
    idx[:, half:], X[:, half:] = idx[:, :half], X[:, :half] ^ 0x8000
    f32 = lambda h: (h.astype(np.uint32) << 16).view(np.float32)
    w, x = np.take_along_axis(f32(cb), idx.astype(np.int64), axis=1), f32(X)

    def in_lanes(w, x):
        lanes = np.zeros((64, M, len(w)), np.float32)
        for g in range(0, (K + 31) // 32, 64):
            for e in range(32):
                k = np.arange(g, g + 64) * 32 + e
                on = k < K
                lanes[on] += x[:, k[on]].T[:, :, None] * w[:, k[on]].T[:, None, :]      # products of bf16 values are exact
        while len(lanes) > 1:
            lanes = lanes[0::2] + lanes[1::2]
        return lanes[0]

    if bits == 1 and K % 32 == 0:      # rows of whole words: sums of x itself, the centroids afterwards
        c = f32(cb).astype(np.float64)
        other = in_lanes(idx.astype(np.float32), x) * (c[:, 1] - c[:, 0]) + in_lanes(np.ones((1, K), np.float32), x) * c[:, 0]
    else:
        other = in_lanes(w, x)
    got = synth.bf16_to_f64(gpu.run_gemm(gpu.dev(oracle.pack(idx, bits)), gpu.dev(cb), X, N, K, bits))
    rms = lambda v: np.sqrt(np.mean(np.square(v.astype(np.float64))))
    print(f"b{bits} K={K}: {rms(got):.3e}, lane per 32 columns {rms(other):.3e}")
    assert rms(got) <= 1.15 * rms(other)
