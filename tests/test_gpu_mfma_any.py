"""The matrix-core kernel for any row length, on the tiled layout at its edges (super-block counts below, at and above the waves
of a workgroup, half a tile left over, every batch group, both weight formats) and with infinite centroids on both layouts."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu

SB = {1: 512, 2: 256, 3: 128, 4: 128}      # columns of a super-block
TILED = kmq.LAYOUT_TILED


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


# (row count, super-blocks, batch): one super-block, odd counts (3, 4 bits: half a tile), primes, one past a multiple of the waves
SHAPES = [(1, 1, 1), (17, 1, 5), (33, 3, 2), (250, 5, 8), (16, 7, 16), (40, 9, 4), (300, 11, 9), (4100, 3, 3), (8209, 5, 7),
          (31, 17, 1), (5000, 19, 6), (19, 43, 16), (600, 83, 12), (90, 89, 1)]


@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("N,blocks,M", SHAPES)
def test_tiled_per_row_vs_oracle(gpu, bits, N, blocks, M):
    K = blocks * SB[bits]
    seed = 11 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits, symmetric=(bits == 1))
    X, p = synth.make_x(seed, 0, M, K), oracle.pack(idx, bits)
    assert M > 4 or kmq.kernel_name(N, K, bits, M, TILED) == f"mfma_any_b{bits}"
    Yg = gpu.run_gemm(gpu.dev(kmq.repack(p, K, bits, TILED)), gpu.dev(cb), X, N, K, bits, TILED)
    gpu.check_against_oracle(Yg, p, cb, X, K, bits, gpu.sample_ranges(N, seed, nblocks=3), label=f"b{bits} {N}x{K} M{M}")


@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("N,blocks,M", [s for s in SHAPES if s[1] <= 31])
def test_tiled_blockscaled_vs_oracle(gpu, bits, N, blocks, M):
    import torch
    K = blocks * SB[bits]
    seed = 13 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_shared_codebook(seed, 0, bits)
    sc, X = synth.make_scales(seed, 0, N, K), synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    Y = torch.full((M, N), 0x7FC1, dtype=torch.int16, device="cuda")
    kmq.gemm_smallbatch_blockscaled(gpu.dev(kmq.repack(p, K, bits, TILED)), gpu.dev(cb), gpu.dev(sc), gpu.dev(X), Y, N, K, M, bits, TILED)
    torch.cuda.synchronize()
    gpu.check_blockscaled_against_oracle(gpu.host_u16(Y), p, cb, sc, X, K, bits, row_ranges=gpu.sample_ranges(N, seed, nblocks=3),
                                         label=f"b{bits} {N}x{K} M{M}")


@pytest.mark.parametrize("bits", (2, 3, 4))
def test_tiled_one_hot_columns_are_bit_exact(gpu, bits):
    """Row m of X is e_k: every column of every position of a tile meets its own weight."""
    N, K, seed = 35, 11 * SB[bits], 50 + bits
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits)
    p = oracle.pack(idx, bits)
    Wd = oracle.dequant(p, cb, K, bits)
    pd, cd = gpu.dev(kmq.repack(p, K, bits, TILED)), gpu.dev(cb)
    for k0 in list(range(0, 256, 16)) + [1024, K - 16]:
        for M in (4, 8):
            X = np.zeros((M, K), dtype=np.uint16)
            X[np.arange(M), k0 + np.arange(M)] = 0x3F80
            assert np.array_equal(gpu.run_gemm(pd, cd, X, N, K, bits, TILED), Wd[:, k0:k0 + M].T), f"k0={k0} M={M}"


@pytest.mark.parametrize("layout,K", [(kmq.LAYOUT_CANONICAL, 333), (kmq.LAYOUT_CANONICAL, 4101), (TILED, 0)])
@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("M", (1, 9))
def test_infinite_centroids(gpu, bits, layout, K, M):
    """Columns a row does not have contribute nothing, also where centroid 0 -- the index of a word's pad bits -- is an infinity
    (rows 0..7: not used by the row), and where it is used the sum is that infinity (rows 8..15; x is positive)."""
    K = K or 11 * SB[bits]
    N, seed = 16, 70 + bits
    idx, cb = np.maximum(synth.make_indices(seed, 0, N, K, bits), 1), synth.make_codebook(seed, 0, N, bits)
    cb[8:, 1:] = cb[8:, 1:] & 0x7FFF
    X = (synth.make_x(seed, 0, M, K) & 0x7FFF).astype(np.uint16) | 0x3000      # positive, not zero
    finite = cb.copy()
    finite[:, 0] = cb[:, 1]
    want = gpu.run_gemm(gpu.dev(oracle.pack(idx, bits)), gpu.dev(finite), X, N, K, bits)
    cb[:, 0] = 0x7F80
    idx[8:, K // 2] = 0
    p = oracle.pack(idx, bits)
    got = gpu.run_gemm(gpu.dev(kmq.repack(p, K, bits, TILED) if layout else p), gpu.dev(cb), X, N, K, bits, layout)
    assert np.all(got[:, 8:] == 0x7F80)
    f = synth.bf16_to_f64
    assert np.all(np.abs(f(got[:, :8]) - f(want[:, :8])) <= 2.0 ** -7 * np.abs(f(want[:, :8])) + 1e-3)


@pytest.mark.parametrize("layout,blocks", [(kmq.LAYOUT_CANONICAL, 1), (kmq.LAYOUT_CANONICAL, 5), (kmq.LAYOUT_CANONICAL, 38), (kmq.LAYOUT_CANONICAL, 39), (TILED, 6)])
@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("M", (1, 9))
def test_infinite_block_scale(gpu, bits, layout, blocks, M):
    """The scale of a row's last block is an infinity, and the last tile has room for blocks that the row does not have: they
    contribute nothing, so that rows of positive weights and x sum to that infinity and the others stay as they are."""
    K = blocks * 64
    if K % (SB[bits] if layout else 64):
        pytest.skip("not a whole super-block")
    N, seed = 33, 90 + bits
    p, cb = oracle.pack(synth.make_indices(seed, 0, N, K, bits), bits), synth.make_shared_codebook(seed, 0, bits) & 0x7FFF
    sc, X = synth.make_scales(seed, 0, N, K) & 0x7FFF, (synth.make_x(seed, 0, M, K) & 0x7FFF).astype(np.uint16) | 0x3000
    stored = gpu.dev(kmq.repack(p, K, bits, TILED) if layout else p)

    def product(scales):
        Y = gpu.dev(np.zeros((M, N), np.uint16))
        kmq.gemm_smallbatch_blockscaled(stored, gpu.dev(cb), gpu.dev(scales), gpu.dev(X), Y, N, K, M, bits, layout)
        return gpu.host_u16(Y)

    want = product(sc)
    sc[3::2, -1] = 0x7F80
    got = product(sc)
    assert np.all(got[:, 3::2] == 0x7F80)
    assert np.array_equal(got[:, [0, 1] + list(range(2, N, 2))], want[:, [0, 1] + list(range(2, N, 2))])
