"""The matrix-core kernel for any row length, many row blocks: however the rows are given to workgroups and waves, the tiles of a long
row are summed in eight chains, so that rows of a matrix of any height beyond 4096 have the same bits."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


# row blocks a CU: 3, 3, 4, 5, 7 (the last workgroup with a part of one, or with one of two); tiles of 256 columns: 17 (whole, with a last one of one column), 18, 20, 23
MANY = [(8200, 4352, 2), (8449, 4097, 6), (12289, 4608, 12), (16400, 5120, 16), (16385, 4353, 3), (24600, 4352, 8), (24577, 5889, 1)]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("N,K,M", MANY)
def test_rows_do_not_depend_on_how_many_there_are(gpu, bits, N, K, M, layout):
    """The first rows of a tall matrix, against the oracle and bit for bit against a product of those 4160 rows alone (which more than
    256 row blocks and eight waves have).  x takes back in its second half what the first gave, so that the bits are those of the
    32-bit sums' rounding."""
    if layout:
        K = K // 512 * 512 + 512                           # (whole super-blocks of every bit-width; an odd number of tiles of 512)
        if K % 1024 == 0:
            K += 512
    few, seed = 4160, 3 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, few, K, bits), synth.make_codebook(seed, 0, few, bits, symmetric=(bits == 1))
    X = synth.make_x(seed, 0, M, K)
    half = K // 2
    idx[:, half:2 * half], X[:, half:2 * half] = idx[:, :half], X[:, :half] ^ 0x8000
    idx, cb = np.resize(idx, (N, K)), np.resize(cb, (N, 1 << bits))      # the same rows again and again
    p = oracle.pack(idx, bits)
    stored = kmq.repack(p, K, bits, layout) if layout else p
    if "mfma_any" not in kmq.kernel_name(N, K, bits, M, layout) or "mfma_any" not in kmq.kernel_name(few, K, bits, M, layout):
        pytest.skip("another kernel's shape")
    tall = gpu.run_gemm(gpu.dev(stored), gpu.dev(cb), X, N, K, bits, layout)
    gpu.check_against_oracle(tall, p, cb, X, K, bits, [(0, 32), (N - 32, N)], label=f"b{bits} {N}x{K} M{M}", strict=False)
    low = kmq.repack(p[:few], K, bits, layout) if layout else p[:few]
    alone = gpu.run_gemm(gpu.dev(low), gpu.dev(cb[:few]), X, few, K, bits, layout)
    assert np.array_equal(tall[:, :few], alone)
    again = N // few * few                                 # a later repetition of the first rows
    assert np.array_equal(tall[:, again:], tall[:, :N - again])


@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("N,K,M", [(8200, 4416, 2), (8449, 4288, 6), (16400, 4800, 16), (24600, 4352, 8)])
def test_block_scaled_rows_do_not_depend_on_how_many_there_are(gpu, bits, N, K, M):
    few, seed = 4160, 5 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, few, K, bits), synth.make_shared_codebook(seed, 0, bits)
    sc, X = synth.make_scales(seed, 0, few, K), synth.make_x(seed, 0, M, K)
    half = K // 128 * 64
    idx[:, half:2 * half], X[:, half:2 * half] = idx[:, :half], X[:, :half] ^ 0x8000
    sc[:, half // 64:2 * half // 64] = sc[:, :half // 64]
    idx, sc = np.resize(idx, (N, K)), np.resize(sc, (N, K // 64))
    p = oracle.pack(idx, bits)
    assert "mfma_any" in kmq.kernel_name_blockscaled(N, K, bits, M) and "mfma_any" in kmq.kernel_name_blockscaled(few, K, bits, M)
    tall = gpu.run_gemm_blockscaled(gpu.dev(p), gpu.dev(cb), gpu.dev(sc), X, N, K, bits)
    gpu.check_blockscaled_against_oracle(tall, p, cb, sc, X, K, bits, row_ranges=[(0, 32), (N - 32, N)], label=f"b{bits} {N}x{K} M{M}", strict=False)
    alone = gpu.run_gemm_blockscaled(gpu.dev(p[:few]), gpu.dev(cb), gpu.dev(sc[:few]), X, few, K, bits)
    assert np.array_equal(tall[:, :few], alone)


@pytest.mark.parametrize("bits,N,K,M", [(1, 300, 10752, 9), (1, 33, 13824, 16), (1, 4090, 15872, 12), (4, 300, 4736, 16), (4, 47, 5504, 9), (4, 33, 16256, 13)])
def test_block_scaled_tiles_of_two_chains(gpu, bits, N, K, M):
    """Few row blocks, instances that eight waves of two chains serve: numbers of tiles below, at and above the sixteen chains' turns."""
    import torch
    seed = 17 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_shared_codebook(seed, 0, bits)
    sc, X = synth.make_scales(seed, 0, N, K), synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    assert kmq.kernel_name_blockscaled(N, K, bits, M, kmq.LAYOUT_TILED) == f"mfma_any_sc_b{bits}"
    Y = torch.full((M, N), 0x7FC1, dtype=torch.int16, device="cuda")
    kmq.gemm_smallbatch_blockscaled(gpu.dev(kmq.repack(p, K, bits, kmq.LAYOUT_TILED)), gpu.dev(cb), gpu.dev(sc), gpu.dev(X), Y, N, K, M, bits, kmq.LAYOUT_TILED)
    torch.cuda.synchronize()
    gpu.check_blockscaled_against_oracle(gpu.host_u16(Y), p, cb, sc, X, K, bits, row_ranges=gpu.sample_ranges(N, seed, nblocks=3), label=f"b{bits} {N}x{K} M{M}")
