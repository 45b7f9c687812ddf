"""Batches on the table kernels of several columns, one shape for each kernel that the rule on rows, row length and batch can pick (two
columns and two or four rows a wave, three and four columns) and that the other column tests do not reach: every column
is the batch-1 result bit for bit, with last groups of columns and rows that are partly empty."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("bits,K,N,M", [
    (1, 1536, 4121, 11), (1, 2048, 1265, 13), (1, 2048, 1769, 13), (1, 2048, 2909, 9), (1, 2048, 4095, 4), (1, 2048, 4095, 8), (1, 2048, 8161, 5),
    (1, 3072, 4095, 4), (1, 3072, 4095, 8), (1, 3072, 8193, 2), (1, 3072, 10989, 5), (1, 3072, 10989, 7), (1, 3072, 12605, 11), (1, 4096, 7353, 7), (1, 6144, 2049, 11),
    (1, 6144, 4095, 2), (1, 6144, 8565, 5), (1, 8192, 929, 11), (1, 8192, 2049, 8), (1, 8192, 2049, 11),
    (2, 1536, 5737, 7), (2, 1536, 6949, 5), (2, 1536, 7353, 7), (2, 2048, 12605, 5), (2, 3072, 2049, 11), (2, 3072, 2801, 3), (2, 6144, 929, 5), (2, 6144, 1041, 7),
    (2, 6144, 1545, 7), (2, 8192, 301, 11), (2, 8192, 817, 10), (2, 8192, 1545, 7), (2, 14336, 313, 13), (2, 14336, 801, 7), (2, 14336, 1201, 2),
    (2, 14336, 1545, 3),
    (3, 2048, 12605, 5), (3, 3072, 1201, 7), (3, 3072, 1377, 7), (3, 4096, 3717, 7), (3, 4096, 6545, 5), (3, 6144, 1801, 3), (3, 6144, 2049, 2), (3, 8192, 1041, 7),
    (3, 8192, 2049, 11), (3, 8192, 2909, 7),
    (4, 1536, 2049, 11), (4, 2048, 1801, 7), (4, 2048, 2049, 11), (4, 2048, 2909, 7), (4, 2048, 4095, 5), (4, 3072, 1545, 7), (4, 4096, 1501, 5),
    (4, 4096, 1545, 7), (4, 6144, 1321, 5), (4, 8192, 705, 7), (4, 8192, 1545, 7)])
def test_columns_equal_batch_1(gpu, bits, K, N, M):
    seed = 43 * bits + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits, symmetric=(bits == 1))
    X = synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    assert kmq.kernel_name(N, K, bits, M).startswith("lut_") and N * K * M > 24 << 20
    pd, cd = gpu.dev(p), gpu.dev(cb)
    Yg = gpu.run_gemm(pd, cd, X, N, K, bits)
    gpu.check_against_oracle(Yg, p, cb, X, K, bits, gpu.sample_ranges(N, seed, nblocks=2), label=f"b{bits} {N}x{K} M{M}")
    for m in range(M):
        assert np.array_equal(Yg[m], gpu.run_gemm(pd, cd, X[m], N, K, bits)[0]), f"column {m}"


@pytest.mark.parametrize("bits,K,N,M", [
    (2, 4096, 1801, 9), (2, 4096, 3717, 3), (2, 4096, 10585, 2), (2, 8192, 301, 11), (2, 8192, 1009, 13), (2, 8192, 2049, 5), (2, 8192, 3201, 3),
    (2, 14336, 301, 6), (2, 14336, 313, 13), (2, 14336, 801, 7), (2, 14336, 1041, 11), (2, 14336, 1201, 2), (2, 14336, 1201, 10), (2, 14336, 1801, 5),
    (3, 2048, 1801, 7), (3, 4096, 3313, 3), (3, 4096, 8193, 2), (3, 4096, 20479, 2), (3, 8192, 301, 11), (3, 8192, 1041, 7), (3, 8192, 10585, 2),
    (3, 14336, 761, 3), (3, 14336, 1545, 7), (3, 14336, 1801, 5),
    (4, 2048, 1801, 7), (4, 2048, 10585, 2), (4, 4096, 1009, 13), (4, 4096, 1501, 5), (4, 4096, 1713, 5), (4, 8192, 301, 11), (4, 8192, 705, 7), (4, 8192, 753, 13),
    (4, 8192, 1801, 2), (4, 8192, 1801, 5), (4, 14336, 801, 5), (4, 14336, 801, 7)])
def test_scaled_columns_equal_batch_1(gpu, bits, K, N, M):
    seed = 47 * bits + K + M
    p = oracle.pack(synth.make_indices(seed, 0, N, K, bits), bits)
    cb, sc, X = synth.make_shared_codebook(seed, 0, bits), synth.make_scales(seed, 0, N, K), synth.make_x(seed, 0, M, K)
    assert kmq.kernel_name_blockscaled(N, K, bits, M).startswith("lut_sc_") and N * K * M > 24 << 20
    pd, cd, sd = gpu.dev(p), gpu.dev(cb), gpu.dev(sc)
    Yg = gpu.run_gemm_blockscaled(pd, cd, sd, X, N, K, bits)
    gpu.check_blockscaled_against_oracle(Yg, p, cb, sc, X, K, bits, gpu.sample_ranges(N, seed, nblocks=2), label=f"sc b{bits} {N}x{K} M{M}")
    for m in range(M):
        assert np.array_equal(Yg[m], gpu.run_gemm_blockscaled(pd, cd, sd, X[m], N, K, bits)[0]), f"column {m}"
