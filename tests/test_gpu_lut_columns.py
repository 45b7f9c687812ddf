"""Batches whose workgroups take two columns (canonical layout, table kernels specialised on K): every column is the batch-1
result bit for bit, with a last pair that is whole or half empty, rows that leave the last row group partly empty, and
odd row counts (columns of Y that start 2-byte aligned)."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


# N * K * M just above the size from which columns are paired (24 * 2^20), one shape per way the rows are split
@pytest.mark.parametrize("bits,K", [(2, 1536), (2, 2048), (2, 4096), (2, 6144), (2, 14336), (3, 1536), (3, 4096), (3, 8192), (3, 14336),
                                    (4, 1536), (4, 3072), (4, 4096), (4, 8192), (4, 14336)])
@pytest.mark.parametrize("M", (2, 7, 16))
def test_columns_equal_batch_1(gpu, bits, K, M):
    N = (25 << 20) // (K * M) | 1
    seed = 31 * bits + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits)
    X = synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    assert kmq.kernel_name(N, K, bits, M).startswith("lut_")
    pd, cd = gpu.dev(p), gpu.dev(cb)
    Yg = gpu.run_gemm(pd, cd, X, N, K, bits)
    gpu.check_against_oracle(Yg, p, cb, X, K, bits, gpu.sample_ranges(N, seed), label=f"b{bits} {N}x{K} M{M}")
    for m in range(M):
        assert np.array_equal(Yg[m], gpu.run_gemm(pd, cd, X[m], N, K, bits)[0]), f"column {m}"


@pytest.mark.parametrize("bits,K", [(2, 2048), (3, 14336), (4, 4096), (4, 14336)])
def test_scaled_columns_equal_batch_1(gpu, bits, K):
    N, M = (25 << 20) // (K * 2) | 1, 2
    seed = 37 * bits + K
    p = oracle.pack(synth.make_indices(seed, 0, N, K, bits), bits)
    cb, sc, X = synth.make_shared_codebook(seed, 0, bits), synth.make_scales(seed, 0, N, K), synth.make_x(seed, 0, M, K)
    args = [gpu.dev(a) for a in (p, cb, sc)]
    outs = []
    for x in (X, X[:1], X[1:]):
        Y = gpu.dev(np.zeros((len(x), N), np.uint16))
        if len(x) == 1:
            kmq.gemv_blockscaled(*args, gpu.dev(x), Y, N, K, bits)
        else:
            kmq.gemm_smallbatch_blockscaled(*args, gpu.dev(x), Y, N, K, len(x), bits)
        outs.append(gpu.host_u16(Y))
    assert np.array_equal(outs[0], np.concatenate(outs[1:]))
