"""Batches whose workgroups take three or four columns (canonical layout, table kernels specialised on K): every column is the
batch-1 result bit for bit, for every way a row is split over lanes and waves, with row counts that leave the last row group
partly empty, columns past the batch, and odd row counts (columns of Y that start 2-byte aligned)."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


# row lengths of one, two, three, four and seven waves along K and 16, 32 and 64 lanes a row; rows for eight waves a CU and more
@pytest.mark.parametrize("bits,K,N", [(1, 1536, 8197), (1, 2048, 8199), (1, 3072, 16389), (1, 4096, 16387), (1, 6144, 8195), (1, 8192, 8197),
                                      (2, 2048, 16389), (2, 3072, 8195), (2, 4096, 8197), (2, 6144, 4099), (2, 8192, 4101), (2, 14336, 4091),
                                      (3, 1536, 8197), (3, 2048, 16389), (3, 3072, 8195), (3, 4096, 8197), (3, 8192, 4101), (3, 14336, 4091),
                                      (4, 1536, 8197), (4, 3072, 4099), (4, 4096, 4101), (4, 6144, 4099), (4, 8192, 4101), (4, 14336, 4091)])
@pytest.mark.parametrize("M", (3, 4, 7))
def test_columns_equal_batch_1(gpu, bits, K, N, M):
    seed = 41 * bits + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits, symmetric=(bits == 1))
    X = synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    assert kmq.kernel_name(N, K, bits, M).startswith("lut_") and N * K * M > 24 << 20
    pd, cd = gpu.dev(p), gpu.dev(cb)
    Yg = gpu.run_gemm(pd, cd, X, N, K, bits)
    gpu.check_against_oracle(Yg, p, cb, X, K, bits, gpu.sample_ranges(N, seed, nblocks=2), label=f"b{bits} {N}x{K} M{M}")
    for m in range(M):
        assert np.array_equal(Yg[m], gpu.run_gemm(pd, cd, X[m], N, K, bits)[0]), f"column {m}"
