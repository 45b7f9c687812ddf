"""The matrix-core kernel for any row length where a row ends inside a piece of eight columns: every length of the last piece, behind
whole tiles, in a lone tile and in rows of fewer than eight columns; one-hot x, so that every last column meets its own weight
and none of the next row's activations."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("bits", (1, 2, 3, 4))
@pytest.mark.parametrize("K", [1, 5, 7, 8, 9, 14, 23, 121, 130, 255] + [512 + e for e in range(1, 10)] + [512 + 131])
@pytest.mark.parametrize("M", (3, 16))
def test_last_columns(gpu, bits, K, M):
    N = 21
    idx, cb = synth.make_indices(150 + K, 0, N, K, bits), synth.make_codebook(150 + K, 0, N, bits)
    p = oracle.pack(idx, bits)
    assert K % 32 == 0 or kmq.kernel_name(N, K, bits, M) == f"mfma_any_b{bits}"
    Wd = oracle.dequant(p, cb, K, bits)
    cols = K - 1 - np.arange(M) % K
    X = np.zeros((M, K), np.uint16)
    X[np.arange(M), cols] = 0x3F80
    Y = gpu.run_gemm(gpu.dev(p), gpu.dev(cb), X, N, K, bits)
    assert np.array_equal(Y, Wd[:, cols].T)
