"""The matrix-core kernel of 8-bit products at the edges of its tiles: row counts about 16, row lengths about 16, 64 and 256 columns and
about the waves' shares, every kind of batch; the columns that a row does not have."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu
BITS = 8


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


def _codebook(seed, N):
    return synth.f32_to_bf16(synth.rng(seed, 0, synth.KIND_CODEBOOK).normal(0.0, 0.02, size=(N, 256)).astype(np.float32))


@pytest.mark.parametrize("N", (1040, 1025, 1039))
@pytest.mark.parametrize("K", (1, 15, 16, 17, 63, 64, 65, 128, 129, 191, 255, 256, 257, 320, 321, 1023, 1281, 2048 + 77, 4096, 4097))
@pytest.mark.parametrize("M", (1, 5, 16))
def test_edges(gpu, N, K, M):
    idx, cb, X = synth.make_indices(84, K, N, K, BITS), _codebook(84 + K, N), synth.make_x(84, K, M, K)
    assert kmq.kernel_name(N, K, BITS, M) == "mfma_b8"
    p = oracle.pack(idx, BITS)
    gpu.check_against_oracle(gpu.run_gemm(gpu.dev(p), gpu.dev(cb), X, N, K, BITS), p, cb, X, K, BITS, label=f"b8 {N}x{K} M{M}")


@pytest.mark.parametrize("K", (3, 7, 18, 250, 4101))
def test_last_columns(gpu, K):
    """One-hot x reads the last columns back exactly; centroid 0, which the pad bits name but no weight has, is an infinity."""
    N, M = 1030, 16
    idx, cb = np.maximum(synth.make_indices(85, K, N, K, BITS), 1), _codebook(85, N)
    cb[:, 0] = 0x7F80
    p = oracle.pack(idx, BITS)
    cols = K - 1 - np.arange(M) % K
    X = np.zeros((M, K), np.uint16)
    X[np.arange(M), cols] = 0x3F80
    Y = gpu.run_gemm(gpu.dev(p), gpu.dev(cb), X, N, K, BITS)
    assert np.array_equal(Y, np.take_along_axis(cb, idx.astype(np.int64), axis=1)[:, cols].T)
