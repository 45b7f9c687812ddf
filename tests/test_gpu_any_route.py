"""Batches of rows that no table kernel is specialised on, just on either side of the line between the table kernel that walks K in rounds
and the matrix-core kernel, against the oracle: last tiles of one word and of all but one, last row blocks of one row and of all but one."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("bits,N,K,M,route", [(1, 448, 1280, 11, "mfma_any"), (1, 449, 2336, 7, "lut_loop"), (1, 1345, 2304, 3, "mfma_any"),
                                              (2, 873, 2496, 15, "lut_loop"), (2, 257, 3104, 4, "lut_loop"), (2, 1359, 2208, 3, "lut_loop"),
                                              (2, 2415, 2208, 3, "mfma_any"), (3, 977, 1632, 3, "lut_loop"), (3, 1345, 6784, 6, "mfma_any"),
                                              (3, 1001, 2848, 2, "lut_loop"), (4, 961, 4544, 6, "lut_loop"), (4, 767, 1120, 8, "lut_loop"),
                                              (4, 513, 1760, 7, "lut_loop"), (4, 1073, 4544, 6, "mfma_any"), (2, 869, 11040, 11, "mfma_any"),
                                              (2, 865, 11040, 11, "lut_loop"), (3, 1209, 11040, 5, "mfma_any"), (3, 1201, 11040, 5, "lut_loop")])
def test_either_side_of_the_line(gpu, bits, N, K, M, route):
    """On the table kernel's side of it a column is, bit for bit, the product with that column alone; x takes back in its second half what the
    first gave there, so that the bits are those of the sums' rounding."""
    assert kmq.kernel_name(N, K, bits, M) == f"{route}_b{bits}"
    seed = 53 * bits + N + K + M
    idx, cb = synth.make_indices(seed, 0, N, K, bits), synth.make_codebook(seed, 0, N, bits, symmetric=(bits == 1))
    X = synth.make_x(seed, 0, M, K)
    p = oracle.pack(idx, bits)
    pd, cd = gpu.dev(p), gpu.dev(cb)
    gpu.check_against_oracle(gpu.run_gemm(pd, cd, X, N, K, bits), p, cb, X, K, bits, [(0, N)], label=f"b{bits} {N}x{K} M{M}")
    if route == "lut_loop":
        half = K // 2
        idx[:, half:2 * half], X[:, half:2 * half] = idx[:, :half], X[:, :half] ^ 0x8000
        pd = gpu.dev(oracle.pack(idx, bits))
        Yg = gpu.run_gemm(pd, cd, X, N, K, bits)
        for m in range(M):
            assert np.array_equal(Yg[m], gpu.run_gemm(pd, cd, X[m:m + 1], N, K, bits)[0])
