"""The shape-agnostic decoder fusions where their workgroups' work changes: rows that end in whole chunks of eight columns or
not, less and more than one chunk a thread, a last workgroup with missing rows; with and without a pair of matrices."""
import pytest

from tests.test_gpu_fused_decoder import _check, _inputs, _run, _swiglu_norm
from tests.test_gpu_swiglu import _check as _check_swiglu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("N,K", [(1, 8), (5, 2047), (3, 2049), (9, 2056), (6, 4109), (2, 8200), (4097, 519), (2049, 1032),
                                 (1, 7), (9, 72), (5, 504), (3, 511), (6, 512), (4099, 100), (5, 513)])      # rows of one wave, and just above
def test_edges(gpu, bits, N, K):
    idx, cb, x, g, res = _inputs(40 * bits + N + K, bits, N, K)
    _check(gpu, _run(gpu, idx, cb, x, bits, g, res), idx, cb, x, bits, g, res, f"b{bits} {N}x{K}")
    _swiglu_norm(gpu, bits, N, K, 41 * bits + N + K)
    _check_swiglu(gpu, bits, N, K, 43 * bits + N + K)
