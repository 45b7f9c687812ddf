"""The row quantiser's histogram kernel at its edges, bit for bit against the fp64 oracle: row lengths around a thread's
piece (16), around what stays in registers (4096, 8192, 16384) and around the 16-bit counters (65535), and rows that it
leaves to the kernel for any data (exponents further apart than its window, or than exact fp64 sums allow)."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import synth
from tests.test_gpu_quantize import run_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


def check(gpu, W, bits, iters):
    print(f"quantize_rows {W.shape} b={bits} iters={iters}", flush=True)
    idx, cb, _, _ = oracle.quantize_rows(W, bits, iters)
    pg, cg = run_rows(gpu, W, bits, iters)
    assert np.array_equal(cg, cb)
    assert np.array_equal(pg, oracle.pack(idx, bits))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 31, 33, 4080, 4095, 4096, 4097, 8192, 8193, 16384, 16385, 65535, 65536])
def test_row_lengths(gpu, K, bits):
    check(gpu, synth.make_dense_weights(80 + bits, K, 3, K), bits, 12 if K <= 20000 else 3)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_rows_of_every_kind(gpu, bits):
    """Side by side in one call: an ordinary row, zeros of both signs, half zeros, one value only (the largest counter
    there is), values 31 octaves apart (the window's last), 32 and 60 apart (the other kernel), huge and tiny scales."""
    K = 4096
    W = synth.make_dense_weights(90, bits, 9, K)
    W[1] = np.where(np.arange(K) % 3 == 0, 0x8000, 0x0000)
    W[2, ::2] = 0
    W[3] = 0xBDCC
    for row, octaves in ((4, 31), (5, 32), (6, 60)):
        W[row] = 0x3F80 | (W[row] & 0x807F)                    # magnitudes in [1, 2)
        W[row, 5::9] = (W[row, 5::9] & 0x807F) | ((127 - octaves) << 7)
    W[7] = (W[7] & 0x807F) | 0x7E00                             # around 1e38
    W[8] = (W[8] & 0x807F) | 0x1000                             # around 1e-29: the window would reach below the normal range
    check(gpu, W[:8], bits, 10)
    check(gpu, np.ascontiguousarray(W[[0, 8, 1]]), bits, 10)


def test_rows_not_aligned(gpu):
    """Odd row lengths start rows on odd half-words."""
    check(gpu, synth.make_dense_weights(95, 0, 37, 1111), 3, 9)
    check(gpu, synth.make_dense_weights(95, 1, 37, 4095), 4, 25)


def test_rows_left_over_run_side_by_side(gpu):
    """Neighbouring rows outside the histogram's window take about as long as one of them."""
    import torch
    from paper_2602_15563_amd import kmq
    bits, N, K, iters = 4, 256, 4096, 8
    times = []
    for rows in (1, 4):
        W = synth.make_dense_weights(97, 0, N, K)
        W[8:8 + rows, 3::500] = (W[8:8 + rows, 3::500] & 0x807F) | (60 << 7)
        Wd = gpu.dev(W)
        packed, cb = torch.empty((N, K * bits // 32), dtype=torch.int32, device="cuda"), torch.empty((N, 1 << bits), dtype=torch.int16, device="cuda")
        took = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            kmq.quantize_rows(Wd, N, K, bits, iters, packed, cb)
            b.record()
            torch.cuda.synchronize()
            took.append(a.elapsed_time(b))
        times.append(sorted(took)[3])
    print(f"one row left over {times[0] * 1e3:.0f} us, four {times[1] * 1e3:.0f} us")
    assert times[1] < 2 * times[0]


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [17, 511, 512, 513])
def test_no_rounds(gpu, bits, K):
    check(gpu, synth.make_dense_weights(98, bits, 9, K), bits, 0)
