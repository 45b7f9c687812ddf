"""Dense weights from packed ones, the wave-per-row-segment kernel (canonical layout, K >= 512) and the rounding of the
block-scaled one: bit for bit, at the edges of chunks and segments and at every alignment of the destination."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K", [(1, 512), (9, 511), (9, 513), (5, 519), (3, 1018), (4, 1024), (9, 1025), (5, 1032), (3, 2041), (2, 4101)])
def test_rows_of_any_length_and_alignment(gpu, N, K, bits):
    import torch
    seed = 41 * bits + N + K
    p = oracle.pack(synth.make_indices(seed, 0, N, K, bits), bits)
    cb = synth.make_codebook(seed, 0, N, bits)
    want = oracle.dequant(p, cb, K, bits)
    pd, cd = gpu.dev(p), gpu.dev(cb)
    for offset in range(8):      # elements from a 16-byte boundary
        buf = torch.full((offset + N * K + 16,), 0x7FC1, dtype=torch.int16, device="cuda")
        kmq.dequant(pd, cd, buf[offset:offset + N * K].view(N, K), N, K, bits)
        got = gpu.host_u16(buf)
        assert np.array_equal(got[offset:offset + N * K].reshape(N, K), want), f"offset {offset}"
        assert (got[:offset] == 0x7FC1).all() and (got[offset + N * K:] == 0x7FC1).all(), f"offset {offset}: wrote outside"


def test_block_scaled_rounding_of_every_scale(gpu):
    """Every bf16 pattern as a scale against centroids that reach ties, subnormal results, overflow and infinities:
    round to nearest even; a NaN keeps its payload and becomes quiet."""
    import torch
    bits, K = 4, 64
    sc = np.arange(1 << 16, dtype=np.uint16).reshape(-1, 1)
    N = len(sc)
    cb = np.array([0x0000, 0x8000, 0x3F80, 0xBF80, 0x3F81, 0x3FC0, 0x4001, 0x3F03, 0x0001, 0x8003, 0x0080, 0x7F7F, 0xFF7F, 0x7F80, 0x3EAB, 0xBDCD], dtype=np.uint16)
    idx = np.tile(np.arange(16, dtype=np.uint8), (N, 4))
    Wd = torch.full((N, K), 0x7FC1, dtype=torch.int16, device="cuda")
    kmq.dequant_blockscaled(gpu.dev(oracle.pack(idx, bits)), gpu.dev(cb), gpu.dev(sc), Wd, N, K, bits)
    got = gpu.host_u16(Wd)
    f32 = lambda h: (h.astype(np.uint32) << 16).view(np.float32)
    with np.errstate(all="ignore"):
        u = (f32(cb)[idx] * f32(sc)).view(np.uint32)      # exact but for over- and underflow
    nan = (u & 0x7FFFFFFF) > 0x7F800000
    want = ((u.astype(np.uint64) + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    assert np.array_equal(got[~nan], want[~nan])
    assert (((got[nan] & 0x7FFF) > 0x7F80) & ((got[nan] & 0x40) != 0)).all()
    payload = np.broadcast_to(sc | 0x40, got.shape)
    of_scale = np.broadcast_to((sc & 0x7FFF) > 0x7F80, got.shape)
    assert np.array_equal(got[of_scale], payload[of_scale])
