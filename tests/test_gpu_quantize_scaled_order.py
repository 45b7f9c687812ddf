"""The tensor quantiser's order of quotients: boundaries among the smallest quotients that it holds (whose octave has only half of
the pairs), every scale mantissa with every weight mantissa, and tensors large enough for wide counters, which have to give
what the same data gives on narrow ones."""
import numpy as np
import pytest

import oracle
from paper_2602_15563_amd import kmq, synth
from tests.test_gpu_quantize import run_blockscaled

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from tests import gpu_util
    return gpu_util


def check(gpu, W, bits, iters):
    idx, cb, sc, _, _ = oracle.quantize_blockscaled(W, bits, iters)
    pg, cg, sg = run_blockscaled(gpu, W, bits, iters)
    assert np.array_equal(sg, sc)
    assert np.array_equal(cg, cb)
    assert np.array_equal(pg, oracle.pack(idx, bits))


@pytest.mark.parametrize("bits", [1, 2, 4])
@pytest.mark.parametrize("neg,pos", [(3, 1), (1, 3), (1, 1), (7, 6), (2, 1)])
def test_boundaries_among_the_smallest_quotients(gpu, bits, neg, pos):
    """Besides the scales only quotients of neg and pos times 2^-32 to 2^-31: the middle boundary comes to lie in the lowest octave
    (2^-32 to 2^-31) or the one above it, on either side of zero, or at zero."""
    rng = np.random.default_rng(11 * neg + pos)
    mant = np.tile(128 + np.arange(128), 4)                # every scale mantissa
    a = rng.integers(128, 256, size=(512, 64))
    sign = rng.random((512, 64)) < 0.5
    f = a * np.where(sign, -float(neg), float(pos)) * 2.0 ** -38
    f = np.where(np.abs(f) < 128 * 2.0 ** -38, 128 * 2.0 ** -38, f)      # (nothing below the window)
    f[:, 0] = mant / 128.0
    check(gpu, synth.f32_to_bf16(f.astype(np.float32)).reshape(8, 4096), bits, 6)


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_every_pair_of_mantissas(gpu, bits):
    """Every quotient of three octaves once, negative ones twice: boundaries fall next to and on many of them."""
    s, a = np.meshgrid(128 + np.arange(128), 128 + np.arange(128), indexing="ij")
    rows = []
    for octave in (1, 2, 5):
        w = a * 2.0 ** -octave
        for sgn in (1.0, -1.0, -1.0):
            v = (w * sgn).reshape(128, 2, 64)
            v[:, :, 0] = 2 * s[:, :1]                      # the block's scale: twice its mantissa
            rows.append(v.reshape(128, 128))
    W = synth.f32_to_bf16(np.concatenate(rows).astype(np.float32)).reshape(-1, 1024)
    check(gpu, W, bits, 15)


@pytest.mark.parametrize("bits", [1, 4])
def test_wide_counters_give_what_narrow_ones_give(gpu, bits):
    """A tensor of 2^24 elements, and sixteen copies of it: counts and sums are sixteen times as large (exactly), means the same."""
    import torch
    n, iters = 4096, 6
    W = torch.from_numpy(synth.make_dense_weights(170, bits, n, n).view(np.int16)).cuda()
    many = W.repeat(16, 1).contiguous()
    outs = []
    for w in (W, many):
        N, K = w.shape
        packed = torch.zeros((N, kmq.words_per_row(bits, K)), dtype=torch.int32, device="cuda")
        cb, sc = torch.zeros(1 << bits, dtype=torch.int16, device="cuda"), torch.zeros((N, K // 64), dtype=torch.int16, device="cuda")
        ws = torch.empty(kmq.quantize_blockscaled_workspace_bytes(), dtype=torch.uint8, device="cuda")
        kmq.quantize_blockscaled(w, N, K, bits, iters, packed, cb, sc, ws)
        outs.append((packed, cb, sc))
    torch.cuda.synchronize()
    (p, c, s), (pm, cm, sm) = outs
    assert torch.equal(c, cm)
    assert torch.equal(s.repeat(16, 1), sm) and torch.equal(p.repeat(16, 1), pm)


@pytest.mark.parametrize("blocks", [128 * 1024, 128 * 1024 + 1, 256 * 1024, 256 * 1024 + 1, 512 * 1024 + 1])
def test_grouping_step_at_its_edges(gpu, blocks):
    """One, two, four and eight blocks a thread of the step that sorts blocks by scale mantissa, the last workgroup full or with one block:
    copies of one block row have that row's codebook and indices, however many there are."""
    import torch
    row = torch.from_numpy(synth.make_dense_weights(180, 2, 1, 64 * 1024).view(np.int16)).cuda().reshape(1024, 64)
    copies, rest = divmod(blocks, 1024)
    W = torch.cat([row.repeat(copies, 1), row[:rest]]) if rest else row.repeat(copies, 1)
    outs = []
    for w, check_rows in ((row, 1024), (W, blocks)):
        N, K, bits = w.shape[0], 64, 2
        packed = torch.zeros((N, 4), dtype=torch.int32, device="cuda")
        cb, sc = torch.zeros(4, dtype=torch.int16, device="cuda"), torch.zeros((N, 1), dtype=torch.int16, device="cuda")
        ws = torch.empty(kmq.quantize_blockscaled_workspace_bytes(), dtype=torch.uint8, device="cuda")
        kmq.quantize_blockscaled(w.contiguous(), N, K, bits, 6, packed, cb, sc, ws)
        outs.append((packed, cb, sc))
    torch.cuda.synchronize()
    (p, c, s), (pm, cm, sm) = outs
    at = torch.arange(blocks, device="cuda") % 1024
    assert torch.equal(sm, s[at])
    if rest == 0:                                          # (one block more moves the means)
        assert torch.equal(c, cm) and torch.equal(pm, p[at])
    else:                                                  # ... by less than a bf16 step, mostly: indices differ where a stored centroid does
        d = (c.int() - cm.int()).abs().max().item()
        assert d <= 1 and (d > 0 or torch.equal(pm, p[at]))


@pytest.mark.parametrize("iters", [3, 5, 6])
def test_a_boundary_that_goes_from_far_elements_to_zero(gpu, iters):
    """2 bits, quotients whose sums are exact in any order.  The middle boundary is 0, then 2^-32, with 32 far elements of 2^-33 below it,
    then 0 again, and the outer boundaries have moved past their last member by then: as many window members lie below every
    boundary as in the round before, but the far elements have changed sides, so it is no fixed point."""
    low = lambda n: [255 * 2.0 ** -12, 255 * 2.0 ** -20, n * 2.0 ** -28, 11 * 2.0 ** -32]
    C = [0.5] * 4 + low(255)                                   # 8 elements, together 2.0625 - 5 * 2^-32
    B = [-v for v in [1 / 16] * 28 + [1 / 32] * 8 + low(251)]      # 40 elements, together -2.0625 + 69 * 2^-32
    f = C + B + [2.0 ** -33] * 32 + [-33 / 64] * 64
    assert sum(C) == 2.0625 - 5 * 2.0 ** -32 and sum(B) == -2.0625 + 69 * 2.0 ** -32
    n = 256 * 64
    f = np.array(f + [-1.0] * (n // 2) + [1.0] * (n - n // 2 - len(f)))
    f = np.random.default_rng(5).permutation(f).reshape(256, 64)
    assert (np.abs(f).max(axis=1) == 1.0).all()
    W = synth.f32_to_bf16(f.astype(np.float32)).reshape(4, 4096)
    assert not np.array_equal(oracle.quantize_blockscaled(W, 2, 2)[1], oracle.quantize_blockscaled(W, 2, 3)[1])
    check(gpu, W, 2, iters)
