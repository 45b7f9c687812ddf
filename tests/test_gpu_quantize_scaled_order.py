"""The tensor quantiser's order of quotients: boundaries among the smallest quotients that it holds (whose octave has only half of
the pairs), every scale mantissa with every weight mantissa, tensors large enough for wide counters, which have to give
what the same data gives on narrow ones, the step that sorts blocks at its edges, and a boundary that leaves the far elements."""
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
    """One, two, four and eight blocks a thread of the step that sorts blocks by scale mantissa, the last workgroup full or with one block.
    Quotients are 1 and -1 except in one block of each workgroup (its first, its last or one between), whose 63 quotients of 15/32 or 1/32 with either
    sign are all that the two middle clusters have: a block that is lost, or counted twice, moves their means by two bf16 steps or more."""
    import torch
    bits, rng = 2, np.random.default_rng(blocks)
    each = 1024 * (1 if blocks <= 128 * 1024 else 2 if blocks <= 256 * 1024 else 4 if blocks <= 512 * 1024 else 8)
    scale = (128 + rng.integers(0, 128, blocks)) / 128.0
    quot = np.where(rng.integers(0, 2, (blocks, 64), dtype=np.int8) == 1, np.float32(1), np.float32(-1))
    groups = range((blocks + each - 1) // each)
    for g in groups:
        first, last = g * each, min((g + 1) * each, blocks) - 1
        at = (first, last, (first + last) // 2)[g % 3]
        quot[at, 1:] = (-1.0 if g & 1 else 1.0) * (15 / 32 if g & 2 else 1 / 32)
        scale[at] = 1.0
    count = {(neg, big): sum((g & 1 == neg) and (g & 2 == 2 * big) for g in groups) for neg in (0, 1) for big in (0, 1)}
    mean = [(count[n, 0] / 32 + count[n, 1] * 15 / 32) / (count[n, 0] + count[n, 1]) for n in (0, 1)]
    idx = (quot > -0.625).astype(np.uint8) + (quot > 0) + (quot > 0.625)
    want = synth.f32_to_bf16(np.array([-1, -mean[1], mean[0], 1], np.float32))
    W = gpu.dev(synth.f32_to_bf16(quot * scale[:, None].astype(np.float32)))
    packed = torch.ones((blocks, 4), dtype=torch.int32, device="cuda")      # (the step's list lies there: an entry that is not written is block 1)
    cb, sc = torch.zeros(4, dtype=torch.int16, device="cuda"), torch.zeros((blocks, 1), dtype=torch.int16, device="cuda")
    ws = torch.empty(kmq.quantize_blockscaled_workspace_bytes(), dtype=torch.uint8, device="cuda")
    kmq.quantize_blockscaled(W, blocks, 64, bits, 6, packed, cb, sc, ws)
    torch.cuda.synchronize()
    assert np.array_equal(gpu.host_u16(sc)[:, 0], synth.f32_to_bf16(scale.astype(np.float32)))
    assert np.array_equal(gpu.host_u16(cb), want)
    assert np.array_equal(packed.cpu().numpy().view(np.uint32), oracle.pack(idx, bits))


def far_then_zero():
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
    return W


@pytest.mark.parametrize("iters", [3, 5, 6])
def test_a_boundary_that_goes_from_far_elements_to_zero(gpu, iters):
    check(gpu, far_then_zero(), 2, iters)


@pytest.mark.parametrize("iters", [2, 3, 6])
def test_wide_counters_with_far_elements(gpu, iters):
    """2^28 elements, copies of the tensor above: searches among far elements in two of the rounds, and every sum exactly as many times as large."""
    import torch
    W, copies = far_then_zero(), 1 << 14
    idx, want, scales, _, _ = oracle.quantize_blockscaled(W, 2, iters)
    w = gpu.dev(W).repeat(copies, 1)
    N, K = w.shape
    packed = torch.zeros((N, kmq.words_per_row(2, K)), dtype=torch.int32, device="cuda")
    cb, sc = torch.zeros(4, dtype=torch.int16, device="cuda"), torch.zeros((N, K // 64), dtype=torch.int16, device="cuda")
    ws = torch.empty(kmq.quantize_blockscaled_workspace_bytes(), dtype=torch.uint8, device="cuda")
    kmq.quantize_blockscaled(w, N, K, 2, iters, packed, cb, sc, ws)
    torch.cuda.synchronize()
    assert np.array_equal(gpu.host_u16(cb), want)
    assert torch.equal(sc, gpu.dev(scales).reshape(W.shape[0], -1).repeat(copies, 1))
    assert torch.equal(packed, gpu.dev(oracle.pack(idx, 2)).reshape(W.shape[0], -1).repeat(copies, 1))
