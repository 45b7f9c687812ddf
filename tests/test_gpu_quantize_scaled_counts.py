"""The tensor quantiser's counting kernels where they can go wrong, against the fp64 oracle: few blocks and many, every scale
mantissa, zeros, boundaries that fall exactly on weights (the first round's do), scales near bf16's smallest, and elements
far below their scale ("far"), alone in a tensor and by the thousand."""
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
    N, K = W.shape
    print(f"quantize_blockscaled {W.shape} b={bits} iters={iters}", flush=True)
    idx, cb, sc, _, vn = oracle.quantize_blockscaled(W, bits, iters)
    pg, cg, sg = run_blockscaled(gpu, W, bits, iters)
    assert np.array_equal(sg, sc)
    assert np.array_equal(cg, cb)
    assert np.array_equal(pg, oracle.pack(idx, bits))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K", [(1, 64), (1, 64 * 63), (1, 64 * 65), (31, 64 * 66), (64, 64 * 65), (700, 6400)])
def test_sizes(gpu, N, K, bits):
    check(gpu, synth.make_dense_weights(110 + bits, N, N, K), bits, 9)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K", [(1, 64), (3, 64), (31, 64), (2, 64 * 64), (1, 64 * 129), (64, 64), (640, 64)])
@pytest.mark.parametrize("iters", [0, 1, 4, 5])
def test_few_rounds_of_small_tensors(gpu, N, K, bits, iters):
    """Up to 128 blocks and 4 rounds one workgroup does everything; around those limits, with zeros, a block of zeros, subnormal
    scales and far elements."""
    W = synth.make_dense_weights(115 + bits, N + iters, N, K)
    W[0, 5::7] &= 0x8000
    if N > 2:
        W[1] = 0
        W[2, 1::3] = (W[2, 1::3] & 0x807F) | (40 << 7)
        W[N // 2] = W[N // 2] & 0x803F
    check(gpu, W, bits, iters)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("iters", [0, 1, 40])
def test_rounds_and_exact_boundaries(gpu, bits, iters):
    """Weights on a coarse grid: many quotients coincide with the evenly spaced starting boundaries."""
    rng = np.random.default_rng(5 + bits)
    W = synth.f32_to_bf16((rng.integers(-16, 17, size=(64, 1024)) / 16.0).astype(np.float32))
    W[:, ::64] = 0x3F80
    W[40:, ::64] = synth.f32_to_bf16(rng.uniform(1.0, 2.0, size=(24, 16)).astype(np.float32))
    check(gpu, W, bits, iters)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_small_scales(gpu, bits):
    """Blocks scaled down to 1e-29 and to the smallest normal numbers, where weights are subnormal, next to ordinary ones."""
    W = synth.make_dense_weights(120, bits, 48, 512)
    f = synth.bf16_to_f32(W).astype(np.float64)
    f[8:16] *= 2.0 ** -100
    f[16:24] *= 2.0 ** -118
    f[24] = 0.0
    check(gpu, synth.f32_to_bf16(f.astype(np.float32)), bits, 12)


@pytest.mark.parametrize("bits", [1, 2, 4])
@pytest.mark.parametrize("share", ["one", "most", "positive"])
def test_far_elements(gpu, bits, share):
    """Elements more than 31 octaves below their scale: one in the tensor; most of it (their own values then make the
    middle centroids and boundaries); all of one sign."""
    W = synth.make_dense_weights(130, bits, 16, 1024)
    rng = np.random.default_rng(6)
    tiny = synth.f32_to_bf16((rng.normal(size=W.shape) * 2.0 ** -45).astype(np.float32))
    if share == "one":
        W[3, 77] = tiny[3, 77]
    else:
        if share == "positive":
            tiny &= 0x7FFF
        keep = np.zeros(W.shape, bool)
        keep[:, ::64] = True
        W = np.where(keep, W, tiny)
    check(gpu, W, bits, 8)


def _with_tiny(W, share, seed):
    """`share` of the elements (never a block's first) moved 40 to 60 octaves down."""
    rng = np.random.default_rng(seed)
    pick = rng.random(W.shape) < share
    pick[:, ::64] = False
    down = rng.integers(40, 61, size=W.shape) << 7
    mag = np.where(pick, np.maximum((W & 0x7FFF).astype(np.int64) - down, 1), W & 0x7FFF)
    out = ((W & 0x8000) | mag).astype(np.uint16)
    first = out[:, ::64]
    first[...] = np.maximum(first & 0x7FFF, 0x3C00)       # every block keeps an ordinary scale
    return out


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("share", [0.0005, 0.3, 1.0])
def test_far_elements_of_many_pieces(gpu, bits, share):
    """More blocks than the tensor is cut into pieces: a few far elements, a third, all but the scales themselves."""
    W = _with_tiny(synth.make_dense_weights(150, bits, 96, 2048), share, 8)
    check(gpu, W, bits, 7)
    a, b = (run_blockscaled(gpu, W, bits, 7) for _ in range(2))
    assert all(np.array_equal(u, v) for u, v in zip(a, b))


def _halfway():
    """16384 positive members, scales 1, without the last one's value halfway between two bf16 values in the mean."""
    W = np.full((4, 4096), 0x3F40, np.uint16)             # 0.75
    W[:, ::64] = 0x3F80                                    # 256 of 1, the scales
    W[0, 1:64] = W[0, 65:127] = 0x3F00                     # 125 of 0.5
    W[3, 4000] = 0
    assert np.sum(synth.bf16_to_f64(W)) == 16384 * (0.75 + 2.0 ** -9)
    return W


def test_far_member_decides_a_tie(gpu):
    """With the far one the mean lies a little above halfway (both sums are exact in 64 bits)."""
    W = _halfway()
    W[3, 4000] = 0x2F00                                    # 2^-33
    assert list(oracle.quantize_blockscaled(W, 1, 1)[1]) == [0xBF00, 0x3F41]
    check(gpu, W, 1, 1)


def test_small_member_decides_a_tie_above_many_others(gpu):
    """The same with a member of 2^-31 and 2^24 members of -1 in the cluster below: a cluster's sum owes nothing to those."""
    W = np.full((4100, 4096), 0xBF80, np.uint16)
    W[:4] = _halfway()
    W[3, 4000] = 0x3000                                    # 2^-31
    assert list(oracle.quantize_blockscaled(W, 1, 1)[1]) == [0xBF80, 0x3F41]
    check(gpu, W, 1, 1)


@pytest.mark.parametrize("bits", [1, 4])
@pytest.mark.parametrize("share", [0.0001, 0.9])
def test_far_elements_cost_no_more_than_a_reading_or_two_a_round(gpu, bits, share):
    """The tensor is searched for them by the whole chip: once for a few of them, at most once a round where they fill clusters of
    their own.  One workgroup's search took 50 to 700 times the call without them."""
    import torch
    N, K, iters = 2048, 4096, 8
    W = synth.make_dense_weights(160, bits, N, K)
    times = []
    for w in (W, _with_tiny(W, share, 9)):
        Wd = gpu.dev(w)
        packed = torch.empty((N, K * bits // 32), dtype=torch.int32, device="cuda")
        cb, sc = torch.empty(1 << bits, dtype=torch.int16, device="cuda"), torch.empty((N, K // 64), dtype=torch.int16, device="cuda")
        ws = torch.empty(kmq.quantize_blockscaled_workspace_bytes(), dtype=torch.uint8, device="cuda")
        run = lambda: kmq.quantize_blockscaled(Wd, N, K, bits, iters, packed, cb, sc, ws)
        run()
        took = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            run()
            b.record()
            torch.cuda.synchronize()
            took.append(a.elapsed_time(b))
        times.append(sorted(took)[2])
    print(f"b{bits} share {share}: {times[0] * 1e3:.0f} us without, {times[1] * 1e3:.0f} us with far elements")
    assert times[1] < (3 if share < 0.5 else 3 + iters) * times[0]


@pytest.mark.parametrize("bits", [1, 4])
@pytest.mark.parametrize("pattern", [0x7F80, 0xFF80, 0x7FC1, 0xFFFF])
def test_non_finite_weight(gpu, bits, pattern):
    """One infinity or NaN in the tensor shows in every centroid; the other blocks keep their scales."""
    for N, iters in ((40, 5), (4, 3)):
        W = synth.make_dense_weights(170, bits, N, 1024)
        sc = run_blockscaled(gpu, W, bits, iters)[2]
        W[3, 700] = pattern
        _, cg, sg = run_blockscaled(gpu, W, bits, iters)
        assert np.all((cg & 0x7FFF) > 0x7F80)
        sc[3, 700 // 64] = pattern & 0x7FFF
        assert np.array_equal(sg, sc)


def test_list_reuse_of_the_output(gpu):
    """The index words hold the sorted block list for a while: nothing of it may be left, and repeats give the same bits."""
    W = synth.make_dense_weights(140, 0, 96, 4096)
    a = run_blockscaled(gpu, W, 1, 6)
    b = run_blockscaled(gpu, W, 1, 6)
    assert all(np.array_equal(u, v) for u, v in zip(a, b))
    assert kmq.quantize_blockscaled_workspace_bytes() % 8 == 0
