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


def test_list_reuse_of_the_output(gpu):
    """The index words hold the sorted block list for a while: nothing of it may be left, and repeats give the same bits."""
    W = synth.make_dense_weights(140, 0, 96, 4096)
    a = run_blockscaled(gpu, W, 1, 6)
    b = run_blockscaled(gpu, W, 1, 6)
    assert all(np.array_equal(u, v) for u, v in zip(a, b))
    assert kmq.quantize_blockscaled_workspace_bytes() % 8 == 0
