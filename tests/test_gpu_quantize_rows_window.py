"""The row quantiser's kernel of four rows a workgroup (2560 rows and more, from 2049 elements on 3000, with fewer than four rounds 9216, at
most 4096 elements) at its edges, bit for bit against the fp64 oracle: row lengths around a thread's piece and a wave's share, row
counts that leave a workgroup partly empty, and rows side by side that go its several ways: elements below its window (a few, sixteen,
seventeen), boundaries among those, counters at and over 255, zeros of both signs, one value only, infinities' neighbours.  Longer
rows, and long ones with few rounds, are the other side of the rule: a workgroup a row."""
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


def bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def check(gpu, W, bits, iters, rows):
    N, K = W.shape
    print(f"quantize_rows {W.shape} b={bits} iters={iters}", flush=True)
    pg, cg = run_rows(gpu, W, bits, iters)
    idx, cb, _, _ = oracle.quantize_rows(np.ascontiguousarray(W[rows]), bits, iters)
    assert np.array_equal(cg[rows], cb)
    assert np.array_equal(pg[rows], oracle.pack(idx, bits))


def check_size(gpu, N, K, bits, iters):
    W = synth.make_dense_weights(120 + bits, K, N, K)
    check(gpu, W, bits, iters, np.unique(np.r_[:9, np.linspace(0, N - 1, 20).astype(int), N - 9:N]))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K", [(2560, 1), (2561, 15), (2562, 16), (2563, 17), (2560, 33), (2561, 1023), (2562, 1041), (3003, 2049), (3003, 4095), (3000, 4096), (3001, 4097),
                                 (2562, 6001), (2563, 8191), (2560, 8192)])
def test_sizes(gpu, N, K, bits):
    check_size(gpu, N, K, bits, 12)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("iters", [0, 1, 3])
@pytest.mark.parametrize("N,K", [(2561, 513), (2562, 529), (2563, 2047), (9215, 2049), (9217, 2049)])
def test_few_rounds(gpu, N, K, iters, bits):
    check_size(gpu, N, K, bits, iters)


def special_rows(K, rng):
    normal = lambda: rng.standard_normal(K) * 0.02
    tiny = lambda n: rng.choice([-1, 1], n) * 2.0 ** rng.uniform(-30, -16, n) * 0.06
    rows = []
    for n in (1, 3, 16, 17, 200):                              # below the window: sixteen of them are met one by one
        r = normal()
        r[0], r[5:5 + n] = 0.06, tiny(n)
        rows.append(r)
    half = (K - 11) // 2
    for signs in ([1] * 5 + [-1] * 5, [1] * 10, [-1] * 10):    # the middle boundary ends up among them
        r = np.zeros(K)
        a = np.abs(normal()[:half]) + 1e-3
        r[:half], r[half:2 * half], r[2 * half:2 * half + 10] = a, -a, np.array(signs) * 2.0 ** rng.uniform(-33, -17, 10) * 0.06
        rows.append(r)
    for _ in range(3):                                         # ... after rounding, too (huge elements of both signs, so that the others are split at 0)
        r = rng.choice([-1, 1], K) * rng.uniform(0.25, 2, K)
        r[1], r[2], r[3:13] = 1500, -1500, rng.choice([-1, 1], 10) * rng.uniform(0.001, 0.06, 10)
        rows.append(r)
    for n in (254, 255, 256, 1000):                            # one value so often
        r = normal()
        r[:min(n, K)] = 0.0123
        rows.append(r)
    for v in (0.0, -0.0, 0.05, -0.05, 3e38, 2e-38, 1e-30):     # nothing else; huge and small
        rows.append(np.full(K, v))
    r = normal(); r[::2] = 0.0; r[1::4] = -0.0; rows.append(r)
    r = normal() * 1e-30; rows.append(r)
    r = np.abs(normal()); rows.append(r); rows.append(-r)
    rows.append(normal() * 2.0 ** rng.integers(-40, 1, K))
    rows.append(np.round(normal() / 0.0006) * 0.0006)
    return bf16(np.array(rows))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [301, 2035, 3001, 4096, 8000])
@pytest.mark.parametrize("iters", [0, 1, 25])
def test_rows_of_every_kind(gpu, K, bits, iters):
    rng = np.random.default_rng(K + bits)
    special = special_rows(K, rng)
    W = synth.make_dense_weights(130 + bits, K, 3001, K)
    at = rng.permutation(3001)[:len(special)]                  # side by side with ordinary rows, any place in a workgroup
    W[at] = special
    check(gpu, W, bits, iters, at)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [1025, 1041, 3001, 4096])
def test_rows_left_early(gpu, K, bits):
    """The look after half of the first pieces (eight of every sixteen elements, the first 1024): equal values and elements below the
    window around what it lets pass, all inside that half or all outside; rows that are left there and rows that are not give the same bits."""
    rng = np.random.default_rng(7 * K + bits)
    inside = np.flatnonzero((np.arange(K) < 1024) & (np.arange(K) % 16 < 8))
    outside = np.setdiff1d(np.arange(K), inside)
    rows = []
    for places in (inside, outside):
        share = 255 * 8 * 64 // K                               # of the half: as many as 255 of the row
        for n in (share - 1, share, share + 1, 254, 255, 256, 257, len(places)):
            r = rng.standard_normal(K) * 0.02
            r[rng.permutation(places)[:n]] = rng.choice([0.0123, -0.0123])
            rows.append(r)
        for n in (1, 16, 17, 40, 256, 300):
            r = rng.standard_normal(K) * 0.02
            at = rng.permutation(places)[:n]
            r[at] = rng.choice([-1, 1], len(at)) * 2.0 ** rng.uniform(-30, -16, len(at)) * 0.06
            rows.append(r)
        for zero in (0.0, -0.0):
            r = rng.standard_normal(K) * 0.02
            r[places] = zero
            rows.append(r)
    W = synth.make_dense_weights(150 + bits, K, 3001, K)
    at = rng.permutation(3001)[:len(rows)]
    W[at] = bf16(np.array(rows))
    check(gpu, W, bits, 12, at)
