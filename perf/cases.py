"""The calls this library is used for, at the sizes it is used at, as timed cases.

A case is a dict of plain values; its "kind" says which part of the path it takes:

  product   y = W x, or Y = X W^T at small batch, one codebook per row: the projections of a decoder, one token
            (M = 1) or a few sequences at a time, on any of the three layouts
  scaled    the same in the tensor-codebook format with one scale per 64 weights
  decoder   one token through a stack of decoder layers, RMSNorm / SwiGLU / residual folded into the products
  dequant   dense bf16 weights from the packed ones: the first half of a large-batch (prompt) product
  quantize  dense bf16 weights to packed indices and codebooks: how the formats are made

Inference replays a HIP graph of one token's (or one batch step's) calls over all layers, every layer with its own
weights, as a serving loop does; "graph": False is a single call launched from Python.  Sizes are those of the
benchmark (bench.py) and of the tests, and generic ones between them.
"""
import math

import torch

from paper_2602_15563_amd import kmq

CANONICAL, TILED, ROWLANE = kmq.LAYOUT_CANONICAL, kmq.LAYOUT_TILED, kmq.LAYOUT_ROWLANE
BLOCK = 64            # weights per scale
TILE_ROWS = 16        # the tiled and row-lane layouts pad rows to this
MOST_BITS = 32 * 14336 * 4096 * 3      # index bits of the largest listed stack of layers
MOST_BATCH = 16


def listed():
    return [
        # a single small product launched from Python: the latency of the call itself (2048 x 2048, the smallest shape of the benchmark)
        dict(name="call_1bit_2048", kind="product", bits=1, N=2048, K=2048, M=1, layout=CANONICAL, layers=1, graph=False),
        # token generation with the up projections of an 8B-sized model at 2 bits, the headline shape, 32 layers
        dict(name="token_2bit_14336x4096", kind="product", bits=2, N=14336, K=4096, M=1, layout=ROWLANE, layers=32, graph=True),
        # attention projections at 4 bits, one token, in the interchange layout
        dict(name="token_4bit_4096", kind="product", bits=4, N=4096, K=4096, M=1, layout=CANONICAL, layers=32, graph=True),
        # a matrix whose sides fit nothing: 3 bits, odd row length, three sequences
        dict(name="ragged_3bit_5001x4101", kind="product", bits=3, N=5001, K=4101, M=3, layout=CANONICAL, layers=16, graph=True),
        # four sequences at 2 bits, weights as the quantiser and kmq_pack leave them
        dict(name="batch4_2bit_4096x14336", kind="product", bits=2, N=4096, K=14336, M=4, layout=CANONICAL, layers=32, graph=True),
        # sixteen sequences at 3 bits on the matrix-core layout: the largest batch the library takes
        dict(name="batch16_3bit_14336x4096", kind="product", bits=3, N=14336, K=4096, M=16, layout=TILED, layers=32, graph=True),
        # one token through the 28 layers of the 3.9B-sized 1-bit decoder, four launches a layer
        dict(name="decoder_1bit_28", kind="decoder", bits=1, hidden=3072, qkv=9216, mlp=8192, layers=28),
        # the block-scaled format at the micro-benchmark's width, one token at 4 bits ...
        dict(name="token_4bit_scaled_8192", kind="scaled", bits=4, N=8192, K=8192, M=1, layout=CANONICAL, layers=8, graph=True),
        # ... and eight sequences at 1 bit
        dict(name="batch8_1bit_scaled_8192", kind="scaled", bits=1, N=8192, K=8192, M=8, layout=CANONICAL, layers=8, graph=True),
        # dense weights for a prompt's matrix product
        dict(name="dense_4bit_scaled_8192", kind="dequant", bits=4, N=8192, K=8192, scaled=True),
        # a layer's matrix quantised row by row, the format of the benchmark
        dict(name="quantize_rows_2bit", kind="quantize", bits=2, N=14336, K=4096, iters=25, scaled=False),
        # a layer's matrix quantised to the tensor-codebook format
        dict(name="quantize_scaled_4bit", kind="quantize", bits=4, N=8192, K=8192, iters=25, scaled=True),
    ]


def _between(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _multiple(n, of):
    return max(of, n // of * of)


def _row_step(bits, layout, scaled):
    """What the row length has to be a multiple of."""
    if layout == TILED:
        return {1: 512, 2: 256, 3: 128, 4: 128}[bits]
    if layout == ROWLANE:
        return 256
    return BLOCK if scaled else 1


def _draw_product(rng, scaled):
    bits = rng.choice([1, 2, 3, 4, 1, 2, 3, 4, 8] if not scaled else [1, 2, 3, 4])
    layouts = [CANONICAL]
    if bits <= 4:
        layouts.append(TILED)
    if bits <= 2 and not scaled:
        layouts.append(ROWLANE)
    layout = rng.choice(layouts)
    N = _between(rng, 1024, 20480)
    K = _between(rng, 1024, 16384)
    step = _row_step(bits, layout, scaled)
    if step == 1 and rng.random() < 0.7:      # most widths are multiples of 64 or 256, some are not
        step = rng.choice([64, 256])
    K = _multiple(K, step)
    if rng.random() < 0.7:
        N = _multiple(N, 64)
    M = 1 if rng.random() < 0.5 else rng.randint(2, MOST_BATCH)
    layers = max(1, min(32, MOST_BITS // (N * K * max(bits, 3))))
    graph = rng.random() < 0.85
    if not graph:
        layers = 1
    return dict(kind="scaled" if scaled else "product", bits=bits, N=N, K=K, M=M, layout=layout, layers=layers, graph=graph)


def draw(rng):
    u = rng.random()
    if u < 0.45:
        return _draw_product(rng, False)
    if u < 0.65:
        return _draw_product(rng, True)
    if u < 0.75:
        hidden = rng.choice([1536, 2048, 3072, 4096, 6144]) if rng.random() < 0.6 else _multiple(_between(rng, 1024, 6144), 128)
        mlp = _multiple(int(hidden * rng.uniform(2.6, 3.6)), 256)
        per_layer = hidden * (3 * hidden + hidden + 3 * mlp)
        bits = rng.choice([1, 2, 3, 4])
        return dict(kind="decoder", bits=bits, hidden=hidden, qkv=3 * hidden, mlp=mlp,
                    layers=max(1, min(28, MOST_BITS // (per_layer * max(bits, 3)))))
    scaled = rng.random() < 0.5
    if u < 0.85:
        N = _between(rng, 1024, 14336)
        K = _multiple(_between(rng, 1024, 8192 * 8192 // N), BLOCK if scaled else rng.choice([1, 8, 64, 64]))
        return dict(kind="dequant", bits=rng.choice([1, 2, 3, 4]), N=N, K=K, scaled=scaled)
    N = _between(rng, 1024, 12288)
    K = _multiple(_between(rng, 1024, min(16384, 8192 * 8192 // N)), BLOCK if scaled else rng.choice([1, 64, 64]))
    return dict(kind="quantize", bits=rng.choice([1, 2, 3, 4]), N=N, K=K, iters=rng.randint(8, 25), scaled=scaled)


# ---- inputs ------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, sigma=1.0):
    return (torch.randn(shape, generator=g, device="cuda") * sigma).to(torch.bfloat16)


def _words(g, shape):
    return torch.randint(-2**31, 2**31, shape, generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def _packed(g, N, K, bits, layout):
    """Uniform random indices of one matrix in `layout`: random words, with the pad bits of a row and the rows of padding cleared."""
    wpr = kmq.words_per_row(bits, K)
    if layout == CANONICAL:
        W = _words(g, (N, wpr))
        used = K * bits - 32 * (wpr - 1)
        if used < 32:
            W[:, -1] &= (1 << used) - 1
        return W
    per_row = K * bits // 32
    W = _words(g, ((N + TILE_ROWS - 1) // TILE_ROWS, per_row * TILE_ROWS))
    live = N % TILE_ROWS
    if live:      # both layouts store a block of 16 rows as pieces of 64 lanes, lane % 16 the row
        size = {TILED: {1: 4, 2: 4, 3: 3, 4: 4}[bits], ROWLANE: 2 * bits}[layout]
        W[-1].view(-1, 4, TILE_ROWS, size)[:, :, live:, :] = 0
    return W


def _row_codebooks(g, N, bits, sigma=0.02):
    if bits == 1:
        t = _normal(g, (N, 1), sigma).abs()
        return torch.cat([-t, t], dim=1).contiguous()
    return _normal(g, (N, 1 << bits), sigma).sort(dim=1).values.contiguous()


def _tensor_codebook(g, bits):
    if bits == 1:
        t = 0.5 + 0.4 * torch.rand(1, generator=g, device="cuda")
        return torch.cat([-t, t]).to(torch.bfloat16)
    return (torch.randn(1 << bits, generator=g, device="cuda") * 0.45).clamp(-1, 1).to(torch.bfloat16).sort().values.contiguous()


def _block_scales(g, N, K):
    """Distributed as the largest magnitude of 64 samples of N(0, 0.02)."""
    u = torch.rand((N, K // BLOCK), generator=g, device="cuda", dtype=torch.float64).clamp_(1e-12, 1 - 1e-12)
    return (0.02 * math.sqrt(2.0) * torch.special.erfinv(u ** (1.0 / BLOCK))).to(torch.bfloat16)


def _dense(g, N, K):
    """Trained-like weights: N(0, 0.02) with a gain of its own for each row."""
    gain = 0.5 + 1.5 * torch.rand((N, 1), generator=g, device="cuda")
    return (torch.randn((N, K), generator=g, device="cuda") * (0.02 * gain)).to(torch.bfloat16)


def _captured(step):
    """`step` once eagerly, then as a HIP graph."""
    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    return graph


def _prepare_product(case, g):
    N, K, M, bits, layout, layers = (case[k] for k in ("N", "K", "M", "bits", "layout", "layers"))
    scaled = case["kind"] == "scaled"
    W = [_packed(g, N, K, bits, layout) for _ in range(layers)]
    C = [_tensor_codebook(g, bits) if scaled else _row_codebooks(g, N, bits) for _ in range(layers)]
    S = [_block_scales(g, N, K) for _ in range(layers)] if scaled else None
    X = [_normal(g, (M, K)) for _ in range(layers)]
    Y = torch.empty((layers, M, N), dtype=torch.bfloat16, device="cuda")
    need = 0 if scaled else kmq.workspace_bytes(N, K, bits, M, layout)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None

    def step():
        for l in range(layers):
            if scaled and M == 1:
                kmq.gemv_blockscaled(W[l], C[l], S[l], X[l], Y[l], N, K, bits, layout, workspace=ws)
            elif scaled:
                kmq.gemm_smallbatch_blockscaled(W[l], C[l], S[l], X[l], Y[l], N, K, M, bits, layout, workspace=ws)
            elif M == 1:
                kmq.gemv(W[l], C[l], X[l], Y[l], N, K, bits, layout, workspace=ws)
            else:
                kmq.gemm_smallbatch(W[l], C[l], X[l], Y[l], N, K, M, bits, layout, workspace=ws)

    return dict(run=_captured(step).replay if case["graph"] else step, keep=(W, C, S, X, ws, step), out=Y)


def _prepare_decoder(case, g):
    h, qkv, mlp, bits, layers = (case[k] for k in ("hidden", "qkv", "mlp", "bits", "layers"))
    eps = 1e-5

    into_stream = 0.02 / math.sqrt(2 * layers)      # what adds to the residual stream is scaled down by depth, as models are

    def matrices(N, K, sigma=0.02):
        return [(_packed(g, N, K, bits, CANONICAL), _row_codebooks(g, N, bits, sigma)) for _ in range(layers)]

    Wq, Wo, Wg, Wu, Wd = matrices(qkv, h), matrices(h, h, into_stream), matrices(mlp, h), matrices(mlp, h), matrices(h, mlp, into_stream)
    gains = [[(1.0 + 0.1 * torch.randn(h, generator=g, device="cuda")).to(torch.bfloat16) for _ in range(2)] for _ in range(layers)]
    hs = torch.empty((layers + 1, h), dtype=torch.bfloat16, device="cuda")      # the residual stream between layers
    hs[0] = _normal(g, (h,))
    mid = torch.empty((layers, h), dtype=torch.bfloat16, device="cuda")
    yq = torch.empty((layers, qkv), dtype=torch.bfloat16, device="cuda")
    ym = torch.empty((layers, mlp), dtype=torch.bfloat16, device="cuda")

    def step():
        for l in range(layers):
            kmq.gemv_fused(*Wq[l], hs[l], yq[l], qkv, h, bits, norm_weight=gains[l][0], eps=eps)
            # attention is not part of this library: its value slice stands in for its output
            kmq.gemv_fused(*Wo[l], yq[l, qkv - h:], mid[l], h, h, bits, residual=hs[l])
            kmq.gemv_swiglu_rmsnorm(*Wg[l], *Wu[l], mid[l], gains[l][1], eps, ym[l], mlp, h, bits)
            kmq.gemv_fused(*Wd[l], ym[l], hs[l + 1], h, mlp, bits, residual=mid[l])

    return dict(run=_captured(step).replay, keep=(Wq, Wo, Wg, Wu, Wd, gains, step), out=(hs, mid, yq, ym))


def _prepare_dequant(case, g):
    N, K, bits = case["N"], case["K"], case["bits"]
    W = _packed(g, N, K, bits, CANONICAL)
    D = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    if case["scaled"]:
        C, S = _tensor_codebook(g, bits), _block_scales(g, N, K)
        return dict(run=lambda: kmq.dequant_blockscaled(W, C, S, D, N, K, bits), out=D)
    C = _row_codebooks(g, N, bits)
    return dict(run=lambda: kmq.dequant(W, C, D, N, K, bits), out=D)


def _prepare_quantize(case, g):
    N, K, bits, iters = case["N"], case["K"], case["bits"], case["iters"]
    D = _dense(g, N, K)
    W = torch.empty((N, kmq.words_per_row(bits, K)), dtype=torch.int32, device="cuda")
    if not case["scaled"]:
        C = torch.empty((N, 1 << bits), dtype=torch.int16, device="cuda")
        return dict(run=lambda: kmq.quantize_rows(D, N, K, bits, iters, W, C), out=(W, C))
    C = torch.empty(1 << bits, dtype=torch.int16, device="cuda")
    S = torch.empty((N, K // BLOCK), dtype=torch.int16, device="cuda")
    ws = torch.empty(kmq.quantize_blockscaled_workspace_bytes(), dtype=torch.uint8, device="cuda")
    return dict(run=lambda: kmq.quantize_blockscaled(D, N, K, bits, iters, W, C, S, ws), out=(W, C, S))


def prepare(case, seed):
    make = {"product": _prepare_product, "scaled": _prepare_product, "decoder": _prepare_decoder,
            "dequant": _prepare_dequant, "quantize": _prepare_quantize}[case["kind"]]
    return make(case, _generator(seed))


def run(state):
    state["run"]()
    return state["out"]


# ---- what a pass cannot do without ----------------------------------------------------------------------

def _matrix_bytes(N, K, bits, scaled):
    words = 4 * N * ((K * bits + 31) // 32)
    return words + (2 * (1 << bits) + 2 * N * (K // BLOCK) if scaled else 2 * N * (1 << bits))


def work(case):
    kind, bits = case["kind"], case["bits"]
    if kind in ("product", "scaled"):
        N, K, M, layers = (case[k] for k in ("N", "K", "M", "layers"))
        return {"bytes": layers * (_matrix_bytes(N, K, bits, kind == "scaled") + 2 * M * (N + K)), "flops": 2 * layers * N * K * M}
    if kind == "decoder":
        h, qkv, mlp, layers = (case[k] for k in ("hidden", "qkv", "mlp", "layers"))
        matrices = [(qkv, h), (h, h), (mlp, h), (mlp, h), (h, mlp)]
        vectors = (2 * h + qkv) + 3 * h + (2 * h + mlp) + (mlp + 2 * h)      # inputs, gains and residuals read, outputs written
        return {"bytes": layers * (sum(_matrix_bytes(N, K, bits, False) for N, K in matrices) + 2 * vectors),
                "flops": 2 * layers * sum(N * K for N, K in matrices)}
    N, K, scaled = case["N"], case["K"], case["scaled"]
    return {"bytes": _matrix_bytes(N, K, bits, scaled) + 2 * N * K, "flops": N * K if scaled else 0}


def tolerance(case):
    """Integers and looked-up values are exact.  A product is a 32-bit sum rounded once to bf16: the sum in 64 bits moves
    single results by one unit in the last place (rel 3e-5, max 6e-3 on the worst of a dozen shapes).  Through a stack of
    layers those single units spread: against the stack in 64 bits with the same roundings of the activations, rel 1.2e-2
    after 28 layers at 1 bit."""
    if case["kind"] in ("dequant", "quantize"):
        return "exact"
    if case["kind"] == "decoder":
        return {"rel": 4e-2}
    return {"rel": 1.2e-4, "max": 2.4e-2}
