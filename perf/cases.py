"""The work a training program has this library do, as cases that can be timed and compared.

Every case is one training step's worth of calls through ``paper_2203_05705_amd.binding``: a layer, a
three-layer perceptron, an LSTM layer or a convolution layer, forward and backward, under the dropout
patterns of the paper.  Sizes follow the benchmark configurations (``bench.py``,
``paper_2203_05705_amd/workloads.py``) and the paper's own tables; ``draw`` spreads over the ranges
between the smallest and the largest of them, ragged sizes included.
"""
import math

import torch

from paper_2203_05705_amd import binding as ard

IN, OUT, WC = ard.IN_COMPACT, ard.OUT_COMPACT, ard.W_COMPACT


def listed():
    return [
        # one small fp32 layer (configuration 1): three calls of a few microseconds, latency and launches
        dict(name="layer_f32_64", family="layer", dtype="f32", B=64, I=784, O=1024, pattern="row", dp=2, dp_in=1),
        # a middle layer whose sizes are multiples of nothing, both sides under a row pattern
        dict(name="layer_ragged_bf16", family="layer", dtype="bf16", B=1027, I=1501, O=1203, pattern="row", dp=3, dp_in=2),
        # a large layer under the tile pattern (configuration 3): matrix-core throughput
        dict(name="layer_tile64_4096", family="layer", dtype="bf16", B=4096, I=4096, O=4096, pattern="tile", tile=64, dp=2, dp_in=1),
        # the headline network (configuration 2), rate 0.5, one grouped launch per dependency level
        dict(name="mlp_row_b1024_bf16", family="mlp", dtype="bf16", B=1024, I=784, H1=2048, H2=2048, O=10, pattern="row", dp=2, dp2=2),
        # the paper's own network, batch and precision (Section 7.2.1), rate 0.7
        dict(name="mlp_row_b128_f32", family="mlp", dtype="f32", B=128, I=784, H1=2048, H2=2048, O=10, pattern="row", dp=3, dp2=3),
        # the largest network of the paper's Table 1, with its 32 x 32 tiles
        dict(name="mlp_tile32_b128_bf16", family="mlp", dtype="bf16", B=128, I=784, H1=4096, H2=4096, O=10, pattern="tile", tile=32, dp=3, dp2=3),
        # the LSTM layer of configuration 4
        dict(name="lstm_1024_b128_bf16", family="lstm", dtype="bf16", T=64, B=128, I=1024, H=1024, pattern="row", dp=2),
        # the LSTM layer of Section 7.2.3: 1500 units, 35 steps, batch 20
        dict(name="lstm_1500_b20_bf16", family="lstm", dtype="bf16", T=35, B=20, I=1500, H=1500, pattern="row", dp=2),
        # a convolution layer with half of its input feature maps dropped (configuration 5)
        dict(name="conv_28_bf16", family="conv", dtype="bf16", N=128, C=256, S=28, Cout=256, k=3, rate=0.5),
        # an early layer of a CIFAR-sized network in fp32
        dict(name="conv_32_f32", family="conv", dtype="f32", N=64, C=64, S=32, Cout=64, k=3, rate=0.5),
        # the sensitivity-aware row pattern of Section 5.2.1 from prediction to gradients
        dict(name="conv_rows_28_bf16", family="rows", dtype="bf16", N=128, C=256, S=28, Cout=256, k=3, x=8),
        # the balanced block pattern of Section 5.2.2: bands of four rows by 64-channel groups
        dict(name="conv_blocks_28_bf16", family="blocks", dtype="bf16", N=128, C=256, S=28, Cout=256, k=3, x=112),
    ]


def _size(rng, lo, hi):
    """A size from lo to hi, even over its logarithm; half of them round, as layer widths mostly are."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        m = 64 if n >= 256 else 8
        n = max(m, n // m * m)
    return min(max(n, lo), hi)


# most arithmetic of a drawn case: the large listed layers for bf16; for fp32, whose matrix rate is a
# sixteenth, as much less
_MOST = {"bf16": 1.6e11, "f32": 1.0e10}


def draw(rng):
    family = rng.choice(("layer", "layer", "layer", "mlp", "mlp", "lstm", "lstm", "conv", "conv", "rows", "blocks"))
    dtype = "f32" if rng.random() < (0.35 if family in ("layer", "mlp", "conv") else 0.2) else "bf16"
    dp = rng.choice((1, 2, 2, 3, 4, 5, 6, 8))
    if family == "layer":
        c = dict(B=_size(rng, 16, 4096), I=_size(rng, 64, 4096), O=_size(rng, 64, 4096), pattern=rng.choice(("row", "row", "tile")), dp=dp)
        c["dp_in"] = rng.choice((1, 2, 3, 4)) if c["pattern"] == "row" else 1
        if c["pattern"] == "tile":
            c["tile"] = rng.choice((32, 64))
        less = "B"
    elif family == "mlp":
        c = dict(B=_size(rng, 16, 1024), I=_size(rng, 100, 3072), H1=_size(rng, 64, 4096), H2=_size(rng, 64, 4096), O=_size(rng, 2, 128),
                 pattern=rng.choice(("row", "row", "tile")), dp=dp, dp2=rng.choice((1, 2, 2, 3, 4, 5, 6, 8)))
        if c["pattern"] == "tile":
            c["tile"] = rng.choice((32, 64))
        less = "B"
    elif family == "lstm":
        c = dict(T=_size(rng, 8, 64), B=_size(rng, 8, 128), I=_size(rng, 128, 1536), H=_size(rng, 128, 1536),
                 pattern=rng.choice(("row", "row", "row", "tile")), dp=rng.choice((1, 2, 2, 3, 4)))
        if c["pattern"] == "tile":
            c["tile"] = 32
        less = "T"
    else:
        # planes of the usual networks' stages and odd ones between them
        c = dict(N=_size(rng, 8, 128), C=_size(rng, 16, 512), S=rng.choice((7, 13, 14, 16, 19, 27, 28, 32, 56)), Cout=_size(rng, 16, 512), k=3)
        if family == "conv":
            c["k"], c["rate"] = rng.choice((3, 3, 3, 5)), rng.choice((0.0, 0.3, 0.5, 0.7))
        elif family == "rows":
            c["x"] = rng.choice((4, 8, c["S"]))
        else:
            c["C"] = 64 * max(1, c["C"] // 64)
            c["x"] = c["S"] * rng.choice((2, 4, 7))
        less = "N"
    c.update(family=family, dtype=dtype)
    while work(c)["flops"] > _MOST[dtype] and c[less] > 8:
        c[less] = max(8, c[less] * 3 // 4)
    while work(c)["flops"] > _MOST[dtype]:
        for n in ("I", "O", "H1", "H2", "H", "C", "Cout"):
            if n in c:
                c[n] = c[n] * 7 // 8 // 64 * 64 if n == "C" and family == "blocks" else c[n] * 7 // 8
    return c


# ---- what a program has in hand before the step -------------------------------------------------------

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


class _Inputs:
    """Seeded tensors on the GPU, rounded once to the case's type."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = _dtype(case)

    def normal(self, shape, scale=1.0):
        return (torch.randn(shape, generator=self.g, device="cuda") * scale).to(self.dtype)

    def uniform(self, shape, lo, hi):
        return (torch.rand(shape, generator=self.g, device="cuda") * (hi - lo) + lo).to(self.dtype)

    def xavier(self, o, i):
        lim = math.sqrt(6.0 / (o + i))
        return self.uniform((o, i), -lim, lim)

    def relu_normal(self, shape):
        return torch.randn(shape, generator=self.g, device="cuda").clamp_(min=0).to(self.dtype)


def _bytes(n):
    return torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")


def _code(case):
    return ard.F32 if case["dtype"] == "f32" else ard.BF16


def _pattern(case, dp, b):
    """(kind, parameters): the pattern of an iteration is two numbers; the program builds it anew per step."""
    if case["pattern"] == "tile":
        return ard.Pattern.tile(dp, b, case["tile"], case["tile"])
    return ard.Pattern.row(dp, b)


def prepare(case, seed):
    return dict(case=case, seed=seed, **_PREPARE[case["family"]](case, seed))


def run(state):
    return _RUN[state["case"]["family"]](state, state["case"])


# ---- one fully connected layer ------------------------------------------------------------------------

def _prepare_layer(case, seed):
    x = _Inputs(case, seed)
    B, I, O = case["B"], case["I"], case["O"]
    po = _pattern(case, case["dp"], 1)
    pi = ard.Pattern.row(case["dp_in"], 1) if case["pattern"] == "row" else None
    n = ard.gemm_workspace_bytes(_code(case), B, I, O, po, pi)
    return dict(X=x.normal((B, I)), W=x.xavier(O, I), dY=x.normal((B, O)), ws=_bytes(n), b=1 + seed % case["dp"], b_in=1 + seed // 7 % case["dp_in"],
                Y=torch.empty((B, O), dtype=x.dtype, device="cuda"), dX=torch.empty((B, I), dtype=x.dtype, device="cuda"),
                dW=torch.empty((O, I), dtype=x.dtype, device="cuda"))


def _run_layer(s, case):
    po = _pattern(case, case["dp"], s["b"])
    pi = ard.Pattern.row(case["dp_in"], s["b_in"]) if case["dp_in"] > 1 else None
    Y = ard.drop_gemm_fwd(s["X"], s["W"], po, pi, relu=True, out=s["Y"], ws=s["ws"])
    dX = ard.drop_gemm_bwd_data(s["dY"], s["W"], po, pi, out=s["dX"], ws=s["ws"])
    dW = ard.drop_gemm_bwd_weight(s["dY"], s["X"], po, pi, out=s["dW"], ws=s["ws"])
    return dict(Y=Y, dX=dX, dW=dW)


# ---- a three-layer perceptron -------------------------------------------------------------------------
# Forward chain, then the backward chain.  The backward pass takes the saved activations from the state, as
# an autograd node does, and not the ones this step's forward pass has just made: a ReLU whose input rounds
# to the other side of zero would otherwise make two correct gradients differ by whole values.

def _prepare_mlp(case, seed):
    x = _Inputs(case, seed)
    B, sizes = case["B"], (case["I"], case["H1"], case["H2"], case["O"])
    X0 = x.uniform((B, sizes[0]), 0.0, 1.0)
    W = [x.xavier(sizes[l + 1], sizes[l]) for l in range(3)]
    b, b2 = 1 + seed % case["dp"], 1 + seed // 7 % case["dp2"]
    row = case["pattern"] == "row"
    k1 = torch.arange(b - 1, sizes[1], case["dp"], device="cuda") if row else slice(None)
    k2 = torch.arange(b2 - 1, sizes[2], case["dp2"], device="cuda") if row else slice(None)
    Y1 = x.relu_normal((B, sizes[1]))[:, k1].contiguous()
    Y2 = x.relu_normal((B, sizes[2]))[:, k2].contiguous()
    dY = x.normal((B, sizes[3]))
    if row:
        Y1, Y2, dY = ard.pad_compact(Y1), ard.pad_compact(Y2), ard.pad_compact(dY)
    pats = (_pattern(case, case["dp"], 1), _pattern(case, case["dp2"], 1))
    outer = (pats[0], pats[1], None)
    inner = (None, pats[0], pats[1]) if row else (None, None, None)
    n = max(ard.gemm_workspace_bytes(_code(case), B, sizes[l], sizes[l + 1], outer[l], inner[l]) for l in range(3))
    return dict(X0=X0, W=W, dY=dY, Y1=Y1, Y2=Y2, b=b, b2=b2, ws=[_bytes(n) for _ in range(3)], dW=[torch.empty_like(w) for w in W])


def _run_mlp(s, case):
    p1, p2 = _pattern(case, case["dp"], s["b"]), _pattern(case, case["dp2"], s["b2"])
    X0, (W1, W2, W3), dY, S1, S2 = s["X0"], s["W"], s["dY"], s["Y1"], s["Y2"]
    ws, (dW1, dW2, dW3) = s["ws"], s["dW"]
    I, H1, H2, O = case["I"], case["H1"], case["H2"], case["O"]
    if case["pattern"] == "tile":   # synapses are dropped, every neuron stays
        Y1 = ard.drop_gemm_fwd(X0, W1, p1, relu=True, ws=ws[0])
        Y2 = ard.drop_gemm_fwd(Y1, W2, p2, relu=True, ws=ws[0])
        with ard.batch():
            ard.drop_gemm_bwd_weight(dY, S2, out=dW3, ws=ws[1])
            Y3 = ard.drop_gemm_fwd(Y2, W3, ws=ws[0])
            dY2 = ard.drop_gemm_bwd_data(dY, W3, relu_src=S2, ws=ws[2])
        with ard.batch():
            ard.drop_gemm_bwd_weight(dY2, S1, p2, out=dW2, ws=ws[1])
            dY1 = ard.drop_gemm_bwd_data(dY2, W2, p2, relu_src=S1, ws=ws[0])
        ard.drop_gemm_bwd_weight(dY1, X0, p1, out=dW1, ws=ws[0])
        return dict(Y1=Y1, Y2=Y2, Y3=Y3, dY1=dY1, dY2=dY2, dW1=dW1, dW2=dW2, dW3=dW3)
    # kept neurons only between the layers; the kept block of W2 is gathered once for both of its products
    with ard.batch():
        W2c = ard.compact_weight(W2, p2, p1)
        Y1 = ard.drop_gemm_fwd(X0, W1, p1, relu=True, flags=OUT, ws=ws[0])
    Y2 = ard.drop_gemm_fwd(Y1, W2c, p2, p1, relu=True, flags=IN | OUT | WC, I=H1, O=H2, ws=ws[0])
    with ard.batch():
        ard.drop_gemm_bwd_weight(dY, S2, None, p2, flags=IN | OUT, I=H2, O=O, out=dW3, ws=ws[1])
        Y3 = ard.drop_gemm_fwd(Y2, W3, None, p2, flags=IN, I=H2, O=O, ws=ws[0])
        dY2 = ard.drop_gemm_bwd_data(dY, W3, None, p2, relu_src=S2, flags=IN | OUT, I=H2, O=O, ws=ws[2])
    with ard.batch():
        ard.drop_gemm_bwd_weight(dY2, S1, p2, p1, flags=IN | OUT, I=H1, O=H2, out=dW2, ws=ws[1])
        dY1 = ard.drop_gemm_bwd_data(dY2, W2c, p2, p1, relu_src=S1, flags=IN | OUT | WC, I=H1, O=H2, ws=ws[0])
    ard.drop_gemm_bwd_weight(dY1, X0, p1, None, flags=OUT, I=I, O=H1, out=dW1, ws=ws[0])
    return dict(Y1=Y1, Y2=Y2, Y3=Y3, dY1=dY1, dY2=dY2, dW1=dW1, dW2=dW2, dW3=dW3)


# ---- an LSTM layer ------------------------------------------------------------------------------------

def _prepare_lstm(case, seed):
    x = _Inputs(case, seed)
    T, B, I, H = case["T"], case["B"], case["I"], case["H"]
    lim = 1.0 / math.sqrt(H)
    n = ard.lstm_workspace_bytes(_code(case), T, B, I, H, _pattern(case, case["dp"], 1))
    f32 = dict(dtype=torch.float32, device="cuda")
    return dict(x=x.normal((T, B, I)), W=x.uniform((4 * H, I + H), -lim, lim), dh=x.normal((T, B, H)), ws=_bytes(n), b=1 + seed % case["dp"],
                out=(torch.empty((T, B, H), dtype=x.dtype, device="cuda"), torch.empty((T, B, H), **f32), torch.empty((T, B, 4 * H), **f32)),
                grads=(torch.empty((T, B, I), dtype=x.dtype, device="cuda"), torch.empty((4 * H, I + H), dtype=x.dtype, device="cuda")))


def _run_lstm(s, case):
    pat = _pattern(case, case["dp"], s["b"])
    h, c, gates = ard.lstm_fwd(s["x"], s["W"], pat, ws=s["ws"], out=s["out"])
    dx, dW = ard.lstm_bwd(s["x"], s["W"], pat, h, c, gates, s["dh"], ws=s["ws"], out=s["grads"])
    return dict(h=h, c=c, gates=gates, dx=dx, dW=dW)


# ---- convolution layers -------------------------------------------------------------------------------

def _prepare_conv(case, seed):
    x = _Inputs(case, seed)
    N, C, S, Co, k = case["N"], case["C"], case["S"], case["Cout"], case["k"]
    n = ard.conv_workspace_bytes(_code(case), N, C, S, S, Co, k, k, 1, k // 2)
    new = lambda *shape: torch.empty(shape, dtype=x.dtype, device="cuda")
    return dict(A=x.relu_normal((N, C, S, S)), Wt=x.normal((Co, C, k, k), math.sqrt(2.0 / (C * k * k))), dY=x.normal((N, Co, S, S)), ws=_bytes(n),
                Y=new(N, Co, S, S), dA=new(N, C, S, S), dWt=new(Co, C, k, k))


def _reuse(case, n_keep=1):
    """The weight gradient takes the grids that the two passes before it left in the workspace (bf16)."""
    return ard.CONV_REUSE_A | ard.CONV_REUSE_DY if case["dtype"] == "bf16" and n_keep > 0 else 0


def _run_conv(s, case):
    A, Wt, dY, ws, k = s["A"], s["Wt"], s["dY"], s["ws"], case["k"]
    n_keep = case["C"] - int(math.floor(case["rate"] * case["C"]))
    sel = ard.conv_select(A, case["rate"], Cout=case["Cout"], ksize=(k, k), pad=k // 2, ws=ws)
    Y = ard.conv_fwd(A, Wt, sel["keep"], n_keep, pad=k // 2, ws=ws, out=s["Y"])
    dA = ard.conv_bwd_data(dY, Wt, sel["keep"], n_keep, A.shape[2:], pad=k // 2, ws=ws, out=s["dA"])
    dWt = ard.conv_bwd_weight(dY, A, sel["keep"], n_keep, ksize=(k, k), pad=k // 2, ws=ws, out=s["dWt"], reuse=_reuse(case, n_keep))
    return dict(mask=sel["mask"], keep=sel["keep"], count=sel["count"], score=sel["score"], Y=Y, dA=dA, dWt=dWt)


# k = 30 % sampled, threshold 0.5, t = 50 %, possibilities 0.3 / 0.7, as in bench.py
_K, _T, _THRESHOLD, _M, _N = 300, 500, 0.5, 0.3, 0.7


def _run_rows(s, case):
    A, Wt, dY, ws, x, k = s["A"], s["Wt"], s["dY"], s["ws"], case["x"], case["k"]
    pred = ard.sens_predict(A, (k, k), 1, k // 2, x, 0, _K, _T, _THRESHOLD, s["seed"], 0)
    pat = ard.sens_row_pattern(pred["sens"], case["S"] * case["S"], x, _M, _N, s["seed"], 0)
    n_keep = int(pat["count"].item())   # the launch sizes of the forward pass depend on it
    Y = ard.conv_fwd_rows(A, Wt, pat, n_keep, pad=k // 2, ws=ws, out=s["Y"])
    dA, dWt = ard.conv_bwd_rows(dY, A, Wt, pat, pad=k // 2, ws=ws, out=(s["dA"], s["dWt"]), reuse=_reuse(case, n_keep))
    return dict(drawn=pred["count"], sens=pred["sens"], mask=pat["mask"], keep=pat["keep"], count=pat["count"], Y=Y, dA=dA, dWt=dWt)


def _run_blocks(s, case):
    A, Wt, dY, ws, x, k = s["A"], s["Wt"], s["dY"], s["ws"], case["x"], case["k"]
    y = 64 * k * k
    pred = ard.sens_predict(A, (k, k), 1, k // 2, x, y, _K, _T, _THRESHOLD, s["seed"], 0)
    pat = ard.sens_block_pattern(pred, True, _M, _N, s["seed"], 0)
    Y = ard.conv_fwd_blocks(A, Wt, pat["keep"], x, y, pad=k // 2, ws=ws, out=s["Y"])
    dA, dWt = ard.conv_bwd_blocks(dY, A, Wt, pat["keep"], x, y, pad=k // 2, ws=ws, out=(s["dA"], s["dWt"]))
    return dict(drawn=pred["count"], sens=pat["sens"], keep=pat["keep"], Y=Y, dA=dA, dWt=dWt)


_PREPARE = dict(layer=_prepare_layer, mlp=_prepare_mlp, lstm=_prepare_lstm, conv=_prepare_conv, rows=_prepare_conv, blocks=_prepare_conv)
_RUN = dict(layer=_run_layer, mlp=_run_mlp, lstm=_run_lstm, conv=_run_conv, rows=_run_rows, blocks=_run_blocks)


# ---- what a pass cannot do without --------------------------------------------------------------------

def work(case):
    """Operations of the kept part of the products; every input read once (its kept part, where the pattern
    is known before it is read) and every output written once, zeros included."""
    e = 4 if case["dtype"] == "f32" else 2
    f = case["family"]
    if f == "layer":
        B, I, O = case["B"], case["I"], case["O"]
        if case["pattern"] == "tile":
            o, i, w = O, I, O * I / case["dp"]
        else:
            o, i = -(-O // case["dp"]), -(-I // case["dp_in"])
            w = o * i
        return dict(flops=6.0 * B * w, bytes=float(e * (B * i + w + B * o + B * O + B * I + O * I)))
    if f == "mlp":
        B, I, O, dp, dp2 = case["B"], case["I"], case["O"], case["dp"], case["dp2"]
        if case["pattern"] == "tile":
            h1, h2, w = case["H1"], case["H2"], (case["H1"] * I / dp, case["H2"] * case["H1"] / dp2, O * case["H2"])
        else:
            h1, h2 = -(-case["H1"] // dp), -(-case["H2"] // dp2)
            w = (h1 * I, h2 * h1, O * h2)
        full = case["H1"] * I + case["H2"] * case["H1"] + O * case["H2"]
        return dict(flops=2.0 * B * (2 * w[0] + 3 * w[1] + 3 * w[2]),
                    bytes=float(e * (B * I + sum(w) + B * O + B * (h1 + h2)   # X0, weights, loss gradient, saved activations
                                     + 2 * B * (h1 + h2) + B * O + full)))    # activations, their gradients, weight gradients
    if f == "lstm":
        T, B, I, H, dp = case["T"], case["B"], case["I"], case["H"], case["dp"]
        if case["pattern"] == "tile":
            k, w = H, 4 * H * (I + H) / dp
        else:
            k = -(-H // dp)
            w = 4 * k * (I + k)
        return dict(flops=6.0 * T * B * w, bytes=float(e * (2 * T * B * I + w + T * B * k + T * B * H + 4 * H * (I + H)) + 4 * T * B * 5 * H))
    N, C, S, Co, k = case["N"], case["C"], case["S"], case["Cout"], case["k"]
    kept = 1.0 - case["rate"] if f == "conv" else 1.0 - _N   # rows and blocks: hardly a band of these inputs is sensitive
    return dict(flops=6.0 * N * S * S * Co * C * k * k * kept, bytes=float(e * (2 * N * C * S * S + 2 * N * Co * S * S + 2 * Co * C * k * k)))


def tolerance(case):
    """Sums of 32-bit products in another order, stored in 32 bits or rounded to bf16 (an LSTM's state is
    rounded at every step).  Masks, lists and counts are whole numbers and exact."""
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
