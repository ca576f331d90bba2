"""The work that a program gives this library, as cases to time and compare.

Each case is one call sequence of `paper_2606_28516_amd.clearmoe` as a vision
transformer's host program makes it: a whole CLEAR-MoE FFN layer with one of
its routers, the dense FFN, a chained stack of layers, the padded-batch
backend, or the route / dispatch / combine steps around experts of the
caller's own.  Shapes are the DeiT widths of the repository's benchmark and
tests, one image up to 256 images of 197 tokens, and ragged ones beside them.

Inputs follow the benchmark's recipe, drawn on the GPU: tokens from a
Gaussian mixture (centres of norm 3, unit noise), router rows near the
centres, N(0, 0.02^2) fc1 / fc2 weights, and for the factors what a truncated
SVD of such an fc2 looks like: rows of Vt and Q of norm 1, columns of US and P
with singular values falling over the rank.
"""
import math

import torch

from paper_2606_28516_amd import clearmoe as cm

IMAGE = 197          # tokens of one 224 x 224 image: 196 patches and the class token


def _layer(name, T, D, H, E, k, r, q, dtype="bf16", router="linear", tau=0.9, hidden=0, stride=0,
           skew=0.0, backend="grouped"):
    return dict(name=name, kind="layer", T=T, D=D, H=H, E=E, k=k, r=r, q=q, dtype=dtype,
                router=router, tau=tau, hidden=hidden, stride=stride, skew=skew, backend=backend)


def listed():
    return [
        # one image through a DeiT-Small-shaped layer: interactive serving,
        # where launches and latency are the whole cost
        _layer("small-top1-1image", IMAGE, 384, 1536, 8, 1, 128, 32),
        # DeiT-Tiny-shaped layer in float32, eight images: the type in which
        # the paper's own models are calibrated and checked
        _layer("tiny-top1-f32", 8 * IMAGE, 192, 768, 4, 1, 64, 16, dtype="f32"),
        # the paper's dispatch micro-benchmark: eight images without class
        # tokens, four experts, top-2, a skewed load
        _layer("small-top2-8images", 8 * 196, 384, 1536, 4, 2, 128, 32, skew=0.4),
        # DeiT-Small-shaped layer, a batch of 64 images: offline inference
        _layer("small-top1-64images", 64 * IMAGE, 384, 1536, 8, 1, 128, 32),
        # the adaptive router (top-1, escalated to top-2 below a confidence)
        _layer("small-adaptive-64images", 64 * IMAGE, 384, 1536, 8, 2, 128, 32, router="adaptive"),
        # the MLP router, with the class tokens on the dense path
        _layer("small-mlp-classtok", 64 * IMAGE, 384, 1536, 8, 1, 128, 32, router="mlp", hidden=64,
               stride=IMAGE),
        # widths and a token count that are no multiples of anything (a pruned
        # model): the generic path on padded copies
        _layer("ragged-top2", 5003, 390, 1550, 6, 2, 100, 27, skew=0.2),
        # the padded-batch backend at the micro-benchmark's larger batch
        _layer("small-top2-padded", 64 * IMAGE, 384, 1536, 4, 2, 128, 32, skew=0.4, backend="padded"),
        # DeiT-Base-shaped layer, 256 images, top-2: the benchmark's headline
        _layer("base-top2-256images", 256 * IMAGE, 768, 3072, 8, 2, 256, 64, skew=0.2),
        # the dense FFN of a DeiT-Base-shaped block, 128 images: the blocks
        # that are not expertised, and what the layer is compared with
        dict(name="base-dense-128images", kind="dense", T=128 * IMAGE, D=768, H=3072, dtype="bf16"),
        # twelve chained DeiT-Small-shaped FFN blocks with the skip connection,
        # the last six CLEAR-MoE with class tokens on the dense path
        dict(name="small-stack-64images", kind="stack", T=64 * IMAGE, D=384, H=1536, E=8, r=128,
             q=32, blocks=12, stride=IMAGE, dtype="bf16"),
        # route, dispatch with rows, gated combine over a million tokens:
        # expert parallelism around the caller's own experts
        dict(name="dispatch-1M", kind="dispatch", T=1 << 20, D=384, E=8, k=2, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["layer"] * 6 + ["f32", "adaptive", "mlp", "ragged", "padded", "dense", "stack",
                       "dispatch"])
    D = rng.choice([192, 384, 384, 768])
    if rng.random() < 0.2:                       # a width in between, whole 16-byte rows
        D = 8 * rng.randint(24, 96)
    H = 4 * D
    E = rng.choice([2, 3, 4, 6, 8])
    r = 32 * max(1, D // 96)                     # a third of the width
    q = 8 * max(1, r // 32)
    # the largest token count that costs no more than the headline case
    most = max(IMAGE, min(256 * IMAGE, int(256 * IMAGE * (768 / D) ** 2 * 0.9)))
    T = _log_int(rng, 64, most)
    skew = round(rng.choice([0.0, 0.2, 0.4, 0.6]), 2)
    k = min(E, rng.choice([1, 1, 2]))
    if kind == "layer":
        c = _layer("", T, D, H, E, k, r, q, skew=skew, stride=rng.choice([0, 0, IMAGE]))
    elif kind == "f32":
        c = _layer("", _log_int(rng, 64, 64 * IMAGE), 192, 768, E, k, 64, 16, dtype="f32", skew=skew)
    elif kind == "adaptive":
        c = _layer("", T, D, H, E, 2, r, q, router="adaptive", tau=round(rng.uniform(0.7, 0.97), 3),
                   skew=skew)
    elif kind == "mlp":
        c = _layer("", min(T, 128 * IMAGE), D, H, E, k, r, q, router="mlp", hidden=8 * max(1, D // 48), skew=skew,
                   stride=rng.choice([0, IMAGE]))
    elif kind == "ragged":
        D = rng.randint(150, 500)
        r = rng.randint(40, D // 3)
        c = _layer("", _log_int(rng, 64, 64 * IMAGE), D, 4 * D - rng.randint(0, 30), E, k, r,
                   max(1, r // 4), skew=skew)
    elif kind == "padded":
        c = _layer("", min(T, 64 * IMAGE), D, H, E, k, r, q, skew=skew, backend="padded")
    elif kind == "dense":
        c = dict(name="", kind="dense", T=T, D=D, H=H, dtype="bf16")
    elif kind == "stack":
        c = dict(name="", kind="stack", T=min(T, 64 * IMAGE), D=D, H=H, E=E, r=r, q=q,
                 blocks=rng.choice([2, 4, 6]), stride=rng.choice([0, IMAGE]), dtype="bf16")
    else:
        c = dict(name="", kind="dispatch", T=_log_int(rng, 1 << 10, 1 << 19), D=D, E=E, k=k,
                 dtype=rng.choice(["bf16", "f32"]))
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed))

    def n(self, *shape):
        return torch.randn(*shape, device="cuda", generator=self.g)


def _tokens(gen, T, D, E, skew):
    """Mixture tokens [T, D] and the cluster centres [E, D]: a share `skew` of
    the tokens from cluster 0 on top of an even spread."""
    c = gen.n(E, D)
    c = 3.0 * c / c.norm(dim=1, keepdim=True)
    w = torch.full((E,), (1.0 - skew) / E, device="cuda")
    w[0] += skew
    lab = torch.multinomial(w, T, replacement=True, generator=gen.g)
    return gen.n(T, D) + c[lab], c


def _factors(gen, D, H, rank):
    """What the SVD of an N(0, 0.02^2) fc2 [D, H] gives: U S [D, rank], V^T
    [rank, H], singular values falling from the largest."""
    top = 0.02 * (math.sqrt(H) + math.sqrt(D))
    s = torch.linspace(top, 0.6 * top, rank, device="cuda") if rank else torch.empty(0, device="cuda")
    return gen.n(D, rank) / math.sqrt(D) * s, gen.n(rank, H) / math.sqrt(H)


def _moe_weights(gen, D, H, E, r, q, dt, differ):
    """One layer's weights.  differ: experts with factors of their own; else
    the shared tail scaled per expert, as the extraction makes them."""
    w = dict(W1=0.02 * gen.n(H, D), b1=0.02 * gen.n(H), b2=0.02 * gen.n(D), W2=0.02 * gen.n(D, H))
    w["US"], w["Vt"] = _factors(gen, D, H, r)
    if differ:
        pq = [_factors(gen, D, H, q) for _ in range(E)]
        w["P"], w["Q"] = torch.stack([a for a, _ in pq]), torch.stack([b for _, b in pq])
    else:
        a, b = _factors(gen, D, H, q)
        s = 1.0 + 0.02 * gen.n(E, 1, 1)
        w["P"], w["Q"] = s * a, b.expand(E, q, H)
    return {n: (t.float() if n in ("b1", "b2") else t.to(dt)).contiguous() for n, t in w.items()}


def _linear(gen, c, dt):
    return (c + 0.1 * gen.n(*c.shape)).to(dt), 0.1 * gen.n(c.shape[0])


def prepare(case, seed):
    gen, dt, T, D = _Gen(seed), _dt(case), case["T"], case["D"]
    st = dict(case=case)
    if case["kind"] == "dense":
        H = case["H"]
        st.update(x=gen.n(T, D).to(dt), W1=(0.02 * gen.n(H, D)).to(dt), b1=0.02 * gen.n(H),
                  W2=(0.02 * gen.n(D, H)).to(dt), b2=0.02 * gen.n(D))
        st["ws"] = cm.alloc_workspace(cm.make_shape(T, D, 1, 1, cm._dt(st["x"]), H=H))
        return st
    E = case["E"]
    x, c = _tokens(gen, T, D, E, case.get("skew", 0.0))
    st["x"] = x.to(dt)
    del x
    code = cm._dt(st["x"])
    if case["kind"] == "dispatch":
        # a router bias of Zipf(1.2) weights skews the expert load
        p = torch.arange(1, E + 1, device="cuda", dtype=torch.float32) ** -1.2
        st["Wg"], _ = _linear(gen, c, dt)
        st["bg"] = torch.log(p / p.sum())
        st["ws"] = cm.alloc_workspace(cm.make_shape(T, D, E, case["k"], code))
        return st
    H, r, q = case["H"], case["r"], case["q"]
    if case["kind"] == "stack":
        keep, layers = [], []
        for b in range(case["blocks"]):
            w = _moe_weights(gen, D, H, E, r, q, dt, False)
            if b < case["blocks"] // 2:
                layers.append(cm.make_stack_layer(w["W1"], w["b1"], w["b2"], W2=w["W2"]))
            else:
                w["Wg"], w["bg"] = _linear(gen, c, dt)
                rt = cm.make_router(w["Wg"], w["bg"], dense_stride=case["stride"],
                                    W2=w["W2"] if case["stride"] else None)
                layers.append(cm.make_stack_layer(w["W1"], w["b1"], w["b2"], US=w["US"], Vt=w["Vt"],
                                                  P=w["P"], Q=w["Q"], router=rt, k=1, W2=w["W2"]))
            keep.append(w)
        st.update(layers=layers, weights=keep)
        n = cm.stack_workspace_bytes(cm.stack_shape(st["x"], H, E, r, q), layers)
        st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return st
    st.update(_moe_weights(gen, D, H, E, r, q, dt, True))
    st["Wg"], st["bg"] = _linear(gen, c, dt)
    if case["router"] == "mlp":
        # hidden units along the linear router's rows, the rest random; the
        # output layer reads unit e for expert e
        h = max(case["hidden"], E)
        lin = st["Wg"].float()
        Wh = gen.n(h, D) / math.sqrt(D)
        Wh[:E] = lin / lin.norm(dim=1, keepdim=True)
        Wo = 0.05 * gen.n(E, h)
        Wo[torch.arange(E), torch.arange(E)] += 2.0
        st.update(Wh=Wh.to(dt), bh=0.02 * gen.n(h), Wg=Wo.to(dt))
    st["linear"] = case["router"] == "linear" and case["stride"] == 0
    if not st["linear"]:
        st["router"] = cm.make_router(st["Wg"], st["bg"], st.get("Wh"), st.get("bh"),
                                      adaptive=case["router"] == "adaptive", tau=case["tau"],
                                      dense_stride=case["stride"],
                                      W2=st["W2"] if case["stride"] else None)
    shape = cm.make_shape(T, D, E, case["k"], code, H=H, r=r, q=q)
    if case["backend"] == "padded":
        st["ws"] = torch.empty(cm.padded_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    else:
        st["ws"] = cm.alloc_workspace(shape)
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    if case["kind"] == "dense":
        return cm.dense_ffn_forward(st["x"], st["W1"], st["b1"], st["W2"], st["b2"], ws=st["ws"])
    if case["kind"] == "stack":
        return cm.stack_forward(st["x"], st["layers"], case["H"], case["E"], case["r"], case["q"],
                                ws=st["ws"])
    if case["kind"] == "dispatch":
        idx, gate = cm.route(st["x"], st["Wg"], st["bg"], case["k"], ws=st["ws"])
        counts, offsets, perm, inv, xperm = cm.dispatch(idx, case["E"], ws=st["ws"], x=st["x"],
                                                        hist_in_ws=True)
        # the experts would run on xperm here
        y = cm.combine(xperm, inv, gate)
        return dict(idx=idx, gate=gate, counts=counts, offsets=offsets, perm=perm, inv=inv,
                    xperm=xperm, y=y)
    w = (st["x"], st["W1"], st["b1"], st["US"], st["Vt"], st["b2"], st["P"], st["Q"])
    if case["backend"] == "padded":
        return cm.ffn_forward_padded(*w, st["Wg"], st["bg"], case["k"], ws=st["ws"])
    if st["linear"]:
        return cm.ffn_forward(*w, st["Wg"], st["bg"], case["k"], ws=st["ws"])
    return cm.ffn_forward_ex(*w, st["router"], case["k"], ws=st["ws"])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _layer_work(T, D, H, E, k, r, q, b, cls, hidden):
    moe = T - cls
    rq = r + k * q
    flops = 2.0 * T * D * H + 2.0 * moe * rq * (H + D) + 2.0 * cls * H * D
    flops += 2.0 * T * D * (hidden or E) + 2.0 * T * hidden * E
    by = b * (2.0 * T * D + H * D + r * (H + D) + E * q * (H + D) + D * (hidden or E) + hidden * E)
    by += 4.0 * (H + D + E) + (b * D * H if cls else 0)
    return by, flops


def work(case):
    b = 4 if case["dtype"] == "f32" else 2
    T, D = case["T"], case["D"]
    if case["kind"] == "dense":
        H = case["H"]
        return dict(bytes=b * (2.0 * T * D + 2.0 * H * D) + 4.0 * (H + D), flops=4.0 * T * D * H)
    if case["kind"] == "dispatch":
        E, k = case["E"], case["k"]
        # x read once, xperm written, read back by the combine, y written;
        # idx, gate, perm and inv written once
        return dict(bytes=b * D * T * (2.0 + 2.0 * k) + 16.0 * T * k + b * E * D,
                    flops=2.0 * T * D * E + 2.0 * T * k * D)
    E, H, r, q = case["E"], case["H"], case["r"], case["q"]
    cls = -(-T // case["stride"]) if case["stride"] else 0
    if case["kind"] == "stack":
        n = case["blocks"]
        # x in, y out, every block's weights once
        dense = n // 2
        wm = _layer_work(T, D, H, E, 1, r, q, b, cls, 0)
        by = b * 2.0 * T * D + dense * (b * 2.0 * H * D + 4.0 * (H + D))
        by += (n - dense) * (wm[0] - b * 2.0 * T * D)
        return dict(bytes=by, flops=dense * 4.0 * T * D * H + (n - dense) * wm[1])
    k = 1 if case["router"] == "adaptive" else case["k"]     # at least one expert a token
    by, fl = _layer_work(T, D, H, E, k, r, q, b, cls, case["hidden"])
    return dict(bytes=by, flops=fl)


def tolerance(case):
    # About four times the relative error against 64 bits measured on an
    # MI355X: bf16 layers 2.9e-3 (the roundings of z, the projections and y),
    # the twelve-block stack 6.0e-3 (they travel through later blocks),
    # float32 layers 4.1e-7.
    if case["kind"] == "dispatch":
        # indices and copied rows are exact; gates (float32) and combined
        # rows (one rounding of an exact sum of two products) may round apart
        return dict(rel=4e-3 if case["dtype"] == "bf16" else 1e-6, max=0.01, differ=0.0)
    if case["dtype"] == "f32":
        return dict(rel=2e-6, max=3e-5)
    if case["kind"] == "stack":
        return dict(rel=2.4e-2, max=0.3)
    return dict(rel=1.2e-2, max=0.15)


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _gelu(v):
    return 0.5 * v * (1.0 + torch.erf(v / math.sqrt(2.0)))


def _topk(logits, k):
    """Experts by logit, largest first, ties to the lower index."""
    v, i = torch.sort(logits, dim=1, descending=True, stable=True)
    return i[:, :k], v[:, :k]


def _moe_exact(x, w, E, idx, gate, cls_rows):
    z = _gelu(x @ w["W1"].double().T + w["b1"].double())
    y = (z @ w["Vt"].double().T) @ w["US"].double().T + w["b2"].double()
    for j in range(idx.shape[1]):
        for e in range(E):
            s = (idx[:, j] == e).nonzero().flatten()
            if s.numel():
                u = gate[s, j:j + 1] * (z[s] @ w["Q"][e].double().T)
                y[s] += u @ w["P"][e].double().T
    if cls_rows is not None:
        y[cls_rows] = z[cls_rows] @ w["W2"].double().T + w["b2"].double()
    return y


def _route_exact(x, w, k, adaptive=False, tau=0.0, mlp=False, stride=0):
    if mlp:
        hr = _gelu(x @ w["Wh"].double().T + w["bh"].double()).to(w["Wh"].dtype).double()
        logits = hr @ w["Wg"].double().T + w["bg"].double()
    else:
        logits = x @ w["Wg"].double().T + w["bg"].double()
    idx, top = _topk(logits, k)
    gate = torch.softmax(top, dim=1)
    if adaptive:
        sure = torch.softmax(logits, dim=1).amax(dim=1) >= tau
        idx, gate = idx.clone(), gate.clone()
        idx[sure, 1] = -1
        gate[sure] = torch.tensor([1.0, 0.0], device="cuda", dtype=torch.float64)
    if stride:
        idx, gate = idx.clone(), gate.clone()
        idx[::stride] = -1
        gate[::stride] = 0.0
    return idx, gate


def exact(case, seed):
    st = prepare(case, seed)
    x = st["x"].double()
    if case["kind"] == "dense":
        z = _gelu(x @ st["W1"].double().T + st["b1"].double())
        return z @ st["W2"].double().T + st["b2"].double()
    if case["kind"] == "dispatch":
        T, k = case["T"], case["k"]
        idx, gate = _route_exact(x, st, k)
        flat = idx.reshape(-1)
        perm = torch.sort(flat, stable=True)[1]
        inv = torch.empty_like(perm)
        inv[perm] = torch.arange(T * k, device="cuda")
        counts = torch.bincount(flat, minlength=case["E"])
        offsets = torch.cat([counts.new_zeros(1), counts.cumsum(0)])
        y = x * gate.sum(1, keepdim=True)
        i32 = torch.int32
        return dict(idx=idx.to(i32), gate=gate, counts=counts.to(i32), offsets=offsets.to(i32),
                    perm=perm.to(i32), inv=inv.to(i32), xperm=st["x"][perm // k], y=y)
    E, stride = case["E"], case["stride"]
    rows = torch.arange(0, case["T"], stride, device="cuda") if stride else None
    if case["kind"] == "stack":
        for b, w in enumerate(st["weights"]):
            if b < case["blocks"] // 2:
                z = _gelu(x @ w["W1"].double().T + w["b1"].double())
                x = x + z @ w["W2"].double().T + w["b2"].double()
            else:
                idx, gate = _route_exact(x, w, 1, stride=stride)
                x = x + _moe_exact(x, w, E, idx, gate, rows)
        return x
    idx, gate = _route_exact(x, st, case["k"], case["router"] == "adaptive", case["tau"],
                             case["router"] == "mlp", stride)
    return _moe_exact(x, st, E, idx, gate, rows)
