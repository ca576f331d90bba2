"""The bfloat16 GEMM's tiles (csrc/gemm_bf16.h) through the dense FFN and the
layers, at the sizes where they can go wrong: one row, one tile and one more
row, rows, widths and k that end inside a tile or a stage, grouped rows, and
each tile (test_gemm_bf16_host.py checks which tiles the sizes select)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_28516_amd import clearmoe as cm
from paper_2606_28516_amd import synth
from tests.parity_util import BF16_FROB_REGRESS, assert_routing, frob_rel, gpu_ffn

pytestmark = pytest.mark.gpu

SIZES = [
    # T, D (k of fc1, columns of fc2), H
    (1, 8, 8),                # smallest
    (64, 64, 64), (65, 72, 72),
    (197, 384, 1536),
    (320, 200, 1560),
    (1000, 384, 1544),
    (3152, 768, 3072),
    (6304, 136, 1032),
    (16384, 96, 1536),        # 768 tiles of 256 x 128: the two-workgroup fc1 tile
    (16421, 96, 1528),        # ... with short last row and column tiles
    (16129, 64, 1536),        # ... one k stage, one row in the last row tile
    (8449, 320, 2944),        # ... an odd number of k stages
    (8192, 1032, 3072),       # ... a last stage of 8 k
    (16003, 1032, 1032),      # 320 x 256 twice, with short last tiles and a last stage of 8 k
    (9003, 520, 1544),        # 256 x 256 with short last tiles
    (2001, 264, 1032),        # fc1 on the deeper 128 x 128 tiles
]


@pytest.mark.parametrize("T,D,H", SIZES)
def test_dense_ffn_tiles(T, D, H):
    g = torch.Generator(device="cuda").manual_seed(T * 31 + D)
    n = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, W1, W2 = n(T, D).bfloat16(), (n(H, D) / D ** 0.5).bfloat16(), (n(D, H) / H ** 0.5).bfloat16()
    b1, b2 = 0.1 * n(H), 0.1 * n(D)
    y = cm.dense_ffn_forward(x, W1, b1, W2, b2).double()
    z = torch.nn.functional.gelu(x.double() @ W1.double().T + b1.double())
    ref = z @ W2.double().T + b2.double()
    # y is rounded once (2^-9 of itself) from a sum over z rounded to bf16
    # (2^-9 of each |z w|; twice that where the float32 z lands on the other
    # side of a tie), plus float32 sums, far below either
    bound = 2.0 ** -8 * (ref.abs() + z.abs() @ W2.double().abs().T) + 1e-6
    assert (y - ref).abs().le(bound).all()
    # the roundings are independent: over the whole result they stay near
    # sqrt(2) 2^-9 / sqrt(3), well under 2^-8
    assert ((y - ref).norm() / ref.norm()).item() <= 2.0 ** -8


# one product of each tile: rows, columns, k; the tile its size selects
TILES = [
    (70, 72, 272),            # 64 x 64
    (4000, 1544, 272),        # 128 x 128
    (2000, 1032, 520),        # 128 x 128, deeper pipeline
    (8000, 1544, 272),        # 256 x 256
    (16000, 1032, 272),       # 320 x 256
    (16000, 1544, 272),       # with a GELU: 256 x 128, two workgroups on a CU
]


@pytest.mark.parametrize("product", ["fc1", "fc2"])
@pytest.mark.parametrize("M,N,K", TILES)
def test_bias_is_added_to_the_finished_sum(M, N, K, product):
    """A sum of 256 terms 2^-6 and, last in k, 2^24, plus a bias of -2^24: every
    partial sum is a float32 value (4 after the small terms, 2^24 + 4 with the
    large one), so the result is 4, exactly, where the bias is added last.
    Next to a bias that comes first, -2^24, each 16 k's quarter is lost."""
    dev = dict(device="cuda")
    if product == "fc1":
        x = torch.ones(M, K, **dev)
        x[:, 256:] = 0
        x[:, -1] = 2.0 ** 12
        W1 = torch.full((N, K), 2.0 ** -6, **dev)
        W1[:, -1] = 2.0 ** 12
        b1, b2 = torch.full((N,), -2.0 ** 24, **dev), torch.zeros(K, **dev)
        h = torch.arange(N, **dev)
        W2 = (h % K == torch.arange(K, **dev)[:, None]).float()      # [K, N]: sums of whole z columns
        want = (4.0 * W2.sum(1)).expand(M, K)                        # GELU(4) rounds to 4
    else:
        # z = 8 in 256 hidden units, 2^12 in the last one (GELU(v) = v there)
        x, W1 = torch.zeros(M, N, **dev), torch.zeros(K, N, **dev)
        b1 = torch.zeros(K, **dev)
        b1[:256] = 8.0
        b1[-1] = 2.0 ** 12
        W2 = torch.full((N, K), 2.0 ** -9, **dev)
        W2[:, -1] = 2.0 ** 12
        b2 = torch.full((N,), -2.0 ** 24, **dev)
        want = torch.full((M, N), 4.0, **dev)
    y = cm.dense_ffn_forward(x.bfloat16(), W1.bfloat16(), b1, W2.bfloat16(), b2)
    assert torch.equal(y.float(), want)


@pytest.mark.parametrize("T,D,H,E,k,r,q", [
    (300, 128, 1024, 4, 1, 40, 0),      # top-1 products without residual columns, N inside a tile
    (300, 128, 1024, 4, 1, 0, 24),      # ... without basis columns
    (300, 128, 1024, 4, 2, 40, 0),      # pair order
    (300, 128, 1024, 4, 2, 0, 24),
    (9001, 520, 1032, 4, 2, 392, 0),    # ... over 256-wide tiles
])
def test_layers_with_an_empty_part(T, D, H, E, k, r, q):
    cfg = synth.LayerConfig("part", T=T, D=D, H=H, E=E, k=k, r=r, q=q, dtype="bf16", seed=T + r + q,
                            residual="random", n_cal=2000)
    L = synth.make_layer(cfg)
    out = gpu_ffn(L)
    rows = np.unique(np.random.default_rng(3).integers(0, T, 400))
    tie = assert_routing(out["idx"], oracle.route(L["x"], L["Wg"], L["bg"], k)[2], k)
    rows = rows[~tie[rows]]
    ref = oracle.ffn_forward_layer(L, rows=rows)["y"]
    assert frob_rel(out["y"][rows], ref) <= BF16_FROB_REGRESS


@pytest.mark.parametrize("T,D,H,stride", [
    (2900, 520, 3072, 700),      # five class rows of z 4.3 MB apart: 512 of them would span 2 GiB
    (6000, 1544, 1032, 2999),    # three of them, 6.2 MB apart
])
def test_class_rows_far_apart(T, D, H, stride):
    """Class tokens with a large stride on the product chain: the dense FFN's
    output in their rows, the routed layer's in the others."""
    cfg = synth.LayerConfig("far", T=T, D=D, H=H, E=4, k=1, r=40, q=24, dtype="bf16", seed=T, residual="random",
                            n_cal=2000)
    L = synth.make_layer(cfg)
    rng = np.random.default_rng(T)
    W2 = synth.to_bf16_bits((rng.standard_normal((D, H)) / H ** 0.5).astype(np.float32))
    d = {n: cm.from_stored(v) for n, v in dict(L, W2=W2).items()
         if n in ("x", "W1", "b1", "US", "Vt", "b2", "P", "Q", "Wg", "bg", "W2")}
    w = [d[n] for n in ("x", "W1", "b1", "US", "Vt", "b2", "P", "Q")]
    y = cm.ffn_forward_ex(*w, cm.make_router(d["Wg"], d["bg"], dense_stride=stride, W2=d["W2"]), 1)
    plain = cm.ffn_forward_ex(*w, cm.make_router(d["Wg"], d["bg"]), 1)
    cls = torch.arange(0, T, stride, device="cuda")
    rest = torch.ones(T, dtype=torch.bool, device="cuda")
    rest[cls] = False
    assert torch.equal(y[rest], plain[rest])
    z = torch.nn.functional.gelu(d["x"][cls].double() @ d["W1"].double().T + d["b1"].double())
    ref = z @ d["W2"].double().T + d["b2"].double()
    # as in test_dense_ffn_tiles: y rounded once from a sum over rounded z
    bound = 2.0 ** -8 * (ref.abs() + z.abs() @ d["W2"].double().abs().T) + 1e-6
    assert (y[cls].double() - ref).abs().le(bound).all()


@pytest.mark.parametrize("T", [3, 16, 40])
def test_dense_ffn_with_weights_of_2_gib(T):
    """Weights past the loads' 32-bit offsets: the general kernel, with 64 x 128
    tiles for few rows and 256 x 128 ones for more."""
    D, H = 16384, 65536
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(T, D, device="cuda", generator=g).bfloat16()
    W1 = torch.empty(H, D, device="cuda", dtype=torch.bfloat16).normal_(0, D ** -0.5, generator=g)
    W2 = torch.empty(D, H, device="cuda", dtype=torch.bfloat16).normal_(0, H ** -0.5, generator=g)
    b1, b2 = 0.1 * torch.randn(H, device="cuda", generator=g), 0.1 * torch.randn(D, device="cuda", generator=g)
    y = cm.dense_ffn_forward(x, W1, b1, W2, b2).double()
    z = torch.nn.functional.gelu(x.double() @ W1.double().T + b1.double())
    W2 = W2.double()
    ref = z @ W2.T + b2.double()
    # as in test_dense_ffn_tiles
    bound = 2.0 ** -8 * (ref.abs() + z.abs() @ W2.abs().T) + 1e-6
    assert (y - ref).abs().le(bound).all()
    assert ((y - ref).norm() / ref.norm()).item() <= 2.0 ** -8


@pytest.mark.parametrize("k,r,q", [(1, 40, 24), (1, 136, 24), (2, 136, 24)])
def test_layers_with_z_of_2_gib(k, r, q):
    """z [T, H] past the loads' 32-bit offsets: the [t|u] products gather its
    rows with the general kernel (128 x 64 and 256 x 128 tiles, grouped, scaled
    columns, parts of B), the others stay with the bfloat16 kernels."""
    T, D, H, E = 16421, 144, 65536, 4
    g = torch.Generator(device="cuda").manual_seed(r + k)
    n = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, W1, b1, b2 = n(T, D).bfloat16(), (n(H, D) / D ** 0.5).bfloat16(), 0.1 * n(H), 0.1 * n(D)
    US, Vt = (n(D, r) / r ** 0.5).bfloat16(), (n(r, H) / H ** 0.5).bfloat16()
    P, Q = (n(E, D, q) / q ** 0.5).bfloat16(), (n(E, q, H) / H ** 0.5).bfloat16()
    Wg, bg = (n(E, D) / D ** 0.5).bfloat16(), 0.1 * n(E)
    idx = torch.empty(T, k, device="cuda", dtype=torch.int32)
    gate = torch.empty(T, k, device="cuda")
    y = cm.ffn_forward(x, W1, b1, US, Vt, b2, P, Q, Wg, bg, k, idx_out=idx, gate_out=gate)
    rows = torch.cat([torch.arange(0, T, 41, device="cuda"), torch.arange(T - 40, T, device="cuda")]).unique()
    ref = _layer_rows(rows, x, W1, b1, US, Vt, b2, P, Q, idx, gate)
    err = (y[rows].double() - ref).norm() / ref.norm()
    assert err.item() <= BF16_FROB_REGRESS


def _layer_rows(rows, x, W1, b1, US, Vt, b2, P, Q, idx, gate):
    """Rows of the layer in 64 bits, with the experts and gates given."""
    z = torch.nn.functional.gelu(x[rows].double() @ W1.double().T + b1.double())
    ref = (z @ Vt.double().T) @ US.double().T + b2.double()
    for j in range(idx.shape[1]):
        for e in range(P.shape[0]):
            at = (idx[rows, j] == e).nonzero().flatten()
            u = gate[rows[at], j:j + 1].double() * (z[at] @ Q[e].double().T)
            ref[at] += u @ P[e].double().T
    return ref


GROUPED = [
    # T, D, H, E, r, q; tiles of the y products (split along k, rows scattered)
    # and of the pair order's [t|u_a|u_b] (parts along n, scaled, rows gathered)
    (11003, 1032, 520, 4, 136, 24, "320", "128 deep"),
    (20011, 776, 520, 4, 264, 72, "128", "256 long"),
]


@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("T,D,H,E,r,q", [c[:6] for c in GROUPED])
def test_grouped_products_on_tall_tiles(T, D, H, E, r, q, k):
    g = torch.Generator(device="cuda").manual_seed(T + k)
    n = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, W1, b1, b2 = n(T, D).bfloat16(), (n(H, D) / D ** 0.5).bfloat16(), 0.1 * n(H), 0.1 * n(D)
    US, Vt = (n(D, r) / r ** 0.5).bfloat16(), (n(r, H) / H ** 0.5).bfloat16()
    P, Q = (n(E, D, q) / q ** 0.5).bfloat16(), (n(E, q, H) / H ** 0.5).bfloat16()
    Wg, bg = (n(E, D) / D ** 0.5).bfloat16(), 0.1 * n(E)
    idx = torch.empty(T, k, device="cuda", dtype=torch.int32)
    gate = torch.empty(T, k, device="cuda")
    y = cm.ffn_forward(x, W1, b1, US, Vt, b2, P, Q, Wg, bg, k, idx_out=idx, gate_out=gate)
    rows = torch.arange(T, device="cuda")
    ref = _layer_rows(rows, x, W1, b1, US, Vt, b2, P, Q, idx, gate)
    err = (y.double() - ref).norm(dim=1) / ref.norm(dim=1)      # every row of every segment
    assert err.max().item() <= BF16_FROB_REGRESS
    # and with the skip connection in the y product
    layer = cm.make_stack_layer(W1, b1, b2, US=US, Vt=Vt, P=P, Q=Q, router=cm.make_router(Wg, bg), k=k)
    skip = cm.stack_forward(x, [layer], H, E, r, q, residual=True)
    assert torch.equal(skip, (x.float() + y.float()).bfloat16())
