"""The skip connection of a stack inside the layers' last kernels: for one
layer it is round(x + round(f)), bit for bit what a pass of its own would give,
over every path that adds it there and those that do not.  And the router's
choice at the widths where its lane count changes."""
import pytest
import torch

from paper_2606_28516_amd import clearmoe as cm

pytestmark = pytest.mark.gpu

CASES = [
    # kind, T, D, H, E, k, r, q, class stride, adaptive
    ("dense", 197, 384, 1536, 4, 1, 32, 8, 0, False),
    ("dense", 4099, 200, 808, 4, 1, 32, 8, 0, False),
    ("moe", 9001, 384, 1536, 8, 1, 128, 32, 197, False),    # fused, class rows in its launch
    ("moe", 9001, 384, 1536, 8, 1, 128, 32, 0, False),      # fused, a pass of its own
    ("moe", 300, 384, 1536, 8, 1, 128, 32, 50, False),      # fused with the hidden split
    ("moe", 1003, 520, 1032, 4, 1, 64, 24, 0, False),       # grouped products
    ("moe", 1003, 520, 1032, 4, 1, 64, 24, 100, False),
    ("moe", 777, 384, 1536, 4, 2, 128, 32, 0, False),       # pair order
    ("moe", 777, 384, 1536, 4, 2, 128, 32, 11, False),
    ("moe", 2000, 384, 1536, 4, 2, 128, 32, 197, True),     # adaptive: fused and pairs
    ("moe", 2000, 520, 1032, 4, 2, 64, 24, 197, True),      # adaptive: products only
    ("moe", 500, 128, 256, 16, 4, 32, 8, 0, False),         # the general path
    ("moe", 300, 128, 256, 4, 1, 0, 0, 0, False),           # no basis, no residual: y = x + b2
    ("moe", 300, 128, 256, 4, 1, 0, 0, 50, False),
    ("moe", 300, 128, 256, 4, 2, 0, 0, 0, False),
    ("moe", 300, 128, 256, 4, 2, 0, 0, 50, True),
]


@pytest.mark.parametrize("kind,T,D,H,E,k,r,q,stride,adaptive", CASES)
def test_skip_is_the_layer_plus_its_input(kind, T, D, H, E, k, r, q, stride, adaptive):
    g = torch.Generator(device="cuda").manual_seed(T + D)
    n = lambda *s: torch.randn(*s, device="cuda", generator=g)
    bf = lambda t: t.bfloat16().contiguous()
    x = bf(n(T, D))
    W1, b1, b2 = bf(n(H, D) / D ** 0.5), 0.1 * n(H), 0.1 * n(D)
    W2 = bf(n(D, H) / H ** 0.5)
    if kind == "dense":
        layers = [cm.make_stack_layer(W1, b1, b2, W2=W2)]
    else:
        US, Vt = bf(n(D, r) / r ** 0.5), bf(n(r, H) / H ** 0.5)
        P, Q = bf(n(E, D, q) / q ** 0.5), bf(n(E, q, H) / H ** 0.5)
        Wg, bg = bf(n(E, D) / D ** 0.5), 0.1 * n(E)
        rt = cm.make_router(Wg, bg, adaptive=adaptive, tau=0.5 if adaptive else 0.0,
                            dense_stride=stride, W2=W2 if stride else None)
        layers = [cm.make_stack_layer(W1, b1, b2, US=US, Vt=Vt, P=P, Q=Q, router=rt, k=k, W2=W2)]
    f = cm.stack_forward(x, layers, H, E, r, q, residual=False)
    y = cm.stack_forward(x, layers, H, E, r, q, residual=True)
    assert torch.isfinite(f.float()).all()
    assert torch.equal(y, (x.float() + f.float()).bfloat16())


@pytest.mark.parametrize("E", [2, 7, 8, 9, 16])
@pytest.mark.parametrize("T", [130, 70001])
def test_router_choice_by_expert_count(E, T):
    D, k = 136, 2
    g = torch.Generator(device="cuda").manual_seed(E * 7 + T)
    x = torch.randn(T, D, device="cuda", generator=g).bfloat16()
    Wg = torch.randn(E, D, device="cuda", generator=g).bfloat16()
    bg = torch.randn(E, device="cuda", generator=g)
    idx, gate = cm.route(x, Wg, bg, k)
    logits = x.double() @ Wg.double().T + bg.double()
    v, i = torch.sort(logits, dim=1, descending=True, stable=True)
    # the router promises the exact choice down to the rounding of a double sum
    sure = (v[:, :k] - v[:, 1:k + 1]).amin(dim=1) > 1e-9 if E > k else (v[:, 0] - v[:, 1]) > 1e-9
    assert sure.float().mean() > 0.99
    assert torch.equal(idx[sure].long(), i[sure][:, :k])
    want = torch.softmax(v[:, :k], dim=1)
    # float32 gates of float32 partial logits: 1e-5 covers their rounding
    assert (gate.double() - want)[sure].abs().max() < 1e-5
