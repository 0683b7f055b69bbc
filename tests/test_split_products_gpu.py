"""The fp32 products that run as six bf16 products of exactly split operands
(duo_prune_layer's Y form, unquantised) at sizes where they take that path, k a
multiple of 256, of 8 and of nothing, with NaN in a workspace's unwritten
memory, and with workspaces that leave the packed operands no room (the fp32
instructions then do the work); and the routes of the same sizes that keep the
fp32 instructions.  Bars: relative Frobenius error 16 sqrt(k) 2^-24
for one product, and between two correct fp32 runs of a chain of them (k = 8200:
8.6e-5)."""

import math

import pytest
import torch

pytestmark = pytest.mark.gpu

KS = [8192, 8200, 8195]


def _bar(k):
    return 16 * math.sqrt(k) * 2.0 ** -24


def _rel(x, r):
    return float((x.double() - r).norm() / r.norm())


def _lower(k, g):
    L = torch.randn((k, k), generator=g, device="cuda").tril_().mul_(1 / 64)
    L.diagonal().abs_().add_(1.0)
    return L


@pytest.mark.parametrize("k", KS)
def test_score_terms(duo_lib, k):
    print("[case] large score terms", k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k)
    L = _lower(k, g)
    G = torch.randn((k, k), generator=g, device="cuda")
    a = torch.rand(k, generator=g, device="cuda") * k
    bad = G.clone()
    i = torch.arange(k, device="cuda")
    below = i[:, None] // 128 > i[None, :] // 128
    bad[below] = float("nan")  # below the diagonal 128-tiles: not read
    Q = G.double().triu_() @ L.double()
    U = Q.triu(1)
    R = U @ L.double().t()
    d = L.diagonal().double()
    fac = 1 / d.square() + a.double() - U.square().sum(1) + 2 * Q.diagonal() / d
    D = torch.full((k, k), 7.0, device="cuda")
    D, f = duo_lib.duo_score_terms(L, bad, a, D=D)
    assert _rel(D.triu(1), R.triu(1)) < _bar(k)
    assert _rel(f, fac) < _bar(k)
    assert (D[below] == 7.0).all()  # below the diagonal 128-tiles: not written
    assert (D.tril()[~below] == 0.0).all()


@pytest.mark.parametrize("quant", [None, (4, 128), (8, 64)])
def test_two_call_route(duo_lib, quant):
    """duo_score_terms and duo_sweep give the bits of duo_prune_layer in the D form,
    a quantised layer's codes among them."""
    n, k = 1000, 8200
    print("[case] two-call route", n, k, quant, flush=True)
    g = torch.Generator(device="cuda").manual_seed(9)
    L = _lower(k, g)
    G = torch.randn((k, k), generator=g, device="cuda").triu_().mul_(1 / k)
    a = torch.full((k,), 50.0, device="cuda")
    W = torch.randn((n, k), generator=g, device="cuda") * 0.02
    one = duo_lib.duo_prune_layer(W, L, G, a, 0.5, 128, quant=quant, form="d")
    D, fac = duo_lib.duo_score_terms(L, G, a)
    two = duo_lib.duo_sweep(W, L, D, fac, 0.5, 128, quant=quant)
    for x, y in zip(one, two):
        assert x is None and y is None or torch.equal(x, y)


@pytest.mark.parametrize("n,k", [(4096, 8192), (4100, 8200), (4099, 8195)])
def test_sweep_y_form(duo_lib, n, k):
    print("[case] split Y form sweep", n, k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + k)
    L = _lower(k, g)
    G = torch.randn((k, k), generator=g, device="cuda").triu_().mul_(1 / k)
    a = torch.full((k,), 50.0, device="cuda")
    W = torch.randn((n, k), generator=g, device="cuda") * 0.02
    keep = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, (k + 31) // 32), generator=g, device="cuda", dtype=torch.int32)
    size = duo_lib.duo_workspace_size(duo_lib.DUO_OP_PRUNE_LAYER, n, k, 0, 128)
    out = []
    for form, nbytes in (("y", size), ("y", size // 2 // 256 * 256), ("d", size)):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")  # NaN
        out.append(duo_lib.duo_prune_layer(W, L, G, a, 0.5, 128, mask_in=keep, ws=ws, form=form)[0].double())
    assert torch.isfinite(out[0]).all()
    assert not torch.equal(out[0], out[1])  # the full workspace took the split path
    for o in out[1:]:
        assert _rel(out[0], o) < _bar(k)
