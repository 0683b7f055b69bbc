"""The fp32 products that run as six bf16 products of exactly split operands:
score terms and Y-form sweep at sizes where they take that path,
k a multiple of 256, of 8 and of nothing, with NaN wherever an operand is not to
be read, and with workspaces that leave the packed operands no room (the fp32
instructions then do the work).  Bars: relative Frobenius error 16 sqrt(k) 2^-24
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
    print("[case] split score terms", k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k)
    L = _lower(k, g)
    G = torch.randn((k, k), generator=g, device="cuda")
    a = torch.rand(k, generator=g, device="cuda") * k
    bad = G.clone()
    i = torch.arange(k, device="cuda")
    bad[i[:, None] // 128 > i[None, :] // 128] = float("nan")  # below the diagonal 128-tiles: not read
    Q = G.double().triu_() @ L.double()
    U = Q.triu(1)
    R = U @ L.double().t()
    d = L.diagonal().double()
    fac = 1 / d.square() + a.double() - U.square().sum(1) + 2 * Q.diagonal() / d
    size = duo_lib.duo_workspace_size(duo_lib.DUO_OP_SCORE_TERMS, 0, k, 0, 0)
    for nbytes in (size, size - 1):  # split, fp32 instructions
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        D = torch.zeros((k, k), device="cuda")
        D, f = duo_lib.duo_score_terms(L, bad, a, D=D, ws=ws)
        assert _rel(D.triu(1), R.triu(1)) < _bar(k)
        assert _rel(f, fac) < _bar(k)


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
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out.append(duo_lib.duo_prune_layer(W, L, G, a, 0.5, 128, mask_in=keep, ws=ws, form=form)[0].double())
    assert torch.isfinite(out[0]).all()
    for o in out[1:]:
        assert _rel(out[0], o) < _bar(k)
