"""Layers whose sizes are no multiples of 64, which run on zero-padded copies:
against the same calls with a workspace that leaves the copies no room (edge
tiles), for every kind of mask, both residual forms, quantisation, scores and
16-bit copies, n or k ragged or both.  With the mask given, both are fp32 runs of
the same algorithm: relative Frobenius difference below 16 sqrt(k) 2^-24 times a
factor 8 for the sums of up to k / 128 blocks that each of them rounds in its own
order; masks of a free selection may differ only where scores are close (at most 2
entries here)."""

import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _terms(duo, k, m, g):
    X = torch.randn((m, k), generator=g, device="cuda") * torch.exp(0.5 * torch.randn(k, generator=g, device="cuda"))
    H = torch.zeros((k, k), device="cuda")
    G = torch.zeros((k, k), device="cuda")
    a = torch.zeros(k, device="cuda")
    duo.duo_hessian_accum(X, H, 0.5 if k > 1 else 0.0, G=G, a=a)  # (half of one channel rounds to all)
    return H, G, a


def _bar(k):
    return 8 * 16 * math.sqrt(k) * 2.0 ** -24


def _rel(x, r):
    return float((x.double() - r.double()).norm() / r.double().norm())


@pytest.mark.parametrize("k", [1, 63, 65, 127, 130, 1000, 1345])
def test_inverse_factor(duo_lib, k):
    print("[case] padded inverse factor", k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k)
    H, _, _ = _terms(duo_lib, k, 3 * k + 8, g)
    wide = torch.full((k, k + 3), 5.0, device="cuda")
    wide[:, :k] = H
    L = H.clone()
    lam, fail = duo_lib.duo_chol_inv(L, 0.01)
    assert fail == -1
    Lw = wide[:, :k]
    duo_lib.duo_chol_inv(Lw, 0.01)
    assert torch.equal(Lw, L) and (wide[:, k:] == 5.0).all()
    Hd = H.double()
    Hd.diagonal().add_(lam)
    Ld = L.double()
    assert torch.equal(Ld, Ld.tril())
    r = Ld.t() @ Hd @ Ld - torch.eye(k, dtype=torch.float64, device="cuda")
    assert float(r.abs().max()) <= 16 * math.sqrt(k) * 2.0 ** -24 * 4
    Hb = -H  # not positive definite: reported, with an index inside the matrix
    Hb.diagonal().abs_()
    if k > 2:
        with pytest.raises(duo_lib.DuoError):
            duo_lib.duo_chol_inv(Hb, 0.0)


@pytest.mark.parametrize("n,k,B,kw", [
    (75, 1000, 64, dict(form="d")), (75, 1000, 64, dict(form="y")), (500, 1000, 128, dict(nm_n=2)),
    (130, 1345, 128, dict()), (1, 200, 128, dict()), (300, 1100, 100, dict(form="y")), (65, 1024, 128, dict(form="y")),
    (128, 1001, 128, dict(form="d")), (200, 1300, 128, dict(quant=(4, 128), form="d")),
    (200, 1300, 128, dict(quant=(4, 128), form="y")), (90, 700, 128, dict(quant=(8, 32))),
])
@pytest.mark.parametrize("forced", [True, False])
def test_prune_layer(duo_lib, n, k, B, kw, forced):
    print("[case] padded prune layer", n, k, B, kw, forced, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + k)
    H, G, a = _terms(duo_lib, k, 4 * k, g)
    duo_lib.duo_chol_inv(H, 0.01)
    W = (torch.randn((n, k + 5), generator=g, device="cuda") * 0.02).bfloat16()[:, :k]
    mask = None
    if forced:
        mask = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, (k + 31) // 32), generator=g, device="cuda", dtype=torch.int32)
    # the old layout's bytes: too small for the copies, enough for the rest
    size = duo_lib.duo_workspace_size(duo_lib.DUO_OP_PRUNE_LAYER, n, k, 0, B)
    kk = max(n, k) * k * 4 + k * 4 + k * k * 4 + 4 * 256
    base = kk + duo_lib.duo_workspace_size(duo_lib.DUO_OP_SWEEP, n, k, 0, B)
    assert base < size
    res = []
    for nbytes in (size, base):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        ws.fill_(0xff)  # NaN wherever the padding is not written
        res.append(duo_lib.duo_prune_layer(W, H, G, a, 0.5, B, mask_in=mask, want_lowp=True, want_scores=True, ws=ws,
                                           **kw))
    p, e = res
    diff = (duo_lib.unpack_mask(p[2], k) != duo_lib.unpack_mask(e[2], k)).sum().item()
    assert diff <= (0 if forced else 2)
    for x, y in zip(p, e):
        if x is not None and x.is_floating_point():
            assert torch.isfinite(x.float()).all()
    if diff == 0 and not kw.get("quant"):
        assert _rel(p[0], e[0]) < _bar(k)
        assert _rel(p[3], e[3]) < 2 * _bar(k)
        assert _rel(p[1].float(), e[1].float()) < 2.0 ** -9
    elif kw.get("quant"):
        # a value next to a rounding boundary may take the next code
        assert _rel(p[0], e[0]) < 2e-2
