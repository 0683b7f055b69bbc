"""Stage 1 at the edges of the Gram kernels' plan: tokens around the 64-token
stages and the pieces that one set of accumulators sums up, tile counts below,
at and above one round of the chip (whole tiles, split tiles, both), with one
stream and two, against float64 sums.  The bar is the one of the stage-1
parity tests: 32-bit sums, entries within 2e-5 (6e-5 for two bf16 streams, whose
residual has 16 significant bits) of sqrt(H_ii H_jj)."""

import pytest
import torch

pytestmark = pytest.mark.gpu


def _terms64(Xs, Xd, p):
    k = Xs.shape[1]
    z = int(p * k + 0.5)
    order = torch.sort(Xs.abs(), dim=1, stable=True).indices[:, :z]
    Xh = Xs.scatter(1, order, 0.0).double()
    dX = Xd.double() - Xh
    return Xh.t() @ Xh, dX.t() @ Xh, dX.square().sum(0)


def _run(duo, k, m, dtype, two, pad=0):
    print("[case] gram plan", k, m, dtype, two, pad, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k + m)
    Xd = torch.randn((m, k + pad), generator=g, device="cuda").to(dtype)
    Xs = (Xd.float() * (1 + 0.1 * torch.randn(Xd.shape, generator=g, device="cuda"))).to(dtype) if two else Xd
    Xd, Xs = Xd[:, :k], Xs[:, :k]
    base = torch.randn((k, k), generator=g, device="cuda")
    H, G, a = (base + base.t()).contiguous(), base.clone(), torch.ones(k, device="cuda")
    H0, G0, a0 = H.double(), G.double(), a.double()
    duo.duo_hessian_accum(Xs, H, 0.5, X_dense=Xd if two else None, G=G, a=a)
    Hr, Gr, ar = _terms64(Xs, Xd, 0.5)
    i = torch.arange(k, device="cuda") // 256
    up = i[:, None] <= i[None, :]
    d = (Hr.diagonal() + 1.0).sqrt()
    bar = (6e-5 if two and dtype == torch.bfloat16 else 2e-5) * d[:, None] * d[None, :]
    assert torch.equal(H, H.t())
    assert ((H.double() - H0 - Hr).abs() <= bar).all()
    dd = (ar + 1.0).sqrt()
    barg = (6e-5 if two and dtype == torch.bfloat16 else 2e-5) * torch.maximum(d, dd)[:, None] * d[None, :]
    assert ((G.double() - G0 - Gr).abs() <= barg)[up].all()
    assert torch.equal(G.double()[~up], G0[~up])  # outside the defined part: untouched
    assert ((a.double() - a0 - ar).abs() <= 2e-5 * (ar + 1.0)).all()


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("k,m", [(256, 1), (512, 33), (520, 63), (512, 65), (1000, 129), (3848, 300), (4096, 200),
                                 (520, 16384), (520, 16417), (264, 40000)])
def test_bf16(duo_lib, k, m, two):
    _run(duo_lib, k, m, torch.bfloat16, two)


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("k,m", [(256, 1), (300, 31), (512, 65), (1000, 129), (4096, 70), (264, 4100), (264, 20000)])
def test_f32(duo_lib, k, m, two):
    _run(duo_lib, k, m, torch.float32, two)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_unaligned(duo_lib, dtype):
    _run(duo_lib, 333, 500, dtype, False, pad=1)
    _run(duo_lib, 333, 500, dtype, True, pad=1)
