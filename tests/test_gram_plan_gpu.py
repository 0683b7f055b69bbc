"""Stage 1 at the edges of the Gram kernels' plan: tokens around the 64-token
stages and the pieces that one set of accumulators sums up, tile counts below,
at and above one round of the chip (whole tiles, split tiles, both), with one
stream and two, H and G together and alone, against float64 sums.  The bar is the one of the stage-1
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


def _forms(duo, k, m, dtype, two):
    """H alone, G alone and all of G, added to by a second call: entries within the
    bar of the sums, and all with the precision of shorter sums (2-norm)."""
    print("[case] gram forms", k, m, dtype, two, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k + m)
    Xd = torch.randn((m, k), generator=g, device="cuda").to(dtype)
    Xs = (Xd.float() * (1 + 0.1 * torch.randn(Xd.shape, generator=g, device="cuda"))).to(dtype) if two else Xd
    Hr, Gr, ar = _terms64(Xs, Xd, 0.5)
    i = torch.arange(k, device="cuda") // 256
    up = i[:, None] <= i[None, :]
    # rounding errors of sums of `run` tokens, 32 (bf16) or 4 tokens a step, none
    # longer than 16384 (4096) here: 2^-24 per step, in quadrature
    steps = min(m, 16384 if dtype == torch.bfloat16 else 4096) / (32 if dtype == torch.bfloat16 else 4)
    bar = 4 * 2.0 ** -24 * steps ** 0.5
    ws = duo.workspace(duo.DUO_OP_HESSIAN, 0, k, m, 0, "cuda")
    for form in ("H", "G", "G full", "H, G full"):
        H, G, a = (torch.zeros(s, device="cuda") for s in ((k, k), (k, k), (k,)))
        for calls in (1, 2):
            ws.fill_(255)
            if form == "H":
                duo.duo_hessian_accum(Xs, H, 0.5, X_dense=Xd if two else None, ws=ws)
            elif form[0] == "H":
                duo.duo_hessian_accum(Xs, H, 0.5, X_dense=Xd if two else None, G=G, a=a, ws=ws, g_full=True)
            else:
                duo.duo_residual_term(Xd, G, a, 0.5, X_src=Xs if two else None, ws=ws, g_full=form == "G full")
            if form[0] == "H":
                assert torch.equal(H, H.t())
                assert (H.double() - calls * Hr).norm() <= bar * calls * Hr.norm(), (form, calls)
            if "G" in form:
                ref = Gr if "full" in form else torch.where(up, Gr, 0.0)
                lo = 2.0 ** -16 if two and dtype == torch.bfloat16 else 0.0
                assert (G.double() - calls * ref).norm() <= (bar + lo) * calls * ref.norm(), (form, calls)
                assert ((a.double() - calls * ar).abs() <= 2e-5 * calls * ar).all()


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("k,m", [(200, 700), (1024, 3001), (1300, 2000), (2816, 4096), (3328, 8200), (4096, 8200),
                                 (4100, 16500)])
def test_forms_bf16(duo_lib, k, m, two):
    _forms(duo_lib, k, m, torch.bfloat16, two)


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("k,m", [(200, 700), (1300, 2000), (2048, 4096), (4096, 8200)])
def test_forms_f32(duo_lib, k, m, two):
    _forms(duo_lib, k, m, torch.float32, two)


def _even_run(k, m, ntiles):
    """Tokens per segment when every tile of a launch is split into the up to eight
    segments that fill rounds of 256 tiles best."""
    def cost(s):
        sums = ntiles * (s + 2) * 65536 * 4 / 4e12 if s > 1 else 0.0
        return -(-ntiles * s // 256) / s * 2 * 65536 * m / 4.5e12 + sums
    return -(-m // min(range(1, 9), key=cost))


@pytest.mark.parametrize("k,m", [(3328, 8200), (3584, 16384)])
def test_run_lengths(duo_lib, k, m):
    """G alone, all of G, and both with H are summed in runs no longer than those of
    a launch whose tiles are all split: the error of independent roundings of `run` /
    32 steps.  The factor is measured: 0.21-0.25 for such runs, 0.40-0.63 for
    unsplit tiles."""
    print("[case] gram run lengths", k, m, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k + m)
    X = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    _, Gr, _ = _terms64(X, X, 0.5)
    i = torch.arange(k, device="cuda") // 256
    t = -(-k // 256)
    half = t * (t + 1) // 2
    for with_h, full in ((False, False), (False, True), (True, True)):
        H, G, a = (torch.zeros(s, device="cuda") for s in ((k, k), (k, k), (k,)))
        if with_h:
            duo_lib.duo_hessian_accum(X, H, 0.5, G=G, a=a, g_full=full)
        else:
            duo_lib.duo_residual_term(X, G, a, 0.5, g_full=full)
        ref = Gr if full else torch.where(i[:, None] <= i[None, :], Gr, 0.0)
        run = _even_run(k, m, (t * t if full else half) + (half if with_h else 0))
        assert (G.double() - ref).norm() <= 0.33 * 2.0 ** -24 * (run / 32) ** 0.5 * ref.norm(), (with_h, full)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_second_chunk(duo_lib, dtype):
    # tokens go through the kernels in chunks of at most 131072
    _run(duo_lib, 264, 131072 + 333, dtype, False)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("k,m", [(520, 3000), (4096, 8200)])
def test_nonfinite_entry(duo_lib, k, m, dtype):
    """One infinite and one NaN entry: H and G are non-finite exactly in the rows and
    columns that the two tokens' products reach, and the sums elsewhere are kept."""
    print("[case] gram non-finite", k, m, dtype, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k)
    X = torch.randn((m, k), generator=g, device="cuda").to(dtype)
    X[m // 3, 5], X[m - 1, k - 2] = float("inf"), float("nan")
    H, G, a = (torch.zeros(s, device="cuda") for s in ((k, k), (k, k), (k,)))
    duo_lib.duo_hessian_accum(X, H, 0.5, G=G, a=a)
    z = int(0.5 * k + 0.5)
    mag = torch.where(X.isnan(), float("inf"), X.abs().float())  # neither is among the smaller half
    drop = torch.zeros((m, k), dtype=torch.bool, device="cuda").scatter(1, torch.sort(mag, dim=1, stable=True).indices[:, :z], True)
    Xh, dX = X.masked_fill(drop, 0.0).double(), X.masked_fill(~drop, 0.0).double()
    i = torch.arange(k, device="cuda") // 256
    up = i[:, None] <= i[None, :]
    for got, ref, part in ((H, Xh.t() @ Xh, torch.ones_like(up)), (G, dX.t() @ Xh, up)):
        assert torch.equal(got.isfinite()[part], ref.isfinite()[part])
        ok = part & ref.isfinite()
        assert ((got.double() - ref).abs()[ok] <= 2e-5 * m).all()
    assert ((a.double() - dX.square().sum(0)).abs() <= 2e-5 * (dX.square().sum(0) + 1.0)).all()
