"""duo_linear at the edges of its three tile sizes: K of one, two, three and five
64-deep stages, M and N around the tile edges, residual (also in place), rows
wider than the operands, outputs that are not 16-byte aligned, against a
float64 product.  Each bf16 output may be one unit off (a rounding boundary)
plus the fp32 accumulation's 1e-5 of the outputs' root mean square."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(duo, m, k, n, res, pad=0, odd=0, inplace=False):
    print("[case] linear tiles", m, k, n, res, pad, odd, inplace, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + 7 * k + 13 * n)
    x = torch.randn((m, k + pad), generator=g, device="cuda").bfloat16()[:, :k]
    w = (torch.randn((n, k + pad), generator=g, device="cuda") * 0.02).bfloat16()[:, :k]
    r = torch.randn((m, n + odd), generator=g, device="cuda").bfloat16()[:, :n] if res else None
    ref = x.double() @ w.double().t()
    if res:
        ref = ref + r.double()
    y = torch.full((m, n + odd), 9.0, dtype=torch.bfloat16, device="cuda")
    out = r if inplace else y[:, :n]
    duo.duo_linear(x, w, R=r, out=out)
    if odd and not inplace:
        assert (y[:, n:] == 9.0).all()
    err = (out.double() - ref).abs()
    tol = 2.0 ** -7 * ref.abs() + 1e-5 * ref.square().mean().sqrt()
    assert (err <= tol).all(), float((err / tol).max())


# 256 and 128 rows per tile
@pytest.mark.parametrize("k", [64, 128, 192, 320])
@pytest.mark.parametrize("m,n", [(4096, 4096), (4097, 3848), (3839, 4104), (129, 257), (127, 1024)])
def test_linear_large_tiles(duo_lib, m, k, n):
    _run(duo_lib, m, k, n, res=False)
    _run(duo_lib, m, k, n, res=True, pad=8, odd=3)
    _run(duo_lib, m, k, n, res=True, inplace=True)


# rows of Y or R that 16-byte accesses cannot take, on the large tiles
@pytest.mark.parametrize("m,n", [(129, 257), (300, 1003), (4097, 4001), (3839, 300)])
def test_linear_large_tiles_narrow_stores(duo_lib, m, n):
    _run(duo_lib, m, 1024, n, res=False)
    _run(duo_lib, m, 1024, n, res=True)
    _run(duo_lib, m, 128, n, res=True, inplace=True)


@pytest.mark.parametrize("m,k,n", [(1, 64, 8), (300, 4096, 520), (257, 72, 256), (255, 128, 257), (4000, 128, 300)])
def test_linear_small_tiles(duo_lib, m, k, n):
    _run(duo_lib, m, k, n, res=True)
    _run(duo_lib, m, k, n, res=False, pad=8, odd=1)
