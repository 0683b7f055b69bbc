"""The decode GEMV around the sizes where its selection changes form (8192 and
16384 channels), both activation types, ties at the threshold, against float64:
every product is exact in fp32 and the sums run over at most k terms, so a row is
within (k + 2) 2^-24 sum |w x|."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("k", [7, 1024, 8192, 8193, 16384, 16385, 20000, 32768])
def test_decode_sizes(duo_lib, k, dtype):
    print("[case] decode sizes", k, dtype, flush=True)
    n, p = 300, 0.5
    g = torch.Generator(device="cuda").manual_seed(k)
    W = (torch.randn((n, k), generator=g, device="cuda") * 0.02).bfloat16()
    keep = torch.rand((n, k), generator=g, device="cuda") < 0.5
    W = torch.where(keep, W, torch.zeros_like(W))
    words = (k + 31) // 32
    b = torch.nn.functional.pad(keep, (0, words * 32 - k)).view(n, words, 32).to(torch.int64)
    w = (b << torch.arange(32, device="cuda")).sum(-1)
    comp = duo_lib.dsc_compress(W, torch.where(w >= 2 ** 31, w - 2 ** 32, w).to(torch.int32))
    for ties in (False, True):
        x = torch.randn(k, generator=g, device="cuda")
        if ties:
            x = (x * 2).round() / 2
        x = x.to(dtype)
        y = duo_lib.dsc_gemv(comp, x, p).double()
        z = int(p * k + 0.5)
        xs = x.clone()
        xs[torch.sort(x.abs(), stable=True).indices[:z]] = 0
        ref = W.double() @ xs.double()
        bound = (k + 2) * 2.0 ** -24 * (W.double().abs() @ xs.double().abs()) + 1e-30
        assert ((y - ref).abs() <= bound).all(), float(((y - ref).abs() / bound).max())
