"""Attention at the edges of its tiles: sequence lengths around the 64-key
blocks and the 64- and 128-query workgroups, both workgroup widths (128 queries
from 512 workgroups up), rows wider than the heads and an output whose rows
are not 8-byte aligned, against the float64 oracle.  The bar is the one of the
block's attention test: two bf16 units (the probabilities are rounded to bf16
on both sides) plus 2^-8 of the outputs' root mean square."""

import numpy as np
import pytest
import torch

from oracle import block_ref as BR

pytestmark = pytest.mark.gpu


def _run(duo, nseq, L, heads, hd, pad, ldo_odd):
    print("[case] attention tiles", nseq, L, heads, hd, pad, ldo_odd, flush=True)
    g = torch.Generator().manual_seed(1000 * L + hd)
    d = heads * hd
    # one allocation of rows wider than the heads: Q, K and V share their stride
    qkv = torch.randn((nseq * L, 3 * d + pad), generator=g).to(torch.bfloat16)
    dev = qkv.cuda()
    q, k, v = (dev[:, i * d:(i + 1) * d] for i in range(3))
    out = torch.full((nseq * L, d + (1 if ldo_odd else 0)), 7.0, dtype=torch.bfloat16, device="cuda")
    duo.duo_attention(q, k, v, nseq, L, heads, hd, out=out[:, :d])
    o = out.cpu().double().numpy()
    if ldo_odd:
        assert (o[:, d] == 7.0).all()
    ref = BR.attention(*(qkv[:, i * d:(i + 1) * d].double().numpy() for i in range(3)), nseq, L, heads, hd)
    err = np.abs(o[:, :d] - ref)
    tol = 2 * 2.0 ** -7 * np.abs(ref) + 2.0 ** -8 * np.sqrt(np.mean(ref * ref))
    assert (err <= tol).all(), float((err / tol).max())


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("nseq,L,heads", [
    (1, 1, 3), (3, 31, 1), (2, 63, 2), (1, 64, 1), (1, 65, 9), (2, 127, 1), (1, 129, 2), (1, 193, 3),  # 64 queries
    (32, 33, 16), (16, 129, 16),                                                                      # 128 queries
])
def test_attention_tile_edges(duo_lib, nseq, L, heads, hd):
    _run(duo_lib, nseq, L, heads, hd, pad=0, ldo_odd=False)


@pytest.mark.parametrize("hd", [64, 128])
def test_attention_strided_rows(duo_lib, hd):
    _run(duo_lib, 2, 100, 3, hd, pad=8, ldo_odd=True)
