"""Attention at the edges of its tiles: sequence lengths around the 64-key
blocks and the 64- and 128-query workgroups, both workgroup widths (128 queries
from 512 workgroups up), rows wider than the heads and an output whose rows
are not 8-byte aligned, against the float64 oracle.  The bar is the one of the
block's attention test, two bf16 units plus 2^-8 of the outputs' root mean square,
plus one rounding of a probability that falls the other way: the oracle rounds
them to bf16 too, a probability next to a rounding boundary may land one unit
(at most 2^-7 of it) off, and its row's outputs move by that times its V."""

import math

import numpy as np
import pytest
import torch

from oracle import block_ref as BR

pytestmark = pytest.mark.gpu


def _one_unit(qkv, nseq, L, heads, hd):
    """2^-7 max_j p_j |v_j| of every output."""
    q, k, v = (x.double().view(nseq, L, heads, hd).transpose(1, 2) for x in qkv[:, :3 * heads * hd].chunk(3, 1))
    P = (q @ k.transpose(2, 3) / hd ** 0.5).masked_fill(torch.ones((L, L), dtype=torch.bool).triu(1), -torch.inf).softmax(-1)
    out = torch.empty_like(q)
    for i in range(L):  # (nseq, heads, keys, hd) of one query at a time
        out[:, :, i] = (P[:, :, i, :i + 1, None] * v[:, :, :i + 1].abs()).amax(2)
    return 2.0 ** -7 * out.transpose(1, 2).reshape(nseq * L, heads * hd).numpy()


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
    tol = 2 * 2.0 ** -7 * np.abs(ref) + 2.0 ** -8 * np.sqrt(np.mean(ref * ref)) + _one_unit(qkv, nseq, L, heads, hd)
    assert (err <= tol).all(), float((err / tol).max())


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("nseq,L,heads", [
    (1, 1, 3), (3, 31, 1), (2, 63, 2), (1, 64, 1), (1, 65, 9), (2, 127, 1), (1, 129, 2), (1, 193, 3),  # 64 queries
    (32, 33, 16), (16, 129, 16),                                                                      # 128 queries
])
def test_attention_tile_edges(duo_lib, nseq, L, heads, hd):
    _run(duo_lib, nseq, L, heads, hd, pad=0, ldo_odd=False)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("nseq,heads", [(1, 5), (1, 7), (1, 8), (3, 3), (2, 7), (1, 15), (2, 8), (1, 41)])
def test_attention_head_counts(duo_lib, nseq, heads, hd):
    # (sequence, head) pairs in groups of eight, left over from them, and seven over
    _run(duo_lib, nseq, 200, heads, hd, pad=0, ldo_odd=False)


@pytest.mark.parametrize("hd", [64, 128])
def test_attention_strided_rows(duo_lib, hd):
    _run(duo_lib, 2, 100, 3, hd, pad=8, ldo_odd=True)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("nseq,L,heads", [(2, 200, 3), (16, 300, 16)])  # 64 and 128 queries per workgroup
@pytest.mark.parametrize("scale", [30.0, 400.0, 2000.0])
def test_attention_large_scores(duo_lib, nseq, L, heads, hd, scale):
    """Scores up to about 1e8 (Q and K of `scale` standard deviations): a row whose
    best key leads by far has one probability of one, and its output is that
    key's V up to the roundings of the probability and of the output to bf16
    (2^-8 each)."""
    print("[case] attention large scores", nseq, L, heads, hd, scale, flush=True)
    g = torch.Generator(device="cuda").manual_seed(L + hd)
    q, k, v = (torch.randn((nseq * L, heads * hd), generator=g, device="cuda") for _ in range(3))
    q, k, v = (q * scale).bfloat16(), (k * scale).bfloat16(), v.bfloat16()
    o = duo_lib.duo_attention(q, k, v, nseq, L, heads, hd)
    later = torch.ones((L, L), dtype=torch.bool, device="cuda").triu(1)
    rows = 0
    for s in range(nseq):
        t = slice(s * L, (s + 1) * L)
        for h in range(heads):
            f = slice(h * hd, (h + 1) * hd)
            S = (q[t, f].double() @ k[t, f].double().t() / hd ** 0.5).masked_fill(later, float("-inf"))
            top, i = S.topk(2, dim=1)
            # a score's own error: hd fp32 roundings of sums of its terms' size
            slack = hd * 2.0 ** -24 * (q[t, f].double().abs() @ k[t, f].double().abs().t()).amax(1) / hd ** 0.5
            clear = top[:, 0] - top[:, 1] > 40 + 2 * slack  # the others weigh less than L e^-40
            rows += int(clear.sum())
            x, y = o[t, f][clear].double(), v[t, f][i[clear, 0]].double()
            assert ((x - y).abs() <= (2.0 ** -7 + 2.0 ** -15) * y.abs() + L * math.exp(-40) * 8).all(), (s, h)
    assert rows > nseq * L * heads // 2


@pytest.mark.parametrize("hd", [64, 128])
def test_attention_nonfinite(duo_lib, hd):
    """Scores of -inf weigh nothing; a row that sees +inf or NaN is NaN, and so is
    one that sees nothing but -inf; other rows are not touched."""
    print("[case] attention non-finite", hd, flush=True)
    L, heads = 150, 2
    g = torch.Generator().manual_seed(hd)
    q, k, v = (torch.randn((L, heads * hd), generator=g).bfloat16() for _ in range(3))
    q[:, 0] = 1.0
    q[100:, 0] = -1.0
    k[70, 0] = float("-inf")          # head 0: -inf for queries 70 .. 99, +inf from 100 on
    q[:3, hd], k[:3, hd] = 1.0, float("-inf")  # head 1: queries 0 .. 2 see only -inf
    q[3:, hd] = 0.25
    k[120, hd + 1] = float("nan")
    o = duo_lib.duo_attention(q.cuda(), k.cuda(), v.cuda(), 1, L, heads, hd).cpu().double()
    later = torch.ones((L, L), dtype=torch.bool).triu(1)
    for h in range(heads):
        f = slice(h * hd, (h + 1) * hd)
        S = (q[:, f].double() @ k[:, f].double().t() / hd ** 0.5).masked_fill(later, float("-inf"))
        ref = S.softmax(-1) @ v[:, f].double()
        assert torch.equal(o[:, f].isnan(), ref.isnan())
        ok = ~ref.isnan()
        # every probability and every output rounded to bf16 (2^-8 relative)
        tol = 2.0 ** -8 * (S.softmax(-1) @ v[:, f].double().abs() + ref.abs()) * 1.01 + 1e-5
        assert ((o[:, f] - ref).abs() <= tol)[ok].all()
