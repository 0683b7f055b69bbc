"""duo_act_sparsify bit for bit against the oracle's rule on the one-pass kernels:
the ends of every register form (one wave per token up to k = 8192, one workgroup
above), magnitude ties across the vectors of a thread, rows wider than k, nothing
and everything dropped, zeros of either sign, and rows that only the two-pass
form takes."""

import numpy as np
import pytest
import torch

from oracle import duo_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,p", [(8, 0.5), (512, 0.5), (520, 0.6), (2056, 0.4), (8192, 0.5), (8200, 0.5), (12288, 0.6),
                                 (12296, 0.5), (16392, 0.3), (24584, 0.5), (32768, 0.5), (11008, 0.0), (11008, 1.0),
                                 (4096, 0.0), (4096, 1.0), (11004, 0.5)])
@pytest.mark.parametrize("pad", [0, 8, 1])
def test_sparsify_bit_exact(duo_lib, k, p, pad):
    print("[case] sparsify", k, p, pad, flush=True)
    g = torch.Generator().manual_seed(k + pad)
    x = torch.randn((5, k + pad), generator=g).to(torch.bfloat16)
    x[1:4] = (x[1:4].float() * 2).round().to(torch.bfloat16) / 2  # many ties
    x[2, ::2] = 0.0
    x[3, ::3] = -0.0
    xd = x.cuda()
    y = torch.full((5, k + pad), 3.0, dtype=torch.bfloat16, device="cuda")
    duo_lib.duo_act_sparsify(xd[:, :k], p, out=y[:, :k])
    y = y.cpu()
    ref = R.sparsify_tokens(x[:, :k].double().numpy(), p)[0]
    assert np.array_equal(y[:, :k].double().numpy(), ref)
    assert (y[:, k:] == 3.0).all()
