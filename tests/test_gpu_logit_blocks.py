"""Gate logits whose workgroups walk the hidden states from blocks of their own (rows whole
multiples of 4 KB apart, more than 16 384 tokens, up to 128 hidden units) against the oracle, with
sizes on both sides of that rule."""

import numpy as np
import pytest
import torch

import paper_2605_14037_amd as spkv
from paper_2605_14037_amd.inputs import to_numpy_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dm,dh,Hk", [(16385, 2048, 64, 1), (20001, 2048, 80, 5), (16600, 6144, 16, 2),
                                        (16511, 4096, 128, 8), (16400, 1920, 128, 3)])
def test_logits_from_a_block_of_its_own(n, dm, dh, Hk):
    """fp32 sums of dm + dh products of unit scale in another order: a few thousand roundings of
    6e-8 add up to less than 1e-5."""
    from oracle.spkv_oracle import utility_logits as oracle_logits
    g = torch.Generator(device="cuda").manual_seed(n + dm + dh)
    x = torch.randn(n, dm, generator=g, device="cuda").to(torch.bfloat16)
    w1 = (torch.randn(dh, dm, generator=g, device="cuda") / dm ** 0.5).to(torch.bfloat16)
    w2 = (torch.randn(Hk, dh, generator=g, device="cuda") / dh ** 0.5).to(torch.bfloat16)
    biases = (torch.randn(dh, generator=g, device="cuda"), torch.randn(Hk, generator=g, device="cuda"))
    rows = np.unique(np.r_[0:300, n - 300:n, np.arange(0, n, 97)])       # ends, and some of every workgroup
    for b1, b2 in (biases, (None, None)):
        got = spkv.utility_logits(x, w1, b1, w2, b2).cpu().numpy()
        ref = oracle_logits(*(None if t is None else to_numpy_f32(t)
                              for t in (x[torch.from_numpy(rows).cuda()], w1, b1, w2, b2)))
        assert np.isfinite(got).all()
        assert np.abs(got[rows] - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())
