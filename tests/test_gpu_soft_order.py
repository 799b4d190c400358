"""GPU parity of spkv_soft_gated_attention where all pairs run on all XCDs, longest spans of every pair
first: numbers of pairs that are no multiple of eight and more than one round of spans (16 tokens each
with groups of 16 heads, 32 with groups of 8), sequences without tokens and much shorter ones, and a
round less, which keeps a pair to an XCD.  Oracle and tolerances of tests/harness.py."""

import pytest

from tests.test_gpu_soft_gated import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts,Hq,Hkv,D,w", [
    ([480, 37, 300], 48, 3, 64, 100),             # 9 pairs, 270 spans
    ([448, 0, 15, 449], 48, 3, 128, 33),          # 12 pairs, 348 spans
    ([450] * 3, 48, 3, 64, 512),                  # 9 pairs, 261 spans, all inside the window
    ([448] * 3, 48, 3, 64, 64),                   # 9 pairs, 252 spans: one round
    ([600, 599], 24, 3, 64, 128),                 # 6 pairs
])
def test_soft_gated_pairs_on_all_xcds(counts, Hq, Hkv, D, w):
    _check(counts, Hq, Hkv, D, w, seed=len(counts) + w)
