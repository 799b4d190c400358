"""GPU parity of long prefill calls whose spans are taken in order of their pairs' lengths (up to 64
pairs), in groups of pairs per XCD: every count of groups, sequences without a token, spans cut into
ranges, one pair more than the order serves.  Oracle and tolerances of tests/harness.py; the grid, which
counts only spans that hold a token, shows that the route is the one named."""

import numpy as np
import pytest

from tests.test_gpu_prefill import _run_prefill
from paper_2605_14037_amd.inputs import small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,ctx,counts,ranges,groups", [
    (1, 9, 300, [497], 1, 1),                                    # one group of nine pairs, a ragged last span
    (2, 8, 700, [300, 277], 1, 2),                               # two groups
    (4, 8, 400, [200, 200, 199, 176], 1, 4),                     # four groups
    (8, 8, 300, [120, 128, 127, 113, 128, 100, 128, 128], 1, 8),   # eight groups, 64 pairs
    (8, 8, 300, [300, 0, 1, 0, 16, 17, 0, 288], 1, 1),           # few of the sequences bring tokens
    (16, 4, 300, [90 + b for b in range(16)], 1, 4),             # 64 pairs, no more groups than heads
    (21, 3, 200, [0 if b % 4 == 1 else 60 + 5 * b for b in range(21)], 1, 1),      # heads that no group divides
    (4, 8, 2200, [144, 0, 3, 0], 3, 1),                          # 80 spans of tokens: ranges, merged in order
    (13, 5, 300, [70] * 13, None, 1),                            # 65 pairs: in turn
])
def test_prefill_spans_in_order(B, Hkv, ctx, counts, ranges, groups):
    G, span = 16, 16                      # tokens of eight waves' 32 columns
    rates = np.random.default_rng(B).permutation(np.tile([1.0, 0.0, 0.7, 0.2], -(-B * Hkv // 4))[:B * Hkv])
    wl = small_workload("order", B, Hkv * G, Hkv, 64, [ctx + 7 * b for b in range(B)], rates.reshape(B, Hkv),
                        window=64, seed=B + Hkv)
    grid = -(-max(counts) // span) * B * Hkv + (-(B * Hkv) % 8) * -(-max(counts) // span)      # in turn
    if ranges is not None:
        each = sum(-(-n // span) for n in counts) * Hkv * ranges // groups       # workgroups of a group
        grid = 8 * 2 * -(-each // (2 * (8 // groups)))                           # two at a time per XCD
    _run_prefill(wl, [counts], sample=120, last_grid=grid, decode_after=1)


@pytest.mark.parametrize("D,window,ctx,n", [(64, 64, 500, 4099), (128, 600, 700, 4099), (128, 600, 40, 4097),
                                            (64, 100, 0, 513), (128, 64, 90, 65), (64, 600, 2000, 601)])
def test_prefill_rows_staged_beside_the_append(D, window, ctx, n):
    """The window is staged while the append counts: chunks whose segments are counted before it (above
    4096 tokens) or by it, leaving ring rows moved by it (long windows) or later, windows that hold
    nothing or a part, chunks of one token more than the window, and decode steps on what is left."""
    wl = small_workload("staged", 2, 4, 2, D, [ctx, ctx // 2], [[0.4, 0.1]], window=window, seed=D + n)
    _run_prefill(wl, [[n, n // 3]], sample=60, decode_after=2)
