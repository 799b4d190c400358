"""Calls are refused by the exact lengths, whichever way the host has learnt them."""

import ctypes

import numpy as np
import pytest
import torch

import paper_2605_14037_amd as spkv
from paper_2605_14037_amd.inputs import TokenStream, small_workload, to_numpy_f32
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_refusals_follow_the_exact_lengths(seed):
    """Prompts, steps, prunes, releases and resets in random order on a small pool: an append is refused exactly
    if the pages that its worst case would need, counted from the lengths as they are, do not fit."""
    B, Hk, w, pool = 3, 2, 16, 900
    rng = np.random.default_rng(seed)
    wl = small_workload("capacity", B, 4, Hk, 64, [0] * B, 0.4, window=w, seed=seed)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, pool_tokens=pool, extra_context=100000), H.make_oracle(wl)
    pages = lambda n: -(-n // 64)
    accepted = refused = 0
    for r in range(150):
        op = rng.choice(["prompt", "prompt", "prompt", "few", "step", "prune", "release", "reset"], p=[.2, .2, .2, .15, .15, .03, .05, .02])
        if op == "prune":
            for tau in (0.7, 0.5):
                cache.set_tau(tau)
                oracle.set_tau(tau)
                if tau == 0.7:
                    cache.prune()
                    oracle.prune()
        elif op == "release":
            b = int(rng.integers(B))
            cache.release_sequence(b)
            oracle.release_sequence(b)
        elif op == "reset":
            cache.reset()
            for b in range(B):
                oracle.release_sequence(b)
        else:
            top = dict(prompt=400, few=17, step=2)[op]
            counts = [int(rng.integers(1, top)) for _ in range(B)]
            k, v, f, cu = stream.next_tokens(counts)
            lens = oracle.kept_len()
            need = 0
            for b in range(B):
                t = oracle.seq_len(b)
                ev = max(0, t + counts[b] - w) - max(0, t - w)
                need += sum(pages(int(lens[b][h]) + ev) for h in range(Hk))
            if need > pages(pool) + B * Hk:
                with pytest.raises(spkv.SPKVError) as e:
                    cache.append(k, v, f, cu)
                assert e.value.code == -3, r
                refused += 1
                b = int(np.argmax(lens.sum(axis=1)))                  # room again
                cache.release_sequence(b)
                oracle.release_sequence(b)
            else:
                cache.append(k, v, f, cu)
                oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
                accepted += 1
    assert accepted > 30 and refused > 5
    assert cache.stats(with_kept_len=True)[1] == oracle.kept_len().tolist()
    q = stream.next_query()
    if all(oracle.seq_len(b) for b in range(B)):
        H.check_output(cache.decode_attention(q), oracle.decode(to_numpy_f32(q))[0])
    cache.close()


def test_destroyed_right_behind_a_prompt():
    """The lengths that a prompt sends to the host go into pinned memory of the cache: destroyed while the
    launches are still on their way, it frees that memory only when they have come."""
    hold = torch.randn(4096, 4096, device="cuda")
    held = []
    for r in range(8):
        cache = spkv.SPKVCache(4, 8, 2, 64, max_context=8192, max_total_kept_tokens=65536, window=64, tau=0.5)
        k = torch.zeros(4 * 700, 2, 64, dtype=torch.bfloat16, device="cuda")
        f = torch.ones(4 * 700, 2, device="cuda")
        for _ in range(r):
            hold = hold @ hold * 1e-3                     # so that the append starts late
        cache.append(k, k, f, [0, 700, 1400, 2100, 2800])
        assert cache.lib.spkv_cache_destroy(cache.handle) == 0       # (close() would wait by itself)
        cache.handle = ctypes.c_void_p()
        held.append((cache.arena, torch.full((1024,), -7, dtype=torch.int32, pin_memory=True)))
    torch.cuda.synchronize()
    assert all(bool((p == -7).all()) for _, p in held)
