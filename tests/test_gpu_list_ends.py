"""Pages are not cleared when they are created, reset or handed out again: whoever lengthens a list clears
the values behind its end.  An arena full of NaN must not show in any attention."""

import numpy as np
import pytest
import torch

import paper_2605_14037_amd as spkv
from paper_2605_14037_amd.inputs import TokenStream, small_workload, to_numpy_f32
from tests import harness as H

pytestmark = pytest.mark.gpu


def _poisoned_cache(wl, pool_tokens, extra):
    cfg = spkv.SPKVConfig(wl.batch, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.window, 0, wl.tau,
                          wl.max_context + extra, pool_tokens)
    poison = torch.full((spkv.required_bytes(cfg),), 255, dtype=torch.uint8, device="cuda")
    at = poison.data_ptr()
    del poison
    cache = H.make_cache(wl, pool_tokens=pool_tokens, extra_context=extra)
    assert cache.arena.data_ptr() == at               # the poisoned block again
    return cache


@pytest.mark.parametrize("D,w,keep", [(128, 32, 1.0), (64, 40, 0.5), (128, 7, 0.8)])
def test_nan_in_unused_pages_never_shows(D, w, keep):
    """Lists lengthened by prompts, short chunks, few-token appends and single steps, past every position of a
    half-page, with recycled pages and after a reset."""
    B, rng = 2, np.random.default_rng(D + w)
    wl = small_workload("poison", B, 8, 2, D, [0] * B, keep, window=w, seed=D + w)
    cache = _poisoned_cache(wl, B * 2 * 1500, 1400)
    for life in range(2):
        stream, oracle = TokenStream(wl, device="cuda"), H.make_oracle(wl)
        for r in range(36):
            kind = ("prompt", "few", "step", "chunk")[int(rng.integers(4))] if r else "prompt"
            n = {"prompt": int(rng.integers(1, 90)), "few": min(w, int(rng.integers(2, 17))),
                 "chunk": min(w, int(rng.integers(2, 17))), "step": 1}[kind]
            counts = [n] * B if kind in ("step", "chunk") else [n, n // 2]
            k, v, f, cu = stream.next_tokens(counts)
            q = stream.next_query(rows=sum(counts))
            if kind == "step":
                out = cache.decode_step(k, v, f, q)
            elif kind == "chunk":
                out = cache.decode_chunk(k, v, f, q, cu)
            else:
                cache.append(k, v, f, cu)
                q = stream.next_query()
            oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
            if kind not in ("step", "chunk"):
                if oracle.seq_len(1) == 0:
                    continue
                out, counts = cache.decode_attention(q), [1] * B
            H.check_output(out, oracle.decode_chunk(to_numpy_f32(q), counts)[0], f"life {life}, {r}: {kind} {counts}")
            if r == 20:
                cache.release_sequence(1)
                oracle.release_sequence(1)
                k, v, f, cu = stream.next_tokens([0, 45])
                H.feed(cache, oracle, k, v, f, cu)
        H.check_state(cache, oracle, wl)
        cache.reset()
    cache.close()
