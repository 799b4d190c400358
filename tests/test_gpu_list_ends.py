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


@pytest.mark.parametrize("option", [None, (spkv.OPT_ITEM_TARGET, 64), (spkv.OPT_STEP_LAUNCHES, 1)])
@pytest.mark.parametrize("D,w", [(128, 64), (64, 70)])
def test_released_window_does_not_show(D, w, option):
    """Infinite values that a released sequence leaves in the window, in every call of the sequence that takes its
    place while its own window is filling: steps fused, apart and static on short lists and split ones, narrow
    and wide chunks."""
    B = 2
    wl = small_workload("released", B, 8, 2, D, [0] * B, 0.5, window=w, seed=D + w)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=600, pool_tokens=8000), H.make_oracle(wl)
    if option is not None:
        cache.set_option(*option)
    for kind in ("step", "attend", "narrow", "wide"):
        k, v, f, cu = stream.next_tokens([w] * B)
        cache.append(k, torch.full_like(v, float("inf")), f, cu)
        for b in range(B):
            cache.release_sequence(b)
            oracle.release_sequence(b)
        for r in range(3):
            counts = {"step": [1, 1], "attend": [2, 1], "narrow": [4, 1 + r], "wide": [9, 5 + r]}[kind]
            k, v, f, cu = stream.next_tokens(counts)
            q = stream.next_query(rows=sum(counts))
            oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
            if kind == "step":
                out = cache.decode_step(k, v, f, q)
            elif kind == "attend":
                cache.append(k, v, f, cu)
                q, counts = stream.next_query(), [1] * B
                out = cache.decode_attention(q)
                static = torch.empty_like(out)
                cache.decode_attention_static(q, static)
                H.check_output(static, oracle.decode_chunk(to_numpy_f32(q), counts)[0], f"static {r}")
            else:
                out = cache.decode_chunk(k, v, f, q, cu)
            H.check_output(out, oracle.decode_chunk(to_numpy_f32(q), counts)[0], f"{kind} {r}")
        H.check_state(cache, oracle, wl)
    cache.close()


@pytest.mark.parametrize("D,w,keep", [(128, 16, 0.5), (64, 33, 0.7)])
def test_pruned_entries_do_not_show(D, w, keep):
    """Entries with infinite values that a prune drops stay behind the new end of the list's last half-page;
    they must not show in attention, nor in that of the tokens that lengthen the list again."""
    B, n = 3, 500
    wl = small_workload("pruned", B, 8, 2, D, [0] * B, keep, window=w, seed=D + w)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=900, pool_tokens=B * 2 * 1000), H.make_oracle(wl)
    counts = [n, n - 37, n - 111]
    k, v, f, cu = stream.next_tokens(counts)
    oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
    bad = v.clone()
    for b in range(B):                                # all that the higher threshold drops, but not the window
        rows = slice(cu[b], cu[b + 1] - w)
        bad[rows][f[rows] < 0.5] = float("inf")
    cache.append(k, bad, f, cu)
    tau = float(torch.sigmoid(torch.tensor(0.5)))
    for c in (cache, oracle):
        c.set_tau(tau)
        c.prune()
    assert any(L % 32 for L in oracle.kept_len().ravel())
    for r, kind in enumerate(["attend", "step", "narrow", "wide", "prefill", "step"]):
        n_new = {"attend": 0, "step": 1, "narrow": 3, "wide": 9, "prefill": 40}[kind]
        q = stream.next_query(rows=B * max(1, n_new))
        if n_new:
            k, v, f, cu = stream.next_tokens([n_new] * B)
            oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
        if kind == "attend":
            out = cache.decode_attention(q)
        elif kind == "step":
            out = cache.decode_step(k, v, f, q)
        else:
            out = (cache.prefill_attention if kind == "prefill" else cache.decode_chunk)(k, v, f, q, cu)
        H.check_output(out, oracle.decode_chunk(to_numpy_f32(q), [max(1, n_new)] * B)[0], f"{r}: {kind}")
    H.check_state(cache, oracle, wl)
    cache.close()
