"""GPU parity of chunks of up to 16 tokens that are attended before their append (decode_chunk, score_chunk
and prefill_attention with more than 16 columns), and of the append of a few tokens, against the oracle."""

import copy

import numpy as np
import pytest
import torch

import paper_2605_14037_amd as spkv
from paper_2605_14037_amd.inputs import TokenStream, small_workload, to_numpy_f32
from tests import harness as H
from tests.test_gpu_parity import _first_kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hk,G,D,w,ctx,n,kernel", [
    (2, 4, 128, 128, [0, 1, 127, 128, 2500], 16, "128, 4, 1, 1"),      # empty, filling and full rings
    (2, 4, 64, 16, [0, 15, 16, 17, 900], 16, "64, 4, 1, 1"),           # the chunk replaces the window
    (2, 3, 128, 100, [33, 99, 100, 101, 700], 7, "128, 2, 1, 1"),      # two waves, 15 of 16 columns
    (1, 6, 64, 33, [5, 32, 33, 34, 1200], 10, "64, 4, 2, 1"),          # two column groups a wave
    (1, 8, 128, 250, [0, 100, 249, 250, 1500], 16, "128, 4, 2, 1"),    # 128 columns: prefill alone takes them
    (1, 16, 64, 1100, [200, 1023, 1025, 1100, 4000], 4, "64, 4, 1, 1")])      # gates past the first 1024 slots
def test_chunks_attended_before_their_append(Hk, G, D, w, ctx, n, kernel):
    """Scored, decoded and prefilled chunks, ragged and with sequences that bring none, against the oracle;
    outputs of a chunk scored first and then decoded are the same bits."""
    B = len(ctx)
    wl = small_workload("direct", B, Hk * G, Hk, D, ctx, 0.4, window=w, seed=w + G)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=100, pool_tokens=B * Hk * 5000), H.make_oracle(wl)
    H.prefill(cache, oracle, stream, wl, 4096)
    held = list(ctx)
    calls = ["decode", "prefill", "decode"] if n * G <= 64 else ["prefill", "prefill"]
    for r, call in enumerate(calls):
        counts = [n] * B if r == 0 else [n, 0, 1, n, max(1, n // 2)]
        k, v, f, cu = stream.next_tokens(counts)
        q = stream.next_query(rows=sum(counts))
        script = ["chunk" if call == "decode" else "prefill", counts]
        assert _first_kernel(cache, wl, held, script) == f"spkv_prefill_attend<{kernel}>"
        trial = copy.deepcopy(oracle)
        trial.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
        ref_out, ref_lse = trial.decode_chunk(to_numpy_f32(q), counts)
        scored = None
        if n * G <= 64:
            scored, lse = cache.score_chunk(k, v, q, cu, want_lse=True)
            H.check_output(scored, ref_out, f"scored {counts}")
            H.check_lse(lse, ref_lse, f"scored {counts}")
            H.check_state(cache, oracle, wl, label="scoring changes nothing")
        args = (k, v, f, q, cu)
        out, lse = (cache.decode_chunk if call == "decode" else cache.prefill_attention)(*args, want_lse=True)
        oracle = trial
        H.check_output(out, ref_out, f"{call} {counts}")
        H.check_lse(lse, ref_lse, f"{call} {counts}")
        H.check_state(cache, oracle, wl, label=f"{call} {counts}")
        held = [h + c for h, c in zip(held, counts)]
    cache.close()


def test_wide_window_in_one_workgroup():
    """512 pairs are not cut into ranges: the workgroup of the one that holds a sequence meets more ring tiles
    than it keeps gates of."""
    B, w, n = 64, 8300, 10
    wl = small_workload("wide", B, 16, 8, 64, [w + 150] + [0] * (B - 1), 0.4, window=w, seed=9)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=100, pool_tokens=8 * 400), H.make_oracle(wl)
    H.prefill(cache, oracle, stream, wl, 4096)
    counts = [n] + [0] * (B - 1)
    k, v, f, cu = stream.next_tokens(counts)
    q = stream.next_query(rows=n)
    assert _first_kernel(cache, wl, list(wl.ctx_lens), ["chunk", counts]) == "spkv_prefill_attend<64, 2, 1, 1>"
    scored = cache.score_chunk(k, v, q, cu)
    out = cache.decode_chunk(k, v, f, q, cu)
    assert torch.equal(scored, out)
    oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
    H.check_output(out, oracle.decode_chunk(to_numpy_f32(q), counts)[0], "wide window")
    cache.close()


def test_stale_ring_slots_do_not_show():
    """A released sequence leaves its rows in the ring; infinite ones must not show in the chunks of the
    sequence that takes its place while its own ring is filling."""
    wl = small_workload("stale", 2, 8, 2, 128, [0, 0], 0.5, window=64, seed=3)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=400, pool_tokens=4000), H.make_oracle(wl)
    k, v, f, cu = stream.next_tokens([64, 64])
    bad = torch.full_like(v, float("inf"))
    cache.append(k, bad, f, cu)
    for b in range(2):
        cache.release_sequence(b)
    for counts in ([9, 16], [16, 5], [1, 16]):
        k, v, f, cu = stream.next_tokens(counts)
        q = stream.next_query(rows=sum(counts))
        out = cache.decode_chunk(k, v, f, q, cu)
        oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
        H.check_output(out, oracle.decode_chunk(to_numpy_f32(q), counts)[0], str(counts))
    H.check_state(cache, oracle, wl)
    cache.close()


@pytest.mark.parametrize("D,w,sinks,keep", [(128, 16, 0, 1.0), (64, 17, 3, 0.5), (128, 60, 20, 0.0), (64, 128, 0, 1.0)])
def test_few_tokens_appended_over_page_boundaries(D, w, sinks, keep):
    """Chunks of 1 to 16 tokens from the empty cache on, across the filling of the window and the pages, with
    recycled pages handed out first; ragged, some sequences bring none."""
    B, rng = 3, np.random.default_rng(w)
    wl = small_workload("few", B, 4, 2, D, [0] * B, keep, window=w, seed=w + D)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=600, pool_tokens=B * 2 * 600), H.make_oracle(wl)
    if sinks:
        cache.set_option(spkv.OPT_SINK_TOKENS, sinks)
        oracle.n_sink = sinks
    else:                                              # pages to recycle
        k, v, f, cu = stream.next_tokens([200, 150, 0])
        cache.append(k, v, f, cu)
        for b in range(B):
            cache.release_sequence(b)
    for r in range(30):
        counts = [int(rng.integers(0, min(16, w) + 1)) for _ in range(B)]
        if r % 7 == 0:
            counts = [min(16, w)] * B
        if sum(counts) == 0:
            continue
        k, v, f, cu = stream.next_tokens(counts)
        H.feed(cache, oracle, k, v, f, cu)
        if r % 5 == 4:
            H.check_state(cache, oracle, wl, label=f"round {r}")
    k, v, f, cu = stream.next_tokens([1] * B)
    q = stream.next_query()
    out = cache.decode_step(k, v, f, q)
    oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
    H.check_output(out, oracle.decode(to_numpy_f32(q))[0], "decode of what was appended")
    H.check_state(cache, oracle, wl)
    cache.close()


@pytest.mark.parametrize("Hk,G,D,n", [(2, 4, 128, 16), (2, 4, 64, 16), (3, 8, 64, 7), (1, 16, 128, 4), (2, 4, 128, 4)])
def test_weights_of_the_chunk_itself_are_32_bit(Hk, G, D, n):
    """Drafts on an empty cache see nothing but each other: with weights and sums in 32 bits an output is the
    64-bit one rounded to bf16, but for those within some 2^-20 of the middle between two (fewer than one
    in 500); with weights of 8 bits one in five is another one."""
    wl = small_workload("own", 4, Hk * G, Hk, D, [0] * 4, 0.5, window=64, seed=D + n)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=100), H.make_oracle(wl)
    counts = [n, n, 1, n - 1]
    k, v, f, cu = stream.next_tokens(counts)
    q = stream.next_query(rows=sum(counts))
    oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
    ref = torch.from_numpy(oracle.decode_chunk(to_numpy_f32(q), counts)[0])
    for out in (cache.score_chunk(k, v, q, cu), cache.decode_chunk(k, v, f, q, cu)):
        other = float((out.cpu() != ref.to(torch.bfloat16)).double().mean())
        assert other < 0.01, other
    cache.close()
