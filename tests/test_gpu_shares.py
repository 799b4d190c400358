"""GPU parity of the single-token and multi-token calls on caches that are cut into equal shares, against the oracle."""

import copy

import numpy as np
import pytest
import torch

from paper_2605_14037_amd.inputs import TokenStream, small_workload, to_numpy_f32
from tests import harness as H
from tests.test_gpu_parity import _first_kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hk,G,D,w,ctx,keep", [
    (9, 1, 4, 128, 100, [9000, 1, 0, 17, 3000, 9001, 20000, 99, 14000], 1.0),         # long and empty lists mixed
    (2, 4, 16, 128, 64, [46000, 29000], 1.0),                                         # few pairs, many partial results each
    (64, 8, 1, 128, 16, [0 if b % 5 == 2 else 7 + 13 * b for b in range(64)], 0.35),  # 512 pairs, most end inside a run
    (23, 3, 5, 128, 2300, [2299 + 37 * b for b in range(23)], 0.2),                   # rings of more half-pages than lists
    (4, 5, 2, 64, 300, [45000, 20100, 39000, 33003], 1.0)])                           # four half-pages in registers
def test_equal_shares(B, Hk, G, D, w, ctx, keep):
    """Steps with and without the predictor, attention, the static variant, drafts and chunks (ragged, some
    sequences bring none), and a step replayed from a graph."""
    rates = np.full((B, Hk), keep)
    if keep < 1:
        rates[:, 0], rates[::3, 1:2] = 1.0, 0.0
    wl = small_workload("shares", B, Hk * G, Hk, D, ctx, rates, window=w, seed=B + D)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl, extra_context=60, pool_tokens=sum(ctx) * Hk + B * Hk * 64), H.make_oracle(wl)
    H.prefill(cache, oracle, stream, wl, 4096)
    held = list(ctx)

    def bring(counts):
        k, v, f, cu = stream.next_tokens(counts)
        return k, v, f, cu, stream.next_query(rows=sum(counts))

    def mirror(k, v, f, cu):
        oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
        for b in range(B):
            held[b] += cu[b + 1] - cu[b]

    def check(got, q, label):
        out, lse = oracle.decode(to_numpy_f32(q))
        H.check_output(got[0], out, label)
        H.check_lse(got[1], lse, label)

    one = [1] * B
    for step in range(2):
        k, v, f, cu, q = bring(one)
        assert _first_kernel(cache, wl, held, ["step"]).startswith("spkv_decode_shares<")
        got = cache.decode_step(k, v, f, q, want_lse=True)
        mirror(k, v, f, cu)
        check(got, q, f"step {step}")

    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(B, 256, generator=g, device="cuda").to(torch.bfloat16)
    w1 = (torch.randn(32, 256, generator=g, device="cuda") / 16).to(torch.bfloat16)
    w2 = (torch.randn(Hk, 32, generator=g, device="cuda") / 4).to(torch.bfloat16)
    k, v, _, cu, q = bring(one)
    assert _first_kernel(cache, wl, held, ["predict", 256, 32]).startswith("spkv_decode_shares_predict<")
    out, lse, logits = cache.decode_step_predict(x, w1, None, w2, None, k, v, q, want_lse=True)
    mirror(k, v, logits, cu)
    check((out, lse), q, "step with the predictor")

    k, v, f, cu, q = bring(one)
    H.feed(cache, None, k, v, f, cu)
    mirror(k, v, f, cu)
    check(cache.decode_attention(q, want_lse=True), q, "attention")
    static, lse = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
    cache.decode_attention_static(q, static, lse)
    check((static, lse), q, "static")

    most = 16 // G
    for counts in ([most if b % 3 else 0 for b in range(B)], [1 + b % most for b in range(B)]):
        k, v, f, cu, q = bring(counts)
        assert _first_kernel(cache, wl, held, ["score", counts]).startswith("spkv_chunk_shares<")
        trial = copy.deepcopy(oracle)
        trial.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
        ref_out, ref_lse = trial.decode_chunk(to_numpy_f32(q), counts)
        for call in (lambda: cache.score_chunk(k, v, q, cu, want_lse=True),
                     lambda: cache.decode_chunk(k, v, f, q, cu, want_lse=True)):
            out, lse = call()
            H.check_output(out, ref_out, f"chunk {counts}")
            H.check_lse(lse, ref_lse, f"chunk {counts}")
        mirror(k, v, f, cu)

    H.check_state(cache, oracle, wl, pairs=[(0, 0), (B - 1, Hk - 1)])       # reads the lengths: nothing on its way
    bufs = [torch.empty_like(t) for t in bring(one)[:3]]
    qs, outs = torch.empty(B, Hk * G, D, dtype=torch.bfloat16, device="cuda"), torch.empty(B, Hk * G, D, dtype=torch.bfloat16, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cache.decode_step(*bufs, qs, out=outs)
    for i in range(4):
        k, v, f, cu, q = bring(one)
        for dst, src in zip(bufs + [qs], (k, v, f, q)):
            dst.copy_(src)
        if i > 0:
            cache.advance(1)
        graph.replay()
        mirror(k, v, f, cu)
        torch.cuda.synchronize()
        H.check_output(outs, oracle.decode(to_numpy_f32(q))[0], f"replay {i}")
    H.check_state(cache, oracle, wl, pairs=[(0, 0), (B - 1, Hk - 1)])
    cache.close()
