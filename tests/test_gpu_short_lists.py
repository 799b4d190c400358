"""GPU parity of the single-token calls on short lists (spkv_decode_short: a workgroup per
(sequence, KV head), one launch), against the fp64 oracle."""

import numpy as np
import pytest
import torch

import paper_2605_14037_amd as spkv
from paper_2605_14037_amd.inputs import TokenStream, small_workload, to_numpy_f32
from tests import harness as H
from tests.test_gpu_parity import _first_kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hk,G,D,w,top", [
    (7, 2, 1, 128, 128, 500), (7, 1, 16, 128, 100, 200), (8, 3, 8, 64, 33, 730), (7, 1, 5, 128, 1, 475),
    (9, 2, 4, 64, 250, 755), (7, 4, 3, 128, 64, 505), (30, 8, 4, 128, 64, 900), (7, 1, 9, 64, 96, 760)])
def test_short_lists_against_the_oracle(B, Hk, G, D, w, top):
    """Sequences from empty to the longest that is taken, list and window ends on and beside the edges of
    half-pages and rounds of waves, heads that keep all, none and some; the fused step from empty and full
    windows (the pair that leaves them kept and dropped), the two-call step, the static variant."""
    rng = np.random.default_rng(B * G + w)
    edges = [0, 1, w - 1, w, w + 1, w + 32, w + 33, top]
    ctx = [min(top, edges[b]) if b < len(edges) else int(rng.integers(top * 9 // 10, top)) for b in range(B)]
    ctx[-1] = top
    keep = np.array([[(1.0, 0.4, 0.0)[(b + h) % 3] if B < 20 else 1.0 for h in range(Hk)] for b in range(B)])
    keep[-1] = 1.0
    wl = small_workload("short", B, Hk * G, Hk, D, ctx, keep, window=w, decode_steps=6, seed=B + w)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl), H.make_oracle(wl)
    H.prefill(cache, oracle, stream, wl, 4096)
    for step in range(5):
        k, v, f, cu = stream.next_tokens([1] * B)
        q = stream.next_query()
        assert "short" in _first_kernel(cache, wl, [c + step for c in ctx], ["step"])
        if step < 4:
            out, lse = cache.decode_step(k, v, f, q, want_lse=True)
            oracle.append(to_numpy_f32(k), to_numpy_f32(v), to_numpy_f32(f), cu)
        else:
            H.feed(cache, oracle, k, v, f, cu)
            out, lse = cache.decode_attention(q, want_lse=True)
        ref_out, ref_lse = oracle.decode(to_numpy_f32(q))
        H.check_output(out, ref_out, f"step {step}")
        H.check_lse(lse, ref_lse, f"step {step}")
    static = torch.empty_like(out)
    cache.decode_attention_static(q, static)
    assert torch.equal(static, out)
    H.check_state(cache, oracle, wl)
    cache.close()


def test_captured_step_outgrows_the_short_lists():
    """A captured step stays right however long the lists get while it is replayed: past the lengths that
    would be chosen for it, and past the 64 pages whose ids a wave holds at a time."""
    n = 4250
    wl = small_workload("growth", 1, 4, 1, 64, [40], 1.0, window=32, decode_steps=n + 2, seed=5)
    stream = TokenStream(wl, device="cuda")
    cache, oracle = H.make_cache(wl), H.make_oracle(wl)
    H.prefill(cache, oracle, stream, wl, 4096)
    k, v, f, cu = stream.next_tokens([n])
    q = stream.next_query()
    ks, vs, fs = k[:1].clone(), v[:1].clone(), f[:1].clone()
    out = torch.empty_like(q)
    assert cache.safe_steps() >= n
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):                     # records the launch; runs nothing
        cache.decode_step(ks, vs, fs, q, out=out)
    done = 0
    for stop in (1, 300, 2100, n):                    # one, 11, 67 and 134 half-pages
        for i in range(done, stop):
            for dst, src in ((ks, k), (vs, v), (fs, f)):
                dst.copy_(src[i:i + 1])
            graph.replay()
        oracle.append(to_numpy_f32(k[done:stop]), to_numpy_f32(v[done:stop]), to_numpy_f32(f[done:stop]), [0, stop - done])
        torch.cuda.synchronize()
        H.check_output(out, oracle.decode(to_numpy_f32(q))[0], f"after {stop} replays")
        done = stop
    cache.advance(n - 1)                              # the captured call itself counted one step
    H.check_state(cache, oracle, wl)
    cache.close()
