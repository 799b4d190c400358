"""Which launches the host side chooses for a call, without a GPU (see tests/recorder)."""

import pytest

from tests.recorder import record


def _uneven(pairs, long):
    """Kept lengths of a cache with one dense head in eight, the others sparse."""
    return [long if p % 8 == 0 else long // 20 for p in range(pairs)]


# ------------------------------------------------------------------ short lists
# (a window of 128 tokens is four half-pages, a list of 32 n keys n more; the step may add a key)
@pytest.mark.parametrize("cfg,kept,short", [
    (dict(batch=4), [12 * 32 - 1] * 32, True), (dict(batch=4), [12 * 32] * 31 + [12 * 32 + 1], False),
    (dict(batch=3, n_q_heads=24, n_kv_heads=3, head_dim=64), [20 * 32 - 1] * 9, True),
    (dict(batch=3, n_q_heads=24, n_kv_heads=3, head_dim=64), [20 * 32 + 1] + [0] * 8, False),
    (dict(batch=2, n_q_heads=16, n_kv_heads=1), [4 * 32 - 1] * 2, True), (dict(batch=2, n_q_heads=16, n_kv_heads=1), [129, 0], False),
    (dict(batch=23), [300] * 184, True), (dict(batch=23), [60 * 32] * 184, False),
    (dict(batch=24), [60 * 32 - 1] * 192, True), (dict(batch=24), [60 * 32 + 1] * 192, False),
    (dict(batch=24), [60 * 32 - 1] * 96 + [25 * 32 - 1] * 96, True), (dict(batch=24), [60 * 32] * 96 + [16 * 32] * 96, False)])
def test_short_lists_are_one_launch(cfg, kept, short):
    """Every single-token call alike; an explicit partition, launch count or timing keeps the split kernel."""
    calls = [["step"], ["attend"], ["static"]]
    fill = [["append", [8192] * cfg["batch"]], ["lengths", kept], ["stats"]]
    got = record(cfg, fill + calls)[2:]
    assert [c.rc for c in got] == [0] * 3
    for c in got:
        names = [n for n, _, _ in c.launches if "copy" not in n]
        assert (len(names) == 1 and names[0].startswith("spkv_decode_short<")) == short, names
    for option in ([1, 64], [5, 1], [5, 4], [6, 2], [6, 1]):
        names = [n for c in record(cfg, fill + [["option"] + option] + calls)[3:] for n, _, _ in c.launches]
        assert names and not any("short" in n for n in names)


@pytest.mark.parametrize("call", [["step"], ["attend"], ["static"]])
@pytest.mark.parametrize("cfg,kept,short,captured", [
    (dict(batch=1), [8 * 32] * 8, True, False), (dict(batch=24), [60 * 32 - 1] * 192, True, False),
    (dict(batch=1, n_q_heads=8, n_kv_heads=2, head_dim=64), [10, 10], True, False),
    (dict(batch=1, window=64), [2 * 32 - 1] * 8, True, True), (dict(batch=1, window=64), [2 * 32 + 1] * 8, True, False)])
def test_captured_short_lists(cfg, kept, short, captured, call):
    """A captured step is replayed on lists that grow: 2 pairs of 64 captured at 24 half-pages took 54 us in one
    workgroup each at 384, 18 split."""
    for capture, want in (([0, 0], short), ([1, 0], captured), ([0, 906], captured)):
        script = [["append", [8192] * cfg["batch"]], ["lengths", kept], ["stats"], ["capture"] + capture, call]
        got = record(cfg, script)[-1]
        names = [n for n, _, _ in got.launches if "copy" not in n]
        assert got.rc == 0 and names[0].startswith("spkv_decode_short<") == want, names


@pytest.mark.parametrize("option", [[2, 1], [3, 1]])
def test_what_times_the_split_kernel_is_given_it(option):
    """Timing and split-only take spkv_decode_attention to the split kernel on short lists too, and the work
    items reported are of the kernel that the next such call takes."""
    fill = [["append", [8192]], ["lengths", [300] * 8], ["stats"]]        # 10 half-pages and the window's 4
    plain = record(dict(batch=1), fill + [["stats"], ["attend"], ["step"]])
    other = record(dict(batch=1), fill + [["option"] + option, ["stats"], ["attend"], ["step"]])[1:]
    assert plain[2].launches[0] == ("items", (8 * 8, 0), 0) and other[2].launches[0] == ("items", (8 * 14, 0), 0)
    assert plain[3].launches[0][0].startswith("spkv_decode_short<")
    assert [n for n, _, _ in other[3].launches if "event" not in n][0].startswith("spkv_decode_split<")
    assert plain[4].launches == other[4].launches and plain[4].launches[0][0].startswith("spkv_decode_short<")


# ------------------------------------------------------------------ gapless numbering
@pytest.mark.parametrize("call", [["step"], ["attend"], ["static"], ["score", [4] * 16], ["predict", 4096, 256]])
def test_unanswered_capture_query_leaves_no_error_behind(call):
    """The runtime may refuse to say whether a stream is being captured (the legacy stream while
    another one is: error 906).  The call must go on, and must not find that error when it asks
    whether its own launches went well."""
    setup = [["append", [8192] * 16], ["lengths", _uneven(128, 6000)], ["attend"], ["capture", 0, 906]]
    got = record(dict(batch=16), setup + [call])[-1]
    assert got.rc == 0
    assert got.launches[0][0] in ("spkv_decode_split_compact<128, 1>", "spkv_decode_split_compact<128, 0>",
                                  "spkv_chunk_split<128, 1, 1>",     # the routes that ask
                                  "spkv_decode_split_predict_compact<128>")


@pytest.mark.parametrize("batch,kept,gapless", [
    (16, _uneven(128, 6000), True), (16, [1500] * 128, False), (4, _uneven(32, 6000), False),
    (128, _uneven(1024, 9000), True), (128, _uneven(1024, 5000), False), (129, _uneven(1032, 9000), False)])
def test_gapless_numbering_of_steps(batch, kept, gapless):
    """Uneven lists take it in every single-token call alike, the step with the predictor inside too
    (64 sequences of 1k-64k with dense and local-only heads: 641 us plain, 512 gapless)."""
    calls = [["step"], ["attend"], ["predict", 4096, 256]]
    got = record(dict(batch=batch, max_total_kept_tokens=1 << 26), [["append", [16384] * batch], ["lengths", kept]] + calls)[1:]
    want = ["spkv_decode_split_compact<128, 1>", "spkv_decode_split_compact<128, 0>", "spkv_decode_split_predict_compact<128>"]
    assert [c.rc for c in got] == [0, 0, 0]
    assert [c.launches[0][0] == w for c, w in zip(got, want)] == [gapless] * 3


@pytest.mark.parametrize("batch,kept,gapless", [
    (48, [150] * 384, False),                        # short lists
    (24, [900] * 192, False),                        # 33 half-pages at most
    (24, [1300] * 192, True),
    (24, [5000 if p % 8 == 0 else 100 for p in range(192)], True),     # uneven
    (10, [2400 if p % 8 == 0 else 800 for p in range(80)], True),
    (10, [1300 if p % 8 == 0 else 1000 for p in range(80)], False),    # even, three half-pages an item
    (8, [1200] * 64, True),                          # few pairs
    (8, [600] * 64, False),
    (49, [4000] * 392, False)])                      # more pairs than it pays for
def test_gapless_numbering_of_drafts(batch, kept, gapless):
    """Few items per compute unit make long chains of short lists (192 pairs of 300 keys: 25 us plain,
    28 gapless); the longer and the more unlike the lists, the more there is to gain (80 pairs of
    200 to 2400 keys: 26.5 plain, 24.8 gapless)."""
    got = record(dict(batch=batch), [["append", [8192] * batch], ["lengths", kept], ["score", [4] * batch]])[-1]
    assert got.rc == 0 and got.launches[0][0] == f"spkv_chunk_split<128, 1, {int(gapless)}>"


# ------------------------------------------------------------------ equal shares
def _unlike(pairs, kept):
    return [kept + p for p in range(pairs)]


@pytest.mark.parametrize("cfg,kept,step,chunk", [
    (dict(batch=4), _unlike(32, 1410), True, True), (dict(batch=4), _unlike(32, 1310), False, True),     # 24 and 20 MiB
    (dict(batch=4), _unlike(32, 1100), False, False), (dict(batch=1), _unlike(8, 36800), True, True),    # few pairs: 144
    (dict(batch=1), _unlike(8, 36600), False, True), (dict(batch=64), _unlike(512, 2000), True, True),
    (dict(batch=64), [2000 + p % 8 for p in range(512)], False, False),                                  # copies
    (dict(batch=65), _unlike(520, 2000), False, False),                                                  # too many pairs
    (dict(batch=16, head_dim=64), _unlike(128, 5000), True, True), (dict(batch=16, head_dim=64), _unlike(128, 4800), False, True),
    (dict(batch=16, head_dim=64), _unlike(128, 2900), False, False)])
def test_large_caches_in_equal_shares(cfg, kept, step, chunk):
    """Every single-token call alike, by the kept bytes; an explicit partition or launch count keeps the items."""
    counts = [4] * cfg["batch"]
    script = [["append", [40000] * cfg["batch"]], ["lengths", kept], ["stats"]]
    calls = [["attend"], ["static"], ["step"], ["predict", 4096, 256], ["score", counts], ["chunk", counts]]
    got = record(dict(cfg, max_total_kept_tokens=1 << 27), script + calls)[2:]
    assert [c.rc for c in got] == [0] * 6
    assert [c.launches[0][0].split("<")[0].endswith(("shares", "shares_predict")) for c in got] == [step] * 4 + [chunk] * 2
    for option in ([1, 64], [5, 1], [5, 4], [6, 1]):
        for c in record(dict(cfg, max_total_kept_tokens=1 << 27), script + [["option"] + option] + calls[:3])[3:]:
            assert not [n for n, _, _ in c.launches if "shares" in n]
    if step:        # a workgroup per run, one for the table, those of the predictor
        assert got[0].launches[0][1][0] == 513 and got[3].launches[0][1][0] == 513 + 64 * -(-cfg["batch"] // 16)


@pytest.mark.parametrize("cfg,kept,waves", [
    (dict(batch=1), _unlike(8, 40000), 16), (dict(batch=3, n_q_heads=12, n_kv_heads=4), _unlike(12, 9000), 4),     # 65, 43 of a list
    (dict(batch=3, n_q_heads=12, n_kv_heads=4), [9000 + 100 * (p == 5) + 2000 * (p == 7) + p for p in range(12)], 16),
    (dict(batch=2), [25000 + p if p % 8 == 0 else 500 for p in range(16)], 16),       # one dense head in eight
    (dict(batch=8), [14000 + p if p % 8 == 0 else 500 for p in range(64)], 16), (dict(batch=4), _unlike(32, 3000), 4),
    (dict(batch=9), [14000 + p if p % 8 == 0 else 500 for p in range(72)], 4)])       # more merging workgroups than compute units
def test_merge_of_equal_shares_follows_the_longest_list(cfg, kept, waves):
    """Waves by the most partial results of one list, not by the mean: 16 pairs of 26 MB, one dense head in eight, took
    17.3 us a step merged by four waves and 15.4 by sixteen."""
    script = [["append", [60000] * cfg["batch"]], ["lengths", kept], ["stats"]]
    calls = [["attend"], ["static"], ["step"], ["predict", 4096, 256]]
    got = record(dict(cfg, max_total_kept_tokens=1 << 26), script + calls)[2:]
    assert [c.rc for c in got] == [0] * 4
    d = f"<128, {waves}, 1>", f"<128, 0, {waves}, 1>", f"<128, 1, {waves}, 1>"
    assert [c.launches[1][0] for c in got] == ["spkv_decode_combine" + d[0]] * 2 + ["spkv_combine_append" + d[1], "spkv_combine_append" + d[2]]


@pytest.mark.parametrize("pairs,kept", [(9, 5300), (12, 3900), (16, 2880), (23, 1950), (47, 850)])
def test_equal_shares_from_one_size_on(pairs, kept):
    """24 MiB whatever the number of pairs above eight, in steps with and without the predictor: 12 pairs of 26 MB 13.7 us
    both ways, with the predictor 15.9 in items and 13.8 in shares."""
    for lists, want in ((_unlike(pairs, kept), False), (_unlike(pairs, kept + 64), True)):
        script = [["append", [60000] * pairs], ["lengths", lists], ["stats"], ["step"], ["attend"], ["predict", 4096, 256]]
        got = record(dict(batch=pairs, n_q_heads=8, n_kv_heads=1, max_total_kept_tokens=1 << 25), script)[2:]
        assert [(c.rc, "shares" in c.launches[0][0]) for c in got] == [(0, want)] * 3


@pytest.mark.parametrize("kept,contexts,shares", [
    (_unlike(64, 3000), [16384] * 64, True),
    ([3000 + p * 5 % 63 for p in range(64)], [16384] * 64, False),                        # two lists of one length, no copies
    ([3000 + p * 5 % 63 for p in range(64)], [16384] * 63 + [16385], True),               # ... of unlike contexts
    ([3000] * 64, [16384 + b for b in range(64)], True)])
def test_sequences_of_equal_lengths_keep_the_items(kept, contexts, shares):
    """One KV head: copies of a sequence cannot be told from two whose contexts and kept lengths coincide."""
    calls = [["step"], ["attend"], ["predict", 4096, 256], ["score", [2] * 64]]
    got = record(dict(batch=64, n_q_heads=4, n_kv_heads=1), [["append", contexts], ["lengths", kept], ["stats"]] + calls)[2:]
    assert [(c.rc, "shares" in c.launches[0][0]) for c in got] == [(0, shares)] * 4


@pytest.mark.parametrize("cfg", [dict(batch=64), dict(batch=4), dict(batch=2)])
def test_calls_in_equal_shares_allocate_nothing(cfg):
    """No item partition is worked out (a vector of all pairs and up to 64 passes over it) only to be dropped."""
    pairs, ones = 8 * cfg["batch"], [4] * cfg["batch"]
    script = [["append", [30000] * cfg["batch"]], ["lengths", _unlike(pairs, 6000)], ["stats"], ["step"], ["allocations"]]
    for call in (["step"], ["attend"], ["static"], ["predict", 4096, 256], ["score", ones], ["chunk", ones]):
        script += [call, ["allocations"]]
    got = record(dict(cfg, max_total_kept_tokens=1 << 27), script)[4:]
    assert [c.rc for c in got[::2]] == [0] * 6 and all("shares" in c.launches[0][0] for c in got[::2])
    assert [c.launches[0][1][0] for c in got[1::2]] == [0] * 6


# ------------------------------------------------------------------ utility predictor
@pytest.mark.parametrize("tokens,d_model,d_hidden,kernel", [
    (4096, 4096, 16, "spkv_predictor_hidden"), (4096, 4096, 48, "spkv_predictor_hidden"),
    (6000, 4096, 32, "spkv_predictor_hidden"), (4096, 1024, 32, "spkv_predictor_hidden"),
    (4096, 4096, 64, "spkv_predictor_gemm<1, 64>"), (12000, 512, 16, "spkv_predictor_gemm<1, 64>"), (2048, 4096, 128, "spkv_predictor_hidden"),
    (4096, 4096, 96, "spkv_predictor_gemm<2, 64>"), (12000, 4096, 16, "spkv_predictor_gemm<1, 64>"),
    (6000, 1024, 32, "spkv_predictor_gemm<1, 64>"), (2048, 4096, 256, "spkv_predictor_gemm<4, 64>"),
    (1400, 4096, 256, "spkv_predictor_gemm<4, 64>"), (32768, 4096, 256, "spkv_predictor_gemm<4, 128>"),
    (8192, 4096, 512, "spkv_predictor_tiled"), (8192, 4096, 272, "spkv_predictor_hidden"),
    (1, 128, 16, "spkv_predictor_hidden"), (1 << 24, 128, 256, "spkv_predictor_gemm<4, 128>")])
def test_predictor_kernel_by_size(tokens, d_model, d_hidden, kernel):
    """The staged kernel costs a fixed time and is for calls whose pair of launches costs more;
    narrow hidden layers took up to twice as long in it at 4096 tokens."""
    got = record(dict(batch=1), [["logits", tokens, d_model, d_hidden, 8]])[0]
    assert got.rc == 0 and got.launches[0][0] == kernel


# ------------------------------------------------------------------ bulk append
@pytest.mark.parametrize("batch,window,piece,ring_workgroups,move", [
    (1, 512, 270, 8, 1), (1, 512, 2048, 8, 1), (32, 256, 270, 4, 1), (16, 512, 700, 1, 0),
    (1, 128, 270, 2, 1), (1, 128, 700, 1, 0), (1, 64, 270, 1, 0), (8, 256, 513, 1, 0),
    (7, 256, 513, 4, 1), (64, 513, 4096, 9, 1)])
def test_bulk_append_who_writes_the_ring(batch, window, piece, ring_workgroups, move):
    """One workgroup per pair works through a long ring slowly: few pairs and single segments have
    it spread over workgroups."""
    got = record(dict(batch=batch, window=window), [["append", [piece] * batch]])[0]
    (ring, _, _), (scatter, grid, _) = got.launches
    assert ring == f"spkv_bulk_ring<128, 0, 1, {move}>" and scatter == "spkv_bulk_scatter<128>"
    assert grid == (-(-piece // 512) + ring_workgroups, batch * 8)


@pytest.mark.parametrize("call", [["append", [4096] * 16], ["prefill", [4096] * 16], ["chunk", [16] * 16]])
def test_lengths_are_sent_without_an_event(call):
    """The launch after an event starts 5 to 6 us late, which every append of a prompt would pay for."""
    script = [["append", [4096] * 16], ["lengths", _uneven(128, 4000)], ["chunk", [16] * 16], call]
    for got in record(dict(batch=16), script):
        assert got.rc == 0 and got.launches and not [n for n, _, _ in got.launches if "event" in n]


@pytest.mark.parametrize("arrived", [0, 1])
@pytest.mark.parametrize("call", [["step"], ["attend"], ["predict", 4096, 256], ["chunk", [4] * 16], ["score", [16] * 16]])
def test_first_call_after_a_prompt_is_not_captured(call, arrived):
    """It needs the lengths, and waits for the stream, which a capture refuses: always, not only while the
    prompt still runs.  Outside a capture the lengths that have arrived will do."""
    prompt = [["lengths", _uneven(128, 6000)], ["prompt_lengths", arrived], ["append", [8192] * 16]]
    assert record(dict(batch=16), prompt + [["capture", 1, 0], ["sync_error", 900], call])[-1].rc != 0
    assert record(dict(batch=16), prompt + [["capture", 0, 906], call])[-1].rc == 0
    assert record(dict(batch=16), prompt + [call])[-1].rc == 0


def test_a_cache_is_destroyed_after_its_copies():
    """The pinned buffer is freed when nothing can write it any more: at once where every copy has arrived,
    behind the device where one has not."""
    def end(script):
        return [n for n, _, _ in record(dict(batch=16), script + [["destroy"]])[-1].launches]
    assert end([]) == ["host_free"]
    assert end([["append", [4096] * 16]]) == ["device_sync", "host_free"]
    assert end([["prompt_lengths", 1], ["append", [4096] * 16]]) == ["host_free"]


def test_reset_is_one_launch():
    """A prompt of a small model is fed in two or three launches a piece: three more for the reset
    were a fifth of the time of feeding 4096 tokens."""
    got = record(dict(batch=1, n_q_heads=8, n_kv_heads=2, head_dim=64), [["append", [4096]], ["reset"]])[1]
    assert got.rc == 0 and [name for name, _, _ in got.launches] == ["spkv_reset"]


# ------------------------------------------------------------------ short chunks
def _chunk_grid(call):
    (got,) = [grid[0] for name, grid, _ in call.launches if name.startswith("spkv_prefill_attend")]
    return got


@pytest.mark.parametrize("batch,tokens,kept,grid", [
    (8, 2000, [60 + p % 8 * 70 for p in range(64)], 64 * 5),       # short lists: ranges of every pair
    (1, 2000, [300] * 8, 8 * 3),
    (16, 400, [10] * 128, 128),                                    # nothing worth cutting
    (16, 32768, [3300 + 7600 * (p % 8) // 7 for p in range(128)], 512),    # heads of unlike lists
    (4, 131072, [2600 + 17000 * (p % 8) // 7 for p in range(32)], 512),
    (8, 32768, [30000 if p == 5 else 500 for p in range(64)], 512),        # one dense head
    (64, 8000, [900] * 512, 512)])                                 # more pairs than are cut
def test_short_chunk_ranges(batch, tokens, kept, grid):
    """Ranges of equal length over all pairs cost every workgroup a search: only where the lists are
    long and unlike enough; and the lengths count, not the bound that a prompt has left (all its
    tokens kept), as soon as a copy of them has arrived."""
    chunk = ["chunk", [16] * batch]
    script = [["append", [tokens] * batch], ["lengths", kept], chunk, chunk, chunk]
    calls = record(dict(batch=batch), script)
    assert _chunk_grid(calls[3]) == grid
    copies = [sum(name in ("copy", "spkv_copy_lengths") for name, _, _ in c.launches) for c in calls]
    assert copies == [0, 0, 1, 0]                  # a single chunk after a prompt is not charged for one


@pytest.mark.parametrize("tokens,attend,merge", [
    (4, "spkv_chunk_split<128, 1, 1>", "spkv_chunk_combine<128>"), (8, "spkv_prefill_attend<128, 2, 1, 1>", "spkv_prefill_combine<128>"),
    (16, "spkv_prefill_attend<128, 4, 1, 1>", "spkv_prefill_combine<128>")])
def test_chunks_are_two_launches(tokens, attend, merge):
    """Attention from the cache as it is, then the merge with the append beside it: staging rows and an
    append of its own were 18 of the 118 us of a 16-token chunk.  Drafts the same without the append."""
    counts = [tokens] * 16
    fill = [["append", [32768] * 16], ["lengths", _uneven(128, 20000)], ["stats"]]
    for call, more in ((["chunk", counts], 128), (["score", counts], 0)):
        names = [(n, grid[0]) for n, grid, _ in record(dict(batch=16), fill + [call])[-1].launches if "copy" not in n]
        assert [n for n, _ in names] == [attend, merge]
        assert names[1][1] == more + 128 * (16 if tokens == 4 else tokens * 4 // 8)
    few = record(dict(batch=16), fill + [["append", counts]])[-1].launches
    assert [n for n, _, _ in few] == ["spkv_append_few<128>"]


@pytest.mark.parametrize("group", [1, 2, 3, 5, 8, 16])
def test_every_chunk_length_needs_no_staging_rows(group):
    """spkv_decode_chunk and spkv_score_chunk bring none: all that they accept is attended before its append."""
    cfg = dict(batch=2, n_q_heads=group, n_kv_heads=1, head_dim=64, window=16)
    counts = [n for n in range(1, 18) if n <= 16 and n * group <= 64]
    script = [[op, [n, 0]] for n in counts for op in ("score", "chunk")]
    for (_, (n, _)), got in zip(script, record(cfg, [["append", [900, 900]], ["stats"]] + script)[2:]):
        names = [x for x, _, _ in got.launches if "copy" not in x]
        assert got.rc == 0 and names[0].startswith("spkv_prefill_attend<64," if n * group > 16 else "spkv_chunk_split<64")
        assert n * group <= 16 or names[0].endswith(", 1>"), names
        assert not [x for x in names if "stage" in x or "bulk" in x]
    assert record(cfg, [["score", [17, 0]]])[0].rc != 0


@pytest.mark.parametrize("call", [["chunk", [16] * 16], ["chunk", [4] * 16], ["step"], ["attend"], ["prefill", [16] * 16]])
def test_lengths_on_their_way_are_not_asked_for_by_event(call):
    """A query of an event is refused while a stream of the process is being captured (error 907) and
    ends that capture: a call that finds a copy of the lengths on its way must be able to go into
    a graph, and beside one."""
    chunk = ["chunk", [16] * 16]
    script = [["append", [32768] * 16], ["lengths", _uneven(128, 20000)], chunk, chunk]
    for capturing in (0, 1):
        got = record(dict(batch=16), script + [["capture", capturing, 0], call])
        assert any("copy" in name for name, _, _ in got[2].launches)        # it is on its way
        assert got[3].rc == 0 and not [n for n, _, _ in got[3].launches if n == "event_query"]


def test_ordered_spans_need_no_room_for_ranges():
    """A ragged call whose longest piece alone counts too many spans to be cut took a workspace of staging rows
    and prefix counts; the spans that hold a token are fewer, and are cut where there is room."""
    counts, at_ks = [1024, 10, 10, 10], 52
    rows = -(-sum(counts) * 8 * 4 // 256) * 256 + 32 * -(-(128 + 1024) // 32) * 32 * 128 * 4
    fill = [["append", [30000] * 4], ["lengths", [6000] * 32], ["stats"], ["watch", "spkv_prefill_attend32", 5, at_ks]]
    for more, ks in (([], 2), ([rows], 1)):
        got = record(dict(batch=4), fill + [["prefill", counts] + more])[-1]
        assert got.rc == 0 and [x for n, (x, _), _ in got.launches if n == "watched"] == [ks]
    assert record(dict(batch=4), fill + [["prefill", counts, rows - 256]])[-1].rc != 0


@pytest.mark.parametrize("batch,tokens,pairs_grid", [(8, 2000, 64 * 8), (1, 500, 8 * 4), (64, 4000, 512)])
def test_short_chunk_right_after_a_prompt(batch, tokens, pairs_grid):
    """The bound alone (nothing copied yet) takes the equal ranges for long lists only."""
    got = record(dict(batch=batch), [["append", [tokens] * batch], ["event_ready", 0], ["chunk", [16] * batch]])[1]
    assert _chunk_grid(got) == pairs_grid


@pytest.mark.parametrize("kept,once", [(100, 0), (340, 0), (400, 1), (3000, 1)])
def test_short_chunk_reads_past_the_caches_by_the_kept_bytes(kept, once):
    """512 pairs of 8000 tokens: 128 MB are 8192 tiles of 32 keys, 16 per pair, five of them the
    window's.  The bound after the prompt (2 GB) must not decide."""
    at_ks, at_once = 52, 60                                        # bytes of SpkvPrefill, argument 5
    for at, want in ((at_ks, [1, 1, 1]), (at_once, [0, 0, once])):
        chunk = ["chunk", [16] * 64]
        script = [["append", [8000] * 64], ["lengths", [kept] * 512], ["watch", "spkv_prefill_attend", 5, at],
                  chunk, chunk, chunk]
        calls = record(dict(batch=64), script)[1:]
        assert [x for c in calls for n, (x, _), _ in c.launches if n == "watched"] == want
