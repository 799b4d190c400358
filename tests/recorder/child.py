"""Runs one script of calls (see __init__.py) against the recording runtime; no GPU, no torch."""

import ctypes as C
import json
import sys


STATS_ITEMS = 100          # offset of n_work_items in spkv_stats_t: twelve 8-byte fields and device_error before it


class Config(C.Structure):
    _fields_ = [("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32),
                ("head_dim", C.c_int32), ("window", C.c_int32), ("page_tokens", C.c_int32),
                ("tau", C.c_float), ("max_context", C.c_int32), ("max_total_kept_tokens", C.c_int64)]


def main():
    rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # before the library: its names win
    lib = C.CDLL(sys.argv[2])
    config, script = json.load(sys.stdin)
    cfg = Config(**{**dict(n_q_heads=32, n_kv_heads=8, head_dim=128, window=128, page_tokens=0, tau=0.5,
                           max_context=1 << 20, max_total_kept_tokens=1 << 23), **config})
    lib.spkv_cache_required_bytes.restype = C.c_size_t
    lib.spkv_prefill_workspace_bytes.restype = C.c_size_t
    lib.spkv_soft_gated_workspace_bytes.restype = C.c_size_t
    lib.spkv_decode_step_predict_workspace_bytes.restype = C.c_size_t
    need = lib.spkv_cache_required_bytes(C.byref(cfg))
    assert need > 0
    at = C.c_void_p(1 << 40)                          # an aligned address that nothing touches
    handle = C.c_void_p()
    assert lib.spkv_cache_create(C.byref(cfg), at, C.c_size_t(need), None, C.byref(handle)) == 0

    def cu(counts):
        got = [0]
        for n in counts:
            got.append(got[-1] + n)
        return (C.c_int32 * len(got))(*got)

    def taken():
        buf, got = C.create_string_buffer(1024), []
        while rt.rec_take(buf, 1024) >= 0:
            name, x, y, b = buf.value.decode().rsplit(" ", 3)
            got.append([name, x, y, b])
        return got

    taken()
    zero, calls = C.c_float(0.0), []
    for op, *a in script:
        if op == "lengths":
            rows = (C.c_int32 * len(a[0]))(*a[0])
            rt.rec_device_bytes(rows, C.c_size_t(4 * len(a[0])))
            continue
        if op == "watch":
            rt.rec_watch(a[0].encode(), a[1], a[2])
            continue
        if op in ("capture", "event_ready", "prompt_lengths", "sync_error"):
            getattr(rt, "rec_" + op)(*a)
            continue
        if op == "allocations":
            calls.append([0, [["allocations", rt.rec_news(), 0, 0]]])
            continue
        if op == "append":
            rc = lib.spkv_append(handle, at, at, at, cu(a[0]), None)
        elif op == "step":
            rc = lib.spkv_decode_step(handle, at, at, at, at, at, None, zero, None)
        elif op == "attend":
            rc = lib.spkv_decode_attention(handle, at, at, None, zero, None)
        elif op == "static":
            rc = lib.spkv_decode_attention_static(handle, at, at, None, zero, None)
        elif op == "predict":
            ws = lib.spkv_decode_step_predict_workspace_bytes(cfg.batch, a[1])
            rc = lib.spkv_decode_step_predict(handle, at, at, None, at, None, a[0], a[1], at, at, at, at, None,
                                              at, at, C.c_size_t(ws), zero, None)
        elif op == "chunk":
            rc = lib.spkv_decode_chunk(handle, at, at, at, at, cu(a[0]), at, None, zero, None)
        elif op == "score":
            rc = lib.spkv_score_chunk(handle, at, at, at, cu(a[0]), at, None, zero, None)
        elif op == "prefill":
            ws = a[1] if len(a) > 1 else lib.spkv_prefill_workspace_bytes(handle, max(a[0]), C.c_int64(sum(a[0])))
            rc = lib.spkv_prefill_attention(handle, at, at, at, at, cu(a[0]), at, None, zero, at, C.c_size_t(ws), None)
        elif op == "soft":
            ws = lib.spkv_soft_gated_workspace_bytes(cfg.batch, cfg.n_kv_heads, cfg.head_dim, cfg.window, max(a[0]))
            rc = lib.spkv_soft_gated_attention(at, at, at, at, cu(a[0]), cfg.batch, cfg.n_q_heads, cfg.n_kv_heads,
                                               cfg.head_dim, cfg.window, at, None, zero, at, C.c_size_t(ws), None)
        elif op == "logits":
            rc = lib.spkv_utility_logits(at, at, None, at, None, at, at, *a, None)
        elif op == "stats":
            buf = (C.c_byte * 4096)()
            rc = lib.spkv_cache_stats(handle, buf, None, None)
            items = C.c_int32.from_buffer(buf, STATS_ITEMS).value
            calls.append([rc, [["items", items, 0, 0]] + taken()])
            continue
        elif op == "reset":
            rc = lib.spkv_cache_reset(handle, None)
        elif op == "destroy":                             # last of a script
            rc = lib.spkv_cache_destroy(handle)
        elif op == "advance":
            rc = lib.spkv_cache_advance(handle, C.c_int64(a[0]))
        elif op == "option":
            rc = lib.spkv_cache_set_option(handle, a[0], C.c_int64(a[1]))
        else:
            raise ValueError(op)
        calls.append([rc, taken()])
    json.dump(calls, sys.stdout)


main()
