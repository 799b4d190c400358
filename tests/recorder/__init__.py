"""Which kernels the library launches for a call, on the CPU: libspkv.so's host code is run in a
process of its own against hip_recorder.cpp, a HIP runtime that writes launches down.

    calls = record(dict(batch=16, ...), [["append", [4096] * 16], ["lengths", [700] * 128], ["step"]])
    calls[-1].rc, calls[-1].launches      # [("spkv_decode_split<128, 1, 1>", (grid x, grid y), block), ...]

Script entries: ["append" | "chunk" | "score" | "prefill", tokens per sequence] (prefill: and the workspace's bytes), ["step"], ["attend"],
["static"], ["predict", d_model, d_hidden], ["stats"], ["reset"], ["logits", tokens, d_model, d_hidden, heads],
["soft", tokens per sequence], ["advance", n], ["option", id, value], ["destroy"] (last; "stats" has an
entry ("items", (n_work_items, 0), 0)), ["allocations"] (an entry ("allocations", (n, 0), 0): what the library has asked of the host's
allocator since the last such entry); and what the runtime answers from
there on: ["lengths", per pair] (any read-back of device lengths), ["capture", status, error],
["prompt_lengths", 0 | 1] (whether what a prompt sends to the host arrives: of lengths set before it),
["sync_error", error] (of waiting for a stream),
["event_ready", 0 | 1] (whether what is enqueued has run when the call returns), ["watch", kernel, argument, byte] (an entry ("watched", (value, 0), 0) before
every launch of that kernel: the int at that byte of that argument).
"""

import collections
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
LIB = os.path.join(ROOT, "paper_2605_14037_amd", "libspkv.so")

Call = collections.namedtuple("Call", "rc launches")
_dir = None


def _runtime():
    global _dir
    if _dir is None:
        _dir = tempfile.TemporaryDirectory(prefix="hip_recorder")
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", os.path.join(HERE, "hip_recorder.cpp"),
                        "-o", os.path.join(_dir.name, "hip_recorder.so")], check=True)
    return os.path.join(_dir.name, "hip_recorder.so")


def _readable(mangled):
    m = re.match(r"_Z(\d+)", mangled)
    if not m:
        return mangled
    at = m.end()
    name, rest = mangled[at:at + int(m.group(1))], mangled[at + int(m.group(1)):]
    args = re.match(r"I((?:L[a-z]\d+E)+)E", rest)
    if not args:
        return name
    return name + "<" + ", ".join(a[1:] for a in re.findall(r"L([a-z]\d+)E", args.group(1))) + ">"


def record(config, script):
    out = subprocess.run([sys.executable, os.path.join(HERE, "child.py"), _runtime(), LIB],
                         input=json.dumps([config, script]), capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    return [Call(rc, [(_readable(n), (int(x), int(y)), int(b)) for n, x, y, b in ls])
            for rc, ls in json.loads(out.stdout)]
