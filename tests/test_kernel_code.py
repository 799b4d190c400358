"""Orders inside a kernel that no run shows reliably, read from the gfx950 code of libspkv.so as it was built
(the test walks the branches of the disassembly; no GPU)."""

import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_14037_amd", "libspkv.so")
LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """{kernel: {address: (mnemonic, branch target or None, next address)}}"""
    if not os.path.exists(LIB) or shutil.which("llvm-objdump", path=LLVM) is None:
        pytest.skip("needs the built library and llvm-objdump")
    at = tmp_path_factory.mktemp("code")
    bundles = str(at / "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={bundles}", LIB, str(at / "copy.so")], check=True)
    data, found, kernels = open(bundles, "rb").read(), -1, {}
    while (found := data.find(b"__CLANG_OFFLOAD_BUNDLE__", found + 1)) >= 0:
        entry = found + 32
        for _ in range(struct.unpack_from("<Q", data, found + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + name]
            entry += 24 + name
            if b"gfx950" not in target:
                continue
            (at / "object").write_bytes(data[found + offset:found + offset + size])
            text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", str(at / "object")], check=True, capture_output=True,
                                  text=True).stdout
            kernels.update(_parse(text))
    assert kernels
    return kernels


def _parse(text):
    kernels, body, start, last = {}, None, 0, None
    for line in text.splitlines():
        if m := re.match(r"([0-9a-f]+) <(.+)>:$", line):
            start, last = int(m.group(1), 16), None
            body = kernels.setdefault(m.group(2), {})
        elif body is not None and (m := re.match(r"\s+(\S+).*// ([0-9A-F]{12}):", line)):
            addr = int(m.group(2), 16)
            to = re.search(r"<[^>+]+(?:\+0x([0-9a-f]+))?>", line) if "branch" in m.group(1) else None
            if last is not None:
                body[last] = body[last][:2] + (addr,)
            body[addr] = (m.group(1), start + int(to.group(1) or "0", 16) if to else None, None)
            last = addr
    return kernels


def _first_stores(body):
    """Addresses of memory writes that some path from the entry reaches before a barrier."""
    todo, seen, stores = [min(body)], set(), []
    while todo:
        addr = todo.pop()
        if addr is None or addr in seen:
            continue
        seen.add(addr)
        op, target, after = body[addr]
        if op == "s_barrier" or op == "s_endpgm":
            continue
        if re.match(r"(global|flat|buffer)_(store|atomic)", op):
            stores.append(hex(addr))
        todo += [target] if op == "s_branch" else [target, after]
    return stores


@pytest.mark.parametrize("kernel", ["spkv_append_stepILi128E", "spkv_combine_appendILi128ELb0ELi4E",
                                    "spkv_combine_appendILi64ELb0ELi4E"])
def test_single_token_append_stores_after_every_wave_has_read(code, kernel):
    """Wave 0 advances the counters, the ring's logit and its rows: a wave that starts late must not find
    them advanced already."""
    bodies = [b for name, b in code.items() if kernel in name]
    assert bodies
    for body in bodies:
        assert any(op == "s_barrier" for op, _, _ in body.values())
        assert _first_stores(body) == []


@pytest.mark.parametrize("head_dim", [128, 64])
def test_soft_gated_loop_lies_where_it_was_measured(code, head_dim):
    """The same instructions took up to 1 % longer at other places in a 32-byte line of instructions.  The
    loop is the one of two half-pages' products."""
    (body,) = [b for name, b in code.items() if f"spkv_prefill_attend32ILi{head_dim}ELb1E" in name]
    heads = {to for at, (_, to, _) in body.items() if to is not None and to <= at
             and sum(to <= a <= at and "mfma" in body[a][0] for a in body) == head_dim // 4}
    assert len(heads) == 1 and heads.pop() % 32 == 16
