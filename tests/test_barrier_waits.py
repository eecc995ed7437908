"""No LDS operation of a wave is in flight at a workgroup barrier, in the built code of
every kernel: past a barrier other waves may overwrite what this one was reading (by
direct loads into the next stage, or a tile's transposition), and a barrier does not
wait by itself.  Walks the control flow of each kernel's disassembly, counting LDS
operations since the last lgkmcnt wait."""
import os
import re
import shutil
import subprocess

import pytest

from tests.test_abi_host_sanitized import _objects

LLVM = "/opt/rocm/llvm/bin"


def kernels(objdump, obj, tmp):
    """{kernel: [(address, mnemonic, operands, branch target or None)]} of an object's gfx950 code."""
    o = shutil.copy(obj, tmp)
    subprocess.run([objdump, "--offloading", o], capture_output=True, check=True)
    code = [os.path.join(tmp, f) for f in os.listdir(tmp) if f.startswith(os.path.basename(o) + ".") and f.endswith("gfx950")]
    got, base = {}, {}
    for f in code:
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", f], capture_output=True, text=True, check=True).stdout
        cur = None
        for line in text.split("\n"):
            m = re.match(r"^([0-9a-f]+) <(.*)>:", line)
            if m:
                cur = m.group(2)
                got[cur], base[cur] = [], int(m.group(1), 16)
                continue
            m = re.match(r"^\s+(\S+)(.*)//\s*([0-9A-F]+):(.*)", line)
            if m and cur:
                t = re.search(r"<(\S+?)(?:\+0x([0-9a-f]+))?>", m.group(4))
                to = base[cur] + int(t.group(2) or "0", 16) if t and t.group(1) == cur else None
                got[cur].append((int(m.group(3), 16), m.group(1), m.group(2), to))
    return got


def in_flight(code):
    """(barriers, the most LDS operations in flight at one)."""
    at = {c[0]: i for i, c in enumerate(code)}
    state, work, most, bars = [-1] * len(code), [(0, 0)], 0, 0
    bars = sum(op == "s_barrier" for _, op, _, _ in code)
    while work:
        i, n = work.pop()
        if i is None or i >= len(code) or state[i] >= n:
            continue
        state[i] = n
        _, op, args, to = code[i]
        if op.startswith("ds_"):
            n = min(n + 1, 99)
        elif op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", args)
            n = min(n, int(m.group(1))) if m else n
        elif op == "s_barrier":
            most = max(most, n)
        if op in ("s_endpgm", "s_setpc_b64"):
            continue
        if op == "s_branch" or op.startswith("s_cbranch"):
            work.append((at.get(to), n))
        if op != "s_branch":
            work.append((i + 1, n))
    return bars, most


def test_nothing_in_flight_at_barriers(tmp_path):
    objdump = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("llvm-objdump not found")
    seen, bad = 0, []
    for obj in _objects():
        for name, code in kernels(objdump, obj, str(tmp_path)).items():
            bars, most = in_flight(code)
            seen += bars
            if most:
                bad.append(f"{most} LDS operations in flight at a barrier of {name}")
    assert seen > 1000
    assert not bad, "\n".join(bad)
