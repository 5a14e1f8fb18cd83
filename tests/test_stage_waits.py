"""The built Group-GEMM kernels wait for every staged k block before the barrier
that publishes it.

A step of the k loop issues the direct-to-LDS loads of the next stage, then the
weight loads of the step after, then waits until at most N loads are left and
passes a barrier.  Vector-memory loads complete in issue order, so the stage has
landed only if at least N load instructions follow its last one on every path.
How many follow is the compiler's doing (it merges adjacent loads), so the count
is read from the generated code."""

import collections
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2505_05799_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
VMEM = ("global_", "buffer_", "scratch_", "flat_")
LANDED = 1 << 30
WINDOW = 14        # instructions between the wait and its barrier, at most


def _objdump():
    for d in ("/opt/rocm/llvm/bin", "/opt/rocm/lib/llvm/bin"):
        if os.path.exists(f"{d}/llvm-objdump"):
            return f"{d}/llvm-objdump"
    return shutil.which("llvm-objdump")


def _code_objects(lib):
    """The gfx950 code objects bundled in the library (one per source file)."""
    b = open(lib, "rb").read()
    at = b.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", b, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", b, p)
            triple = b[p + 24:p + 24 + tlen]
            p += 24 + tlen
            if b"gfx950" in triple and size:
                yield b[at + off:at + off + size]
        at = b.find(MAGIC, at + len(MAGIC))


def _kernels(text):
    """(name, [(address, instruction, encoding)]) of every function."""
    name, ins = None, []
    for line in text.splitlines():
        m = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:", line)
        if m:
            if name:
                yield name, ins
            name, ins = m[1], []
        elif line.startswith("\t") and name:
            t, _, c = line.partition("//")
            a, _, enc = c.strip().partition(":")
            ins.append((int(a, 16), t.strip(), int(enc.split()[0], 16)))
    if name:
        yield name, ins


def _short_waits(ins):
    """(stage waits examined, [(address, loads that may follow the stage, N)])."""
    n = len(ins)
    index = {a: i for i, (a, _, _) in enumerate(ins)}
    kind, succ = [None] * n, [()] * n       # kind: "stage", "load", "barrier" or a wait's count
    for i, (a, t, enc) in enumerate(ins):
        op, _, args = t.partition(" ")
        nxt = (i + 1,) if i + 1 < n else ()
        simm = (enc & 0xFFFF) - ((enc & 0x8000) << 1)
        succ[i] = nxt
        if op == "s_branch":
            succ[i] = (index[a + 4 + 4 * simm],)
        elif op.startswith("s_cbranch"):
            succ[i] = nxt + (index[a + 4 + 4 * simm],)
        elif op == "s_endpgm":
            succ[i] = ()
        elif op == "s_setpc_b64":           # a branch out of the short form's range
            j = i
            while not ins[j][1].startswith("s_getpc_b64 " + args.strip()):
                j -= 1
                assert i - j < 6
            assert ins[j + 1][1].startswith("s_add_u32")
            d = int(ins[j + 1][1].split(",")[-1], 0)
            succ[i] = (index[ins[j + 1][0] + d - ((d & 0x80000000) << 1)],)
        if op.startswith("global_load_lds"):
            kind[i] = "load" if "sc1" in args else "stage"     # (sc1: a finisher's partial sums)
        elif op.startswith(VMEM):
            kind[i] = "load"
        elif op == "s_barrier":
            kind[i] = "barrier"
        elif op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", args)
            kind[i] = int(m[1]) if m else (0 if "cnt" not in args else None)
    stage_waits = set()
    for i in range(n):
        if kind[i] == "barrier":
            for j in range(i - 1, max(i - WINDOW, 0), -1):
                if type(kind[j]) is int:
                    if kind[j] > 0:
                        stage_waits.add(j)
                elif kind[j] is not None or ins[j][1].startswith("ds_"):
                    break
    starts = sorted({0} | {s for i in range(n) if succ[i] != (i + 1,) for s in (*succ[i], i + 1) if s < n})
    block = {s: (s, e) for s, e in zip(starts, starts[1:] + [n])}
    # least number of loads issued since the last stage load, over all paths
    # (LANDED: none outstanding)
    state = {0: LANDED}
    seen, short = set(), {}

    def run(b, c):
        for i in range(*block[b]):
            k = kind[i]
            if k == "stage":
                c = 0
            elif k == "load":
                c = min(c + 1, LANDED)
            elif type(k) is int:
                if i in stage_waits:
                    seen.add(i)
                    # (c = 0: a wait of the compiler's own right behind a tile entry's load)
                    if 0 < c < k:
                        short[i] = (ins[i][0], c, k)
                if k <= c:
                    c = LANDED
        return c

    todo = collections.deque([0])
    while todo:
        b = todo.popleft()
        c = run(b, state[b])
        for s in succ[block[b][1] - 1]:
            if c < state.get(s, LANDED + 1):
                state[s] = c
                todo.append(s)
    return len(seen), list(short.values())


def test_every_stage_lands_before_its_barrier(tmp_path):
    objdump = _objdump()
    if not objdump:
        pytest.skip("no llvm-objdump")
    found, checked = [], 0
    for i, code in enumerate(_code_objects(build.LIB)):
        if b"group_gemm" not in code:
            continue
        f = tmp_path / f"{i}.elf"
        f.write_bytes(code)
        text = subprocess.run([objdump, "-d", str(f)], capture_output=True, text=True, check=True).stdout
        for name, ins in _kernels(text):
            n, short = _short_waits(ins)
            checked += n
            found += [(name, hex(a), f"{c} loads behind the stage, wait for {k}") for a, c, k in short]
    assert checked >= 12 * 20, checked       # 12 kernels, 11 kinds in several configurations each
    assert not found, found
