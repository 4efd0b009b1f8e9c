"""The compiled kernels of libqap.so, read back as assembly: a wave comes to a barrier only
after a wait for its own LDS operations.  (The wait that __syncthreads stands for is one the
compiler may drop, and in block-form kernels it dropped it at the head of a loop: other waves
could read what a write had not reached yet, or write what a read had not fetched.)"""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2307_11248_amd import qap

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump"))
                if p and os.path.exists(p)), None)


def unwaited(code):
    """Addresses of the barriers that some path reaches with an LDS operation of the wave not
    waited for.  `code`: (address, operation, operands) of one function, in order."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    succ = []
    for i, (a, op, args) in enumerate(code):
        nxt = [i + 1] if i + 1 < len(code) else []
        if op in ("s_branch",) or op.startswith("s_cbranch"):
            to = a + 4 + 4 * ((int(args.split()[0]) + 0x8000) % 0x10000 - 0x8000)
            nxt = ([] if op == "s_branch" else nxt) + [at[to]]
        elif op in ("s_endpgm", "s_setpc_b64"):
            nxt = []
        succ.append(nxt)
    seen = [set() for _ in code]          # the states (pending or not) an operation was reached in
    work, bad = [(0, False)], set()
    while work:
        i, pending = work.pop()
        if pending in seen[i]:
            continue
        seen[i].add(pending)
        a, op, args = code[i]
        if op.startswith("ds_"):
            pending = True
        elif op == "s_waitcnt" and (args.split("//")[0].strip() == "0" or "lgkmcnt(0)" in args):
            pending = False
        elif op == "s_barrier" and pending:
            bad.add(a)
        work.extend((j, pending) for j in succ[i])
    return bad


def functions(text):
    name, code = None, []
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
        if m:
            if name:
                yield name, code
            name, code = m.group(1), []
            continue
        m = re.match(r"\t(\w+)(.*?)// ([0-9A-F]+):", line)
        if m:
            code.append((int(m.group(3), 16), m.group(1), m.group(2).strip()))
    if name:
        yield name, code


def test_the_check_finds_a_dropped_wait():
    loop = [(0, "s_waitcnt", "lgkmcnt(0)"), (4, "s_barrier", ""), (8, "ds_read_b32", "v0, v0"),
            (12, "s_waitcnt", "lgkmcnt(0)"), (16, "ds_write_b32", "v1, v0"), (20, "s_cbranch_scc1", "65531"),
            (24, "s_endpgm", "")]
    assert unwaited(loop) == {4}           # the branch goes to the barrier
    loop[5] = (20, "s_cbranch_scc1", "65530")
    assert unwaited(loop) == set()         # to the wait before it


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_barriers_wait_for_lds_operations(tmp_path):
    lib = shutil.copy(qap.LIB_PATH, str(tmp_path / "libqap.so"))
    subprocess.check_call([OBJDUMP, "--offloading", lib], cwd=str(tmp_path), stdout=subprocess.DEVNULL)
    objs = [p for p in sorted(glob.glob(str(tmp_path / "*gfx950"))) if os.path.getsize(p)]
    assert objs
    kernels, barriers, bad = 0, 0, {}
    for p in objs:
        text = subprocess.run([OBJDUMP, "-d", p], capture_output=True, text=True, check=True).stdout
        for name, code in functions(text):
            kernels += 1
            barriers += sum(op == "s_barrier" for _, op, _ in code)
            b = unwaited(code)
            if b:
                bad[name] = sorted(hex(x) for x in b)
    assert kernels > 50 and barriers > 500
    assert not bad, bad
