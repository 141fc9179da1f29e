"""What the compiler made of a barrier that counts LDS accesses (host only: the
built library is disassembled).

The wavefronts that take the rows of a tile finish wait at a block's end for the
store of the block's bits, not for the loads of the next block behind it:
s_waitcnt lgkmcnt(4), then s_barrier.  LDS accesses of a wavefront complete in
order, so this is right if at least four loads follow the last store on every
path to it."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def kernels(text):
    """name -> [(label or None, instruction text)] of a disassembly with labels."""
    out, body, label = {}, None, None
    for line in text.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:$", line)
        if m and not re.fullmatch(r"L\d+", m.group(1)):
            body, label = out.setdefault(m.group(1), []), None
        elif m:
            label = m.group(1)
        elif line.startswith("\t") and body is not None:
            body.append((label, line.split("//")[0].strip()))
            label = None
    return out


def fewest_loads_behind_a_store(code, at, enough=4):
    """Over all paths to instruction `at`: the fewest LDS loads since the last LDS
    store (at most `enough`; paths without a store count as enough)."""
    into = {}
    for i, (_, ins) in enumerate(code):
        m = re.match(r"s_c?branch\S*\s+(L\d+)", ins)
        if m:
            into.setdefault(m.group(1), []).append(i)
    worst, seen, todo = enough, set(), [(at, 0)]
    while todo:
        i, n = todo.pop()
        if (i, n) in seen or n >= enough:
            continue
        seen.add((i, n))
        label = code[i][0]
        before = list(into.get(label, [])) if label else []
        if i > 0 and not re.match(r"s_(branch|endpgm|setpc)", code[i - 1][1]):
            before.append(i - 1)
        for p in before:
            ins = code[p][1]
            if re.match(r"ds_(write|add|max|min|or|and)", ins):
                worst = min(worst, n)
            else:
                todo.append((p, n + (1 if ins.startswith("ds_read") else 0)))
    return worst


def check(lib, tmp):
    so = shutil.copy(lib, tmp)
    subprocess.check_call([OBJDUMP, "--offloading", os.path.basename(so)], cwd=tmp, stdout=subprocess.DEVNULL)
    found, bad = 0, []
    for f in sorted(os.listdir(tmp)):
        if "gfx950" not in f:
            continue
        text = subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", f], cwd=tmp, text=True)
        for name, code in kernels(text).items():
            for i in range(len(code) - 1):
                if code[i][1] == "s_waitcnt lgkmcnt(4)" and code[i + 1][1] == "s_barrier":
                    found += 1
                    if fewest_loads_behind_a_store(code, i) < 4:
                        bad.append((name, i))
    return found, bad


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_four_loads_follow_the_store_a_counting_barrier_waits_for(tmp_path):
    found, bad = check(os.path.join(ROOT, "paper_1307_7820_amd", "libnf.so"), str(tmp_path))
    assert found >= 2 * 20  # both word counts in k_tile<1..9>, k_stage<1..9, 0>, k_stage<8, 1..2>
    assert bad == []
