"""Counted waits, in the code that the compiler made (no GPU).

k_backward_dq waits for the copies of its second block while the kept weights of the next pair, asked for after them, stay in
flight: `s_waitcnt vmcnt(5)` stands for four asynchronous copies and one ordinary load, the metadata.  The copies are
assembly statements and keep their order.  The load is the compiler's to move: issued before the copies that are waited for, or
after the wait, it would leave one of these outstanding.  So it is looked up in the built library: in the kernel's loop it has to
stand among the last five loads of a basic block, and no other load may come between these and the wait.
"""
import os
import re
import shutil
import subprocess

import pytest

import paper_2203_00091_amd as dfss

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
pytestmark = pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(dfss.library_path())),
                                reason="needs llvm-objdump and the built library")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: [(address, instruction, address it may branch to or None), ...]} of every k_backward_dq."""
    d = tmp_path_factory.mktemp("code")
    shutil.copy(dfss.library_path(), d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    found = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        if b"k_backward_dq" not in (d / f).read_bytes():
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"([0-9a-f]{16}) <(\S+)>:", line)
            if m:
                name, base = m[2], int(m[1], 16)
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):.*?(?:<\S+?\+0x([0-9a-f]+)>)?$", line)
            if m and name and "k_backward_dq" in name:
                found.setdefault(name, []).append((int(m[2], 16), m[1], base + int(m[3], 16) if m[3] and "branch" in m[1] else None))
    return found


def _copies_stay_behind_the_wait(code):
    """None, or what is wrong."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    after = []      # of every instruction: those that may follow
    for i, (_, x, to) in enumerate(code):
        # (s_cbranch_execnz stands for a jump: a wave that runs has lanes)
        n = [] if x.startswith(("s_endpgm", "s_branch", "s_cbranch_execnz")) else [i + 1]
        after.append([j for j in n + ([at[to]] if to is not None else []) if j < len(code)])
    starts = {0} | {j for i, js in enumerate(after) if code[i][2] is not None for j in js} | \
             {i + 1 for i, (_, x, _) in enumerate(code) if "branch" in x and i + 1 < len(code)}

    def kind(i):    # C: asynchronous copy, L: ordinary load, S: store
        m = re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)(_lds)?", code[i][1])
        return "" if not m else "C" if m[3] else "L" if m[2] == "load" else "S"

    def reach(i):
        seen, todo = set(), list(after[i])
        while todo:
            j = todo.pop()
            if j not in seen:
                seen.add(j)
                todo += after[j]
        return seen

    loads = [i for i in range(len(code)) if kind(i) == "L" and i in reach(i)]
    if len(loads) != 1:
        return f"{len(loads)} ordinary loads in the loop"
    end = loads[0]
    while end + 1 not in starts:
        end += 1
    begin = loads[0]
    while begin not in starts:
        begin -= 1
    block = [i for i in range(begin, end + 1) if kind(i)]
    if sorted(kind(i) for i in block[-5:]) != ["C"] * 4 + ["L"]:
        return "the block of the load ends in " + "".join(kind(i) for i in block)
    # on the way to the counted wait
    waits, seen, todo = 0, set(), [(j, False) for j in after[end]]
    while todo:
        j, more = todo.pop()
        if (j, more) in seen:
            continue
        seen.add((j, more))
        m = re.match(r"s_waitcnt.*vmcnt\((\d+)\)", code[j][1])
        if m and int(m[1]) == 0:
            continue
        if m:
            if int(m[1]) != 5 or more:
                return f"{code[j][1]} {'behind another load' if more else ''}"
            waits += 1
            continue
        todo += [(k, more or kind(j) != "") for k in after[j]]
    return None if waits else "no counted wait behind the load"


def test_the_load_that_the_wait_counts_is_where_it_is_counted(kernels):
    assert len(kernels) >= 12
    for name, code in kernels.items():
        assert _copies_stay_behind_the_wait(code) is None, name


def test_a_load_elsewhere_is_found(kernels):
    """The check itself: the load hoisted out of its place, or sunk behind the wait."""
    for name, code in kernels.items():
        texts = [x for _, x, _ in code]
        wait = max(i for i, x in enumerate(texts) if x == "s_waitcnt vmcnt(5)")
        load = max(i for i, x in enumerate(texts[:wait]) if x.startswith("global_load_dwordx4"))
        copies = [i for i in range(load) if texts[i].startswith("global_load_lds")]

        def with_load_at(j):
            return [(a, texts[load] if i == j else "s_nop 0" if i == load else x, to) for i, (a, x, to) in enumerate(code)]

        assert _copies_stay_behind_the_wait(with_load_at(load)) is None, name
        assert _copies_stay_behind_the_wait(with_load_at(wait + 1)) is not None, name
        assert _copies_stay_behind_the_wait(with_load_at(copies[-5] - 1)) is not None, name
