"""CPU-side check of the sweep's compiled code (csrc/sweep.hip, cross-compiled for gfx950): the waits for the second chunk's keys.

A workgroup's eight waves move the keys of the first two chunks, and leave the prologue by a barrier that waits for all but the second
chunk's.  Waves 0-3 read these between the second and the third barrier after it, and waves 4-7, which form nothing before the first of
them, come to their first sums only behind the second: they have to wait for their part by itself.  Whether a transfer is late is a matter
of the memory, so no run can be relied on to show that a wait is missing: what is looked at is the code.  (Waves 0-3 wait with their first
sums; halves of workgroups move their own keys.)
"""
import os
import re
import subprocess

import pytest

from paper_2510_09309_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def assembly():
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "sweep.hip"), "-o", "-"],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return res.stdout


def kernel(assembly, d):
    """The instructions of sweep_kernel<d, false>, and where its labels are among them."""
    name = r"_ZN\S*sweep_kernelILi%dELb0E\S*" % d
    body = re.search(r"^%s:.*?\n(.*?)^\.Lfunc_end" % name, assembly, re.S | re.M).group(1)
    code, labels = [], {}
    for line in body.split("\n"):
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            labels[line[:-1]] = len(code)
        elif line and not line.startswith("."):
            code.append(line)
    return code, labels


def late_paths(code, labels, start):
    """Barriers that a path from `start` meets as its second without having waited for what is in flight at `start`, and without having
    formed anything before its first.  (Whatever a branch depends on, both ways are looked at.)"""
    todo, seen, late = [(start, 0, 0)], set(), set()
    while todo:
        at, met, issued = todo.pop()       # issued: memory accesses since `start`
        while (at, met, issued) not in seen:
            seen.add((at, met, issued))
            op = code[at]
            if op == "s_endpgm" or (met == 0 and op.startswith("v_mfma")):
                break
            if op == "s_barrier":
                met += 1
                if met == 2:
                    late.add(at)
                    break
            elif re.match(r"(global|buffer|flat|scratch)_", op):
                issued = min(issued + 1, 63)
            elif op.startswith("s_waitcnt"):
                count = re.search(r"vmcnt\((\d+)\)", op)
                if count and int(count.group(1)) <= issued:
                    break
            elif op.startswith("s_branch"):
                at = labels[op.split()[1]]
                continue
            elif op.startswith("s_cbranch"):
                todo.append((labels[op.split()[1]], met, issued))
            else:
                assert not re.match(r"s_(setpc|swappc|call)", op), op
            at += 1
    return late


@pytest.mark.parametrize("d", [128, 64])
def test_second_chunks_keys_are_waited_for_before_the_second_barrier(assembly, d):
    code, labels = kernel(assembly, d)
    moves = 128 // 8 * d * 2 // 1024                    # transfers of 1 KiB per wave and chunk
    prologue = [i for i, op in enumerate(code)
                if op == "s_waitcnt vmcnt(%d) lgkmcnt(0)" % (1 + moves) and code[i + 1] == "s_barrier"]
    assert len(prologue) == 1
    assert late_paths(code, labels, prologue[0] + 2) == set()
