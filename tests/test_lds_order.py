"""The loads into LDS that a counted wait leaves in flight are the youngest
ones in the built kernels. A GEMM tile with a ring of LDS stages waits with
``vmcnt(n)``, which lets the last n loads issued stay in flight; a load that
the compiler moved behind them would be read before it has landed. The order
is a property of the machine code, so it is read off the library built here.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_22335_amd", "libvla.so")
LLVM = "/opt/rocm/llvm/bin/"

LOAD = re.compile(r"buffer_load_dwordx4 v\d+, (s\[\d+:\d+\]), 0 offen lds")
WAIT = re.compile(r"s_waitcnt vmcnt\((\d+)\)")
TILE = re.compile(r"k_gemmItLi(\d+)ELi(\d+)ELi64ELi2ELi2ELi1ELi0ELb1EL\w+?ELi([34])EEE")


def segments(lines):
    """The LDS loads (their buffer resources, in issue order) before each
    counted wait, back to the wait or barrier before it: [(loads, n)]. (A wait
    that leaves all of them in flight is for an older load.)"""
    out, cur = [], []
    for ln in lines:
        ld, wt = LOAD.search(ln), WAIT.search(ln)
        if ld:
            cur.append(ld.group(1))
        elif wt and int(wt.group(1)) < len(cur):
            if int(wt.group(1)):
                out.append((cur, int(wt.group(1))))
            cur = []
        elif "s_barrier" in ln:
            cur = []
    return out


def check_ring3(lines, la, lb):
    """Activations one K-tile ahead, weights two: a step issues its la
    activation loads, then its lb weight loads, and its wait leaves the
    weights in flight."""
    seg = segments(lines)
    assert len(seg) == 4, "four steps in a round"
    for loads, n in seg:
        a, w = loads[0], loads[-1]
        assert n == lb and a != w and loads == [a] * la + [w] * lb, (n, loads)


def check_ring4(lines, la, lb):
    """Whole K-tiles, three in flight: a wait leaves two tiles' loads (a step
    issues one tile's, in any order among themselves); the prologue issues
    three tiles one after another."""
    seg = segments(lines)
    assert len(seg) == 1, "the prologue"
    loads, n = seg[0]
    a, w = loads[0], loads[-1]
    assert n == 2 * (la + lb) and a != w and loads == ([a] * la + [w] * lb) * 3, (n, loads)
    assert sum(bool(m) and int(m.group(1)) == n for m in map(WAIT.search, lines)) >= 4, "four steps in a round"


def test_counted_waits_in_built_kernels(tmp_path):
    tools = [LLVM + t for t in ("llvm-objdump", "llvm-readelf")]
    if not os.path.exists(LIB) or not all(shutil.which(t) for t in tools):
        pytest.skip("library or LLVM tools not here")
    lib = shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([tools[0], "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    seen = set()
    for obj in sorted(p for p in os.listdir(tmp_path) if p.endswith("gfx950")):
        sym = subprocess.run([tools[1], "-sW", obj], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for name in re.findall(r"FUNC.*\s(\S*k_gemm\S+)", sym):
            m = TILE.search(name)
            if not m:
                continue
            text = subprocess.run([tools[0], "-d", "--no-show-raw-insn", f"--disassemble-symbols={name}", obj],
                                  cwd=tmp_path, check=True, capture_output=True, text=True).stdout.splitlines()
            bm, bn, stages = (int(x) for x in m.groups())
            (check_ring3 if stages == 3 else check_ring4)(text, bm // 32, bn // 32)
            seen.add((bm, bn, stages))
    assert seen == {(320, 128, 3), (64, 64, 4)}


def test_check_sees_a_moved_load():
    """The checks refuse a listing in which one weight load went out before
    the last activation load, or one tile's load into another tile's group."""
    ld = lambda r: f"buffer_load_dwordx4 v2, s[{r}:{r + 3}], 0 offen lds"
    step = lambda seq: [ld(r) for r in seq] + ["s_waitcnt vmcnt(2) lgkmcnt(0)", "s_barrier"]
    good = step([12, 12, 12, 16, 16])
    check_ring3(good * 4, 3, 2)
    with pytest.raises(AssertionError):
        check_ring3(good * 3 + step([12, 12, 16, 12, 16]), 3, 2)
    step = lambda seq: [ld(r) for r in seq] + ["s_waitcnt vmcnt(4) lgkmcnt(0)", "s_barrier"]
    loop = step([16, 12]) * 4
    check_ring4(step([12, 16] * 3) + loop, 1, 1)
    with pytest.raises(AssertionError):
        check_ring4(step([12, 12, 16, 16, 12, 16]) + loop, 1, 1)
