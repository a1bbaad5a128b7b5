"""The cloud projection's one-wave kernels issue their LDS reads as inline asm
whose waits come later, which the compiler cannot see: no instruction may touch
the registers of a read that is still in flight.  Checked on the assembly that
the compiler makes of them, over every path of the control flow (LDS reads
complete in order, so a wait for at most n leaves the newest n)."""

import os
import re
import subprocess

import pytest

from paper_2607_13093_amd import build

REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
LGKM = re.compile(r"lgkmcnt\((\d+)\)")


def _regs(text):
    out = set()
    for f, lo, hi, one in REG.findall(text):
        out.update((f, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return frozenset(out)


def _parse(lines):
    """(label -> index, [(op, operands, line)])"""
    labels, ops = {}, []
    for ln in lines:
        ln = ln.split(";")[0].strip()
        if ln.endswith(":"):
            labels[ln[:-1]] = len(ops)
        elif ln and not ln.startswith("."):
            op, _, rest = ln.partition(" ")
            ops.append((op, rest, ln))
    return labels, ops


def early_uses(lines):
    """Lines of a kernel that touch a register whose LDS read may not have landed."""
    labels, ops = _parse(lines)
    bad, seen, todo = {}, set(), [(0, ())]
    while todo:
        i, fly = todo.pop()
        while i < len(ops) and (i, fly) not in seen:
            seen.add((i, fly))
            op, rest, ln = ops[i]
            flying = frozenset().union(*fly)
            if op == "s_waitcnt":
                m = LGKM.search(rest)
                left = int(m.group(1)) if m else 0 if rest.strip() == "0" else len(fly)
                fly = fly[max(0, len(fly) - left):] if left else ()
            elif _regs(rest) & flying:
                bad[i] = ln
            if op.startswith("ds_"):
                # (a store or atomic without a result occupies a place too)
                fly += (_regs(rest.split(",")[0]) if "read" in op or "rtn" in op else frozenset(),)
            if op.startswith("s_endpgm"):
                break
            if op.startswith(("s_branch", "s_cbranch")):
                to = labels[rest.strip()]
                if op == "s_branch":
                    i = to
                    continue
                todo.append((to, fly))
            i += 1
    return [bad[i] for i in sorted(bad)]


def test_the_check_finds_a_missing_wait():
    good = ["k:", "ds_read_b128 v[0:3], v9 offset:16", "ds_read_b128 v[4:7], v9", "s_waitcnt lgkmcnt(1)",
            "v_add_u32 v8, v0, v3", "s_cbranch_scc0 .L", "v_mov_b32 v10, 0", ".L:", "s_waitcnt lgkmcnt(0)",
            "v_and_b32 v5, 4, v4", "s_endpgm"]
    assert early_uses(good) == []
    early = good[:6] + ["v_mov_b32 v6, 0"] + good[7:]
    assert early_uses(early) == ["v_mov_b32 v6, 0"]
    assert early_uses(good[:8] + good[9:]) == ["v_and_b32 v5, 4, v4"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "mfma.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    r = subprocess.run([build.hipcc(), *flags, "--offload-device-only", "-S",
                        os.path.join(build.CSRC, "mfma.hip"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read().split("\n")


@pytest.mark.parametrize("stages", [2, 3])
def test_one_wave_kernels_wait_for_their_reads(assembly, stages):
    name = f"_ZN3sph9k_mfma_w1ILi0ELi{stages}EEEvNS_8MfmaArgsE"
    start = next(i for i, ln in enumerate(assembly) if ln.startswith(name + ":"))
    end = next(i for i in range(start, len(assembly)) if assembly[i].startswith(".Lfunc_end"))
    body = assembly[start:end]
    assert sum("ds_read_b128" in ln for ln in body) > 64
    assert early_uses(body) == []
