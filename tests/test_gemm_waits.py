"""Waits around the workgroup barriers of the grouped GEMMs, checked on the
listing the compiler makes of moe_forward.hip.  Loads from memory straight into
LDS and the bare s_barrier of the K loops leave the waits to the source, and a
missing one only shows when a wave is late, so no run on a GPU can show that
they are all there."""
import os
import re
import subprocess

import pytest

from paper_2607_17154_amd import build

if not os.path.exists(build.HIPCC):  # pragma: no cover
    pytest.skip("no hipcc", allow_module_level=True)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: instruction lines and labels} of every kernel."""
    out = str(tmp_path_factory.mktemp("listing") / "moe_forward.s")
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "moe_forward.hip"),
                                                      "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found = {}
    for m in re.finditer(r"^(_Z\w+):.*?\n(.*?)^\.Lfunc_end\d+:", open(out).read(), re.M | re.S):
        lines = (s.split(";")[0].strip() for s in m.group(2).split("\n"))
        found[m.group(1)] = [s for s in lines if s and (not s.startswith(".") or s.endswith(":"))]
    return found


def _violations(lines, step):
    """Instructions at which `step(instruction, state) -> (state, wrong)` is wrong
    on some path through the kernel, which starts in state 0."""
    label = {s[:-1]: i for i, s in enumerate(lines) if s.endswith(":")}
    seen, todo, bad = set(), [(0, 0)], set()
    while todo:
        at = todo.pop()
        if at in seen:
            continue
        seen.add(at)
        i, state = at
        op = lines[i].split()[0]
        state, wrong = step(lines[i], state)
        if wrong:
            bad.add((i, lines[i]))
        if op.startswith(("s_branch", "s_cbranch")):
            todo.append((label[lines[i].split()[1]], state))
        if op not in ("s_branch", "s_endpgm"):
            todo.append((i + 1, state))
    return sorted(bad)


def _waits(s, counter):
    return s.startswith("s_waitcnt") and counter + "(0)" in s


def _is_lds_load(s):
    return s.startswith("buffer_load") and s.split()[-1] == "lds"


def _tile_change(s, state):
    """state 1: loads into LDS may be in flight; 2: this wave's have arrived, the
    other waves' may not have.  A new load in state 2 can be overtaken by another
    wave's old one, since which rows a wave loads depends on the tile's height."""
    if _is_lds_load(s):
        return 1, state == 2
    if state == 1 and _waits(s, "vmcnt"):
        return 2, False
    if state == 2 and s == "s_barrier":
        return 0, False
    return state, False


@pytest.mark.parametrize("name", ["ggemm_bf16ILi0E", "ggemm_bf16ILi1E"])    # (the fp32 tiles of a launch have one height)
def test_a_tile_loads_after_every_wave_has_drained_the_last_one(kernels, name):
    lines = next(v for k, v in kernels.items() if name in k)
    assert any(map(_is_lds_load, lines)) and "s_barrier" in lines
    assert _violations(lines, _tile_change) == []


def _lds_write(s, state):
    """state 1: a write to LDS may be outstanding; a barrier then lets other waves read the old value."""
    if s.startswith("ds_write"):
        return 1, False
    if _waits(s, "lgkmcnt"):
        return 0, False
    return state, state == 1 and s == "s_barrier"


@pytest.mark.parametrize("name", ["ggemm_bf16ILi0E", "ggemm_bf16ILi1E", "ggemm_f32ILi0E", "ggemm_f32ILi1E",
                                  "ggemm_thinILi0E", "ggemm_thinILi1E"])
def test_lds_writes_are_done_before_a_barrier(kernels, name):
    lines = next(v for k, v in kernels.items() if name in k)
    assert any(s.startswith("ds_write") for s in lines) and "s_barrier" in lines
    assert _violations(lines, _lds_write) == []
