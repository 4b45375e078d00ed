"""The build's check of register spills: what it finds in a disassembly, and that
no kernel of this build spills where it is not expected."""
import glob
import os

import pytest

from paper_2003_09145_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def _asm(*ops, name="_Z1kv", branch=None):
    # one instruction a line at 4-byte steps from 0x1000; `branch`: (index, target index)
    lines = [f"0000000000001000 <{name}>:"]
    for i, op in enumerate(ops):
        to = f" <{name}+0x{4 * branch[1]:x}>" if branch and branch[0] == i else ""
        lines.append(f"\t{op:<58} // {0x1000 + 4 * i:012X}: BF800000{to}")
    return "\n".join(lines)


STORE, JOIN = "scratch_store_dwordx2 off, v[2:3], off offset:8", "s_or_b64 exec, exec, s[8:9]"


@pytest.mark.parametrize("asm,want", [
    # at a join, before the lanes rejoin
    (_asm("s_cbranch_execz 2", "v_nop", STORE, STORE, JOIN, branch=(0, 2)), {"_Z1kv": 2}),
    (_asm("v_nop", STORE, "v_nop", JOIN), {"_Z1kv": 1}),
    # after it, in the diverged part, in another block
    (_asm("s_cbranch_execz 1", "v_nop", JOIN, STORE, branch=(0, 2)), {}),
    (_asm("s_cbranch_execz 1", STORE, JOIN, branch=(0, 2)), {}),
    (_asm(STORE, "s_cbranch_execz 1", "v_nop", JOIN, branch=(1, 3)), {}),
    # other widenings of a mask that is no join
    (_asm(STORE, "s_or_b64 s[0:1], s[0:1], s[8:9]"), {})])
def test_narrow_stores(asm, want):
    assert build.narrow_stores(asm) == want


def test_no_unexpected_spill_in_this_build():
    objects = sorted(glob.glob(os.path.join(build.OBJ, "*.o")))
    if len(objects) != len(build.sources()):
        pytest.skip("no objects of this build")
    spills, narrow = build.check_spills(objects)
    assert narrow == {}
    assert [k for k in spills if not k.startswith(build.SPILLING)] == []
