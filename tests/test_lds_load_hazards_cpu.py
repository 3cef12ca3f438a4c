"""The direct-to-LDS loads are inline assembly, which the compiler's hazard pass does not look into, so the wait states that gfx9
asks for are checked in the built code: one between a scalar write of m0 and the load that takes its LDS address from it, five
between a vector instruction that writes a scalar register and a load that uses it as its base."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_03383_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def hazards(listing):
    """(number of direct-to-LDS loads, offending lines) of a disassembly."""
    loads, bad = 0, []
    m0_written, states, vector_written = None, 0, {}  # wait state of the last m0 write, of every SGPR's last write by a vector op
    for line in listing.splitlines():
        text = line.split("//")[0].strip()
        if not line.startswith("\t") or not text:
            m0_written, vector_written = None, {}  # a label: where control comes from is not known
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op.startswith("global_load_lds") or (op.startswith("buffer_load") and rest.split()[-1:] == ["lds"]):
            loads += 1
            if m0_written is not None and states - m0_written < 2:
                bad.append("m0: " + text)
            for lo, hi in re.findall(r"s\[(\d+):(\d+)\]", rest):
                if any(states - vector_written.get(s, -99) <= 5 for s in range(int(lo), int(hi) + 1)):
                    bad.append("base: " + text)
        if op.startswith("s_") and args[0] == "m0":
            m0_written = states
        if op.startswith("v_"):
            for a in args[:2]:
                m = re.fullmatch(r"s(\d+)|s\[(\d+):(\d+)\]", a)
                if m and (a is args[0] or op.startswith(("v_add_co", "v_sub_co", "v_addc", "v_subb", "v_div_scale"))):
                    lo = int(m.group(1) or m.group(2))
                    for s in range(lo, int(m.group(3) or lo) + 1):
                        vector_written[s] = states
        states += 1 + (int(args[0], 0) if op == "s_nop" else 0)
    return loads, bad


def test_the_check_sees_both_hazards():
    def listing(*ops):
        return "".join(f"\t{o} // 0\n" for o in ops)

    load = "global_load_lds_dwordx4 v1, s[4:5]"
    assert hazards(listing("s_add_i32 m0, s1, 0x100", load))[1] == ["m0: " + load]
    assert hazards(listing("s_add_i32 m0, s1, 0x100", "s_nop 0", load)) == (1, [])
    assert hazards(listing("v_readfirstlane_b32 s5, v2", "s_nop 3", load))[1] == ["base: " + load]
    assert hazards(listing("v_readfirstlane_b32 s5, v2", "s_nop 4", load)) == (1, [])


def test_built_library_keeps_the_wait_states(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    lib = shutil.copy(binding.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    total = 0
    for obj in glob.glob(str(tmp_path / "*gfx950")):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        loads, bad = hazards(out)
        total += loads
        assert not bad, (os.path.basename(obj), len(bad), bad[:3])
    assert total > 100  # the many-row GEMMs' loads
