"""Wait states of gfx950 in the built kernels' code: a VALU instruction may
read an SGPR that another VALU instruction wrote, and a DPP operand may read a
VGPR, only two wait states after the write.  The compiler keeps these apart in
its own code but neither looks into inline assembly nor counts its writes, so
the built library's own kernels are disassembled and every instruction is
checked against the ones before it."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_1702_07961_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
CARRY = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64_")   # two results


def registers(operand):
    m = re.fullmatch(r"([vs])(\d+)", operand) or re.fullmatch(r"([vs])\[(\d+):(\d+)\]", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[len(m.groups())]) + 1)}
    return {("s", "vcc")} if operand in ("vcc", "vcc_lo", "vcc_hi") else set()


def violations(lines):
    """(writer, reader) of every pair that is too close, in the order of the code."""
    found, recent, at = [], [], 0   # recent: (position, results, text) of VALU instructions
    for line in lines:
        if line.endswith(">:"):
            recent = []
            continue
        text = line.split("//")[0].strip()
        name, _, rest = text.partition(" ")
        if not re.fullmatch(r"[a-z][a-z0-9_]*", name):
            continue
        if name == "s_nop":
            at += int(rest, 0) + 1
            continue
        if name.startswith("v_") and name != "v_nop":
            ops = [registers(o.split()[0].strip("-|")) if o.strip() else set() for o in rest.split(",")]
            results = 2 if CARRY.match(name) else 1
            reads = set().union(*ops[results:]) if ops[results:] else set()
            if re.match(r"v_cndmask_b32_(e32|dpp|sdwa)", name):
                reads.add(("s", "vcc"))
            dpp = ops[1] if re.search(r"quad_perm:|row_|wave_", rest) and len(ops) > 1 else set()
            for pos, wrote, writer in recent:
                if at - pos - 1 < 2 and any(r[0] == "s" or r in dpp for r in wrote & reads):
                    found.append((writer, text))
            recent = [w for w in recent if at - w[0] <= 2] + [(at, set().union(*ops[:results]), text)]
        at += 1
    return found


def test_the_check_itself():
    near = ["v_sub_co_u32_e32 v2, vcc, s26, v2", "s_nop 0", "v_subb_co_u32_e32 v3, vcc, v1, v4, vcc"]
    assert len(violations(near)) == 1
    assert not violations([near[0], "s_nop 1", near[2]])
    assert len(violations(["v_min_u32_e32 v1, v2, v3", "v_mov_b32_dpp v4, v1 row_ror:8 row_mask:0xf"])) == 1
    assert not violations(["v_min_u32_e32 v1, v2, v3", "v_add_u32_e32 v4, v1, v2"])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_wait_states_of_the_built_kernels(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    shutil.copy(build.LIB, tmp_path / "libmms.so")
    subprocess.check_call([OBJDUMP, "--offloading", "libmms.so"], cwd=tmp_path, stdout=subprocess.DEVNULL)
    code = sorted(glob.glob(str(tmp_path / f"*{build.ARCH}")))
    assert code, "no device code in the library"
    kernels, found = 0, []
    for path in code:
        lines = subprocess.check_output([OBJDUMP, "-d", f"--mcpu={build.ARCH}", path], text=True).splitlines()
        kernels += sum(line.endswith(">:") for line in lines)
        found += violations(lines)
    assert kernels >= 30
    assert not found, f"{len(found)} pairs too close, first: {found[0]}"
