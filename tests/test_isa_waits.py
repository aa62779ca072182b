"""Wait states of the built gfx950 code (CPU): the kernels issue their loads
to LDS from inline assembly, which the compiler's hazard handling does not look
into.  Two rules of the instruction set are checked on the disassembly of the
library built here from source:

* a scalar write of M0 needs one wait state before a load to LDS reads it;
* a vector instruction's write of a scalar register needs five wait states
  before a vector memory instruction reads that register (the loads' base)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_12505_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


def _sgprs(operand):
    m = re.match(r"s\[(\d+):(\d+)\]$", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"s(\d+)$", operand)
    return {int(m[1])} if m else set()


def hazards(lines):
    """(violations, loads to LDS seen) of an llvm-objdump listing."""
    bad, loads, recent = [], 0, []   # recent: (opcode, operands), oldest first
    for line in lines:
        text = line.split("//")[0].strip()
        if not text or text.endswith(":"):
            recent = [] if text.endswith(">:") else recent
            continue
        op, _, rest = text.partition(" ")
        operands = [o.strip().split(" ")[0] for o in rest.split(",")]
        if "_load_lds_" in op:
            loads += 1
            base = set().union(*(_sgprs(o) for o in operands))
            waited = 0
            for past, past_operands in reversed(recent):
                if waited < 1 and past.startswith("s_") and past_operands[0] == "m0":
                    bad.append(f"{past} m0 -> {text}")
                if waited < 5 and past.startswith("v_") and _sgprs(past_operands[0]) & base:
                    bad.append(f"{past} {past_operands[0]} -> {text}")
                waited += 1 + (int(past_operands[0], 0) if past == "s_nop" else 0)
        recent = (recent + [(op, operands)])[-6:]
    return bad, loads


def test_rules_on_hand_written_listings():
    mov, load = "\ts_mov_b32 m0, s4", "\tglobal_load_lds_dwordx4 v1, s[2:3]"
    assert len(hazards([mov, load])[0]) == 1
    assert hazards([mov, "\ts_nop 0", load]) == ([], 1)
    assert hazards([mov, "\ts_cmp_lt_i32 s5, 1", "\ts_cbranch_scc1 1", load]) == ([], 1)
    lane = "\tv_readlane_b32 s3, v9, 0"
    assert len(hazards([lane, mov, "\ts_nop 2", load])[0]) == 1
    assert hazards([lane, mov, "\ts_nop 3", load]) == ([], 1)
    assert hazards(["\tv_readlane_b32 s4, v9, 0", mov, "\ts_nop 0", load]) == ([], 1)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump of the ROCm toolchain")
def test_loads_to_lds_have_their_wait_states(tmp_path):
    shutil.copy(build.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    objects = [f for f in os.listdir(tmp_path) if f.endswith(build.ARCH) and os.path.getsize(tmp_path / f)]
    assert objects, "no device code in the library"
    total = 0
    for name in objects:
        with subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", name], cwd=tmp_path, stdout=subprocess.PIPE,
                              text=True) as proc:
            bad, loads = hazards(proc.stdout)
        assert proc.returncode == 0
        assert not bad, f"{len(bad)} in {name}, first: {bad[0]}"
        total += loads
    assert total > 0, "no load to LDS found: the check has lost its subject"
