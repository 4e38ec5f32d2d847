"""The direct global -> LDS loads (lds_dma.h) are written as inline assembly, so the compiler's hazard recogniser does not see
them.  What the architecture asks for in front of such a load, checked on every path of the assembly that the compiler
makes of the three files that use them:
  - one wait state between a scalar write of M0 (the load's LDS address) and the load,
  - five between a vector instruction that writes a scalar register and a memory instruction that reads it (the load's
    base address comes from readfirstlane).
M0 cannot be named as clobbered (the compiler reserves it and writes it itself right before its own uses), so no
instruction of the compiler's may rely on it either."""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2603_05353_amd import build
from tests.test_attention_split import kernel_instructions, reachable

FILES = {"attention_mfma": 150, "attention_full": 150, "score_mfma": 1500}  # and at least so many direct loads
pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc in this environment")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    folder = tmp_path_factory.mktemp("asm")

    def compiled(name):
        out = folder / f"{name}.s"
        subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, f"{name}.hip"), "-o", str(out)],
                       check=True, capture_output=True, timeout=600)
        return out.read_text()

    with cf.ThreadPoolExecutor(3) as ex:
        return dict(zip(FILES, ex.map(compiled, FILES)))


def scalar_registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand) or re.fullmatch(r"s(\d+)()", operand)
    if m:
        return set(range(int(m[1]), int(m[2] or m[1]) + 1))
    return {operand} if operand in ("m0", "vcc", "vcc_lo", "vcc_hi") else set()


def hazards(text):
    found, loads = [], 0
    for name in re.findall(r"^(_Z\S+):", text, re.M):
        ins, after = kernel_instructions(text, re.escape(name))
        loads += sum(op.startswith("global_load_lds") for op, _, _ in ins)
        for i, (op, args, by_hand) in enumerate(ins):
            if "m0" in args and not by_hand:
                found.append(("compiler uses m0", ins[i]))
            if op.startswith("s_") and args[0] == "m0":
                found += [("m0", ins[i], ins[j]) for j in reachable(ins, after, i, 1) if "_lds_" in ins[j][0]]
            if op.startswith("v_") and (written := scalar_registers(args[0])):
                found += [("scalar base", ins[i], ins[j]) for j in reachable(ins, after, i, 5)
                          if ins[j][0].startswith(("global_", "buffer_", "scratch_", "flat_"))
                          and any(scalar_registers(a.split(" ")[0]) & written for a in ins[j][1])]
    return found, loads


@pytest.mark.parametrize("name", FILES)
def test_wait_states_before_direct_loads(assembly, name):
    found, loads = hazards(assembly[name])
    assert loads >= FILES[name] and not found, (loads, len(found), found[:4])


def test_the_scan_sees_missing_wait_states(assembly):
    text = assembly["attention_full"]
    assert hazards(text.replace("s_nop 0\n\tglobal_load_lds", "global_load_lds"))[0]
    load = re.search(r"\tglobal_load_lds_dwordx4 v\d+, s\[(\d+):\d+\]", text)
    assert hazards(text.replace(load[0], f"\tv_readfirstlane_b32 s{load[1]}, v0\n\ts_nop 0\n{load[0]}", 1))[0]
