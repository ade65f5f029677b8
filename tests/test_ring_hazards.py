"""The ring kernel's MFMAs are inline assembly, which hides them from the compiler's hazard handling (mfma_in_place,
gemm_ring.hip).  What the padding there relies on is read off the assembly of a build with the library's flags: no vector
instruction writes an operand right in front of an MFMA, and none touches an accumulator before its MFMA is through."""
import os
import re
import subprocess

from paper_2303_06182_amd import build

READ_WAIT = 2     # wait states from a vector write to an MFMA that reads it
RESULT_WAIT = 19  # from an MFMA to a vector access of its result: what the longest one of 16 passes takes, these have 8


def registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([va])(\d+)$", operand)
    return {(m[1], int(m[2]))} if m else set()


def instructions(text):
    """(mnemonic, operands) in program order; a label as None, which a fall through runs past."""
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"\.?[\w$.]+:$", line):
            yield None
        elif line and not line.startswith("."):
            name, _, rest = line.partition(" ")
            yield name, [o.strip() for o in rest.split(",")] if rest else []


def wait_states(ins):
    return int(ins[1][0], 0) + 1 if ins[0] == "s_nop" else 1


def hazards(text):
    """(MFMAs looked at, descriptions of the hazards found)"""
    prog, found, n = [i for i in instructions(text) if i], [], 0
    vector = lambda i: i[0].startswith("v_") and not i[0].startswith("v_mfma")
    for at, (name, ops) in enumerate(prog):
        if not name.startswith("v_mfma"):
            continue
        n += 1
        reads, result = set().union(*map(registers, ops[1:4])), registers(ops[0])
        waited = 0
        for other in reversed(prog[max(0, at - READ_WAIT):at]):
            if waited >= READ_WAIT:
                break
            if vector(other) and registers(other[1][0]) & reads:
                found.append("%s in front of %s" % (other, ops))
            waited += wait_states(other)
        waited = 0
        for other in prog[at + 1:at + 1 + RESULT_WAIT]:
            if waited >= RESULT_WAIT or other[0] in ("s_endpgm", "s_branch"):
                break
            if not other[0].startswith("v_mfma") and set().union(*map(registers, other[1])) & result:
                found.append("%s behind %s" % (other, ops))
            waited += wait_states(other)
    return n, found


def test_the_check_finds_what_it_is_for():
    mfma = "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[16:19], v[0:3]\n"
    assert hazards("\tv_mov_b32_e32 v9, v40\n" + mfma)[1] and hazards("\tv_mov_b32_e32 v9, v40\n.LBB0_1:\n\ts_nop 0\n" + mfma)[1]
    assert hazards("\tv_mov_b32_e32 v9, v40\n\ts_nop 1\n" + mfma) == (1, [])
    assert hazards(mfma + "\ts_nop 15\n\tv_add_f32_e32 v50, v3, v51\n")[1]
    assert hazards(mfma + "\ts_nop 15\n\ts_nop 15\n\tv_add_f32_e32 v50, v3, v51\n") == (1, [])


def test_no_hazard_in_the_ring_kernel(tmp_path):
    out = tmp_path / "ring.s"
    cmd = [build._hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm_ring.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    n, found = hazards(out.read_text())
    assert n > 1000 and not found, found[:5]
