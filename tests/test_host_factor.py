"""The factor's hand-written cross-lane instructions, read in the assembly the library is built from: a value takes two wait
states from the vector instruction that writes it to one that reads it across lanes, and the compiler does not look into their text."""
import os
import re
import subprocess

import paper_2306_03078_amd.build as build

WAIT_STATES = 2


def _registers(operand):
    m = re.match(r"-?\|?v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"-?\|?v(\d+)\b", operand)
    return {int(m.group(1))} if m else set()


def _too_early(assembly):
    """The cross-lane reads of a register that a vector instruction wrote fewer than WAIT_STATES before, and how many there are in all."""
    written, now, bad, seen = {}, 0, [], 0
    for line in assembly.splitlines():
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        if "row_newbcast" in text or "dpp" in op:
            seen += 1
            # (the operand across lanes is the first source)
            if any(now - written.get(r, -WAIT_STATES) < WAIT_STATES for r in _registers(operands[1])):
                bad.append(text)
        now += int(operands[0]) + 1 if op == "s_nop" else 1
        if op.startswith("v_") and not op.startswith("v_cmp"):
            written.update({r: now for r in _registers(operands[0])})
        assert not op.startswith("v_cmpx")           # (a vector instruction that writes EXEC needs more)
    return bad, seen


def test_values_read_across_lanes_have_had_their_wait_states(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = str(tmp_path / "factor.s")
    subprocess.run([hipcc, *build.FLAGS, "--cuda-device-only", "-S", "-o", out, os.path.join(build.CSRC, "spqr_factor.hip")], check=True,
                   capture_output=True, timeout=120)
    with open(out) as f:
        assembly = f.read()
    bad, seen = _too_early(assembly)
    assert not bad, bad[:5]
    assert seen >= 1000                              # 16 steps of up to 31 such instructions, four panels, two kernels
    assert _too_early(re.sub(r"^\s*s_nop.*$", "", assembly, flags=re.M))[0]          # the waits are what keeps them apart
