"""Wait states around the asynchronous global -> LDS copies, in the built library.

The copies are inline assembly, which the compiler takes as it stands: unlike for
its own instructions it adds no wait state in front of them.  gfx950 needs one
between a write of M0, which holds a copy's LDS address, and the copy, and five
between a vector instruction that writes a scalar register and a memory instruction
that takes it as its base address.  Without the first, a copy can land where the one
before it did.
"""
import os
import re
import subprocess

import pytest

from _code_objects import code_objects, library, tool

OBJDUMP = tool("llvm-objdump")
M0_STATES, SADDR_STATES = 1, 5


def registers(operand):
    """The scalar registers of an operand such as s4 or s[4:5]."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


def violations(lines):
    """(copies seen, [(line, what it lacks)]) of a disassembly, in program order."""
    copies, bad = 0, []
    m0_age = 99
    age = {}  # scalar register -> wait states since a vector instruction wrote it
    for line in lines:
        text = line.split("//")[0].strip()
        if not text or text.endswith(":") or text.startswith("Disassembly"):
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op.startswith("global_load_lds"):
            copies += 1
            if m0_age < M0_STATES:
                bad.append((text, "a wait state after the write of m0"))
            saddr = args[-1].split()[0]
            if any(age.get(r, 99) < SADDR_STATES for r in registers(saddr)):
                bad.append((text, "wait states after the vector write of its base"))
        states = int(args[0], 0) + 1 if op == "s_nop" else 1
        m0_age += states
        for r in list(age):
            age[r] += states
            if age[r] >= SADDR_STATES:
                del age[r]
        if op.startswith(("s_", "v_")) and args[0] == "m0" and not op.startswith("s_cmp"):
            m0_age = 0
        if op.startswith("v_"):
            for r in registers(args[0]):
                age[r] = 0
    return copies, bad


def test_missing_wait_states_are_seen():
    copy = "global_load_lds_dwordx4 v1, s[2:3]"
    assert violations(["s_mov_b32 m0, s5", copy])[1]
    assert not violations(["s_mov_b32 m0, s5", "s_nop 0", copy])[1]
    assert not violations(["s_add_i32 m0, s5, 16", "v_add_u32_e32 v1, v2, v3", copy])[1]
    assert violations(["v_readfirstlane_b32 s3, v7", "s_mov_b32 m0, s5", "s_nop 2", copy])[1]
    assert not violations(["v_readfirstlane_b32 s3, v7", "s_mov_b32 m0, s5", "s_nop 3", copy])[1]
    assert violations(["v_readfirstlane_b32 m0, v7", copy])[1]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler in this image")
def test_copies_of_the_built_library_have_their_wait_states(tmp_path):
    copies = 0
    for i, code in enumerate(code_objects(library())):
        obj = tmp_path / f"{i}.co"
        obj.write_bytes(code)
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], capture_output=True,
                             text=True, check=True).stdout
        n, bad = violations(out.splitlines())
        copies += n
        assert not bad, f"code object {i}: {len(bad)} of {n} copies, the first: {bad[0]}"
    assert copies > 0
