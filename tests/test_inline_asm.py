"""Inline assembly in the kernels, checked in the compiler's own listing.

The compiler keeps the wait states that gfx950 needs between its own
instructions, but sees neither into an asm statement nor across its edge: there
the source has to keep them.  Every kernel is compiled to a listing (no GPU) and
the neighbours of its asm statements are checked."""
import os
import re
import subprocess

import pytest

from paper_1503_07192_amd import build as B

SOURCES = ["fw.hip", "hier.hip", "kernels.hip", "range.hip"]


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    """Per source: the kernels' instructions as (name, operands, in an asm
    statement) and what the compiler said."""
    out = {}
    for src in SOURCES:
        asm = str(tmp_path_factory.mktemp("asm") / (src + ".s"))
        cmd = [c for c in B.command(asm) if not c.endswith(".hip") and c != "-shared"]
        r = subprocess.run(cmd + ["--offload-device-only", "-S", os.path.join(B.CSRC, src)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        out[src] = (kernels(open(asm)), r.stderr)
    return out


def kernels(lines):
    out, cur, inside = {}, None, False
    for line in lines:
        if ";;#ASMSTART" in line or ";;#ASMEND" in line:
            inside = "START" in line
            continue
        label = re.match(r"(_Z\w+):", line)
        if label:
            cur = out.setdefault(label.group(1), [])
        text = line.split(";")[0].strip()
        if cur is None or not text or text[0] == "." or text.endswith(":"):
            continue
        name, _, rest = text.partition(" ")
        cur.append((name, [x.strip() for x in rest.split(",")], inside))
    return out


def scalars(operand):
    """The scalar registers an operand names."""
    m = re.match(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"s(\d+)$", operand)
    if m:
        return {int(m.group(1))}
    return {"vcc"} if operand.startswith("vcc") else set()


def test_scalar_results_of_vector_instructions_are_waited_for(listings):
    """Two wait states between a vector instruction that writes a scalar
    register or vcc and a vector instruction that reads it."""
    seen, bad = 0, []
    for src in SOURCES:
        for kernel, code in listings[src][0].items():
            recent = []  # (wait states since, scalars written, in asm, name)
            for name, ops, inside in code:
                if name == "s_nop":
                    recent = [(t + int(ops[0]) + 1, *r) for t, *r in recent]
                    continue
                if name.startswith("v_"):
                    read = set().union(*[scalars(o.split(" ")[0]) for o in ops[1:]])
                    for t, written, asm, writer in recent:
                        if t < 2 and written & read and (asm or inside):
                            bad.append((src, kernel, writer, name, ops))
                recent = [(t + 1, *r) for t, *r in recent if t < 2]
                if name.startswith("v_"):
                    recent.append((0, scalars(ops[0]), inside, name))
                seen += inside
    assert seen > 1000  # the statements were found
    assert not bad, bad[:4]


def test_m0_belongs_to_the_asm_statements(listings):
    """The statements that load to LDS write m0, a reserved register that no
    clobber list may name: no instruction of the compiler's may rely on it, and
    the compiler has nothing to say about them."""
    for src in SOURCES:
        code, said = listings[src]
        assert "inline-asm" not in said, said.split("\n")[0]
        for kernel, ins in code.items():
            used = [(name, ops) for name, ops, inside in ins if "m0" in ops and not inside]
            loads = [name for name, _, inside in ins if inside and name.startswith("global_load_lds")]
            assert not (loads and used), (kernel, used[:3])


def test_occupancy_targets_are_met(listings):
    for src in SOURCES:
        assert "occupancy" not in listings[src][1], listings[src][1]


def test_loops_unroll_as_asked(listings):
    for src in SOURCES:
        assert "not unrolled" not in listings[src][1], listings[src][1]
