"""Wait states in the library's gfx950 code.

On gfx950 a vector instruction that writes a scalar register (a comparison, a
carry out, a lane read) must be two wait states ahead of a vector instruction
that reads that register (as a carry in, a lane mask or an operand): nearer,
the reader can take the old value, with no error.  The compiler keeps the
distance for the instructions it emits, but it does not look into inline
assembly.  The built library's device code is disassembled and every such pair
in straight-line code is measured."""
import os
import re
import shutil
import subprocess

import pytest

from paper_cs_0608108_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 2

# vector instructions whose scalar result is not their first operand
_SECOND = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_u32|v_div_scale_|v_mad_(u|i)64_")
_RANGE = re.compile(r"^s\[(\d+):(\d+)\]$")
_ONE = re.compile(r"^s(\d+)$")


def _scalars(op):
    """The scalar registers an operand names."""
    op = op.strip().lstrip("-").strip("|")
    if op.startswith("vcc"):
        return {"vcc"}
    m = _RANGE.match(op)
    if m:
        return {f"s{i}" for i in range(int(m.group(1)), int(m.group(2)) + 1)}
    m = _ONE.match(op)
    return {op} if m else set()


def _split(ins):
    """(mnemonic, scalar registers written, scalar registers read) of a vector
    instruction."""
    name, _, rest = ins.partition(" ")
    ops = [o for o in rest.split(",")]
    ops = [o.strip().split(" ")[0] for o in ops if o.strip()]
    out = set(_scalars(ops[0])) if ops else set()
    at = 1
    if _SECOND.match(name):
        out |= _scalars(ops[1])
        at = 2
    read = set()
    for o in ops[at:]:
        read |= _scalars(o)
    if name.startswith(("v_div_fmas", "v_cndmask_b32_e32", "v_cndmask_b32_dpp", "v_cndmask_b32_sdwa")):
        read.add("vcc")
    return name, out, read


def short_waits(lines):
    """(function, writer, reader, wait states between) of each pair closer than
    WAIT_STATES; a function's code is read in order."""
    found, func, recent = [], "", []  # recent: (wait states ago, registers, instruction)
    for line in lines:
        if line.endswith(">:"):
            func, recent = line, []
            continue
        ins = line.split("//")[0].strip()
        if not ins or ins.startswith(("/", "Disassembly")):
            continue
        states = 1
        if ins.startswith("s_nop"):
            states = int(ins.split()[1], 0) + 1
        elif ins.startswith("v_"):
            name, out, read = _split(ins)
            for ago, regs, writer in recent:
                if regs & read:
                    found.append((func, writer, ins, ago))
            recent = [(a + 1, r, w) for a, r, w in recent if a + 1 < WAIT_STATES]
            if out:
                recent.append((0, out, ins))
            continue
        recent = [(a + states, r, w) for a, r, w in recent if a + states < WAIT_STATES]
    return found


@pytest.mark.parametrize("text, n", [
    (["v_cmp_lt_u32_e64 s[4:5], v0, v1", "v_addc_co_u32_e64 v2, s[6:7], 0, v2, s[4:5]"], 1),
    (["v_cmp_lt_u32_e32 vcc, v0, v1", "v_mov_b32_e32 v3, v4", "v_cndmask_b32_e32 v2, v3, v4, vcc"], 1),
    (["v_cmp_lt_u32_e32 vcc, v0, v1", "s_nop 1", "v_cndmask_b32_e32 v2, v3, v4, vcc"], 0),
    (["v_readfirstlane_b32 s8, v0", "v_add_u32_e32 v1, s8, v1"], 1),
    (["v_add_co_u32_e32 v0, vcc, v1, v2", "v_mov_b32_e32 v3, v4", "s_nop 0",
      "v_addc_co_u32_e32 v1, vcc, v3, v4, vcc"], 0),
])
def test_reader_finds_short_waits(text, n):
    assert len(short_waits(["<f>:"] + text)) == n


def test_scalar_results_wait_before_vector_reads(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no AMDGPU disassembler")
    if not os.path.exists(build.LIB):
        build.build()
    lib = shutil.copy(build.LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    objs = [f for f in os.listdir(tmp_path) if build.ARCH in f]
    assert objs
    found, seen = [], 0
    for f in objs:
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / f)], check=True, capture_output=True,
                           text=True)
        lines = [ln.strip() for ln in r.stdout.splitlines()]
        seen += sum(ln.startswith("v_") for ln in lines)
        found += short_waits(lines)
    assert seen > 100000, seen
    assert not found, f"{len(found)} short waits, the first: {found[:5]}"
