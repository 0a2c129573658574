"""Wait states between dependent instructions of the gfx950 code (CPU: hipcc cross-compiles).

The hardware does not hold back an instruction that uses a scalar register too soon after
certain instructions that wrote it; the compiler puts independent instructions or s_nop between
the two, but does not look into inline assembly.  Each source is compiled to assembly and every
pair that needs a distance is checked in the order of the listing, whoever wrote it:

  * a vector instruction that reads a scalar (vcc or s registers) written by a vector
    instruction: two wait states;
  * a vector-memory instruction whose address or data scalars were written by a vector
    instruction: five;
  * a load that goes directly to LDS after a write of m0, its address there: one.
"""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_23019_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


def scalars(operand):
    """Scalar registers named by an operand: 's12', 's[4:5]', 'vcc', 'm0'."""
    operand = operand.strip()
    if operand in ("vcc", "m0"):
        return {operand}
    m = re.match(r"^s(\d+)$", operand)
    if m:
        return {int(m.group(1))}
    m = re.match(r"^s\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


def instructions(text):
    """(function, line number, mnemonic, operands) of a listing, in its order."""
    name = None
    for i, line in enumerate(text.split("\n")):
        line = line.split(";")[0].rstrip()
        m = re.match(r"^(_Z\S+):", line)
        if m:
            name = m.group(1)
        if line.startswith("\t") and not line.startswith("\t."):
            parts = line.split(None, 1)
            yield name, i + 1, parts[0], [x for x in (parts[1] if len(parts) > 1 else "").split(",")]


def vector_writes(op, args):
    """Scalars that a vector instruction writes."""
    if re.match(r"v_(cmp|readlane|readfirstlane)", op):
        return scalars(args[0])
    if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64_", op):
        return scalars(args[1])
    return set()


def vector_reads(op, args):
    skip = 1 if re.match(r"v_(cmp|readlane|readfirstlane)", op) else 2 if vector_writes(op, args) else 1
    return set().union(*[scalars(a) for a in args[skip:]]) if len(args) > skip else set()


def too_soon(text):
    """Pairs with fewer wait states between them than they need."""
    found = []
    written = {}  # scalar -> wait states since a vector instruction wrote it
    m0 = 9        # wait states since m0 was written
    where = None
    for name, line, op, args in instructions(text):
        if name != where:
            written, m0, where = {}, 9, name
        if op.startswith("v_"):
            if any(written.get(r, 9) < 2 for r in vector_reads(op, args)):
                found.append((name, line, op, args))
        elif op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            used = set().union(*[scalars(a.split()[0]) for a in args if a.strip()])
            if any(written.get(r, 9) < 5 for r in used) or ("_lds_" in op and m0 < 1):
                found.append((name, line, op, args))
        states = int(args[0], 0) + 1 if op == "s_nop" else 1
        m0 += states
        for r in written:
            written[r] += states
        if op.startswith("v_"):
            for r in vector_writes(op, args):
                written[r] = 0
        elif op.startswith("s_") and args and not op.startswith(("s_cmp", "s_nop", "s_bitcmp")):
            for r in scalars(args[0]):
                written.pop(r, None)  # rewritten by a scalar instruction
            if "m0" in scalars(args[0]):
                m0 = 0
    return found


def listing(source, tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    from paper_2606_23019_amd import build
    out = str(tmp_path / "out.s")
    subprocess.run([HIPCC] + [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")] + [
        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-S", "-o", out,
        os.path.join(CSRC, source)], check=True, capture_output=True)
    return open(out).read()


def test_the_check_sees_what_it_looks_for():
    def one(*lines):
        return len(too_soon("_Zk:\n" + "\n".join("\t" + x for x in lines)))
    cmp, use = "v_cmp_le_f32_e32 vcc, v1, v2", "v_addc_co_u32_e32 v0, vcc, v0, v0, vcc"
    other = "v_mov_b32_e32 v5, v6"
    assert one(cmp, use) == 1 and one(cmp, other, use) == 1 and one(cmp, "s_nop 0", use) == 1
    assert one(cmp, "s_nop 1", use) == 0 and one(cmp, other, other, use) == 0
    assert one("v_cmp_le_f32_e64 s[4:5], v1, v2", other, "v_cndmask_b32_e64 v0, v1, v2, s[4:5]") == 1
    assert one("v_readlane_b32 s7, v1, 3", "v_add_u32_e32 v1, s7, v1") == 1
    assert one("v_readlane_b32 s7, v1, 3", "v_add_u32_e32 v1, s8, v1") == 0
    load = "global_load_lds_dwordx4 v2, s[6:7]"
    assert one("s_mov_b32 m0, s3", load) == 1 and one("s_add_i32 m0, s3, 0x400", load) == 1
    assert one("s_mov_b32 m0, s3", "s_nop 0", load) == 0
    assert one("s_mov_b32 m0, s3", "global_load_dword v2, v3, s[6:7]") == 0
    assert one("v_readfirstlane_b32 s7, v1", "s_nop 3", load) == 1
    assert one("v_readfirstlane_b32 s7, v1", "s_nop 4", load) == 0


@pytest.mark.parametrize("source", ["prepass.hip", "mask_inst.hip", "fidelity.hip", "resize.hip",
                                    "attn_fwd.hip"])
def test_wait_states(source, tmp_path):
    found = too_soon(listing(source, tmp_path))
    assert not found, "%d pairs, the first: %s" % (len(found), found[:3])
