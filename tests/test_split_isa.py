"""The static checks of test_kernel_isa on the kernels whose items are shared by several slots."""

import re
from collections import Counter

from test_kernel_isa import HIPCC, SRC, ROOT

import os
import subprocess

import pytest


@pytest.fixture(scope="module")
def split_kernels(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    from paper_2606_23019_amd import build
    out = str(tmp_path_factory.mktemp("isa") / "attn.s")
    subprocess.run([HIPCC] + [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")] + [
        "-I", os.path.join(ROOT, "include"), "-I", os.path.dirname(SRC), "--cuda-device-only", "-S",
        "-o", out, SRC], check=True, capture_output=True)
    text = open(out).read()
    names = sorted(set(re.findall(r"^(_ZN2sa\S+bsattn_(?:mask_)?split_kernel\S+):", text, re.M)))
    code = {n: text[text.index("\n%s:" % n):] for n in names}
    code = {n: c[:c.index(".Lfunc_end")].split("\n") for n, c in code.items()}
    meta = {re.search(r"\.name:\s+(\S+)", b).group(1): b
            for b in text.split("  - .agpr_count")[1:] if ".name:" in b}
    return code, meta


def test_split_kernels_found(split_kernels):
    code, _ = split_kernels
    # 128-row items in two parts: two key block sizes x two head dims, bf16 or fp32 out, and the
    # square ones maskless; 64-row items in two and four: (64, 64) x two head dims and (64, 128)
    # with d = 64, bf16 or fp32 out, and the square ones maskless
    walks = [n for n in code if "mask_split" in n]
    assert len(code) - len(walks) == (4 * 2 + 2) + 2 * (3 * 2 + 2), sorted(code)
    # the walk off the mask, one item a workgroup: the masked ones in two and four parts
    assert len(walks) == 4 * 2 + 3 * 2, walks


def test_split_kernels_keep_no_scratch_and_only_copies_in_loops(split_kernels):
    code, meta = split_kernels
    for name, lines in code.items():
        for key in ("vgpr_spill_count", "private_segment_fixed_size"):
            assert int(re.search(r"\.%s:\s+(\d+)" % key, meta[name]).group(1)) == 0, (name, key)
        # the outermost loops; the one over key blocks has the most lines, those before it walk
        # the mask row (Q's loads may stand between)
        spans = []
        for i, line in enumerate(lines):
            m = re.match(r"^\.L(BB\d+_\d+):.*Loop Header: Depth=1", line)
            if m:
                at = [j for j, l in enumerate(lines) if "Header=%s " % m.group(1) in l] + [i]
                hi = max(at) + 1
                while hi < len(lines) and not re.match(r"^\.LBB|^; %bb", lines[hi]):
                    hi += 1
                spans.append(lines[min(at):hi])
        inside = max(spans, key=len)
        assert any("v_mfma" in l for l in inside) and any("v_exp" in l for l in inside), name
        ops = Counter(l.split()[0] for l in inside
                      if re.match(r"^\s+(global_|buffer_|scratch_|flat_)", l))
        assert set(ops) == {"global_load_lds_dwordx4"}, (name, dict(ops))
