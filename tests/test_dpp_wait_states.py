"""The Cholesky kernel's multiply-adds with a DPP operand are inline assembly, so the compiler does not see that the
register such an instruction reads across lanes must not have been written by a vector instruction within the two wait
states before it.  The source keeps that distance; a copy the register allocator puts there would break it silently.
This reads the assembly of the kernel as it is built."""
import os
import re
import subprocess

import pytest

from paper_2106_13308_amd import build as bd

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


def _regs(op):
    m = re.fullmatch(r"-?\|?v\[(\d+):(\d+)\]\|?", op) or re.fullmatch(r"-?\|?v(\d+)()\|?", op)
    return set() if not m else set(range(int(m[1]), int(m[2] or m[1]) + 1))


def hazards(asm):
    """(DPP instructions from inline assembly, those whose source was written less than two wait states before)"""
    seen, bad, recent = 0, [], []  # recent: (wait states ago, registers), a label counts as writing everything
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"[.\w$]+:$", line):
            recent = [(0, None)]
            continue
        m = re.match(r"([a-z]\w+)\s*(.*)", line)
        if not m:
            continue
        name, ops = m[1], [o.strip() for o in m[2].split(",")]
        if name == "v_fmac_f64_dpp":
            seen += 1
            src = _regs(ops[1])
            assert src, line
            bad += [line for _, r in recent if r is None or r & src]
        states = int(ops[0], 0) + 1 if name == "s_nop" else 1
        recent = [(a + states, r) for a, r in recent if a + states < 2]
        if name.startswith("v_"):
            w = _regs(ops[0]) | (_regs(ops[1]) if "swap" in name else set())
            recent.append((0, w))
    return seen, bad


def test_checker_finds_planted_hazards():
    use = "v_fmac_f64_dpp v[2:3], -v[4:5], v[6:7] row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
    for before, ok in (("v_mov_b32_e32 v5, v9\n", False), ("v_mul_f64 v[4:5], v[4:5], v[0:1]\nv_mov_b32_e32 v8, v9\n", False),
                       ("v_mov_b32_e32 v5, v9\ns_nop 0\n", False), ("v_mov_b32_e32 v5, v9\ns_nop 1\n", True),
                       ("v_mul_f64 v[4:5], v[4:5], v[0:1]\nv_mov_b32_e32 v8, v9\nv_mov_b32_e32 v8, v9\n", True),
                       ("ds_read_b64 v[4:5], v9\n", True), (".LBB0_1:\n", False), ("v_swap_b32 v9, v4\n", False)):
        seen, bad = hazards(before + use)
        assert seen == 1 and (not bad) == ok, before


def test_no_hazard_in_the_build(tmp_path):
    src, out = os.path.join(bd.CSRC, "chol.hip"), str(tmp_path / "chol.s")
    subprocess.run([bd.hipcc(), *bd.FLAGS, *bd.FILE_FLAGS.get("chol.hip", []), "-S", "--offload-device-only", src, "-o", out],
                   check=True, capture_output=True)
    seen, bad = hazards(open(out).read())
    assert seen > 100 and not bad, bad[:5]
