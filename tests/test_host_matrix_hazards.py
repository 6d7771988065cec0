"""Matrix instructions issued from inline assembly: the compiler pads neither what they read nor what they write, so the
built code itself is looked at (gfx950, the bf16 products of eight passes that are issued so).  A source written by an ordinary vector instruction needs two
wait states in between, a result eleven before anything but a product may touch it.  What the compiler puts in front of such a
product on its own account -- a copy between the register files, a packed weight that it makes as late as it can -- shows here
first, and on the GPU as wrong values."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_26289_amd import binding as dk

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
PRODUCT, SOURCE_WAIT, RESULT_WAIT = "v_mfma_f32_32x32x16_bf16", 2, 11
_REG = re.compile(r"-?\|?([va])(?:\[(\d+):(\d+)\]|(\d+))")


def _regs(text):
    m = _REG.match(text.strip())
    if not m:
        return frozenset()
    lo, hi = (int(m.group(2)), int(m.group(3))) if m.group(2) else (int(m.group(4)),) * 2
    return frozenset((m.group(1), i) for i in range(lo, hi + 1))


def _writes_reads(op, args):
    regs = [_regs(a) for a in args]
    rest = frozenset().union(*regs[1:])
    if op.startswith(("v_permlane32_swap", "v_swap")):
        return regs[0] | regs[1], regs[0] | regs[1]
    if op.startswith(("v_cmp", "v_readfirstlane", "v_readlane")):
        return frozenset(), rest
    if op.startswith("v_fmac"):
        return regs[0], rest | regs[0]
    if op.startswith(("v_", "ds_read", "global_load_dword", "flat_load", "scratch_load")):
        return regs[0], rest
    return frozenset(), rest | (regs[0] if regs else frozenset())  # stores, and loads into LDS


def hazards(lines):
    """(line, what) of every product too close to what made its sources, or to what touches its result"""
    found, recent = [], []  # recent: (operation, registers written, wait states), oldest first
    for line in lines:
        line = line.split("//")[0].strip()
        if not line or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            recent = []
            continue
        if op == "s_nop":
            recent = recent[-RESULT_WAIT:] + [(op, frozenset(), int(rest, 0) + 1)]
            continue
        product = op.startswith("v_mfma")
        writes = frozenset()
        if op.startswith(("v_", "ds_", "global_", "flat_", "scratch_")):
            writes, reads = _writes_reads(op, rest.split(","))
            wait = 0
            for was, wrote, states in reversed(recent):
                if op == PRODUCT and wait < SOURCE_WAIT and was.startswith("v_") and not was.startswith("v_mfma") and wrote & reads:
                    found.append((line, f"source written by {was} {wait} wait states before"))
                if not product and was == PRODUCT and wait < RESULT_WAIT and wrote & (reads | writes):
                    found.append((line, f"result of {was} {wait} wait states before"))
                wait += states
                if wait >= RESULT_WAIT:
                    break
        recent = recent[-RESULT_WAIT:] + [(op, writes, 1)]
    return found


def test_the_check_sees_what_it_is_for():
    mfma = "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"
    assert hazards(["v_cvt_pk_bf16_f32 v9, v1, v2", "s_nop 0", mfma])
    assert not hazards(["v_cvt_pk_bf16_f32 v9, v1, v2", "s_nop 1", mfma])
    assert hazards(["v_accvgpr_write_b32 a3, v1", mfma])
    assert hazards([mfma, "s_nop 9", "v_accvgpr_read_b32 v1, a15"])
    assert not hazards([mfma, "s_nop 10", "v_accvgpr_read_b32 v1, a15"])
    assert not hazards([mfma, mfma, "v_mov_b32_e32 v4, v3"])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_product_of_the_built_library_is_too_close_to_its_operands(tmp_path):
    lib = shutil.copy(dk.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    products, bad = 0, []
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / name)], check=True, capture_output=True, text=True).stdout
        lines = [x for x in text.splitlines() if x.startswith("\t") or x.endswith(">:")]
        products += sum("v_mfma" in x for x in lines)
        bad += [(name, *h) for h in hazards(lines)]
    assert products > 1000  # (the disassembly is that of the kernels)
    assert not bad, bad[:5]
