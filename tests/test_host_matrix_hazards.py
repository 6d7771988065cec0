"""Matrix instructions whose operands or results pass through inline assembly: the compiler pads neither, so the built code
itself is looked at (gfx950, the bf16 products of eight passes).  A source written by an ordinary vector instruction needs two
wait states in between, a result twelve before anything but a product that adds to it may touch it (what the compiler puts
there itself where it sees both sides: s_nop 11).  What it puts in front of such a product on its own account -- a copy between
the register files, a packed weight that it makes as late as it can -- shows here first, and on the GPU as wrong values; so does
a reader that stands on the far side of a branch, or at the head of a loop whose end is a product."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_26289_amd import binding as dk

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
PRODUCT, SOURCE_WAIT, RESULT_WAIT = "v_mfma_f32_32x32x16_bf16", 2, 12
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


class _Step:
    """One instruction: its registers, the wait states it stands for, and the instructions that may come next."""

    def __init__(self, line):
        self.line = line
        self.op, _, rest = line.partition(" ")
        self.product, self.next = self.op.startswith("v_mfma"), []
        self.states = int(rest, 0) + 1 if self.op == "s_nop" else 1
        self.target = rest.strip() if self.op.startswith(("s_branch", "s_cbranch")) else None
        self.ends = self.op in ("s_branch", "s_endpgm", "s_setpc_b64")
        self.writes = self.reads = self.factors = frozenset()
        if self.op.startswith(("v_", "ds_", "global_", "flat_", "scratch_")):
            args = rest.split(",")
            self.writes, self.reads = _writes_reads(self.op, args)
            self.factors = _regs(args[1]) | _regs(args[2]) if self.product else frozenset()


def _program(lines):
    steps, labels = [], {}
    for line in lines:
        line = line.split("//")[0].strip()
        if line.endswith(":"):
            labels[line[:-1].split()[-1].strip("<>")] = len(steps)
        elif line:
            steps.append(_Step(line))
    for i, s in enumerate(steps):
        if not s.ends and i + 1 < len(steps):
            s.next.append(steps[i + 1])
        if s.target is not None and labels[s.target] < len(steps):
            s.next.append(steps[labels[s.target]])
    return steps


def hazards(lines):
    """(line, what) of every product too close, on any way through the code, to what made its sources, and of everything
    too close to the product whose result it touches"""
    found = []
    for was in _program(lines):
        result = was.op == PRODUCT
        source = was.op.startswith("v_") and not was.product and bool(was.writes)
        limit = RESULT_WAIT if result else SOURCE_WAIT if source else 0
        ways, seen = [(n, 0) for n in was.next if limit], {}
        while ways:
            s, wait = ways.pop()
            if wait >= limit or seen.get(id(s), limit) <= wait:
                continue
            seen[id(s)] = wait
            if source and s.op == PRODUCT and was.writes & s.reads:
                found.append((s.line, f"source written by {was.op} {wait} wait states before"))
            touched = s.factors if s.product else s.reads | s.writes
            if result and was.writes & touched:
                found.append((s.line, f"result of {was.op} {wait} wait states before"))
            ways += [(n, wait + s.states) for n in s.next]
    return found


def test_the_check_sees_what_it_is_for():
    mfma = "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"
    assert hazards(["v_cvt_pk_bf16_f32 v9, v1, v2", "s_nop 0", mfma])
    assert not hazards(["v_cvt_pk_bf16_f32 v9, v1, v2", "s_nop 1", mfma])
    assert hazards(["v_accvgpr_write_b32 a3, v1", mfma])
    assert hazards([mfma, "s_nop 10", "v_accvgpr_read_b32 v1, a15"])
    assert not hazards([mfma, "s_nop 11", "v_accvgpr_read_b32 v1, a15"])
    assert hazards([mfma, "v_mfma_f32_32x32x16_bf16 a[16:31], v[4:7], a[8:11], a[16:31]"])
    assert not hazards([mfma, mfma, "v_mov_b32_e32 v4, v3"])


def test_the_check_follows_branches():
    mfma, read, wait = "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "v_accvgpr_read_b32 v1, a15", "s_nop 11"
    assert hazards([mfma, "s_cbranch_vccnz L1", wait, "<L1>:", read])  # the wait is on one way only
    assert not hazards([mfma, wait, "s_cbranch_vccnz L1", "s_nop 0", "<L1>:", read])
    assert hazards(["<L0>:", read, wait, mfma, "s_cbranch_scc1 L0", "s_endpgm"])  # once round the loop
    assert not hazards(["<L0>:", read, mfma, wait, "s_cbranch_scc1 L0", "s_endpgm"])
    assert not hazards([mfma, "s_branch L2", "<L1>:", read, "<L2>:", "s_endpgm"])
    assert hazards(["v_accvgpr_write_b32 a3, v1", "s_branch L2", "<L1>:", "s_endpgm", "<L2>:", mfma])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_product_of_the_built_library_is_too_close_to_its_operands(tmp_path):
    lib = shutil.copy(dk.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    products, bad = 0, []
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(tmp_path / name)], check=True,
                              capture_output=True, text=True).stdout
        kernels = [[]]  # (labels are numbered anew in every kernel)
        for x in text.splitlines():
            if re.match(r"[0-9a-f]+ <(?!L\d+>)", x):
                kernels.append([])
            elif x.startswith("\t") or x.endswith(">:"):
                kernels[-1].append(x)
        products += sum("v_mfma" in x for k in kernels for x in k)
        bad += [(name, *h) for k in kernels for h in hazards(k)]
    assert products > 1000  # (the disassembly is that of the kernels)
    assert not bad, bad[:5]
