"""The video kernel's inline-asm MFMAs (the accumulators of O and the row sums):
the compiler's hazard recogniser does not see them, so the distances that
matrix instructions need are kept by the source's order and its drains.  This
compiles the kernels to assembly and measures those distances along every path
around each such MFMA, in wait states (one an instruction, k + 1 for s_nop k,
which is no more than the hardware takes):

- a vector instruction that writes an operand comes at least 2 ahead;
- its result (8 passes) is not touched by any other kind of instruction, nor
  taken as a factor by an MFMA, nor as part of another accumulator, for 11;
- its factors are not results of an MFMA of the last 11."""
import os
import re
import subprocess

import pytest

from paper_2607_04443_amd import _build

VALU_TO_MFMA, MFMA_RESULT = 2, 11


def _regs(text):
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo, hi = (int(m.group(4)),) * 2 if m.group(4) else (int(m.group(2)), int(m.group(3)))
        out.update((m.group(1), i) for i in range(lo, hi + 1))
    return out


class Ins:
    def __init__(self, text, in_asm, line):
        self.op, rest = (text.split(None, 1) + [""])[:2]
        self.text, self.in_asm, self.line, self.target = text, in_asm, line, rest.strip()
        self.mfma = self.op.startswith("v_mfma")
        t = re.split(r",(?![^\[]*\])", rest)
        first, others = _regs(t[0]), _regs(",".join(t[1:]))
        vector = self.op.startswith(("v_", "ds_", "global_", "buffer_", "flat_", "scratch_"))
        self.touched = first | others if vector else set()
        self.written = first if self.op.startswith("v_") else set()
        if "swap" in self.op:
            self.written = first | others
        self.states = int(self.target, 0) + 1 if self.op == "s_nop" else 1
        if self.mfma:
            self.d, self.c = first, _regs(t[3])
            self.ab = _regs(t[1]) | _regs(t[2])


def hazards(asm):
    """(asm MFMAs seen, faults) of an assembly text."""
    ins, labels, in_asm = [], {}, False
    for n, raw in enumerate(asm.splitlines(), 1):
        t = raw.strip()
        if t.startswith(";;#ASM"):
            in_asm = t.startswith(";;#ASMSTART")
            continue
        m = re.match(r"([\w.$]+):", raw)
        if m:
            labels[m.group(1)] = len(ins)
            continue
        t = t.split(";")[0].strip()
        if t and not t.startswith("."):
            ins.append(Ins(t, in_asm, n))
    after, before = [[] for _ in ins], [[] for _ in ins]
    for i, x in enumerate(ins):
        to = [] if x.op in ("s_endpgm", "s_branch") else [i + 1]
        if x.op == "s_branch" or x.op.startswith("s_cbranch"):
            to.append(labels[x.target])
        for j in to:
            if j < len(ins):
                after[i].append(j)
                before[j].append(i)

    def near(i, edges, limit, stop):
        best, todo = {}, [(j, 0) for j in edges[i]]
        while todo:
            j, d = todo.pop()
            if d >= limit or best.get(j, limit) <= d:
                continue
            best[j] = d
            if not stop(ins[j]):
                todo += [(k, d + ins[j].states) for k in edges[j]]
        return [(ins[j], d) for j, d in best.items()]

    found, n_asm = [], 0
    for i, x in enumerate(ins):
        if not (x.mfma and x.in_asm):
            continue
        n_asm += 1
        for y, d in near(i, before, MFMA_RESULT, lambda y: False):
            if y.mfma and y.d & x.ab:
                found.append((y.line, y.text, x.line, x.text, d))
            elif not y.mfma and d < VALU_TO_MFMA and y.written & (x.ab | x.c):
                found.append((y.line, y.text, x.line, x.text, d))
        for y, d in near(i, after, MFMA_RESULT, lambda y: y.mfma and y.d == x.d):
            clash = (y.ab & x.d or (y.c & x.d and y.c != x.d) or (y.d & x.d and y.d != x.d)) if y.mfma else y.touched & x.d
            if clash:
                found.append((x.line, x.text, y.line, y.text, d))
    return n_asm, found


MFMA = ";;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]\n\t;;#ASMEND\n"


@pytest.mark.parametrize("text,faults", [
    ("\tv_mov_b32_e32 v5, v1\n\ts_nop 0\n" + MFMA, 1),
    ("\tv_mov_b32_e32 v5, v1\n\ts_nop 1\n" + MFMA, 0),
    ("\tv_accvgpr_write_b32 a2, v1\n" + MFMA, 1),
    (MFMA + "\ts_nop 9\n\tv_accvgpr_read_b32 v0, a3\n", 1),
    (MFMA + "\ts_nop 10\n\tv_accvgpr_read_b32 v0, a3\n", 0),
    (MFMA + "\ts_cbranch_scc1 .L1\n\ts_nop 15\n.L1:\n\tglobal_store_dwordx4 v20, a[0:3], s[0:1]\n", 1),
    (MFMA + "\tv_mfma_f32_16x16x32_bf16 v[12:15], v[20:23], a[0:3], 0\n", 1),
    (MFMA + "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[20:23], v[8:11], a[0:3]\n", 0),
    ("\tv_mfma_f32_16x16x32_bf16 v[8:11], v[20:23], v[24:27], 0\n\ts_nop 7\n" + MFMA, 1),
    (".L2:\n" + MFMA + "\tv_mov_b32_e32 v9, v1\n\ts_branch .L2\n", 1),
])
def test_planted_hazards_are_found(text, faults):
    n, found = hazards(text)
    assert n == 1 and len(found) == faults, found


def test_no_hazard_around_the_inline_asm_mfmas(tmp_path):
    out = tmp_path / "kernels.asm"
    subprocess.run([_build._hipcc()] + _build.HIP_FLAGS + ["-x", "hip", "--offload-device-only", "-S",
                   os.path.join(_build.CSRC, "kernels.hip"), "-o", str(out)], check=True, capture_output=True)
    n, found = hazards(out.read_text())
    assert n > 500, n  # (three wave widths in two kernels)
    assert not found, found[:5]
