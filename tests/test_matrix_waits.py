"""The kernels whose matrix instructions are written as assembly (mfma_acc):
the compiler does not know the wait states that follow them, so nothing but
another matrix instruction may touch an accumulator within the longest of
them.  Where the compiler copies or spills accumulators in a loop it does
exactly that; this reads the assembly of the library's own sources."""
import os
import re
import subprocess

import pytest

from paper_2609_06072_amd import build as b

WAITS = 19   # states from a matrix instruction of 16 passes to a read of its result


def _regs(text):
    regs = set()
    for lo, hi in re.findall(r"\ba\[(\d+):(\d+)\]", text):
        regs |= set(range(int(lo), int(hi) + 1))
    return regs | {int(r) for r in re.findall(r"\ba(\d+)\b", text)}


def _parse(text):
    """(instructions, label -> index) of a function; an instruction is
    (opcode, text, written as assembly)."""
    ins, labels, in_asm = [], {}, False
    for line in text.split("\n"):
        line = line.strip()
        if line.startswith(";"):
            in_asm = "ASMSTART" in line or (in_asm and "ASMEND" not in line)
            continue
        line = line.split(";")[0].strip()
        m = re.match(r"^(\S+):$", line)
        if m:
            labels[m.group(1)] = len(ins)
        elif line and not line.startswith("."):
            ins.append((line.split()[0], line, in_asm))
    return ins, labels


def too_close(text):
    """Instructions that touch an accumulator within WAITS states of the
    assembly-written matrix instruction that wrote it, along any path."""
    ins, labels = _parse(text)
    found = []
    for i, (op, line, in_asm) in enumerate(ins):
        if not (in_asm and op.startswith("v_mfma")):
            continue
        acc = _regs(line.split(",")[0])
        work, seen = [(i + 1, 0)], {}
        while work:
            j, t = work.pop()
            if t >= WAITS or j >= len(ins) or seen.get(j, WAITS) <= t:
                continue
            seen[j] = t
            o, l, _ = ins[j]
            if not o.startswith("v_mfma") and _regs(l) & acc:
                found.append(f"{line}  ->  {l}")
                continue
            if o == "s_endpgm":
                continue
            step = int(l.split()[1]) + 1 if o == "s_nop" else 1
            if "branch" in o:
                work.append((labels[l.split()[1]], t + step))
            if o != "s_branch":
                work.append((j + 1, t + step))
    return found


def _functions(asm):
    for m in re.finditer(r"^(_Z\S+):", asm, re.M):
        end = asm.find(".Lfunc_end", m.start())
        if end > 0:
            yield m.group(1), asm[m.end():end]


@pytest.mark.parametrize("source", ["moe_gemm.hip", "cka.hip"])
def test_accumulators_rest(source, tmp_path):
    out = tmp_path / "k.s"
    subprocess.run([b.hipcc(), *b.HIPFLAGS, "--cuda-device-only", "-S", os.path.join(b.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    n = 0
    for name, text in _functions(out.read_text()):
        ins, _ = _parse(text)
        n += sum(a and op.startswith("v_mfma") for op, _, a in ins)
        bad = too_close(text)
        assert not bad, f"{name}: {len(bad)}, first {bad[0]}"
    assert n > 0


def test_sources_with_assembly_matrix_instructions():
    """Every source that uses mfma_acc is in the list above."""
    using = [s for s in map(os.path.basename, b.sources())
             if "mfma_acc(" in open(os.path.join(b.CSRC, s)).read()]
    assert sorted(using) == ["cka.hip", "moe_gemm.hip"]


MFMA = "\t;;#ASMSTART\n\ts_nop 1\n\tv_mfma_f32_16x16x32_bf16 a[8:11], v[0:3], v[4:7], a[8:11]\n\t;;#ASMEND\n"


@pytest.mark.parametrize("after,bad", [
    ("\tscratch_store_dwordx4 off, a[8:11], off\n", True),
    ("\tscratch_store_dwordx4 off, a[12:15], off\n", False),
    ("\ts_nop 15\n\ts_nop 15\n\tv_accvgpr_read_b32 v0, a9\n", False),
    ("\ts_nop 15\n\tv_accvgpr_read_b32 v0, a9\n", True),
    ("\ts_cbranch_scc1 .L1\n\ts_endpgm\n.L1:\n\tv_accvgpr_mov_b32 a20, a10\n", True),
    ("\ts_branch .L1\n\tv_accvgpr_write_b32 a8, 0\n.L1:\n\ts_endpgm\n", False),
    ("\tv_mfma_f32_16x16x32_bf16 a[8:11], v[0:3], v[4:7], a[8:11]\n\ts_endpgm\n", False),
])
def test_checker(after, bad):
    assert bool(too_close(MFMA + after)) == bad
