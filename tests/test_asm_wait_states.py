"""Wait states around inline assembly, read off the assembly the compiler writes for gfx950 (no GPU needed).

The hardware does not interlock every pair of dependent instructions; the compiler puts the missing wait
states in front of the instructions it emits itself, but it does not look inside inline assembly. On every path
  - inline assembly is not the first to touch the result of a matrix instruction: a compiler instruction
    that reads or overwrites the accumulator, and so waits for it, comes before it;
  - a scalar register that a vector instruction has written is read by a memory instruction of inline
    assembly five wait states later at the earliest, by a vector instruction of it two;
  - a vector register that inline assembly has written is read by a lane permute two wait states later at
    the earliest, by a lane read one;
  - a matrix instruction of inline assembly continues a sum that a matrix instruction has begun only in the very registers of
    it, and reads operands that a vector instruction has written two wait states later at the earliest;
  - where inline assembly names accumulation registers, nothing the compiler emits touches any."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2508_21058_amd import build

_REG = re.compile(r"(?<![\w.])([vsa])(?:\[(0x[0-9a-f]+|\d+)(?::(0x[0-9a-f]+|\d+))?\]|(\d+)(?!\w))")


def _regs(text):
    out = set()
    for kind, lo, hi, one in _REG.findall(text):
        out |= {(kind, i) for i in range(int(lo or one, 0), int(hi or lo or one, 0) + 1)}
    return out


def _kernels(text):
    """{function: [(line, op, args, inside inline assembly)]}; a label is an instruction named "label"."""
    fns, fn, inline = {}, None, False
    for no, raw in enumerate(text.splitlines(), 1):
        line = raw.strip()
        if line.startswith((";;#ASMSTART", ";;#ASMEND")):
            inline = line.startswith(";;#ASMSTART")
            continue
        line = line.split(";")[0].strip()
        label = re.match(r"([\w.$]+):$", line)
        if label and label[1].startswith("_Z"):
            fn = fns.setdefault(label[1], [])
        elif label and label[1].startswith(".Lfunc_end"):
            fn = None
        elif label and fn is not None:
            fn.append((no, "label", label[1], False))
        elif fn is not None and re.match(r"(v|s|ds|global|buffer|flat|scratch)_", line):
            op, _, args = line.partition(" ")
            fn.append((no, op, args, inline))
    return fns


def _written_read(op, args):
    """Registers an instruction writes and reads (the first operand is the destination where there is one)."""
    if op.startswith(("global_store", "buffer_store", "scratch_store", "flat_store", "ds_write", "global_load_lds", "s_cmp", "s_cbranch")):
        return set(), _regs(args)
    if op.startswith("v_permlane"):
        return _regs(args), _regs(args)
    parts = re.split(r",(?![^\[]*\])", args)
    carry = op.startswith(("v_add_co", "v_sub_co", "v_addc_co", "v_subb_co", "v_mad_u64", "v_mad_i64", "v_div_scale"))
    n = 2 if carry else 1
    return _regs(",".join(parts[:n])), _regs(",".join(parts[n:]))


class _Pending:
    """What may be outstanding in front of an instruction, over all paths that lead to it."""

    def __init__(self, matrix=(), scalar=(), vector=(), operand=()):
        self.matrix = set(matrix)          # register tuples of matrix results nobody has waited for
        self.scalar = dict(scalar)         # scalar registers a vector instruction wrote: wait states since (< 5)
        self.vector = dict(vector)         # vector registers inline assembly wrote: wait states since (< 2)
        self.operand = dict(operand)       # vector registers a vector instruction wrote: wait states since (< 2)

    def copy(self):
        return _Pending(self.matrix, self.scalar, self.vector, self.operand)

    def merge(self, other):
        out = _Pending(self.matrix | other.matrix, self.scalar, self.vector, self.operand)
        for mine, more in ((out.scalar, other.scalar), (out.vector, other.vector), (out.operand, other.operand)):
            for r, age in more.items():
                mine[r] = min(mine.get(r, age), age)
        return out

    def __eq__(self, other):
        return other is not None and (self.matrix, self.scalar, self.vector, self.operand) == (other.matrix, other.scalar, other.vector, other.operand)

    def step(self, op, args, inline):
        """Moves past one instruction; returns what is wrong with it."""
        if op == "label":
            return []
        written, read = _written_read(op, args)
        touched = {t for t in self.matrix if (written | read) & set(t)}
        # (a product into the registers of another goes on with its sum: the ones here name them as their third operand too)
        chained = tuple(sorted(written)) if inline and op.startswith("v_mfma") else None
        bad = ["touches a matrix result first"] if inline and touched - {chained} else []
        if chained and any(self.operand.get(r, 9) < 2 for r in read):
            bad.append("reads an operand less than two wait states after a vector instruction wrote it")
        need = 2 if op.startswith("v_") else 5 if op.startswith(("global_", "buffer_", "flat_", "scratch_")) else 0
        if inline and any(self.scalar.get(r, 9) < need for r in read):
            bad.append(f"reads a scalar register less than {need} wait states after a vector instruction wrote it")
        need = 2 if op.startswith("v_permlane") else 1 if op.startswith(("v_readlane", "v_readfirstlane")) else 0
        if any(self.vector.get(r, 9) < need for r in read):
            bad.append(f"reads a register less than {need} wait states after inline assembly wrote it")
        passed = int(args, 0) + 1 if op == "s_nop" else 1
        self.scalar = {r: n + passed for r, n in self.scalar.items() if n + passed < 5 and r not in written}
        self.vector = {r: n + passed for r, n in self.vector.items() if n + passed < 2 and r not in written}
        self.operand = {r: n + passed for r, n in self.operand.items() if n + passed < 2 and r not in written}
        if passed > 15:                    # outlasts the products here, of eight passes at most (32x32x16 in bf16); not one of sixteen
            self.matrix.clear()
        self.matrix -= touched
        if op.startswith("v_mfma"):
            self.matrix.add(tuple(sorted(written)))
        if op.startswith("v_"):
            self.scalar.update({r: 0 for r in written if r[0] == "s"})
            self.vector.update({r: 0 for r in written if r[0] == "v" and inline})
            if not op.startswith("v_mfma"):
                self.operand.update({r: 0 for r in written if r[0] == "v"})
        return bad


def _violations(ins):
    """Forward data flow over the instructions of one function."""
    at = {a: i for i, (_, op, a, _) in enumerate(ins) if op == "label"}
    succ = []
    for i, (_, op, args, _) in enumerate(ins):
        follow = [i + 1] if i + 1 < len(ins) else []
        if op == "s_branch":
            follow = [at[args]]
        elif op.startswith("s_cbranch"):
            follow = follow + [at[args]]
        elif op == "s_endpgm":
            follow = []
        succ.append(follow)
    leaders = {0} | set(at.values()) | {j for i, f in enumerate(succ) if f != [i + 1] for j in f + [i + 1]}
    state, work, bad = {0: _Pending()}, [0], set()
    while work:
        i = start = work.pop()
        cur = state[start].copy()
        while True:
            no, op, args, inline = ins[i]
            bad |= {(no, op, args, why) for why in cur.step(op, args, inline)}
            if succ[i] != [i + 1] or i + 1 in leaders:
                break
            i += 1
        for j in succ[i]:
            new = cur.merge(state[j]) if j in state else cur
            if new != state.get(j):
                state[j] = new.copy()
                work.append(j)
    return sorted(bad)


def _named_accumulators(ins):
    """Compiler instructions that touch accumulation registers in a function whose inline assembly names some."""
    def touches(op, args):
        return op != "label" and any(r[0] == "a" for r in _regs(args))
    if not any(inline and touches(op, args) for _, op, args, inline in ins):
        return []
    return [(no, op, args, "touches accumulation registers that inline assembly names")
            for no, op, args, inline in ins if not inline and touches(op, args)]


def _check(text):
    return {f: v for f, ins in _kernels(text).items() if ins for v in [_violations(ins) + _named_accumulators(ins)] if v}


_MFMA = "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], 0\n"
_ASM = "\t;;#ASMSTART\n\t%s\n\t;;#ASMEND\n"
_SUM = "v_mfma_f32_32x32x16_bf16 a[0:0xf], v[16:19], v[20:23], a[0:0xf]"
_BASE = "\tv_readfirstlane_b32 s8, v40\n\tv_readfirstlane_b32 s9, v41\n"
_COPY = "s_mov_b32 m0, s4\n\ts_nop %d\n\tglobal_load_lds_dwordx4 v42, s[8:9]"


@pytest.mark.parametrize("body,found", [
    (_MFMA + _ASM % "v_max_f32 v30, 0xff800000, v3", True),
    (_MFMA + "\ts_nop 7\n\tv_mov_b32_e32 v31, v3\n" + _ASM % "v_max_f32 v30, 0xff800000, v4", False),
    (_MFMA + _ASM % "v_max_f32 v30, 0xff800000, v33", False),
    # a branch around the one instruction that waits
    (_MFMA + "\ts_cbranch_execz .LBB0_1\n\tv_mov_b32_e32 v31, v3\n.LBB0_1:\n" + _ASM % "v_max_f32 v30, 0xff800000, v4", True),
    # round a loop
    ("\ts_mov_b32 s0, 0\n.LBB0_1:\n" + _ASM % "v_max_f32 v30, 0xff800000, v4" + _MFMA + "\ts_cbranch_scc1 .LBB0_1\n", True),
    (_ASM % _SUM + _ASM % _SUM, False),
    (_ASM % _SUM + _ASM % "v_accvgpr_read_b32 v30, a[3]", True),
    (_ASM % _SUM + _ASM % "s_nop 15" + _ASM % "v_accvgpr_read_b32 v30, a[3]", False),
    (_ASM % _SUM + _ASM % _SUM.replace("[0:0xf]", "[8:23]"), True),
    ("\tv_mov_b32_e32 v20, v1\n" + _ASM % _SUM, True),
    ("\tv_mov_b32_e32 v20, v1\n" + _ASM % ("s_nop 1\n\t" + _SUM), False),
    (_ASM % _SUM + "\tv_accvgpr_write_b32 a200, v1\n", True),
    (_BASE + _ASM % (_COPY % 0), True),
    (_BASE + _ASM % (_COPY % 3), False),
    (_BASE + "\ts_add_u32 s8, s8, s6\n\ts_addc_u32 s9, s9, 0\n" + _ASM % (_COPY % 0), False),
    (_ASM % "v_max_f64 v[2:3], v[4:5], v[6:7]" + "\tv_permlane32_swap_b32_e32 v2, v3\n", True),
    (_ASM % "v_max_f64 v[2:3], v[4:5], v[6:7]" + "\ts_nop 1\n\tv_permlane32_swap_b32_e32 v2, v3\n", False),
])
def test_the_reader_sees_planted_faults(body, found):
    assert bool(_check("_Zkernel: ; @_Zkernel\n" + body + "\ts_endpgm\n")) == found


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_no_unguarded_inline_assembly(tmp_path):
    def assemble(unit):
        out = str(tmp_path / (unit + ".s"))
        subprocess.run(["hipcc", *build.FLAGS, *build.UNIT_FLAGS.get(unit, []), "--cuda-device-only", "-S", os.path.join(build.CSRC, unit + ".hip"), "-o", out],
                       check=True, capture_output=True)
        return open(out).read()

    units = [u for u in build.UNITS if u != "moc_api"]         # (no kernels there)
    with ThreadPoolExecutor(max_workers=6) as ex:
        texts = dict(zip(units, ex.map(assemble, units)))
    assert sum(len(_kernels(t)) for t in texts.values()) > 50, "the assembly was not understood"
    bad = {u: v for u, t in texts.items() for v in [_check(t)] if v}
    assert not bad, "\n".join(f"{u} {f[:70]} line {no}: {op} {args}: {why}"
                              for u, fs in bad.items() for f, v in fs.items() for no, op, args, why in v[:3])
