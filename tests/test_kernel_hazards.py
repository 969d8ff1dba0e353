"""The matrix ops of the 256 x 256 tiles are inline assembly, for which the compiler adds no wait states (no GPU).  In every GEMM kernel, along every path
of its control flow: no vector instruction writes an operand of a matrix op within the two wait states before it, and nothing but a matrix op reads
or writes the result of an inline one before it is there."""
import re

import pytest

UNITS = ["k_fwd", "k_bwd", "k_wgrad", "k_dense_a", "k_dense_b", "k_fp8", "k_fp8_rowwise", "k_probe"]
WAIT = 2
# The ISA guide's table for this family: a vector, LDS or memory instruction that reads or overwrites a matrix result waits 5, 7, 11 or 19 states, by
# the op's 2, 4, 8 or 16 passes; one more on gfx950.  The inline ops have 4 or 8 passes.
DRAIN = 12


def _registers(operand):
    m = re.fullmatch(r"([va])(\d+)|([va])\[(\d+):(\d+)\]", operand)
    if not m:
        return frozenset()
    return frozenset([(m[1], int(m[2]))] if m[1] else [(m[3], i) for i in range(int(m[4]), int(m[5]) + 1)])


class _Op:
    __slots__ = ("text", "name", "states", "matrix", "inline", "writes", "reads", "goes", "falls")

    def __init__(self, text, inline):
        self.text, self.inline = text, inline
        self.name, _, rest = text.partition(" ")
        operands = [a.strip().split(" ")[0] for a in rest.split(",")]
        self.states = int(rest.split()[0]) + 1 if self.name == "s_nop" else 1
        self.matrix = "mfma" in self.name or "smfmac" in self.name
        regs = [_registers(a) for a in operands]
        stores = "store" in self.name or self.name.startswith("ds_write")
        self.writes = frozenset() if stores or not regs else regs[0]
        self.reads = frozenset().union(*(regs if stores or self.matrix else regs[1:]))
        self.goes = operands[0] if self.name.startswith("s_cbranch") or self.name == "s_branch" else None
        self.falls = self.name not in ("s_branch", "s_endpgm", "s_setpc_b64")


def _kernels(text):
    """Each function's instructions, its labels (name -> index of the next instruction)."""
    ops, labels, inline = [], {}, False
    for line in text.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
            continue
        x = line.split(";")[0].strip()
        if x.startswith(".Lfunc_end"):
            yield ops, labels
            ops, labels = [], {}
        elif x.endswith(":"):
            labels[x[:-1]] = len(ops)
        elif x and x[0] != ".":
            ops.append(_Op(x, inline))
    if ops:
        yield ops, labels


def _hazards(text):
    """(matrix ops, those with an operand written too shortly before, inline ones whose result is touched too shortly after)"""
    count, early, late = 0, [], []
    for ops, labels in _kernels(text):
        after = [[*([i + 1] if o.falls and i + 1 < len(ops) else []), *([labels[o.goes]] if o.goes in labels and labels[o.goes] < len(ops) else [])] for i, o in enumerate(ops)]
        before = [[] for _ in ops]
        for i, js in enumerate(after):
            for j in js:
                before[j].append(i)

        def walk(start, edges, limit, hit):
            seen, todo = {}, [(j, 0) for j in edges[start]]
            while todo:
                j, waited = todo.pop()
                if waited >= limit or seen.get(j, limit) <= waited:
                    continue
                seen[j] = waited
                if hit(ops[j]):
                    return True
                todo += [(k, waited + ops[j].states) for k in edges[j]]
            return False

        for i, o in enumerate(ops):
            if not o.matrix:
                continue
            count += 1
            used = o.reads | o.writes
            if walk(i, before, WAIT, lambda p: p.name.startswith("v_") and not p.matrix and bool(p.writes & used)):
                early.append(o.text)
            if o.inline and walk(i, after, DRAIN, lambda p: not p.matrix and bool((p.reads | p.writes) & o.writes)):
                late.append(o.text)
    return count, early, late


@pytest.mark.parametrize("unit", UNITS)
def test_no_operand_or_result_is_touched_too_close_to_a_matrix_op(assembly, unit):
    ops, early, late = _hazards(assembly[unit])
    assert ops > 500 and not early and not late, (unit, ops, early[:5], late[:5])


def test_the_check_finds_hazards():
    near = "v_mov_b32_e32 v5, v9\n\ts_nop 0\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[2:5], v[6:9], a[0:3]\n"
    far = near.replace("s_nop 0", "s_nop 1")
    assert len(_hazards(near)[1]) == 1 and _hazards(far) == (1, [], [])
    # the write stands at the end of a loop's body, the op at its head
    loop = ".LBB0_1:\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[2:5], v[6:9], a[0:3]\n\tv_mov_b32_e32 v7, v1\n\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n"
    assert len(_hazards(loop)[1]) == 1
    assert _hazards(loop.replace("\ts_cbranch", "\ts_nop 0\n\ts_cbranch"))[1] == []
    # a result read, overwritten or stored too early after an inline op, also across a branch
    inline = "\t;;#ASMSTART\n\tv_smfmac_f32_16x16x64_bf16 a[0:3], v[2:5], v[6:13], v20\n\t;;#ASMEND\n%s\ts_endpgm\n"
    for touch in ("v_accvgpr_read_b32 v1, a2", "v_accvgpr_write_b32 a3, v1", "scratch_store_dwordx2 off, a[0:1], off", "ds_write_b32 v1, a0"):
        assert len(_hazards(inline % f"\ts_nop {DRAIN - 2}\n\t{touch}\n")[2]) == 1, touch
        assert _hazards(inline % f"\ts_nop {DRAIN - 1}\n\t{touch}\n")[2] == [], touch
    assert len(_hazards(inline % "\ts_branch .LBB0_9\n\ts_endpgm\n.LBB0_9:\n\tv_accvgpr_read_b32 v1, a0\n")[2]) == 1
    # the next op takes the same accumulators
    assert _hazards(inline % "\tv_smfmac_f32_16x16x64_bf16 a[0:3], v[2:5], v[6:13], v20\n")[2] == []
