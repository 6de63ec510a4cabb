"""Wait states around the matrix instructions that gemm_large.hip writes out as inline assembly.

The compiler keeps the distances that the hardware asks of the program around its own matrix instructions, but does not look into
inline assembly.  Checked here on the code it generates for every instantiation, along every path of control flow:

  * two wait states between a vector-ALU write of a register and a matrix instruction that reads it (for gfx950 the compiler
    puts an s_nop 1 there itself when the product is its own builtin);
  * no other instruction reads or writes an accumulation register that a matrix instruction wrote less than 20 wait states ago
    (the longest such distance, behind a 16-pass instruction; these have fewer passes).

A wait state is an instruction, or N + 1 of them for s_nop N.  Needs hipcc and no GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_26606_amd import build

VALU_TO_MATRIX = 2
MATRIX_TO_OTHER = 20
_REG = re.compile(r"^(?:([va])(\d+)|([va])\[(\d+):(\d+)\])$")


def _regs(operand):
    m = _REG.match(operand.strip())
    if not m:
        return frozenset()
    if m.group(1):
        return frozenset([(m.group(1), int(m.group(2)))])
    return frozenset((m.group(3), i) for i in range(int(m.group(4)), int(m.group(5)) + 1))


class _Ins:
    def __init__(self, text):
        self.text = text
        op, _, rest = text.partition(" ")
        self.op = op
        ops = [_regs(o.split(" ")[0] if not o.strip().startswith(("v[", "a[")) else o.strip().split(" ")[0])
               for o in (x.strip() for x in rest.split(","))] if rest else []
        self.regs = frozenset().union(*ops) if ops else frozenset()
        self.matrix = op.startswith(("v_mfma", "v_smfmac"))
        self.valu = op.startswith("v_") and not self.matrix
        # (compares and lane reads write scalar registers; a swap writes both of its operands)
        self.writes = (ops[0] if self.valu and ops else frozenset()) | (ops[1] if op.startswith("v_swap") else frozenset())
        self.reads = frozenset().union(*ops[1:4]) if self.matrix else frozenset()
        self.wrote = ops[0] if self.matrix else frozenset()
        self.states = int(rest, 0) + 1 if op == "s_nop" else 1
        self.ends = op in ("s_branch", "s_endpgm", "s_setpc_b64")
        self.target = rest.strip() if op.startswith(("s_cbranch", "s_branch")) else None


def _functions(asm):
    """name -> list of (instructions, labels before them): one flat list per function, labels as indices into it."""
    out, cur = {}, None
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        m = re.match(r"^(\S+):$", line)
        if m and m.group(1).startswith("_Z"):
            cur = out[m.group(1)] = ([], {})
        elif m and cur is not None:
            cur[1][m.group(1)] = len(cur[0])
        elif cur is not None and re.match(r"^(v_|s_|ds_|buffer_|global_|flat_|scratch_)", line):
            cur[0].append(_Ins(line))
        elif line.startswith(".section") or line.startswith(".end_amdhsa_kernel"):
            cur = None
    return out


def _backwards(ins, preds, at, limit):
    """Every instruction that can run less than `limit` wait states before ins[at]."""
    seen, todo = {}, [(p, 0) for p in preds[at]]
    while todo:
        i, away = todo.pop()
        if away >= limit or seen.get(i, limit) <= away:
            continue
        seen[i] = away
        todo += [(p, away + ins[i].states) for p in preds[i]]
    return seen


def violations(asm):
    """-> ({function: [what]}, number of matrix instructions looked at)"""
    bad, looked = {}, 0
    for name, (ins, labels) in _functions(asm).items():
        if not any(i.matrix for i in ins):
            continue
        preds = [[] for _ in ins]
        for i, x in enumerate(ins):
            if not x.ends and i + 1 < len(ins):
                preds[i + 1].append(i)
            if x.target is not None and labels.get(x.target, len(ins)) < len(ins):
                preds[labels[x.target]].append(i)
        for i, x in enumerate(ins):
            if x.matrix:
                looked += 1
                for j, away in _backwards(ins, preds, i, VALU_TO_MATRIX).items():
                    if ins[j].writes & x.reads:
                        bad.setdefault(name, []).append("%s | %d wait state(s) | %s" % (ins[j].text, away, x.text))
            elif any(r[0] == "a" for r in x.regs):
                for j, away in _backwards(ins, preds, i, MATRIX_TO_OTHER).items():
                    if ins[j].wrote & x.regs:
                        bad.setdefault(name, []).append("%s | %d wait state(s) | %s" % (ins[j].text, away, x.text))
    return bad, looked


def test_the_check_sees_a_missing_wait_state():
    text = """_Zk:
    s_mov_b32 s0, 0
    v_mov_b32_e32 v3, v9
    %s
    v_mfma_f32_16x16x32_f16 a[0:3], v[0:3], v[4:7], a[0:3]
    %s
    v_accvgpr_read_b32 v8, a2
    s_endpgm
"""
    drained = "s_nop 15\n    s_nop 15"
    assert violations(text % ("s_nop 1", drained)) == ({}, 1)
    assert len(violations(text % ("s_nop 0", drained))[0]["_Zk"]) == 1
    assert len(violations(text % ("s_nop 1", "s_nop 7"))[0]["_Zk"]) == 1
    loop = """_Zk:
.L1:
    v_mfma_f32_16x16x32_f16 a[0:3], v[0:3], v[4:7], a[0:3]
    s_nop 3
    v_mov_b32_e32 v4, v9
    s_cbranch_scc1 .L1
    s_endpgm
"""
    assert len(violations(loop)[0]["_Zk"]) == 1


def test_wait_states_before_and_behind_the_products(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc to compile the kernels with")
    out = str(tmp_path / "gemm_large.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    p = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm_large.hip"), "-o", out],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    bad, looked = violations(open(out).read())
    assert looked > 46 * 100                          # every instantiation has hundreds
    assert not bad, "%d places in %d kernels, e.g. %s: %s" % (sum(map(len, bad.values())), len(bad), *next(iter(bad.items())))
