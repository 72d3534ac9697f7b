"""Checks on the assembly of the kernels that name registers in inline assembly (csrc/k_mlp_acc.hip, k_mlp_acc3.hip).

Their second layer accumulates in the accumulation registers, which the compiler believes free, and their matrix products
are written out, so the compiler does not know how long a product's result takes.  Both hold as long as the compiler keeps
its own values in vector registers and its own instructions away from fresh results; another compiler version or one more live value can end
that without a word.  ``check`` reads what the compiler wrote and raises ``RuntimeError`` when one of these does not hold:

* no spilled vector register and no scratch memory, and no accumulation register outside inline assembly;
* nothing but a product that accumulates into them touches a product's results within MFMA_WAIT wait states of it (the result of
  an 8-pass product; a product that follows another issues 8 wait states behind it), on every path through a branch;
* no product reads what a vector instruction wrote less than VALU_WAIT wait states before.
"""
from __future__ import annotations

import re

MFMA_PASSES, MFMA_WAIT, VALU_WAIT = 8, 12, 2
_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|\[?(\d+)\]?)(?![\w.])")
_SPAN = 96          # instructions behind a branch target that are looked at with the state of the branch


def _regs(text):
    out = set()
    for kind, lo, hi, one in _REG.findall(text):
        lo, hi = (int(lo), int(hi)) if lo else (int(one), int(one))
        out.update((kind, n) for n in range(lo, hi + 1))
    return out


def parse(asm):
    """(instructions, labels): instructions are (opcode, [operand, ...], inside inline assembly, line number)."""
    ins, labels, inline = [], {}, False
    for no, line in enumerate(asm.splitlines(), 1):
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
            continue
        line = line.split(";")[0].split("//")[0].strip()
        m = re.match(r"([.\w$]+):$", line)
        if m:
            labels[m.group(1)] = len(ins)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" " if " " in line else "\t")
            op, _, more = op.partition("\t")
            ins.append((op, [t.strip() for t in (more + " " + rest).strip().split(",")], inline, no))
    return ins, labels


class _State:
    def __init__(self, other=None):
        self.t = other.t if other else 0
        self.last = other.last if other else -MFMA_PASSES               # issue of the last product
        self.mfma = dict(other.mfma) if other else {}                   # register -> issue of the product that writes it
        self.valu = dict(other.valu) if other else {}                   # register -> issue of the vector instruction that wrote it

    def step(self, op, args, no):
        if op.startswith("v_mfma"):
            at = max(self.t, self.last + MFMA_PASSES)
            d, a, b, c = (_regs(x) for x in args[:4])
            fresh = {r for r in a | b | (c - d) | (d - c) if r in self.mfma and at - self.mfma[r] - 1 < MFMA_WAIT}
            if fresh:
                raise RuntimeError(f"line {no}: a product takes operands from another one's fresh results {sorted(fresh)[:4]}")
            young = {r for r in a | b | c if r in self.valu and at - self.valu[r] - 1 < VALU_WAIT}
            if young:
                raise RuntimeError(f"line {no}: a product reads {sorted(young)[:4]} right behind the vector instruction that writes it")
            self.last, self.t = at, at + 1
            for r in d:
                self.mfma[r] = at
                self.valu.pop(r, None)
            return
        touched = set().union(*(_regs(x) for x in args)) if args else set()
        fresh = {r for r in touched if r in self.mfma and self.t - self.mfma[r] - 1 < MFMA_WAIT}
        if fresh:
            raise RuntimeError(f"line {no}: {op} touches a product's fresh results {sorted(fresh)[:4]}")
        if op.startswith("v_"):
            for r in _regs(args[0]):
                self.valu[r] = self.t
        self.t += int(args[0], 0) + 1 if op == "s_nop" else 1


def check(asm, name="assembly"):
    """Raise RuntimeError where `asm`, the device assembly of one of these units, breaks what the kernels rely on."""
    for what in (".vgpr_spill_count:", ".private_segment_fixed_size:"):
        found = re.findall(re.escape(what) + r"\s+(\d+)", asm)
        if not found or any(int(n) for n in found):
            raise RuntimeError(f"{name}: {what} {found}, wanted 0 (a spill takes accumulation registers)")
    ins, labels = parse(asm)
    if not any(op.startswith("v_mfma") for op, _, _, _ in ins):
        raise RuntimeError(f"{name}: no matrix product found")
    try:
        state, branches = _State(), []
        for i, (op, args, inline, no) in enumerate(ins):
            if not inline and any(k == "a" for x in args for k, _ in _regs(x)):
                raise RuntimeError(f"line {no}: the compiler uses an accumulation register ({op} {', '.join(args)})")
            state.step(op, args, no)
            if re.match(r"s_c?branch", op):
                branches.append((labels[args[0]], _State(state)))
        for start, at in branches:
            for op, args, _, no in ins[start:start + _SPAN]:
                at.step(op, args, no)
                if op in ("s_branch", "s_endpgm"):
                    break
    except RuntimeError as e:
        raise RuntimeError(f"{name}: {e}") from None
