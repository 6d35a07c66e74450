"""Scan of compiled gfx950 assembly for the wait states that matrix instructions need.

The compiler inserts them for instructions that it knows; for a v_mfma inside an asm
statement it knows neither its latency nor that it is one, so whatever it places between
such an instruction and the next ordinary use of its registers is checked here, along
every path through the code (`hazards`):

* an accumulator written by an asm v_mfma is touched by no instruction but another v_mfma
  for RESULT wait states (the longest that any matrix instruction of this chip needs);
* a register written by a vector instruction is read by no asm v_mfma for OPERAND wait
  states.

An instruction counts one wait state, s_nop N counts N + 1.
"""
import re

RESULT = 19          # a 16-pass matrix instruction's result
OPERAND = 2          # a vector ALU result read as a matrix operand

_REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for kind, one, lo, hi in _REG.findall(text):
        for i in range(int(one or lo), int(one or hi) + 1):
            out.add((kind, i))
    return out


class _Ins:
    __slots__ = ("op", "text", "line", "dst", "regs", "asm", "target")

    def __init__(self, text, line, asm):
        self.text, self.line, self.asm = text, line, asm
        self.op, _, rest = text.partition(" ")
        ops = rest.split(",")
        self.regs = _regs(rest)
        # the first operand is written by vector ALU and matrix instructions; loads
        # announce theirs through the wait counters
        self.dst = _regs(ops[0]) if self.op.startswith("v_") else set()
        self.target = ops[0].strip() if self.op.startswith(("s_branch", "s_cbranch")) else None

    @property
    def mfma(self):
        return self.op.startswith("v_mfma")

    def states(self):
        return int(self.text.split()[1], 0) + 1 if self.op == "s_nop" else 1


def functions(asm):
    """{name: (instructions, {label: index})} of every kernel in an assembly listing."""
    out, cur, labels, in_asm = {}, None, {}, False
    for n, raw in enumerate(asm.splitlines(), 1):
        if "ASMSTART" in raw:
            in_asm = True
        elif "ASMEND" in raw:
            in_asm = False
        s = raw.split(";")[0].strip()
        if not s:
            continue
        m = re.match(r"([\w.$]+):$", s)
        if m:
            if not m.group(1).startswith(".L"):
                cur, labels = [], {}
                out[m.group(1)] = (cur, labels)
            elif cur is not None:
                labels[m.group(1)] = len(cur)
            continue
        if s.startswith(".") or cur is None:
            if s.startswith((".section", ".rodata")):
                cur = None
            continue
        for part in s.split("\\n"):
            cur.append(_Ins(re.sub(r"\s+", " ", part.strip()), n, in_asm))
    return {k: v for k, v in out.items() if v[0]}


def _walk(ins, labels, start, budget, bad):
    """Instructions reachable from after `start` within `budget` wait states for which
    bad(instruction) holds; a path ends where bad returns None."""
    found, best, todo = [], {}, [(start + 1, budget)]
    while todo:
        i, left = todo.pop()
        if i >= len(ins) or left <= 0 or best.get(i, 0) >= left:
            continue
        best[i] = left
        x = ins[i]
        b = bad(x)
        if b is None:
            continue
        if b:
            found.append(x)
        if x.op == "s_endpgm":
            continue
        if x.target is not None and x.target in labels:
            todo.append((labels[x.target], left - 1))
        if x.op != "s_branch":
            todo.append((i + 1, left - x.states()))
    return found


def hazards(asm):
    """(kernel, line, text, line of the later instruction, its text) of every pair of
    instructions closer than allowed; the number of asm v_mfma seen."""
    out, seen = [], 0
    for name, (ins, labels) in functions(asm).items():
        if not any(x.asm and x.mfma for x in ins):
            continue
        for i, x in enumerate(ins):
            if x.asm and x.mfma:
                seen += 1
                dst = x.dst
                # a later v_mfma on the same accumulator is ordered by the hardware
                hit = _walk(ins, labels, i, RESULT,
                            lambda y: None if y.mfma and y.dst == dst else
                            bool(y.regs & dst) and not (y.mfma and y.dst == dst))
            elif x.op.startswith("v_") and not x.mfma and x.dst:
                dst = x.dst
                hit = _walk(ins, labels, i, OPERAND,
                            lambda y: y.asm and y.mfma and bool(y.regs & dst))
            else:
                continue
            out += [(name, x.line, x.text, y.line, y.text) for y in hit]
    return out, seen
