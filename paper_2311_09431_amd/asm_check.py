"""What the compiler cannot check in the kernels' inline assembly, read from the assembly that the build
assembles (build.py; a build with a finding fails).

 * Accumulators by number: a kernel that keeps values in the accumulation registers between its asm statements
   only declares them as overwritten there.  Nothing tells the compiler that they live, so an instruction of its
   own that names one is a wrong result.
 * Matrix instructions of asm statements, which the compiler's hazard recogniser does not see: a vector
   instruction that writes an operand wants 2 wait states before the matrix instruction reads it, and a result
   wants 11 (8 passes + 3) before any other instruction names it or another product has it as a factor (adding to
   it may follow at once: that wait is the hardware's).  An instruction passes one wait state, s_nop n passes
   n + 1, and a matrix instruction as many as the one before it in the pipeline has passes (8 for 32 x 32 x 16).
"""
import re
from functools import cached_property

RESULT_WAIT, OPERAND_WAIT, PASSES = 11, 2, 8
_NUMBER = r"(0x[0-9a-f]+|\d+)"         # (constants of asm statements above 64 are printed in hex)
_REG = re.compile(r"\b([va])(?:\[%s:%s\]|\[%s\]|(\d+))(?![\w.])" % (_NUMBER, _NUMBER, _NUMBER))
_OPERAND_END = re.compile(r",(?![^\[]*\])")


def registers(text):
    out = set()
    for kind, lo, hi, boxed, one in _REG.findall(text):
        out.update((kind, i) for i in (range(int(lo, 0), int(hi, 0) + 1) if lo else (int(boxed or one, 0),)))
    return out


class Instruction:
    def __init__(self, text, line, by_hand):
        self.text, self.line, self.by_hand = text, line, by_hand
        self.next, self.before = [], []
        self.op, _, self.rest = text.partition(" ")
        self.matrix = self.op.startswith(("v_mfma", "v_smfmac"))
        self.vector = self.op.startswith("v_") and not self.matrix
        if self.op == "s_nop":
            self.wait = int(self.rest, 0) + 1
        else:
            self.wait = PASSES if self.matrix else 1

    @cached_property
    def names(self):
        return registers(self.rest)

    @cached_property
    def writes(self):       # of a vector or matrix instruction: the first operand, of a swap both
        return self.names if "swap" in self.op else registers(_OPERAND_END.split(self.rest)[0])

    @cached_property
    def reads(self):
        return registers(",".join(_OPERAND_END.split(self.rest)[1:]))

    @cached_property
    def factors(self):      # of a matrix instruction: what it multiplies
        return registers(",".join(_OPERAND_END.split(self.rest)[1:3]))


def functions(text):
    """name -> instructions, each with those that may follow it"""
    out, name, body, labels, by_hand = {}, None, [], {}, False
    for number, raw in enumerate(text.splitlines(), 1):
        line = raw.strip()
        if line.startswith(";;#ASM"):
            by_hand = line.startswith(";;#ASMSTART")
            continue
        line = line.split(";")[0].split("//")[0].strip()
        if line.endswith(":"):
            label = line[:-1]
            if not label.startswith("."):
                name, body, labels = label, [], {}
                out[name] = (body, labels)
            elif name:
                labels[label] = len(body)
            continue
        if name and line and not line.startswith("."):
            body.append(Instruction(re.sub(r"\s+", " ", line), number, by_hand))
    for body, labels in out.values():
        for i, x in enumerate(body):
            follow = [i + 1] if x.op not in ("s_branch", "s_endpgm", "s_setpc_b64") else []
            if x.op.startswith(("s_branch", "s_cbranch")):
                follow.append(labels[x.rest])
            for y in follow:
                if y < len(body):
                    x.next.append(body[y])
                    body[y].before.append(x)
    return {n: b for n, (b, _) in out.items()}


def _near(start, way, limit, bad):
    """Instructions before or after `start` (way), fewer than `limit` wait states apart, for which bad() holds."""
    found, seen, todo = [], {}, [(x, 0) for x in getattr(start, way)]
    while todo:
        x, apart = todo.pop()
        if seen.get(x, limit) <= apart:
            continue
        seen[x] = apart
        if bad(x):
            found.append(x)
        else:
            todo += [(y, apart + x.wait) for y in getattr(x, way)]
    return found


def check(text, numbered=()):
    """Findings, as lines of text.  numbered: parts of the names of kernels with accumulators by number."""
    findings = []
    bodies = functions(text)
    for part in numbered:
        of = [n for n in bodies if part in n]
        if not any(x.by_hand and x.matrix and any(k == "a" for k, _ in x.writes) for n in of for x in bodies[n]):
            findings.append("%s: no kernel with accumulators by number" % part)
        findings += ["%s, line %d: %s names an accumulator" % (n, x.line, x.text) for n in of for x in bodies[n]
                     if not x.by_hand and any(k == "a" for k, _ in x.names)]
    for name, body in bodies.items():
        for x in body:
            if not (x.matrix and x.by_hand):
                continue
            for y in _near(x, "before", OPERAND_WAIT, lambda y: y.vector and y.writes & x.reads):
                findings.append("%s, line %d: %s reads what was just written: %s" % (name, x.line, x.text, y.text))
            for y in _near(x, "next", RESULT_WAIT, lambda y: (y.factors if y.matrix else y.names) & x.writes):
                findings.append("%s, line %d: %s has not landed for: %s" % (name, x.line, x.text, y.text))
    return findings
