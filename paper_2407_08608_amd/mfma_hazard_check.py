"""Static check of compiled gfx950 assembly: hand-written instructions and their neighbours keep their distance.

Some kernels issue `v_mfma_*` through inline assembly so that the accumulator lands in ordinary
registers.  The compiler's hazard recogniser does not look inside inline assembly, so nothing
stops it from scheduling, right behind such an MFMA, an instruction that reads or overwrites the
registers the MFMA is still going to write (a register-allocator copy is enough).  On this
hardware that is silent data corruption, not an error.  The kernels place explicit waits; this
script proves, on the assembly the build actually produced, that they suffice.

For every MFMA between `;;#ASMSTART` and `;;#ASMEND` whose destination is a VGPR range it walks
forward through the listing in its printed order, and additionally along every branch that is taken while
the result is not yet safe (a loop's back-edge, a forward branch that skips the wait), counting wait
states (one per instruction, N + 1 for `s_nop N`), and reports any non-MFMA
instruction that names a register of that range, and any MFMA that takes it as an A or B operand,
before `need` wait states have passed.  A following MFMA that accumulates into exactly the same
range is the hardware-interlocked case and is allowed.

The same holds ahead of such an MFMA: an ordinary vector instruction that writes one of its A, B or
accumulator registers (again, a copy the register allocator makes is enough) must be two wait states away
from it, the distance the compiler keeps in front of MFMAs of its own.  Those writes are followed over
branches in the same way.

The 8-pass 32x32x16 MFMA needs 11 wait states before a VALU read of its result and the 16-pass
32x32x64 e4m3 MFMA 19; the compiler leaves 12 (20) or more in the code it schedules itself, and those
are the defaults here.

`check_loads` does the same for hand-written memory instructions: a scalar register that one of them reads (its resource)
must not have been written by a vector instruction in the five wait states before it.  Such writes are rarely in the source;
a scalar register that was spilled comes back through v_readlane, which the compiler may put right ahead of the
assembly that uses it.
"""
import re
import sys

_REG_RANGE = re.compile(r"\b([va])\[(\d+):(\d+)\]")
_REG_ONE = re.compile(r"\b([va])(\d+)\b")
VALU_WRITE_STATES = 2  # between a vector instruction's write of a register and an MFMA that reads it


def _registers(text):
    """Vector registers named in `text`: ("v", n) and, of the accumulation half, ("a", n)."""
    out = set()
    for m in _REG_RANGE.finditer(text):
        out.update((m.group(1), n) for n in range(int(m.group(2)), int(m.group(3)) + 1))
    for m in _REG_ONE.finditer(text):
        out.add((m.group(1), int(m.group(2))))
    return out


def _vgprs(text):
    return {r for r in _registers(text) if r[0] == "v"}


def _valu_writes(op, args):
    """Registers that a vector instruction other than an MFMA writes (empty for anything else)."""
    if not op.startswith("v_") or op.startswith("v_mfma"):
        return set()
    operands = args.split(",")
    return _registers(",".join(operands[:2]) if "swap" in op else operands[0])  # swaps write both operands


def _parse(raw):
    """(op, args, wait states) of an instruction line, or None for anything else."""
    text = raw.split(";")[0].strip()
    if not text or text.startswith(".") or text.endswith(":"):
        return None
    op = text.split()[0]
    args = text[len(op):]
    return text, op, args, (int(args.strip()) + 1 if op == "s_nop" else 1)


def _walk(lines, labels, func, start, pending, written, track_new, need, need_16_pass, horizon, problems, depth):
    """Walks `lines` (of one function) from index `start` in listing order.  `pending` holds [registers,
    wait states so far, wait states required] of hand-written MFMAs whose results are not yet safe, `written`
    [registers, wait states so far] of vector instructions whose results an MFMA may not read yet.  With
    track_new the walk covers the function and registers every such instruction it meets; without, it
    only follows the entries it was given until they are safe.  A branch taken with entries still pending
    is followed to its target with a copy of them (the listing order alone would miss the reader at a loop
    head behind a back-edge, or behind a forward branch that skips the wait)."""
    in_asm = False
    for idx in range(start, len(lines)):
        ln, raw = lines[idx]
        stripped = raw.strip()
        if stripped.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if stripped.startswith(";;#ASMEND"):
            in_asm = False
            continue
        parsed = _parse(raw)
        if parsed is None:
            continue
        text, op, args, states = parsed
        if op.startswith("v_mfma"):
            parts = [a.strip() for a in args.split(",")]
            dst, ab = _vgprs(parts[0]), _vgprs(parts[1]) | _vgprs(parts[2])
            src_c = _vgprs(parts[3]) if len(parts) > 3 else set()
            for regs, waited, req in pending:
                if regs & ab and waited < req:
                    problems.append((func, ln, text, waited))
                if regs & src_c and regs != src_c and waited < req:
                    problems.append((func, ln, text, waited))
            if in_asm:
                read = _registers(",".join(parts[1:]))
                problems.extend((func, ln, text, waited) for regs, waited in written if regs & read)
            pending = [[regs, waited + states, req] for regs, waited, req in pending]
            if track_new and in_asm and dst:
                pending = [p for p in pending if p[0] != dst]
                pending.append([dst, 0, need_16_pass if "f8f6f4" in op else need])
        else:
            touched = _vgprs(args)
            for regs, waited, req in pending:
                if regs & touched and waited < req:
                    problems.append((func, ln, text, waited))
            pending = [[regs, waited + states, req] for regs, waited, req in pending]
            if op.startswith("s_cbranch") or op == "s_branch":
                unsafe = [list(p) for p in pending if p[1] < p[2]]
                recent = [[regs, waited + states] for regs, waited in written if waited + states < VALU_WRITE_STATES]
                target = labels.get(args.strip())
                if (unsafe or recent) and target is not None and depth < 4:
                    _walk(lines, labels, func, target, unsafe, recent, False, need, need_16_pass, horizon, problems,
                          depth + 1)
                if op == "s_branch" and not track_new:
                    return  # an unconditional branch: the followed entries continue at the target only
        pending = [p for p in pending if p[1] < horizon]
        written = [[regs, waited + states] for regs, waited in written if waited + states < VALU_WRITE_STATES]
        if track_new and _valu_writes(op, args):
            written.append([_valu_writes(op, args), 0])
        if not track_new and not written and all(p[1] >= p[2] for p in pending):
            return


def _functions(asm_text):
    """(name, numbered lines, label -> index) of every function of a listing."""
    funcs, cur = [], None
    for raw in asm_text.split("\n"):
        m = re.match(r"^(_Z\w+):", raw)
        if m:
            cur = (m.group(1), [], {})
            funcs.append(cur)
            continue
        if cur is None:
            continue
        name, lines, labels = cur
        lab = re.match(r"^(\.\w+):", raw)
        if lab:
            labels[lab.group(1)] = len(lines)
        lines.append((len(lines) + 1, raw))
    return funcs


def check(asm_text, need=12, need_16_pass=20, horizon=64):
    """Returns a list of (function, line number within the function, instruction, wait states so far)."""
    problems = []
    for name, lines, labels in _functions(asm_text):
        _walk(lines, labels, name, 0, [], [], True, need, need_16_pass, horizon, problems, 0)
    return sorted(set(problems), key=problems.index)


SGPR_LOAD_STATES = 5  # between a vector instruction's write of a scalar register and a memory instruction that reads it
_SGPR = re.compile(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _sgprs(text):
    out = set()
    for m in _SGPR.finditer(text):
        out.update(range(int(m.group(1)), int(m.group(2)) + 1) if m.group(1) else [int(m.group(3))])
    return out


def _walk_loads(lines, labels, func, start, written, track_new, problems, depth):
    """As _walk, for scalar registers written by vector instructions: `written` holds [registers, wait states so far]."""
    in_asm = False
    for idx in range(start, len(lines)):
        ln, raw = lines[idx]
        stripped = raw.strip()
        if stripped.startswith((";;#ASMSTART", ";;#ASMEND")):
            in_asm = stripped.startswith(";;#ASMSTART")
            continue
        parsed = _parse(raw)
        if parsed is None:
            continue
        text, op, args, states = parsed
        if in_asm and op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            read = _sgprs(args)
            problems.extend((func, ln, text, waited) for regs, waited in written if regs & read)
        written = [[regs, waited + states] for regs, waited in written if waited + states < SGPR_LOAD_STATES]
        if op.startswith("v_") and track_new:
            operands = args.split(",")
            regs = _sgprs(",".join(operands[:2 if "_co_" in op or "div_scale" in op else 1]))
            if regs:
                written.append([regs, 0])
        if op.startswith("s_cbranch") or op == "s_branch":
            target = labels.get(args.strip())
            if written and target is not None and depth < 4:
                _walk_loads(lines, labels, func, target, written, False, problems, depth + 1)
            if op == "s_branch":
                written = []  # what follows is reached by other branches only
        if not track_new and not written:
            return


def check_loads(asm_text):
    """Hand-written memory instructions that read a scalar register too soon after a vector instruction wrote it, as check()
    reports."""
    problems = []
    for name, lines, labels in _functions(asm_text):
        _walk_loads(lines, labels, name, 0, [], True, problems, 0)
    return sorted(set(problems), key=problems.index)


def main(argv):
    bad = 0
    for path in argv[1:]:
        listing = open(path).read()
        for func, ln, text, waited in check(listing) + check_loads(listing):
            print(f"{path}: {func} +{ln}: `{text}` only {waited} wait states after the write of its registers")
            bad += 1
    return 1 if bad else 0


if __name__ == "__main__":
    sys.exit(main(sys.argv))
