"""Build-time check of the distance between an MFMA or a dot product and the first use of its result.

The matrix cores write the result of v_mfma_f32_32x32x16_* (eight passes) without an interlock: any
instruction but the next accumulation into the same registers has to stay twelve wait states behind.
The compiler keeps that distance on straight paths.  Behind a branch its count has come out short (three
or four states) for scores that live in accumulation registers, that a scheduling directive moved, or
that a conditional block reads first thing; single scores were then stale.  This script walks every path
behind every MFMA of the device assembly, counts one state per instruction (s_nop: its operand + 1), and
fails the build where an instruction touches the result too early.

A dot product (v_dot2c) likewise delivers its result without an interlock: another kind of instruction has to stay
three wait states behind.  The kernels issue theirs inside inline assembly, of which the compiler keeps no distance,
and it moves what reads the result up to the last of them unless the wait there names the register.
"""
import re
import sys

MFMA = re.compile(r"v_mfma_f32_32x32x16_(bf16|f16)\b")
STATES = 12
DOT = re.compile(r"v_dot2c?_")
DOT_STATES = 3


def _registers(operand):
    out = set()
    for m in re.finditer(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", operand):
        lo, hi = (m.group(2),) * 2 if m.group(2) else (m.group(3), m.group(4))
        out.update((m.group(1), i) for i in range(int(lo), int(hi) + 1))
    return frozenset(out)


def _functions(text):
    """name -> list of (line number, opcode, operand texts); a label is (line number, None, [name])."""
    out, body = {}, None
    for ln, line in enumerate(text.splitlines(), 1):
        t = line.strip()
        if t.startswith(".type") and "@function" in t:
            body = out.setdefault(t.split()[1].split(",")[0], [])
        elif t.startswith(".Lfunc_end"):
            body = None
        elif body is not None:
            label = re.match(r"(\.L\w+):", t)
            code = t.split(";")[0].strip()
            if label:
                body.append((ln, None, [label.group(1)]))
            elif code and code[0] not in ".;" and not code.endswith(":"):
                op, _, rest = code.partition(" ")
                body.append((ln, op, [x.strip() for x in rest.split(",")] if rest else []))
    return out


def _early_use(body, used, labels, start, result, states):
    """Index of an instruction that touches `result` fewer than `states` wait states behind `start`, or None."""
    def used_as_operand(args):
        accumulator = _registers(args[3]) & result
        return (_registers(args[1]) | _registers(args[2])) & result or (accumulator and accumulator != result)

    dot = DOT.match(body[start][1])
    paths, seen = [(start + 1, 0)], set()
    while paths:
        j, waited = paths.pop()
        while j < len(body) and waited < states and (j, waited) not in seen:
            seen.add((j, waited))
            _, op, args = body[j]
            if op is None:
                j += 1
                continue
            if op == "s_endpgm":
                break
            if op == "s_nop":
                waited += int(args[0], 0)  # and one more below
            elif op.startswith("s_branch") or op.startswith("s_cbranch"):
                paths.append((labels[args[0]], waited + 1))
                if op.startswith("s_branch"):
                    break
            elif used[j] & result and dot:
                if op == body[start][1] and _registers(args[0]) == result and not _registers(" ".join(args[1:3])) & result:
                    break  # the sum goes on: checked by itself
                return j
            elif used[j] & result:
                if op.startswith("v_mfma") and _registers(args[0]) == result and not used_as_operand(args):
                    break  # the same registers again, in the matrix cores' own order: checked by itself
                return j
            waited += 1
            j += 1
    return None


def check(text):
    problems = []
    for name, body in _functions(text).items():
        labels = {args[0]: i for i, (_, op, args) in enumerate(body) if op is None}
        used = [frozenset() if op is None else _registers(" ".join(args)) for _, op, args in body]
        for i, (ln, op, args) in enumerate(body):
            if op is None or not (op.startswith("v_mfma") or DOT.match(op)):
                continue
            if not (MFMA.match(op) or DOT.match(op)):
                problems.append(f"{name}: line {ln}: no wait states known for {op}")
                continue
            at = _early_use(body, used, labels, i, _registers(args[0]), DOT_STATES if DOT.match(op) else STATES)
            if at is not None:
                problems.append(f"{name}: line {ln}: {op} {args[0]} is used too early by line {body[at][0]}: "
                                f"{body[at][1]} {', '.join(body[at][2])}")
    return problems


if __name__ == "__main__":
    found = check(open(sys.argv[1]).read())
    print(f"{len(found)} problem(s)")
    for f in found[:20]:
        print(f)
    sys.exit(1 if found else 0)
