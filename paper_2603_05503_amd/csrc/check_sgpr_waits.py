"""Build-time check of the distance between a scalar register written by a vector instruction and a memory
instruction that reads it.

A vector-memory instruction that takes its address or descriptor from scalar registers reads them without an
interlock: five wait states have to lie between it and a vector instruction (v_readfirstlane, v_readlane, a
comparison) that wrote them.  The compiler keeps that distance for its own instructions, not for those inside inline
assembly, where the kernels issue their tile loads and the stores and loads of cut rows.  This script walks every path
behind such a write in the device assembly, counts one state per instruction (s_nop: its operand + 1), and fails the
build where a memory instruction reads the register too early.
"""
import re
import sys

STATES = 5
VMEM = re.compile(r"(buffer|global|flat|scratch)_")


def _sgprs(text):
    out = set()
    for m in re.finditer(r"\bs(?:(\d+)\b|\[(\w+):(\w+)\])", text):
        lo, hi = (m.group(1),) * 2 if m.group(1) else (m.group(2), m.group(3))
        out.update(range(int(lo, 0), int(hi, 0) + 1))
    return out


def _functions(text):
    """name -> list of (line number, opcode, operands); a label is (line number, None, name)."""
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
                body.append((ln, None, label.group(1)))
            elif code and code[0] not in ".;" and not code.endswith(":"):
                op, _, rest = code.partition(" ")
                body.append((ln, op, rest.strip()))
    return out


def check(text):
    problems = []
    for name, body in _functions(text).items():
        labels = {rest: i for i, (_, op, rest) in enumerate(body) if op is None}
        for i, (ln, op, rest) in enumerate(body):
            if op is None or not op.startswith("v_"):
                continue
            written = _sgprs(rest.split(",")[0])
            if op.startswith(("v_add_co", "v_sub_co", "v_addc_co", "v_subb_co", "v_div_scale", "v_mad_u64", "v_mad_i64")):
                written |= _sgprs(",".join(rest.split(",")[:2]))
            if not written:
                continue
            paths, seen = [(i + 1, 0, frozenset(written))], set()
            while paths:
                j, waited, live = paths.pop()
                while j < len(body) and waited < STATES and live and (j, waited, live) not in seen:
                    seen.add((j, waited, live))
                    at, o, args = body[j]
                    if o is None:
                        j += 1
                        continue
                    if VMEM.match(o) and _sgprs(args) & live:
                        problems.append(f"{name}: line {ln}: {op} {rest} is read too early by line {at}: {o} {args}")
                        break
                    if o == "s_endpgm":
                        break
                    if o == "s_nop":
                        waited += int(args, 0)
                    elif o.startswith(("s_branch", "s_cbranch")):
                        paths.append((labels[args.split(",")[-1].strip()], waited + 1, live))
                        if o == "s_branch":
                            break
                    elif o.startswith("s_") and not o.startswith(("s_waitcnt", "s_barrier", "s_cmp", "s_bitcmp")):
                        live = live - _sgprs(args.split(",")[0])  # written again by the scalar unit: interlocked
                    waited += 1
                    j += 1
    return problems


if __name__ == "__main__":
    found = check(open(sys.argv[1]).read())
    print(f"{len(found)} problem(s)")
    for f in found[:20]:
        print(f)
    sys.exit(1 if found else 0)
