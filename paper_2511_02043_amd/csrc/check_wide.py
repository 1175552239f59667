"""Checks the assembly of the dK/dV kernels with 64 keys per wave: python3 check_wide.py FILE.s

Their LDS reads and accumulating MFMAs are asm statements, so the compiler neither waits for the ones nor keeps wait states for the others: no
instruction may touch the destination of a read that has not landed, and none may write an operand of an MFMA within two wait states before
it.  Both follow from where the compiler puts its copies, so the build looks at what it made of them."""
import re
import sys


def registers(operand):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", operand)
    if m:
        return {(m[1], n) for n in range(int(m[2]), int(m[3]) + 1)}
    m = re.fullmatch(r"([va])(\d+)", operand)
    return {(m[1], int(m[2]))} if m else set()


def faults(text, states=2):
    """What breaks either rule.  Reads return in order: `queue` holds the destinations of those in flight, and of a branch's two
    ways the one with more of them counts where they meet."""
    found, queue, written, at, at_label, reached = [], [], {}, 0, {}, True
    for number, raw in enumerate(text.split("\n"), 1):
        line = raw.split(";")[0].strip()
        label = re.fullmatch(r"([\w.$]+):", line)
        if label:
            if not label[1].startswith("."):         # a function
                queue, written, reached, at_label = [], {}, True, {}
            other = at_label.get(label[1])
            if other is not None and (not reached or len(other) > len(queue)):
                queue = other
            at_label[label[1]] = None                # behind us: a branch to it goes back
            reached = True
            continue
        if not line or line.startswith("."):
            continue
        op, *rest = line.split(None, 1)
        operands = re.findall(r"[va]\[\d+:\d+\]|\b[va]\d+\b|[^,\s]+", rest[0]) if rest else []
        at += int(operands[0]) + 1 if op == "s_nop" else 1
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", line)
            if m:
                queue = queue[max(0, len(queue) - int(m[1])):]
            continue
        if op.startswith(("s_cbranch", "s_branch")):
            target = operands[0]
            if target in at_label and at_label[target] is None:
                if queue:
                    found.append((number, "reads in flight past the loop's end"))
            elif len(queue) >= len(at_label.get(target, [])):
                at_label[target] = list(queue)
            reached = op != "s_branch"
            continue
        used = set().union(*(registers(x) for x in operands))
        found += [(number, "in flight since line %d: %s" % (n, line)) for n, dst in queue if dst & used]
        if op.startswith("ds_read"):
            queue.append((number, registers(operands[0])))
        elif op.startswith(("ds_", "s_load")):
            queue.append((number, set()))
        if op.startswith("v_mfma"):
            for r in registers(operands[1]) | registers(operands[2]):
                if at - written.get(r, -99) - 1 < states:
                    found.append((number, "%s%d written just before: %s" % (*r, line)))
        elif op.startswith("v_") and operands:
            written.update({r: at for r in registers(operands[0])})
    return found


if __name__ == "__main__":
    text = open(sys.argv[1]).read()
    if "ds_read_b64_tr_b16" not in text or "v_mfma_f32_32x32x16_bf16" not in text:
        sys.exit(sys.argv[1] + ": no assembly of the kernels")
    wrong = faults(text)
    for number, what in wrong[:20]:
        print("%s:%d: %s" % (sys.argv[1], number, what))
    sys.exit(1 if wrong else 0)
