"""Checks the compiled code of the attention with 64 rows a wavefront: its products, exponentials, sums and packs are
assembly text, which the compiler does not space out by itself.  Between a vector write of a matrix product's operand
and the product lie two issue states (instructions, or as much s_nop), between an exponential and a use of its result one.
Behind a product of eight passes twelve before its result is used outside the matrix pipe, as the factor of another product or
as part of an addend that is not just the result, and seven before its addend is written over: the distances that the
compiler keeps for gfx950 where it sees the product (s_nop 11 and s_nop 6)."""
import re

KERNELS = ["flash_wide_kernelILi0E", "flash_wide_kernelILi1E", "flash_wide_kernelILi2E", "flash_both_wide_kernelILi0E",
           "flash_both_wide_kernelILi1E"]


def registers(operand):
    operand = operand.strip().lstrip("-|").rstrip("|")
    m = re.match(r"([av])\[(\d+):(\d+)\]", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([av])(\d+)\b", operand)
    return {(m[1], int(m[2]))} if m else set()


def parse(text, kernel):
    """Instructions of a kernel: their text, (opcode, register sets of the operands), and where every label stands."""
    body = re.search(r"^_Z\d+" + kernel + r"[^\n:]*:.*?\.Lfunc_end", text, re.S | re.M)[0]
    texts, ins, label = [], [], {}
    for line in body.split("\n")[1:]:
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            label[line[:-1]] = len(ins)
        elif line and not line.startswith((".", "#")):
            op, *rest = line.split(None, 1)
            texts.append(line)
            ins.append((op, [registers(x) for x in rest[0].split(",")] if rest else []))
    return texts, ins, label


def following(texts, ins, label, i, budget):
    """Instructions that may run within `budget` issue states behind instruction i, along every path."""
    todo, seen, out = [(i + 1, 0)], {}, []
    while todo:
        k, passed = todo.pop()
        while k < len(ins) and passed < budget and seen.get(k, budget) > passed:
            seen[k] = passed
            out.append(k)
            op = ins[k][0]
            passed += int(texts[k].split()[1], 0) + 1 if op == "s_nop" else 1
            if op.startswith("s_cbranch"):
                todo.append((label[texts[k].split()[1]], passed))
            k = label[texts[k].split()[1]] if op == "s_branch" else len(ins) if op == "s_endpgm" else k + 1
    return out


def hazards(text, kernel):
    texts, ins, label = parse(text, kernel)
    found = []
    for i, (op, ops) in enumerate(ins):
        if op.startswith("v_mfma"):
            for k in following(texts, ins, label, i, 12):
                if ins[k][0].startswith("v_mfma"):
                    _, a, b, c = ins[k][1][:4]
                    if (a | b) & ops[0] or (c & ops[0] and c != ops[0]):
                        found.append(("product", texts[i], texts[k]))
                elif ins[k][0].startswith(("v_", "ds_", "buffer_", "global_")) and any(x & ops[0] for x in ins[k][1]):
                    found.append(("result", texts[i], texts[k]))
            found += [("addend", texts[i], texts[k]) for k in following(texts, ins, label, i, 7)
                      if ins[k][0].startswith("v_") and not ins[k][0].startswith(("v_mfma", "v_cmp")) and ins[k][1][0] & ops[3]]
        elif op.startswith("v_") and not op.startswith("v_cmp"):
            found += [("operand", texts[i], texts[k]) for k in following(texts, ins, label, i, 2)
                      if ins[k][0].startswith("v_mfma") and any(x & ops[0] for x in ins[k][1][1:])]
        if op.startswith("v_exp"):
            found += [("exponential", texts[i], texts[k]) for k in following(texts, ins, label, i, 1)
                      if ins[k][0].startswith("v_") and any(x & ops[0] for x in ins[k][1][1:])]
    return found, sum(op.startswith("v_mfma") for op, _ in ins), texts


def check(text):
    """Raises where a kernel of KERNELS breaks a distance or lives in scratch memory."""
    for kernel in KERNELS:
        found, _, texts = hazards(text, kernel)
        if found or any(t.startswith("scratch_") for t in texts):
            raise RuntimeError(f"{kernel}: instructions too close, or scratch memory: {found[:5]}")
