"""The compiled code of the attention with 64 rows a wavefront: its products, exponentials, sums and packs are
assembly text, which the compiler does not space out by itself.  Between a vector write of a matrix product's operand
and the product lie two instructions (or as much s_nop), between a product of eight passes and a use of its result
outside the matrix pipe eleven, and between an exponential and a use of its result one."""
import os
import re
import subprocess

import pytest

from paper_2502_14317_amd.build import CSRC, HIPCC_FLAGS, INCLUDE

KERNELS = ["flash_wide_kernelILi0E", "flash_wide_kernelILi1E", "flash_wide_kernelILi2E", "flash_both_wide_kernelILi0E",
           "flash_both_wide_kernelILi1E"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "prefill_attn.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *HIPCC_FLAGS, "-I", INCLUDE, "-I", CSRC, "--cuda-device-only", "-S",
                    os.path.join(CSRC, "prefill_attn.hip"), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    return out.read_text()


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
            found += [("result", texts[i], texts[k]) for k in following(texts, ins, label, i, 11)
                      if ins[k][0].startswith(("v_", "ds_", "buffer_", "global_")) and not ins[k][0].startswith("v_mfma")
                      and any(x & ops[0] for x in ins[k][1])]
        elif op.startswith("v_") and not op.startswith("v_cmp"):
            found += [("operand", texts[i], texts[k]) for k in following(texts, ins, label, i, 2)
                      if ins[k][0].startswith("v_mfma") and any(x & ops[0] for x in ins[k][1][1:])]
        if op.startswith("v_exp"):
            found += [("exponential", texts[i], texts[k]) for k in following(texts, ins, label, i, 1)
                      if ins[k][0].startswith("v_") and any(x & ops[0] for x in ins[k][1][1:])]
    return found, sum(op.startswith("v_mfma") for op, _ in ins), texts


@pytest.mark.parametrize("kernel", KERNELS)
def test_spacing_of_the_assembly_text(assembly, kernel):
    found, n_mfma, texts = hazards(assembly, kernel)
    assert n_mfma >= 150                                     # the loops are there
    assert not found, found[:5]
    # and nothing lives in scratch memory
    assert not any(t.startswith("scratch_") for t in texts)


def test_the_check_sees_a_product_too_close():
    text = "\n".join(["_Z1flash_x:", "v_accvgpr_mov_b32 a0, a64", "s_nop 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]",
                      "s_branch .LBB0_2", ".LBB0_1:", "v_exp_f32 v1, v2", "v_add_f32 v3, v3, v1", "s_endpgm",
                      ".LBB0_2:", "s_nop 8", "v_accvgpr_read_b32 v9, a3", "s_branch .LBB0_1", ".Lfunc_end0:"])
    found, _, _ = hazards(text, "flash_x")
    assert sorted(x[0] for x in found) == ["exponential", "operand", "result"]
