"""The distances between instructions in the compiled code of the attention with 64 rows a wavefront, whose products,
exponentials, sums and packs are assembly text (spacing.py says which; the build refuses code that breaks one)."""
import os
import subprocess

import pytest

from paper_2502_14317_amd.build import CSRC, HIPCC_FLAGS, INCLUDE
from paper_2502_14317_amd.spacing import KERNELS, check, hazards

@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "prefill_attn.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *HIPCC_FLAGS, "-I", INCLUDE, "-I", CSRC, "--cuda-device-only", "-S",
                    os.path.join(CSRC, "prefill_attn.hip"), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    return out.read_text()


@pytest.mark.parametrize("kernel", KERNELS)
def test_spacing_of_the_assembly_text(assembly, kernel):
    found, n_mfma, texts = hazards(assembly, kernel)
    assert n_mfma >= 150                                     # the loops are there
    assert not found, found[:5]
    # and nothing lives in scratch memory
    assert not any(t.startswith("scratch_") for t in texts)


def kinds(lines):
    found, _, _ = hazards("\n".join(["_Z1flash_x:", *lines, "s_endpgm", ".Lfunc_end0:"]), "flash_x")
    return sorted({x[0] for x in found})


PRODUCT = "v_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], v[24:27], v[40:55]"


def test_the_build_refuses_it(assembly):
    check(assembly)
    kernel = KERNELS[1]
    at = assembly.index("v_mfma", assembly.index(f"{kernel}", assembly.index("flash_wide_kernel")))
    end = assembly.index("\n", at)
    result = assembly[at:end].split(None, 1)[1].split(",")[0]
    first = result[0] + result[2:].split(":")[0]
    planted = f"\n\tv_accvgpr_read_b32 v0, {first}" if first[0] == "a" else f"\n\tv_mov_b32_e32 v0, {first}"
    with pytest.raises(RuntimeError):
        check(assembly[:end] + planted + assembly[end:])


def test_the_check_sees_a_product_too_close():
    assert kinds(["v_accvgpr_mov_b32 a0, a64", "s_nop 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]",
                  "s_branch .LBB0_2", ".LBB0_1:", "v_exp_f32 v1, v2", "v_add_f32 v3, v3, v1", "s_endpgm",
                  ".LBB0_2:", "s_nop 8", "v_accvgpr_read_b32 v9, a3", "s_branch .LBB0_1"]) == ["exponential", "operand", "result"]


@pytest.mark.parametrize("kind,line,states", [
    ("result", "v_add_f32 v60, v61, v3", 12),
    ("result", "v_mov_b32 v3, v61", 12),
    ("product", "v_mfma_f32_32x32x16_bf16 v[64:79], v[0:3], v[24:27], v[40:55]", 12),
    ("product", "v_mfma_f32_32x32x16_bf16 v[64:79], v[24:27], v[12:15], v[40:55]", 12),
    ("product", "v_mfma_f32_32x32x16_bf16 v[64:79], v[20:23], v[24:27], v[4:19]", 12),
    ("addend", "v_mov_b32 v55, v61", 7),
])
def test_the_check_counts_to_the_state(kind, line, states):
    assert kinds([PRODUCT, f"s_nop {states - 2}", line]) == [kind]           # one state short
    assert kinds([PRODUCT, f"s_nop {states - 1}", line]) == []
    assert kinds([PRODUCT, "v_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], v[24:27], v[0:15]"]) == []     # in place: no wait
