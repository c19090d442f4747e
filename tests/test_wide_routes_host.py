"""Which calls the attention with 64 query rows a wavefront gets: every case of the GPU tests that are about it, and the
lines of the rule on either side."""
import ctypes

import pytest

import paper_2502_14317_amd as pc
import test_gpu_attention_error
import test_gpu_large_values
import test_gpu_layer_call
import test_gpu_wide_attn
import test_gpu_wide_images


def internal(name, types):
    f = getattr(pc.lib(), f"_Z{len(name)}{name}{types}")
    f.argtypes = [{"i": ctypes.c_int, "x": ctypes.c_longlong}[t] for t in types]
    return f


local = internal("pc_flash_wide", "iiiii")                  # heads of a workgroup, or 0
images = internal("pc_flash_wide_images", "iiiiixi")
parts = internal("pc_flash_parts", "iiiiix")
both_parts = internal("pc_flash_both_parts", "iiiiiixi")


def over_images(B, n_q, S, k_t, H_q, H_kv, tail=False, own=False):
    """(64 rows a wavefront?, parts) of a block of rows over segments of the 8-bit cache."""
    tiles = (S + tail) * -(-k_t // 64) + own * -(-n_q // 64)
    n = parts(B, n_q, H_q, H_kv, 128, tiles)
    return images(B, n_q, H_q, H_kv, 128, tiles, n), n


@pytest.mark.parametrize("case", test_gpu_wide_attn.CASES, ids=str)
def test_local_cases(case):
    C, w, wq, Hq, Hkv, _ = case
    assert local(C, w + wq, Hq, Hkv, 128) == {8: 8, 4: 4, 6: 2, 1: 1, 3: 1}[Hq // Hkv]


def test_other_local_cases():
    assert local(8, 1290, 8, 1, 128) == 8                   # references that move inside a long sequence
    assert local(12, 1350 + 203, 32, 8, 128) == 4           # edges of the window
    for C, w, wq, Hq, Hkv in test_gpu_large_values.CASES:
        assert (local(C, w + wq, Hq, Hkv, 128) > 0) == (w > 200)
    for C, w, wq, Hq, Hkv, D, share in test_gpu_attention_error.CASES:
        assert (local(C, w + wq, Hq, Hkv, D) > 0) == (share < 1.1)


def test_layer_cases():
    cut = []
    for C, w, wq, Hq, Hkv, D, _, kc, kt, _, _ in test_gpu_layer_call.WIDE:
        assert local(C, w + wq, Hq, Hkv, D) == {4: 4, 6: 2, 8: 8, 1: 1}[Hq // Hkv]
        tiles = kc * -(-kt // 64) + -(-wq // 64)
        cut.append(both_parts(C, w + wq, wq, Hq, Hkv, D, tiles, parts(1, wq, Hq, Hkv, D, tiles)) > 1)
    assert cut == [False, False, True, True]
    assert not any(local(c[0], c[1] + c[2], c[3], c[4], c[5]) for c in test_gpu_layer_call.CASES)


@pytest.mark.parametrize("case", test_gpu_wide_images.CASES, ids=str)
def test_image_cases(case):
    wide, n = over_images(*case[:8])
    assert wide and (n > 1) == (case[1] == 17)


def test_other_image_cases():
    B, n_q, S, kt, Hkv, _ = test_gpu_attention_error.IMAGES
    assert over_images(B, n_q, S, kt, 2 * Hkv, Hkv) == (1, 4) and over_images(B, n_q, S, kt, 8 * Hkv, Hkv) == (1, 1)
    cases = [(B, 128, S, 500, G * Hkv, Hkv, False, True) for B, G, S, Hkv in test_gpu_large_values.IMAGES]
    assert [over_images(*c) for c in cases] == [(1, 1), (1, 2), (1, 2)]


def test_lines_of_the_rules():
    assert not local(36, 4096, 32, 8, 64) and not local(1, 2500, 32, 8, 128) and local(1, 2561, 32, 8, 128)
    assert [local(36, n, 32, 8, 128) for n in (1279, 1280, 1281, 1344, 1345, 1408, 1409, 1983, 1984)] == [0, 0, 4, 4, 0, 0, 4, 4, 4]
    assert [local(36, n, 8, 1, 128) for n in (1280, 1281, 1376, 1377, 1408)] == [0, 8, 8, 0, 0]
    assert [local(36, n, 12, 6, 128) for n in (1300, 3071, 3072)] == [0, 0, 2]
    assert [local(36, n, 32, 32, 128) for n in (4096, 7679, 7680)] == [0, 0, 1]
    # blocks of 256 packed rows, 257 workgroups of 128, 64 tiles, 32 a part
    assert images(4, 512, 32, 8, 128, 64, 1) and not images(4, 512, 32, 8, 128, 63, 1)
    assert images(4, 512, 32, 8, 128, 64, 2) and not images(4, 512, 32, 8, 128, 63, 2) and not images(4, 512, 32, 8, 64, 64, 2)
    assert not images(4, 544, 32, 8, 128, 64, 2) and not images(1, 512, 32, 8, 128, 64, 2)
