"""The 8-bit cache's codes at the edges of the quantisation's units (4 KiB of codes) and over the range of scales,
with zeros of both signs, infinities and NaN: bit for bit against the definition in float32 (quotient, clamp to
+-448 with NaN to the lowest, round to nearest even), with and without the maxima handed in."""
import numpy as np
import pytest
import torch

import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc
from workloads import bf16_bits_to_f64
from helpers import bits_to_dev, fp8_rows_view

pytestmark = pytest.mark.gpu


def _codes(x, amax):
    scale = np.where(amax > 0, amax / np.float32(448), np.float32(1)).astype(np.float32)      # NaN: 1
    y = (x / scale[..., None, None]).astype(np.float32)
    y = np.fmin(np.fmax(y, np.float32(-448)), np.float32(448))
    return scale, torch.from_numpy(y).to(torch.float8_e4m3fn).view(torch.uint8).numpy()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("k_t", [1, 31, 32, 33, 64, 65, 200])
def test_quantize_units_and_scales(k_t, D):
    print("quantize", k_t, D, flush=True)
    B, S, Hkv = 2, 8, 2
    r = np.random.default_rng([91, k_t, D])
    # per segment an exponent of the largest value: the reciprocal holds for scales within 2^+-60 only
    top = np.array([0, -133 + 12, -70, -52, -51, 68, 69, 127])
    bits = [None, None]
    for w in range(2):
        x = r.standard_normal((B, S, Hkv, k_t, D)) * np.exp2(top[None, :, None, None, None] - 3.0)
        x = torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16).copy()
        x[r.random(x.shape) < 0.02] = 0x8000                                  # -0
        x[r.random(x.shape) < 0.02] = 0x0001                                  # smallest subnormal
        x[0, 0, 0, -1, 5] = 0x7f80                                            # inf: the segment's scale is inf
        x[1, 0, 1, 0, 3] = 0xffc1                                             # NaN: its scale is 1
        bits[w] = x
    sl = np.maximum(k_t - r.integers(0, 3, size=(B, S)), 0).astype(np.int32)
    dead = np.arange(k_t)[None, None, None, :, None] >= sl[:, :, None, None, None]
    with np.errstate(all="ignore"):
        x32 = [bf16_bits_to_f64(b).astype(np.float32) for b in bits]
        live = [np.where(dead, np.uint16(0), b & 0x7fff).reshape(B, S, Hkv, -1).max(axis=-1) for b in bits]
        amax = [(m.astype(np.uint32) << 16).view(np.float32) for m in live]
        want = [_codes(x, m) for x, m in zip(x32, amax)]
        # a maximum below the largest value (the caller's): clamped, infinities too
        low = [np.where(np.isfinite(m), m * np.float32(0.37), np.float32(2)).astype(np.float32) for m in amax]
        want_low = [_codes(x, m) for x, m in zip(x32, low)]
    src, dsl = [bits_to_dev(b) for b in bits], torch.from_numpy(sl).cuda()
    for given, ref in ((None, want), (amax, want), (low, want_low)):
        k8, v8 = fp8_alloc(B, S, Hkv, k_t, D).fill_(0x55), fp8_alloc(B, S, Hkv, k_t, D).fill_(0x55)
        sc = [torch.empty((B, S, Hkv), dtype=torch.float32, device="cuda") for _ in range(2)]
        if given is None:
            pc.pc_kv_quantize_fp8(*src, dsl, B, S, k_t, Hkv, D, k8, v8, *sc)
        else:
            pc.pc_kv_quantize_fp8_amax(*src, *[torch.from_numpy(m).cuda() for m in given], dsl, B, S, k_t, Hkv, D, k8, v8, *sc)
        torch.cuda.synchronize()
        for w, c8, s, (scale, codes) in zip("kv", (k8, v8), sc, ref):
            np.testing.assert_array_equal(s.cpu().numpy(), scale)
            got = fp8_rows_view(w, c8, k_t, D, padded=True).cpu().numpy()
            np.testing.assert_array_equal(got[..., :k_t, :], np.where(dead, 0, codes))
            assert (got[..., k_t:, :] == 0).all()


@pytest.mark.parametrize("with_max", [False, True])
def test_quantize_above_the_last_level_cache(with_max):
    """More than 256 MiB of rows (loads with the non-temporal hint) against each sequence by itself."""
    B, S, Hkv, k_t, D = 3, 8, 8, 4096, 128
    print("quantize large", with_max, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    src = [torch.randn((B, S, Hkv, k_t, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2)]
    amax = [x.abs().amax(dim=(3, 4)).float() for x in src]

    def run(x, m):
        n = x[0].shape[0]
        c = [fp8_alloc(n, S, Hkv, k_t, D).fill_(0x55) for _ in range(2)]
        s = [torch.empty((n, S, Hkv), device="cuda") for _ in range(2)]
        if with_max:
            pc.pc_kv_quantize_fp8_amax(*x, *m, None, n, S, k_t, Hkv, D, *c, *s)
        else:
            pc.pc_kv_quantize_fp8(*x, None, n, S, k_t, Hkv, D, *c, *s)
        torch.cuda.synchronize()
        return c + s

    whole = run(src, amax)
    for b in range(B):
        one = run([x[b:b + 1].contiguous() for x in src], [m[b:b + 1].contiguous() for m in amax])
        for x, y in zip(whole, one):
            assert torch.equal(x[b:b + 1], y)
