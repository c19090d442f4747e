"""Attention of many rows with values of 2^90: the sums of probabilities times values stay within fp32, also where logits rise
far above a row's first ones, in the kernels of 32 and of 64 query rows a wavefront (whose references stay up to 2^90 behind).

Logits are known exactly: only the slowest pair of a head is used, which the largest angle here, 7757 * 1e30^(-1 + 2 / 128) <
1e-25, leaves as it is.  Scaling values by a power of two changes no rounding, so the bounds are those of values of at most 6:
the bf16 roundings of a probability and of the output (2^-9 each) and fp32 sums."""
import numpy as np
import pytest
import torch

import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import assert_close, bits_to_dev, dev_bf16_to_f64, fp8_from_rows

pytestmark = pytest.mark.gpu

D = 128
BIG = 2.0 ** 90
SCALE_LOG2 = np.log2(np.e) / np.sqrt(D)
LEVELS = {                                                  # logits of the quarters of the keys, log2 units
    "flat": [0.0, 0.0, 0.0, 0.0],
    "behind": [0.0, 40.0, 80.0, 80.0],
    "moves, then behind": [0.0, 100.0, 104.0, 180.0],
    "behind, then moves": [0.0, 80.0, 180.0, 180.0],
}


def as_multiplied(q):                                       # scale * log2(e) in, rounded to bf16 once
    return bf16_bits_to_f64(f32_to_bf16_bits((q * SCALE_LOG2).astype(np.float32)))


def expected(s, v):
    m = s.max(axis=1, keepdims=True)
    p = np.exp2(s - m)
    z = p.sum(axis=1, keepdims=True)
    return (p / z) @ v, (m + np.log2(z))[:, 0] * np.log(2.0)


# C, w, wq, H_q, H_kv
CASES = [
    (2, 200, 57, 4, 2),                                     # 32 rows a wavefront
    (8, 1250, 31, 8, 1),                                    # 64: 8, 4 and one head a workgroup
    (6, 1220, 61, 12, 3),
    (2, 7700, 57, 7, 7),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("name", LEVELS)
def test_chunk_prefill(name, case):
    C, w, wq, Hq, Hkv = case
    print("large values", name, case, flush=True)
    L = w + wq
    r = np.random.default_rng([74, L, len(name)])
    q, k = np.zeros((C, L, Hq, D), np.float32), np.zeros((C, L, Hkv, D), np.float32)
    q[..., D // 2 - 1] = r.choice([1.0, 0.5, -1.0], size=(C, L, Hq)) / SCALE_LOG2
    j = np.arange(L)
    k[:, :, :, D // 2 - 1] = np.array(LEVELS[name])[4 * j // L][None, :, None]
    k[-1, :, 0] = 0.0                                       # one group whose references have nothing to move for
    qb, kb = f32_to_bf16_bits(q), f32_to_bf16_bits(k)
    v = bf16_bits_to_f64(f32_to_bf16_bits(np.clip(r.standard_normal((C, L, Hkv, D)), -6, 6).astype(np.float32)))
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, 1, 1.0e30)
    o = torch.full((C, L, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((C, Hq, L), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_prefill_workspace_bytes(shape))
    pc.pc_chunk_prefill_attn(shape, bits_to_dev(qb), bits_to_dev(kb), bits_to_dev(f32_to_bf16_bits((v * BIG).astype(np.float32))),
                             o, lse, None, None, None, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    qs, kf = as_multiplied(bf16_bits_to_f64(qb)[..., D // 2 - 1]), bf16_bits_to_f64(kb)[..., D // 2 - 1]
    rows = np.unique(np.concatenate([[0, 31, 32, 63, 64, L - 1], r.integers(0, L, size=250)]))
    for c, h in [(0, 0), (0, Hq - 1), (C - 1, 1), (C - 1, Hq - 1)]:
        g = h // (Hq // Hkv)
        s = np.where(j[None, :] <= rows[:, None], qs[c, rows, h, None] * kf[c, None, :, g], -np.inf)
        ref, ref_lse = expected(s, v[c, :, g])
        assert_close(dev_bf16_to_f64(o[c, rows, h]) / BIG, ref, 6 * 2.0 ** -9, 2.0 ** -8, f"o[{c}, {h}]")
        assert_close(lse[c, h, rows].cpu().numpy(), ref_lse, 1e-4, 1e-6, f"lse[{c}, {h}]")


IMAGES = [(4, 8, 9, 16), (2, 8, 33, 16), (4, 2, 33, 32)]    # B, G, S, H_kv: one part; two; groups of two


@pytest.mark.parametrize("B,G,S,Hkv", IMAGES)
@pytest.mark.parametrize("name", ["flat", "behind", "moves", "every step"])
def test_block_over_the_8_bit_cache(name, B, G, S, Hkv):
    """Tile images, 64 rows a wavefront: every segment rises from its first keys on, the next one's keys higher, segments of
    odd length among them; then the causal block itself, whose first keys' logits are 0."""
    n_q, kt = 128, 500
    Hq = G * Hkv
    print("large values over images", name, B, G, S, flush=True)
    r = np.random.default_rng([75, G, len(name)])
    gen = torch.Generator(device="cuda").manual_seed(G + len(name))
    level = np.array([0.0, 112.0, 224.0, 448.0] if name == "moves" else LEVELS.get(name, LEVELS["flat"]))
    lens = r.integers(300, kt + 1, size=(B, S))
    j = np.arange(kt)
    rise = 8.0 * (j // 32) if name == "every step" else level[4 * j // kt]      # exact in E4M3
    grow = 1.0 + np.arange(S) if name == "moves" else 12.0 + np.arange(S) if name == "every step" else np.ones(S)
    rise = bf16_bits_to_f64(f32_to_bf16_bits((grow[:, None] * rise[None]).astype(np.float32)))
    q = np.zeros((B, n_q, Hq, D), np.float32)
    q[..., D // 2 - 1] = r.choice([1.0, 0.5, 0.25], size=(B, n_q, Hq)) / SCALE_LOG2
    qb = f32_to_bf16_bits(q)
    k = torch.zeros((B, S, Hkv, kt, D), device="cuda")
    k[..., D // 2 - 1] = torch.tensor(rise[0] / grow[0], device="cuda", dtype=torch.float32)
    v = torch.randn((B, S, Hkv, kt, D), generator=gen, device="cuda").to(torch.float8_e4m3fn)
    dev = [fp8_from_rows("k", k.to(torch.float8_e4m3fn).view(torch.uint8)), fp8_from_rows("v", v.view(torch.uint8))]
    ones = torch.ones((B, S, Hkv), device="cuda")
    slf_k = torch.zeros((B, n_q, Hkv, D), dtype=torch.bfloat16, device="cuda")
    slf_k[..., D // 2 - 1] = torch.tensor(level[4 * np.arange(n_q) // n_q], device="cuda").to(torch.bfloat16)[None, :, None]
    slf_v = torch.randn((B, n_q, Hkv, D), generator=gen, device="cuda").to(torch.bfloat16)
    o = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, n_q, S, kt, 0, Hq, Hkv, D, True))
    k_scale = ones * torch.tensor(grow, device="cuda", dtype=torch.float32)[None, :, None]
    pc.pc_parallel_attn_fp8(bits_to_dev(qb), *dev, k_scale.contiguous(), ones * BIG, torch.tensor(lens, dtype=torch.int32, device="cuda"), None, None, None,
                            0, B, n_q, S, kt, Hq, Hkv, D, 0, 1.0e30, 0.0, o, lse, ws, k_self=slf_k, v_self=(slf_v.float() * BIG).to(torch.bfloat16))
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    qs, t = as_multiplied(bf16_bits_to_f64(qb)[..., D // 2 - 1]), np.arange(n_q)
    for b, h in [(0, 0), (0, Hq - 1), (B - 1, Hq // 2)]:
        g = h // G
        key = np.concatenate([rise[s, :n] for s, n in enumerate(lens[b])] + [level[4 * t // n_q]])
        val = np.concatenate([v[b, s, g, :n].float().cpu().numpy() for s, n in enumerate(lens[b])] + [slf_v[b, :, g].float().cpu().numpy()])
        s = qs[b, :, h, None] * key[None]
        s[:, -n_q:][t[None] > t[:, None]] = -np.inf
        ref, ref_lse = expected(s, val.astype(np.float64))
        assert_close(dev_bf16_to_f64(o[b, :, h]) / BIG, ref, 6 * 2.0 ** -9, 2.0 ** -8, f"o[{b}, {h}]")
        assert_close(lse[b, h].cpu().numpy(), ref_lse, 1e-4, 1e-6, f"lse[{b}, {h}]")
