"""Local attention with 64 query rows a wavefront (long sequences of head_dim 128, many of them): heads packed 8, 4, 2
or 1 to a workgroup, groups beyond a multiple of 8 (dealt to all XCDs), Q tiles and key tiles cut off by
a sequence's end, sequences far shorter than the call's, and references that move inside a sequence."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu


def prefill(C, w, wq, Hq, Hkv, q, k, v, base, lens=None):
    L = w + wq
    shape = pc.make_shape(C, w, wq, Hq, Hkv, 128, 1, base)
    o = torch.full((C, L, Hq, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((C, Hq, L), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_prefill_workspace_bytes(shape))
    ws.fill_(0xFF)                                          # NaN patterns: nothing may be read before it is written
    dev = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    pc.pc_chunk_prefill_attn(shape, bits_to_dev(q), bits_to_dev(k), bits_to_dev(v), o, lse, None, None, None, ws, chunk_lens=dev)
    torch.cuda.synchronize()
    return o, lse


# C, w, wq, H_q, H_kv, context rows (None: full)
CASES = [
    (8, 1250, 31, 8, 1, None),                              # 8 heads x 32 positions; 1281 rows: one row in the last Q tile
    (8, 1270, 74, 8, 1, [1270, 0, 1, 600, 1206, 1207, 64, 1238]),   # sequences that end at, before and behind tile edges
    (6, 1220, 61, 12, 3, None),                             # 4 heads x 64 positions; 18 groups: two dealt to all XCDs
    (12, 1283, 13, 8, 2, [1283, 2, 1200, 40, 900, 500, 51, 1139, 755, 1, 0, 321]),
    (5, 3030, 58, 12, 2, None),                             # groups of 6: 2 heads x 128 positions, three workgroups a Q tile
    (5, 3000, 108, 12, 2, [3000, 19, 20, 916, 2872]),
    (2, 7700, 57, 7, 7, None),                              # one head x 256 positions
    (2, 7700, 61, 9, 3, [7700, 3]),                         # groups of 3: one head too; a short sequence next to a long one
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(x) for x in c[:5]) + ("" if c[5] is None else "-short"))
def test_wide_attention_edges(case):
    C, w, wq, Hq, Hkv, lens = case
    print("wide attention", case, flush=True)
    L = w + wq
    r = np.random.default_rng([91, C, w, Hq, Hkv])
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((C, L, h, 128), dtype=np.float32))
    q, k, v = mk(Hq), mk(Hkv), mk(Hkv)
    if lens is not None:                                     # rows behind a sequence (64.0 throughout) must not count
        for c, n in enumerate(lens):
            q[c, n + wq:], k[c, n + wq:], v[c, n + wq:] = 0x4280, 0x4280, 0x4280
    o, lse = prefill(C, w, wq, Hq, Hkv, q, k, v, 1.0e4, lens)
    for c in range(C):
        n = (w if lens is None else lens[c]) + wq
        rows = np.unique(np.clip(np.concatenate([[0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 255, 256, n // 2, n - 65, n - 33, n - 32, n - 2, n - 1],
                                                 r.integers(0, n, size=6)]), 0, n - 1))
        pos = np.arange(n)
        kf = oracle.rope(bf16_bits_to_f64(k[c, :n]), pos, 1.0e4)
        vf = bf16_bits_to_f64(v[c, :n])
        qf = oracle.rope(bf16_bits_to_f64(q[c, rows]), rows, 1.0e4)
        for h in range(Hq):
            g = h // (Hq // Hkv)
            s = qf[:, h] @ kf[:, g].T / np.sqrt(128.0)
            s[pos[None, :] > rows[:, None]] = -np.inf
            m = s.max(axis=1, keepdims=True)
            p = np.exp(s - m)
            z = p.sum(axis=1, keepdims=True)
            assert_close(dev_bf16_to_f64(o[c, rows, h]), p @ vf[:, g] / z, O_ATOL, O_RTOL, f"o[{c}, :, {h}]")
            assert_close(lse[c, h, rows].cpu().numpy(), (m + np.log(z))[:, 0], LSE_ATOL, 1e-3, f"lse[{c}, {h}]")
        # every row of the sequence is written, none behind it
        assert torch.isfinite(o[c, :n].float()).all() and torch.isfinite(lse[c, :, :n]).all()
        assert torch.isnan(o[c, n:].float()).all() and torch.isnan(lse[c, :, n:]).all()


J = np.arange(1290)
LEVELS = {                                                  # a key's logit for a query of 1, log2 units
    "every step": 128.0 * (J // 32),
    "every tile's second half": 128.0 * ((J + 32) // 64),
    "two steps in turn": np.select([J < 160, J < 192, J < 544, J < 576], [0.0, 100.0, 200.0, 300.0], 400.0),
    # a lane's 16 keys add up to more than 2^90 above 86
    "just below and above the window": np.select([J < 40, J < 270, J < 611, J < 900], [0.0, 80.0, 86.0, 86.5], 180.0),
    "beyond the range of exp2": np.where(J < 77, 0.0, np.where(J < 700, 300.0, 900.0)),
    "one key": np.where(J == 95, 100.0, np.where(J == 800, 200.0, 0.0)),
    "last key": np.where(J == 1289, 200.0, 0.0),
}


@pytest.mark.parametrize("name", LEVELS)
def test_reference_moves_inside_a_long_sequence(name):
    """As in the attention with 32 rows: logits known exactly, since only the slowest pair of a head is used, which
    the rotation by 1290 * 1e30^(-1 + 2 / 128) < 1e-25 leaves as it is, and a query is one value times one key value.
    Bounds: the bf16 roundings of a probability and of the output (2^-9 each, of at most max |v| < 5.5), fp32 sums."""
    print("reference moves", name, flush=True)
    C, wq, Hq, Hkv, D = 8, 40, 8, 1, 128
    L = 1290
    r = np.random.default_rng([92, len(name)])
    q, k = np.zeros((C, L, Hq, D), np.float32), np.zeros((C, L, Hkv, D), np.float32)
    scale = 1.0 / np.sqrt(D)
    size = r.choice([1.0, 0.5, 0.25, -1.0], size=(C, L, Hq))
    q[..., D // 2 - 1] = size / (scale * np.log2(np.e))
    k[:, :, :, D // 2 - 1] = LEVELS[name][None, :, None]
    k[1::2] = 0.0                                           # every other sequence has nothing to move for
    qb, kb = f32_to_bf16_bits(q), f32_to_bf16_bits(k)
    vb = f32_to_bf16_bits(r.standard_normal((C, L, Hkv, D)).astype(np.float32))
    o, lse = prefill(C, L - wq, wq, Hq, Hkv, qb, kb, vb, 1.0e30)
    qs = bf16_bits_to_f64(f32_to_bf16_bits((bf16_bits_to_f64(qb)[..., D // 2 - 1] * (scale * np.log2(np.e))).astype(np.float32)))
    kf, v = bf16_bits_to_f64(kb)[..., D // 2 - 1], bf16_bits_to_f64(vb)
    for c, h in [(0, 0), (0, 1), (0, 6), (1, 3), (4, 2), (6, 7)]:
        s = np.where(J[None, :] <= J[:, None], qs[c, :, h, None] * kf[c, None, :, 0], -np.inf)
        m = s.max(axis=1, keepdims=True)
        p = np.exp2(s - m)
        z = p.sum(axis=1, keepdims=True)
        assert_close(dev_bf16_to_f64(o[c, :, h]), (p / z) @ v[c, :, 0], 5.5 * 2.0 ** -9, 2.0 ** -8, f"o[{c}, {h}]")
        assert_close(lse[c, h].cpu().numpy(), (m + np.log2(z))[:, 0] * np.log(2.0), 1e-4, 1e-6, f"lse[{c}, {h}]")
