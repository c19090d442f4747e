"""Global attention of a block of query rows (the tile kernel over row-major segments): edges of the
64-key tiles, of the 128 packed (query, head) rows of a workgroup and of the runs the keys are cut
into, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu

# B, n_q, S, k_t, H_q, H_kv, D, lengths (None: full; else drawn, 0 among them), per head, self, q_pos0
CASES = [
    (1, 17, 1, 1, 1, 1, 64, None, 0, False, -1),           # one key, one workgroup of 17 rows
    (1, 32, 1, 63, 4, 1, 128, None, 0, True, 100),         # 128 packed rows exactly, a ragged tile
    (1, 33, 2, 64, 4, 1, 128, None, 0, True, 100),         # 132 rows: the second tile holds 4
    (2, 43, 3, 65, 6, 2, 64, "drawn", 0, True, 777),       # group of 3: 129 rows
    (1, 128, 2, 128, 2, 2, 128, None, 0, True, 5),         # one head a group, tiles full
    (1, 129, 0, 64, 2, 2, 64, None, 0, True, 0),           # self segment only
    (1, 300, 5, 200, 3, 3, 128, "drawn", 1, True, 9),      # per-head lengths, causal diagonal over 3 tiles
    (3, 40, 70, 31, 4, 2, 64, "drawn", 0, False, 31),      # more segments than lanes, all of them masked tiles
    (1, 64, 8, 700, 8, 2, 128, "drawn", 0, True, 8000),    # many parts for few rows
    (1, 64, 2, 96, 8, 2, 128, "zero", 0, False, 3),        # no key at all: zeros and -inf
    (1, 40, 2, 96, 4, 4, 64, "zero", 0, True, 3),          # nothing but the self segment
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(x) for x in c[:7]) + f"-{c[7]}-{int(c[8])}{int(c[9])}")
def test_tile_attention_edges(case):
    B, n_q, S, kt, Hq, Hkv, D, lens, per_head, with_self, q_pos0 = case
    print("tile attention", case, flush=True)
    r = np.random.default_rng([61, B, n_q, S, kt, Hq, D])
    mk = lambda *shape, gain=1.0: f32_to_bf16_bits((gain * r.standard_normal(shape)).astype(np.float32))
    # logits of standard deviation 1: the operands' bf16 rounding stays below half the tolerance
    q, kc, vc = mk(B, n_q, Hq, D), mk(B, max(S, 1), Hkv, kt, D), mk(B, max(S, 1), Hkv, kt, D)
    ks, vs = mk(B, n_q, Hkv, D), mk(B, n_q, Hkv, D)
    sl = None
    if lens is not None:
        shape = (B, S, Hkv) if per_head else (B, S)
        sl = r.integers(0, kt + 1, size=shape).astype(np.int32) if lens == "drawn" else np.zeros(shape, np.int32)
        if lens == "drawn":
            sl[0, 0], sl[0, -1] = kt, 0
    # rows behind a segment's length hold nothing: they must not reach the result
    kc_dev, vc_dev = bits_to_dev(kc), bits_to_dev(vc)
    if sl is not None:
        for b, s in np.ndindex(B, S):
            for g in range(Hkv):
                n = sl[b, s, g] if per_head else sl[b, s]
                kc_dev[b, s, g, n:] = float("nan")
                vc_dev[b, s, g, n:] = float("nan")
    out = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, n_q, S, kt, Hq, Hkv, D, with_self))
    ws.fill_(0xFF)                                          # NaN patterns: nothing may be read before it is written
    pc.pc_parallel_attn(bits_to_dev(q), kc_dev, vc_dev, None if sl is None else torch.from_numpy(sl).cuda(),
                        bits_to_dev(ks) if with_self else None, bits_to_dev(vs) if with_self else None, B, n_q, S, kt,
                        Hq, Hkv, D, q_pos0, 1.0e4, 0.0, out, lse, ws, seg_len_per_head=per_head)
    torch.cuda.synchronize()
    for b in range(B):
        qf = bf16_bits_to_f64(q[b])
        if q_pos0 >= 0:
            qf = oracle.rope(qf, q_pos0 + np.arange(n_q), 1.0e4)
        K, V = bf16_bits_to_f64(kc[b])[:S], bf16_bits_to_f64(vc[b])[:S]
        for g in range(Hkv):
            heads = slice(g * (Hq // Hkv), (g + 1) * (Hq // Hkv))
            n = np.full(S, kt) if sl is None else (sl[b, :, g] if per_head else sl[b])
            if not with_self and int(np.sum(n)) == 0:
                assert torch.all(out[b, :, heads] == 0) and torch.all(torch.isneginf(lse[b, heads]))
                continue
            ro, rl = oracle.global_attention_concat(
                qf[:, heads], K[:, g:g + 1], V[:, g:g + 1], seg_len=n.astype(np.int64),
                k_self=bf16_bits_to_f64(ks[b])[:, g:g + 1] if with_self else None,
                v_self=bf16_bits_to_f64(vs[b])[:, g:g + 1] if with_self else None)
            assert_close(dev_bf16_to_f64(out[b, :, heads]), ro, O_ATOL, O_RTOL, f"out[b={b}, g={g}]")
            assert_close(lse[b, heads].cpu().numpy().T, rl, LSE_ATOL, 1e-3, f"lse[b={b}, g={g}]")


# chunks, H_kv, H_q, D, w, w_q: (chunk, KV head) groups per XCD, batches of them and the rest
@pytest.mark.parametrize("C,Hkv,Hq,D,w,wq", [
    (57, 1, 16, 64, 150, 50),       # 7 groups per XCD in batches of 4 and 3, one group dealt to all
    (3, 3, 3, 128, 130, 40),        # one group per XCD, one dealt to all
    (2, 2, 8, 64, 300, 20),         # fewer groups than XCDs
    (24, 1, 1, 128, 129, 1),        # three groups of two Q tiles, one batch
])
def test_local_attention_group_order(C, Hkv, Hq, D, w, wq):
    print("group order", C, Hkv, Hq, D, w, wq, flush=True)
    r = np.random.default_rng([64, C, Hkv, Hq, D, w])
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((C, w + wq, h, D)).astype(np.float32))
    q, k, v = mk(Hq), mk(Hkv), mk(Hkv)
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, 1, 1.0e4)
    o = torch.full((C, w + wq, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((C, Hq, w + wq), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_prefill_workspace_bytes(shape))
    pc.pc_chunk_prefill_attn(shape, bits_to_dev(q), bits_to_dev(k), bits_to_dev(v), o, lse, None, None, None, ws)
    torch.cuda.synchronize()
    pos = np.arange(w + wq)
    for c in range(C):
        ro, rl = oracle.local_attention(oracle.rope(bf16_bits_to_f64(q[c]), pos, 1.0e4),
                                        oracle.rope(bf16_bits_to_f64(k[c]), pos, 1.0e4), bf16_bits_to_f64(v[c]))[:2]
        assert_close(dev_bf16_to_f64(o[c]), ro, O_ATOL, O_RTOL, f"o[c={c}]")
        assert_close(lse[c].cpu().numpy().T, rl, LSE_ATOL, 1e-3, f"lse[c={c}]")
