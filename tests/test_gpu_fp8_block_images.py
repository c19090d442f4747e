"""A block of query rows over the 8-bit cache: the tile images that the attention reads, at the edges of the
64-key tiles and 32-key blocks, with rows behind the lengths that hold NaN."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import f32_to_bf16_bits, bf16_bits_to_f64
from helpers import (O_ATOL, O_RTOL, LSE_ATOL, bits_to_dev, dev_bf16_to_f64, assert_close, fp8_rows_view, fp8_from_rows)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n_q,S,kt,Hq,Hkv,D,tail_cap,with_self,per_head", [
    (1, 17, 1, 1, 2, 2, 64, 0, True, False),
    (2, 33, 3, 31, 4, 4, 128, 1, True, True),
    (1, 64, 2, 33, 8, 2, 128, 63, False, True),
    (1, 65, 3, 64, 8, 2, 64, 64, True, False),
    (2, 129, 2, 97, 6, 2, 128, 65, True, True),
    (1, 40, 4, 130, 8, 8, 64, 0, False, True),
    (1, 200, 0, 64, 4, 1, 128, 127, True, False),
    (1, 300, 5, 352, 4, 2, 128, 0, True, True),
])
def test_block_over_fp8_cache_at_tile_edges(B, n_q, S, kt, Hq, Hkv, D, tail_cap, with_self, per_head):
    print(f"fp8 images: B={B} n_q={n_q} S={S} kt={kt} H={Hq}/{Hkv} D={D} tail={tail_cap} self={with_self}", flush=True)
    r = np.random.default_rng([81, n_q, kt])
    mk = lambda shape, s=1.0: f32_to_bf16_bits((r.standard_normal(shape) * s).astype(np.float32))
    nan16 = np.uint16(0x7fc0)
    q = mk((B, n_q, Hq, D))
    # |value| < 4, both signs
    codes = {w: (r.integers(0, 0x48, size=(B, S, Hkv, kt, D)) + 0x80 * r.integers(0, 2, size=(B, S, Hkv, kt, D))).astype(np.uint8) for w in "kv"}
    scale = {w: r.uniform(0.2, 0.9, size=(B, S, Hkv)).astype(np.float32) for w in "kv"}
    sl = np.minimum(kt, r.integers(0, kt + 33, size=(B, S, Hkv) if per_head else (B, S))).astype(np.int32)
    if S:
        sl.reshape(-1)[0] = kt
    sl_h = sl if per_head else np.repeat(sl[..., None], Hkv, axis=2)
    dead = np.arange(kt)[None, None, None, :] >= sl_h[..., None]
    dev = {}
    for w in "kv":
        poisoned = codes[w].copy()
        poisoned[dead] = 0x7f                                              # NaN
        dev[w] = fp8_from_rows(w, torch.from_numpy(poisoned)).cuda()
    tail = tl = None
    if tail_cap:
        tail = {w: mk((B, Hkv, tail_cap, D)) for w in "kv"}
        tl = r.integers(1, tail_cap + 1, size=(B,)).astype(np.int32)
        tl[0] = tail_cap if B == 1 else max(1, tail_cap - 1)
        for w in "kv":
            for b in range(B):
                tail[w][b, :, tl[b]:] = nan16
    self_rows = {w: mk((B, n_q, Hkv, D)) for w in "kv"} if with_self else None
    out = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, n_q, S, kt, tail_cap, Hq, Hkv, D, with_self))
    ws.view(torch.uint8).fill_(0xff)                                       # NaN wherever nothing was written
    pc.pc_parallel_attn_fp8(bits_to_dev(q), dev["k"], dev["v"], torch.from_numpy(scale["k"]).cuda(),
                            torch.from_numpy(scale["v"]).cuda(), torch.from_numpy(sl).cuda() if S else None,
                            bits_to_dev(tail["k"]) if tail_cap else None, bits_to_dev(tail["v"]) if tail_cap else None,
                            torch.from_numpy(tl).cuda() if tail_cap else None, tail_cap, B, n_q, S, kt, Hq, Hkv, D,
                            50, 1.0e4, 0.0, out, lse, ws, seg_len_per_head=int(per_head),
                            k_self=bits_to_dev(self_rows["k"]) if with_self else None,
                            v_self=bits_to_dev(self_rows["v"]) if with_self else None)
    torch.cuda.synchronize()
    pad = max(kt, tail_cap)
    for b in range(B):
        n = S + (1 if tail_cap else 0)
        kd, vd = np.zeros((n, Hkv, pad, D)), np.zeros((n, Hkv, pad, D))
        lens = np.zeros((n, Hkv), dtype=np.int64)
        lens[:S] = sl_h[b]
        for x, w in ((kd, "k"), (vd, "v")):
            if S:
                x[:S, :, :kt] = oracle.dequantize_kv_fp8(codes[w][b], scale[w][b])
            if tail_cap:
                x[S, :, :tl[b]] = bf16_bits_to_f64(tail[w][b, :, :tl[b]])
        if tail_cap:
            lens[S] = tl[b]
        qf = oracle.rope(bf16_bits_to_f64(q[b]), 50 + np.arange(n_q), 1.0e4)
        one = lambda w: bf16_bits_to_f64(self_rows[w][b]) if with_self else None
        ro, rl = oracle.global_attention_concat(qf, kd, vd, seg_len=lens, k_self=one("k"), v_self=one("v"))
        assert_close(dev_bf16_to_f64(out[b]), ro, O_ATOL, O_RTOL, f"out[b={b}]")
        assert_close(lse[b].cpu().numpy().T, rl, LSE_ATOL, 1e-3, f"lse[b={b}]")
