"""The 16-bit tail of the 8-bit decoding call: in the 8-bit segments' launch with up to 4 columns or where
there are at most 256 of their workgroups, in a launch of its own otherwise.  Both ways against the oracle, on
either side of the line.

Inputs: logits of standard deviation 1.  The rounding of the rotated query to bf16 moves a logit by
2^-9 / sqrt(3) = 1.1e-3 rms and an output by that times sqrt(sum p^2), 2e-4 over the 60 or more keys
here, so half a million outputs stay far inside 2e-2.  (At a standard deviation of 3 a row's weight sits
on one or two keys, the output moves by 3.4e-3 rms, and 6 of those reach the tolerance.)"""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu


# batch, H_q, H_kv, D, query rows, tail capacity, launches; 64 keys: one workgroup a (sequence, KV head)
@pytest.mark.parametrize("B,Hq,Hkv,D,n_q,cap,launches", [
    (257, 4, 1, 64, 1, 40, 1),
    (256, 5, 1, 64, 1, 40, 1),
    (257, 5, 1, 64, 1, 40, 2),
    (129, 16, 2, 128, 1, 33, 2),
    (65, 12, 4, 128, 5, 64, 2),          # 15 columns
    (257, 16, 1, 64, 1, 0, 1),           # no tail
])
def test_tail_launch(B, Hq, Hkv, D, n_q, cap, launches):
    print("tail launch", B, Hq, Hkv, D, n_q, cap, flush=True)
    S, kt, pos0 = 1, 64, 5000
    r = np.random.default_rng([74, B, Hq, D])
    mk = lambda *shape: f32_to_bf16_bits(r.standard_normal(shape).astype(np.float32))
    q, kc, vc = mk(B, n_q, Hq, D), mk(B, S, Hkv, kt, D), mk(B, S, Hkv, kt, D)
    k_tail, v_tail = mk(B, 1, Hkv, max(cap, 1), D), mk(B, 1, Hkv, max(cap, 1), D)
    tail_len = r.integers(1, cap + 1, size=B).astype(np.int32) if cap else None
    k8, v8 = fp8_alloc(B, S, Hkv, kt, D), fp8_alloc(B, S, Hkv, kt, D)
    ks = torch.empty((B, S, Hkv), dtype=torch.float32, device="cuda")
    vs = torch.empty_like(ks)
    pc.pc_kv_quantize_fp8(bits_to_dev(kc), bits_to_dev(vc), None, B, S, kt, Hkv, D, k8, v8, ks, vs)
    out = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, n_q, S, kt, cap, Hq, Hkv, D))
    tail = (bits_to_dev(k_tail), bits_to_dev(v_tail), torch.from_numpy(tail_len).cuda()) if cap else (None, None, None)
    pc.pc_profile_begin()
    try:
        pc.pc_parallel_attn_fp8(bits_to_dev(q), k8, v8, ks, vs, None, *tail, cap, B, n_q, S, kt, Hq, Hkv, D, pos0,
                                1.0e4, 0.0, out, lse, ws)
        torch.cuda.synchronize()
    finally:
        pc.pc_profile_end()
    names = [name for name, _ in pc.pc_profile_records()]
    assert names.count("decode_attn_fp8_kernel") == 1
    assert names.count("decode_attn_kernel") == launches - 1
    for b in range(B):
        rk8, rks, rv8, rvs = oracle.quantize_kv_fp8(bf16_bits_to_f64(kc[b]), bf16_bits_to_f64(vc[b]), None)
        pad = max(kt, cap)
        K, V, n = np.zeros((S + 1, Hkv, pad, D)), np.zeros((S + 1, Hkv, pad, D)), np.array([kt, 0])
        K[:S, :, :kt], V[:S, :, :kt] = oracle.dequantize_kv_fp8(rk8, rks), oracle.dequantize_kv_fp8(rv8, rvs)
        if cap:
            K[S, :, :cap], V[S, :, :cap] = bf16_bits_to_f64(k_tail[b, 0]), bf16_bits_to_f64(v_tail[b, 0])
            n[S] = tail_len[b]
        qf = oracle.rope(bf16_bits_to_f64(q[b]), pos0 + np.arange(n_q), 1.0e4)
        ro, rl = oracle.global_attention_concat(qf, K, V, seg_len=n)
        assert_close(dev_bf16_to_f64(out[b]), ro, O_ATOL, O_RTOL, f"out[b={b}]")
        assert_close(lse[b].cpu().numpy().T, rl, LSE_ATOL, 1e-3, f"lse[b={b}]")
