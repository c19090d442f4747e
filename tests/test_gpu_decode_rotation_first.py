"""Few query rows: rotated by the split-KV kernel up to 512 workgroups, by a launch in front beyond; the
results on either side of the line against the oracle, which launches ran, and the same bits from both
ways for the sequences that two calls share."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eight_bit", [False, True], ids=["16bit", "8bit"])
@pytest.mark.parametrize("Hq,Hkv,D", [(4, 1, 64), (12, 2, 128)])
def test_rotation_first_beyond_512_workgroups(Hq, Hkv, D, eight_bit):
    S, kt, pos0 = 1, 64, 70001                           # 64 keys: one workgroup a (sequence, KV head)
    most = 512 // Hkv                                    # sequences of the largest call that rotates in the kernel
    r = np.random.default_rng([76, Hq, D])
    mk = lambda *shape: f32_to_bf16_bits(r.standard_normal(shape).astype(np.float32))
    q, kc, vc = mk(most + 1, 1, Hq, D), mk(most + 1, S, Hkv, kt, D), mk(most + 1, S, Hkv, kt, D)
    results = []
    for B, first in ((most, 0), (most + 1, 1)):
        print("rotation first", Hq, Hkv, D, eight_bit, B, flush=True)
        out = torch.full((B, 1, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((B, Hq, 1), float("nan"), dtype=torch.float32, device="cuda")
        dq, dk, dv = bits_to_dev(q[:B]), bits_to_dev(kc[:B]), bits_to_dev(vc[:B])
        if eight_bit:
            k8, v8 = fp8_alloc(B, S, Hkv, kt, D), fp8_alloc(B, S, Hkv, kt, D)
            ks = torch.empty((B, S, Hkv), dtype=torch.float32, device="cuda")
            vs = torch.empty_like(ks)
            pc.pc_kv_quantize_fp8(dk, dv, None, B, S, kt, Hkv, D, k8, v8, ks, vs)
            ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, 1, S, kt, 0, Hq, Hkv, D))
            call = lambda: pc.pc_parallel_attn_fp8(dq, k8, v8, ks, vs, None, None, None, None, 0, B, 1, S, kt, Hq, Hkv,
                                                   D, pos0, 5.0e5, 0.0, out, lse, ws)
        else:
            ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, 1, S, kt, Hq, Hkv, D, False))
            call = lambda: pc.pc_parallel_attn(dq, dk, dv, None, None, None, B, 1, S, kt, Hq, Hkv, D, pos0, 5.0e5, 0.0,
                                               out, lse, ws)
        ws.fill_(0xFF)
        pc.pc_profile_begin()
        try:
            call()
            torch.cuda.synchronize()
        finally:
            pc.pc_profile_end()
        assert [name for name, _ in pc.pc_profile_records()].count("rope_q_kernel") == first
        results.append((out, lse))
        for b in (0, most // 2, B - 1):
            K, V = bf16_bits_to_f64(kc[b]), bf16_bits_to_f64(vc[b])
            if eight_bit:
                rk8, rks, rv8, rvs = oracle.quantize_kv_fp8(K, V, None)
                K, V = oracle.dequantize_kv_fp8(rk8, rks), oracle.dequantize_kv_fp8(rv8, rvs)
            qf = oracle.rope(bf16_bits_to_f64(q[b]), pos0 + np.arange(1), 5.0e5)
            ro, rl = oracle.global_attention_concat(qf, K, V, seg_len=np.array([kt]))
            assert_close(dev_bf16_to_f64(out[b]), ro, O_ATOL, O_RTOL, f"out[b={b}]")
            assert_close(lse[b].cpu().numpy().T, rl, LSE_ATOL, 1e-3, f"lse[b={b}]")
    assert torch.equal(results[0][0], results[1][0][:most]) and torch.equal(results[0][1], results[1][1][:most])
