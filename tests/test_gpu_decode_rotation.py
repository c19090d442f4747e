"""The split-KV kernels rotate the query rows themselves: every shape of their column tile (query rows x
heads of a group, 1 to 16), the 16-bit and the 8-bit cache with its tail in one launch, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu

# B, n_q, H_q, H_kv, D, S, k_t, tail capacity (8-bit cache), q_pos0
CASES = [
    (1, 1, 1, 1, 64, 1, 33, 1, 0),            # one column; position 0
    (2, 1, 16, 1, 128, 2, 64, 40, 70000),     # sixteen heads of one group, a far position
    (1, 5, 6, 2, 64, 3, 50, 0, 9),            # 15 columns of three heads x five rows; no tail
    (1, 16, 2, 2, 128, 1, 100, 65, 123),      # sixteen rows of one head
    (3, 2, 12, 3, 64, 0, 32, 70, 1000),       # no segments: the tail alone
]


# (a 16-bit call without segments has no keys)
@pytest.mark.parametrize("case,eight_bit", [(c, e) for c in CASES for e in (False, True) if e or c[5] > 0],
                         ids=lambda x: "x".join(str(y) for y in x) if isinstance(x, tuple) else ("8bit" if x else "16bit"))
def test_few_rows_rotated_in_the_kernel(case, eight_bit):
    B, n_q, Hq, Hkv, D, S, kt, cap, pos0 = case
    print("decode rotation", case, eight_bit, flush=True)
    r = np.random.default_rng([63, B, n_q, Hq, D, S])
    mk = lambda *shape: f32_to_bf16_bits(r.standard_normal(shape).astype(np.float32))
    q, kc, vc = mk(B, n_q, Hq, D), mk(B, S, Hkv, kt, D), mk(B, S, Hkv, kt, D)
    kt8, vt8 = mk(B, 1, Hkv, max(cap, 1), D), mk(B, 1, Hkv, max(cap, 1), D)
    tail_len = r.integers(1, cap + 1, size=B).astype(np.int32) if cap else None
    out = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    if eight_bit:
        k8, v8 = fp8_alloc(B, max(S, 1), Hkv, kt, D), fp8_alloc(B, max(S, 1), Hkv, kt, D)
        ks = torch.ones((B, max(S, 1), Hkv), dtype=torch.float32, device="cuda")
        vs = torch.ones_like(ks)
        if S:
            pc.pc_kv_quantize_fp8(bits_to_dev(kc), bits_to_dev(vc), None, B, S, kt, Hkv, D, k8, v8, ks, vs)
        ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, n_q, S, kt, cap, Hq, Hkv, D))
        pc.pc_parallel_attn_fp8(bits_to_dev(q), k8, v8, ks, vs, None, bits_to_dev(kt8) if cap else None,
                                bits_to_dev(vt8) if cap else None,
                                torch.from_numpy(tail_len).cuda() if cap else None, cap, B, n_q, S, kt, Hq, Hkv, D,
                                pos0, 1.0e4, 0.0, out, lse, ws)
    else:
        ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, n_q, S, kt, Hq, Hkv, D, False))
        pc.pc_parallel_attn(bits_to_dev(q), bits_to_dev(kc), bits_to_dev(vc), None, None, None, B, n_q, S, kt,
                            Hq, Hkv, D, pos0, 1.0e4, 0.0, out, lse, ws)
    torch.cuda.synchronize()
    for b in range(B):
        K, V, n = bf16_bits_to_f64(kc[b]), bf16_bits_to_f64(vc[b]), np.full(S, kt)
        if eight_bit:
            if S:
                rk8, rks, rv8, rvs = oracle.quantize_kv_fp8(K, V, None)
                K, V = oracle.dequantize_kv_fp8(rk8, rks), oracle.dequantize_kv_fp8(rv8, rvs)
            if cap:
                pad = max(kt, cap)
                K2, V2 = np.zeros((S + 1, Hkv, pad, D)), np.zeros((S + 1, Hkv, pad, D))
                K2[:S, :, :kt], V2[:S, :, :kt] = K, V
                K2[S, :, :cap], V2[S, :, :cap] = bf16_bits_to_f64(kt8[b, 0]), bf16_bits_to_f64(vt8[b, 0])
                K, V, n = K2, V2, np.append(n, tail_len[b])
        qf = oracle.rope(bf16_bits_to_f64(q[b]), pos0 + np.arange(n_q), 1.0e4)
        ro, rl = oracle.global_attention_concat(qf, K, V, seg_len=n.astype(np.int64))
        assert_close(dev_bf16_to_f64(out[b]), ro, O_ATOL, O_RTOL, f"out[b={b}]")
        assert_close(lse[b].cpu().numpy().T, rl, LSE_ATOL, 1e-3, f"lse[b={b}]")
