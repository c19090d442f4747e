"""The tile kernel's query operand, bit for bit: rotated at its position and multiplied by
scale * log2(e) in 64 bits, rounded to fp32 and then to bf16 (a row that arrives rotated is only
multiplied and rounded).  One key, 1 in one dimension and 0 elsewhere, makes the row's logsumexp
that dimension's operand times log 2, so the operand can be read back from it: the operand is a
bf16 value, the logsumexp is off by at most a few 2^-24 of it, and the nearest bf16 value to the
quotient is the operand itself."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import bits_to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n_q,q_pos0,eight_bit", [
    (128, 2048, 7680, False), (64, 3000, 0, False), (128, 300, 900000, True), (64, 129, -1, False)])
def test_query_operand_is_rounded_once_from_64_bits(D, n_q, q_pos0, eight_bit):
    print("query operand", D, n_q, q_pos0, eight_bit, flush=True)
    H, base = D, 5.0e5                       # head h reads dimension h
    r = np.random.default_rng([71, D, n_q])
    q = f32_to_bf16_bits(r.standard_normal((1, n_q, H, D)).astype(np.float32))
    key = np.zeros((1, 1, H, 1, D), dtype=np.float32)
    key[0, 0, np.arange(H), 0, np.arange(H)] = 1.0
    k = bits_to_dev(f32_to_bf16_bits(key))
    out = torch.empty((1, n_q, H, D), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, H, n_q), float("nan"), dtype=torch.float32, device="cuda")
    if eight_bit:                            # the key as the tail segment, no 8-bit segments
        ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(1, n_q, 0, 1, 1, H, H, D))
        one = torch.ones((1,), dtype=torch.int32, device="cuda")
        dummy = torch.zeros((16,), dtype=torch.uint8, device="cuda")
        scale = torch.ones((16,), dtype=torch.float32, device="cuda")
        pc.pc_parallel_attn_fp8(bits_to_dev(q), dummy, dummy, scale, scale, None, k, k, one, 1, 1, n_q, 0, 1, H, H, D,
                                q_pos0, base, 0.0, out, lse, ws)
    else:
        ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(1, n_q, 1, 1, H, H, D, False))
        pc.pc_parallel_attn(bits_to_dev(q), k, k, None, None, None, 1, n_q, 1, 1, H, H, D, q_pos0, base, 0.0, out,
                            lse, ws)
    torch.cuda.synchronize()
    x = bf16_bits_to_f64(q[0])
    if q_pos0 >= 0:
        x = oracle.rope(x, q_pos0 + np.arange(n_q), base)
    x = x[:, np.arange(H), np.arange(H)]                                 # [n_q, H]: head h, dimension h
    mul = np.float32(np.float32(1.0) / np.sqrt(np.float32(D))) * np.float32(1.4426950408889634)
    want = f32_to_bf16_bits((x * np.float64(mul)).astype(np.float32))
    got = f32_to_bf16_bits((lse[0].cpu().numpy().T.astype(np.float64) / np.log(2.0)).astype(np.float32))
    assert int((got != want).sum()) == 0
