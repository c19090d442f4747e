"""Local attention with logits at the edges of the window of a row's softmax reference in the kernel of 64 query rows a
wavefront, a lane's step sum of 2^90: just inside it the probabilities are as large as they get and nothing moves, just
outside the step is taken anew.  The kernel of 32 rows (short rows), whose references move from 2^8 on, gets the same logits.

Logits are known exactly, as in test_gpu_reference_moves.py: the slowest pair of a head, which the largest angle here,
1553 * 1e30^(-1 + 2 / 128) < 2e-26, leaves as it is.  What is left are the bf16 roundings of a probability and of the output
(2^-9 each, of at most max |v| < 6) and fp32 sums."""
import numpy as np
import pytest
import torch

import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu

D = 128
STEPS = {                                                   # logits of the row's four quarters of keys, log2 units
    "inside": [0.0, 40.0, 85.0, 85.5],                      # 16 keys a lane: 2^89.5
    "at the edge": [0.0, 85.5, 86.0, 86.5],
    "outside": [0.0, 88.0, 91.0, 180.0],
    "inside, then outside": [0.0, 85.0, 174.0, 175.0],
}


@pytest.mark.parametrize("C,w,wq,Hq,Hkv", [(2, 200, 57, 4, 2), (12, 1350, 203, 32, 8)])
@pytest.mark.parametrize("name", STEPS)
def test_edges_of_the_window(name, C, w, wq, Hq, Hkv):
    print("reference window", name, C, w, flush=True)
    L = w + wq
    r = np.random.default_rng([73, L, len(name)])
    q, k = np.zeros((C, L, Hq, D), np.float32), np.zeros((C, L, Hkv, D), np.float32)
    scale = 1.0 / np.sqrt(D)
    size = r.choice([1.0, 0.5, -1.0], size=(C, L, Hq))
    q[..., D // 2 - 1] = size / (scale * np.log2(np.e))
    level = np.array(STEPS[name])[4 * np.arange(L) // L]
    k[:, :, :, D // 2 - 1] = level[None, :, None]
    qb, kb = f32_to_bf16_bits(q), f32_to_bf16_bits(k)
    vb = f32_to_bf16_bits(np.clip(r.standard_normal((C, L, Hkv, D)), -6, 6).astype(np.float32))
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, 1, 1.0e30)
    o = torch.full((C, L, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((C, Hq, L), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_prefill_workspace_bytes(shape))
    pc.pc_chunk_prefill_attn(shape, bits_to_dev(qb), bits_to_dev(kb), bits_to_dev(vb), o, lse, None, None, None, ws)
    torch.cuda.synchronize()
    assert not torch.isnan(o).any() and not torch.isnan(lse).any()
    qs = bf16_bits_to_f64(f32_to_bf16_bits((bf16_bits_to_f64(qb)[..., D // 2 - 1] * (scale * np.log2(np.e))).astype(np.float32)))
    kf = bf16_bits_to_f64(kb)[..., D // 2 - 1]
    j = np.arange(L)
    for c, h in [(0, 0), (0, Hq - 1), (C - 1, 1), (C - 1, Hq - 2)]:
        g = h // (Hq // Hkv)
        s = np.where(j[None, :] <= j[:, None], qs[c, :, h, None] * kf[c, None, :, g], -np.inf)
        m = s.max(axis=1, keepdims=True)
        p = np.exp2(s - m)
        z = p.sum(axis=1, keepdims=True)
        assert_close(dev_bf16_to_f64(o[c, :, h]), (p / z) @ bf16_bits_to_f64(vb)[c, :, g], 6 * 2.0 ** -9, 2.0 ** -8, f"o[{c}, {h}]")
        assert_close(lse[c, h].cpu().numpy(), (m + np.log2(z))[:, 0] * np.log(2.0), 1e-4, 1e-6, f"lse[{c}, {h}]")
