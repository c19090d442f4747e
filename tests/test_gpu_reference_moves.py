"""Local attention where the softmax reference has to move behind a row's first 32 keys: the step whose maximum exceeds
it by more than 8 (log2 units) moves it there and rescales what the row has so far.

The logits are known exactly: only the slowest pair of every head is used, which a rotation by the largest angle
here, 257 * 1e30^(-1 + 2 / D) < 1e-25, leaves as it is, and a query is one value times one key value.  What is left are
the bf16 roundings of a probability and of the output (2^-9 each, of at most max |v| < 5) and fp32 sums."""
import numpy as np
import pytest
import torch

import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import assert_close, bits_to_dev, dev_bf16_to_f64

pytestmark = pytest.mark.gpu

L = 257                                                     # four 64-key tiles and one key, two or three Q tiles
J = np.arange(L)
LEVELS = {                                                  # a key's logit for a query of 1, log2 units
    "every step": 10.0 * (J // 32),
    "every tile's second half": 12.0 * ((J + 32) // 64),
    "just below and above the window": np.select([J < 40, J < 70, J < 101, J < 160], [0.0, 4.0, 8.0, 8.0625], 17.0),
    "beyond the range of exp2": np.where(J < 77, 0.0, np.where(J < 200, 300.0, 900.0)),
    "one key": np.where(J == 95, 40.0, np.where(J == 192, 90.0, 0.0)),
    "last key": np.where(J == L - 1, 200.0, 0.0),
    "falling": 250.0 - J // 4 * 4.0,
}


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name", LEVELS)
def test_reference_moves_inside_a_sequence(name, D):
    print("reference moves", name, D, flush=True)
    C, w, wq, Hq, Hkv = 2, 200, L - 200, 4, 2
    r = np.random.default_rng([71, D, len(name)])
    q, k = np.zeros((C, L, Hq, D), np.float32), np.zeros((C, L, Hkv, D), np.float32)
    scale = 1.0 / np.sqrt(D)
    size = r.choice([1.0, 0.5, 0.25, -1.0], size=(C, L, Hq))    # rows of one wavefront differ in whether they move
    q[..., D // 2 - 1] = size / (scale * np.log2(np.e))
    k[:, :, :, D // 2 - 1] = LEVELS[name][None, :, None]
    k[1, :, 1] = 0.0                                        # and one group has nothing to move for
    qb, kb = f32_to_bf16_bits(q), f32_to_bf16_bits(k)
    vb = f32_to_bf16_bits(r.standard_normal((C, L, Hkv, D)).astype(np.float32))
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, 1, 1.0e30)
    o = torch.full((C, L, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((C, Hq, L), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_prefill_workspace_bytes(shape))
    pc.pc_chunk_prefill_attn(shape, bits_to_dev(qb), bits_to_dev(kb), bits_to_dev(vb), o, lse, None, None, None, ws)
    torch.cuda.synchronize()
    # the query as the kernel multiplies it: scale * log2(e) in, rounded to bf16 once
    qs = bf16_bits_to_f64(f32_to_bf16_bits((bf16_bits_to_f64(qb)[..., D // 2 - 1] * (scale * np.log2(np.e))).astype(np.float32)))
    kf, v = bf16_bits_to_f64(kb)[..., D // 2 - 1], bf16_bits_to_f64(vb)
    for c, h in np.ndindex(C, Hq):
        g = h // (Hq // Hkv)
        s = np.where(J[None, :] <= J[:, None], qs[c, :, h, None] * kf[c, None, :, g], -np.inf)
        m = s.max(axis=1, keepdims=True)
        p = np.exp2(s - m)
        z = p.sum(axis=1, keepdims=True)
        assert_close(dev_bf16_to_f64(o[c, :, h]), (p / z) @ v[c, :, g], 5 * 2.0 ** -9, 2.0 ** -8, f"o[{c}, {h}]")
        assert_close(lse[c, h].cpu().numpy(), (m + np.log2(z))[:, 0] * np.log(2.0), 1e-4, 1e-6, f"lse[{c}, {h}]")
