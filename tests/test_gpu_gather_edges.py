"""The gather at the edges of its units (a wavefront takes 4, 8 or 16 rows of 128 values, 8, 16 or 32 of 64,
of one segment): bit for bit against the rule written out in numpy, maxima included, with skipped segments, token indices
outside the source and buffers pre-filled to show stray writes."""
import numpy as np
import pytest
import torch

import paper_2502_14317_amd as pc

from helpers import bits_to_dev, dev_to_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,Hkv", [(1, 3, 1), (40, 15, 4)], ids=["few segments", "many segments"])   # 1, and 2 or 4, rows a thread
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("k", [1, 3, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 65])
def test_gather_unit_edges(B, S, Hkv, D, k):
    print("gather", B, S, Hkv, D, k, flush=True)
    C, rows = 4, 70
    r = np.random.default_rng([75, B, S, D, k])
    finite = lambda *shape: (r.integers(0, 0x7f80, size=shape) | (r.integers(0, 2, size=shape) << 15)).astype(np.uint16)
    src_k, src_v = finite(B, C, rows, Hkv, D), finite(B, C, rows, Hkv, D)
    chunk = r.integers(-1, C, size=(B, S)).astype(np.int32)
    tok = np.stack([np.sort(r.permutation(rows)[:k]) for _ in range(B * S * Hkv)]).reshape(B, S, Hkv, k).astype(np.int32)
    tok[..., -1] = np.where(r.random((B, S, Hkv)) < 0.5, -1, tok[..., -1])
    fill = np.uint16(0x4242)
    kd = bits_to_dev(np.full((B, S, Hkv, k, D), fill))
    vd = bits_to_dev(np.full((B, S, Hkv, k, D), fill))
    ka = torch.full((B, S, Hkv), -5.0, dtype=torch.float32, device="cuda")
    va = torch.full((B, S, Hkv), -5.0, dtype=torch.float32, device="cuda")
    pc.pc_gather_kv_amax(bits_to_dev(src_k), bits_to_dev(src_v), torch.from_numpy(chunk).cuda(),
                         torch.from_numpy(tok).cuda(), B, C, rows, S, Hkv, k, D, kd, vd, ka, va)
    kd2, vd2 = torch.full_like(kd, 0), torch.full_like(vd, 0)
    kd2.view(torch.int16).fill_(0x4242); vd2.view(torch.int16).fill_(0x4242)
    pc.pc_gather_kv(bits_to_dev(src_k), bits_to_dev(src_v), torch.from_numpy(chunk).cuda(),
                    torch.from_numpy(tok).cuda(), B, C, rows, S, Hkv, k, D, kd2, vd2)
    torch.cuda.synchronize()
    for src, dst, dst2, amax in ((src_k, kd, kd2, ka), (src_v, vd, vd2, va)):
        want, want_max = np.full((B, S, Hkv, k, D), fill), np.full((B, S, Hkv), -5.0, dtype=np.float32)
        for b, s in np.ndindex(B, S):
            if chunk[b, s] < 0:
                continue
            for g in range(Hkv):
                t = tok[b, s, g]
                x = src[b, chunk[b, s], np.maximum(t, 0), g]
                x[t < 0] = 0
                want[b, s, g] = x
                want_max[b, s, g] = (x.astype(np.uint32) & 0x7fff).max().astype(np.uint32).__lshift__(16).view(np.float32)
        assert np.array_equal(dev_to_bits(dst), want) and np.array_equal(dev_to_bits(dst2), want)
        assert np.array_equal(amax.cpu().numpy(), want_max)
