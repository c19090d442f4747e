"""Few-row attention and a decoding step of more than 2^24 output rows (2^20 sequences x 20 heads), where one
workgroup of 256 threads a row would pass the launch's limit of 2^32 threads in one grid dimension.  One key a KV head: every
output row is that key's value, exactly."""
import pytest
import torch

import paper_2502_14317_amd as pc

pytestmark = pytest.mark.gpu

B, HQ, HKV, D = 1 << 20, 20, 2, 64


def _check(out, lse, v):
    torch.cuda.synchronize()
    out = out.view(B, HKV, HQ // HKV, D)
    for g in range(HKV):
        for h in range(HQ // HKV):
            assert torch.equal(out[:, g, h], v[:, g])
    assert torch.isfinite(lse).all()


def _inputs():
    gen = torch.Generator(device="cuda").manual_seed(8)
    mk = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)
    out = torch.full((B, 1, HQ, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, HQ, 1), float("nan"), dtype=torch.float32, device="cuda")
    return mk(B, 1, HQ, D), mk(B, 1, HKV, 1, D), mk(B, 1, HKV, 1, D), out, lse


def test_attention_of_more_than_2_24_rows():
    print("many rows: attention", flush=True)
    q, kc, vc, out, lse = _inputs()
    ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, 1, 1, 1, HQ, HKV, D, False))
    pc.pc_parallel_attn(q, kc, vc, None, None, None, B, 1, 1, 1, HQ, HKV, D, -1, 1.0e4, 0.0, out, lse, ws)
    _check(out, lse, vc[:, 0, :, 0])


def test_step_of_more_than_2_24_rows():
    print("many rows: step", flush=True)
    q, k, v, out, lse = _inputs()
    k, v = k.view(B, 1, HKV, D), v.view(B, 1, HKV, D)
    kc, vc = (torch.zeros((B, 1, HKV, 1, D), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    lens = torch.zeros((B, 1), dtype=torch.int32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_decode_step_workspace_bytes(B, 1, 1, HQ, HKV, D))
    pc.pc_decode_step(q, k, v, B, 1, 1, HQ, HKV, D, -1, 1.0e4, 0.0, kc, vc, lens, out, lse, ws)
    _check(out, lse, v[:, 0])
    assert torch.equal(kc.view_as(k), k) and torch.equal(vc.view_as(v), v) and (lens == 1).all()
