"""The gather on both sides of the size above which its stores carry the non-temporal hint (256 MiB of K and V):
bit for bit against an index_select, maxima included."""
import pytest
import torch

import paper_2502_14317_amd as pc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [4096, 4097], ids=["256 MiB", "above"])
def test_gather_around_the_last_level_cache(k):
    B, S, Hkv, D, C, rows = 2, 8, 8, 128, 8, 5000
    print("gather", k, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(k)
    src = [torch.randn((B, C, rows, Hkv, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2)]
    chunk = torch.rand((B, C), generator=gen, device="cuda").argsort(dim=1).to(torch.int32).contiguous()
    tok = torch.rand((B, S, Hkv, rows), generator=gen, device="cuda").argsort(dim=-1)[..., :k].contiguous()
    dst = [torch.empty((B, S, Hkv, k, D), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    amax = [torch.empty((B, S, Hkv), device="cuda") for _ in range(2)]
    pc.pc_gather_kv_amax(*src, chunk, tok.to(torch.int32), B, C, rows, S, Hkv, k, D, *dst, *amax)
    torch.cuda.synchronize()
    for x, d, m in zip(src, dst, amax):
        for b in range(B):
            for s in range(S):
                rows_bsg = x[b, int(chunk[b, s])].transpose(0, 1)                        # [H_kv, rows, D]
                want = torch.gather(rows_bsg, 1, tok[b, s][..., None].expand(-1, -1, D))
                assert torch.equal(d[b, s].view(torch.int16), want.view(torch.int16))
                assert torch.equal(m[b, s], want.abs().amax(dim=(1, 2)).float())
