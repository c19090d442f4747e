"""A block of query rows over the 8-bit cache whose widening launch, a workgroup for every query row and every tile, has more
than 2^24 workgroups of 256 threads (2^32 threads, a grid dimension's limit) although neither has by itself.  One key counts a
sequence: every output row is that key's value, exactly, and the logsumexp its logit."""
import pytest
import torch

import paper_2502_14317_amd as pc
from helpers import LSE_ATOL, fp8_from_rows

pytestmark = pytest.mark.gpu

N_Q, D, KT = 1024, 64, 64


@pytest.mark.parametrize("B", [16380])
def test_more_than_2_24_rows_and_tiles(B):
    assert B * N_Q < 1 << 24 and B * N_Q + B > 1 << 24     # a tile a sequence
    print("fp8 block, many rows", B, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(9)
    q = torch.randn((B, N_Q, 1, D), generator=gen, device="cuda", dtype=torch.bfloat16)
    rows, dev = [], []
    for w in "kv":
        codes = torch.full((B, 1, 1, KT, D), 0x7f, dtype=torch.uint8, device="cuda")           # NaN behind the key that counts
        codes[..., 0, :] = (torch.randint(0, 0x48, (B, 1, 1, D), generator=gen, device="cuda")
                            + 0x80 * torch.randint(0, 2, (B, 1, 1, D), generator=gen, device="cuda")).to(torch.uint8)
        rows.append(codes[:, 0, 0, 0].view(torch.float8_e4m3fn).float())
        dev.append(fp8_from_rows(w, codes))
    ones = torch.ones((B, 1, 1), device="cuda")
    lens = torch.ones((B, 1), dtype=torch.int32, device="cuda")
    out = torch.full((B, N_Q, 1, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, 1, N_Q), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, N_Q, 1, KT, 0, 1, 1, D))
    ws.fill_(0xFF)                                          # NaN wherever nothing was written
    pc.pc_profile_begin()
    try:
        pc.pc_parallel_attn_fp8(q, *dev, ones, ones, lens, None, None, None, 0, B, N_Q, 1, KT, 1, 1, D, -1, 1.0e4, 0.0, out, lse, ws)
        torch.cuda.synchronize()
    finally:
        pc.pc_profile_end()
    assert [name for name, _ in pc.pc_profile_records()].count("fp8_images_kernel") == 1
    assert torch.equal(out[:, :, 0].float(), rows[1][:, None].expand(B, N_Q, D))
    for b0 in range(0, B, 1024):
        ref = (q[b0:b0 + 1024, :, 0].float() * rows[0][b0:b0 + 1024, None]).sum(dim=-1) / 8.0
        assert ((lse[b0:b0 + 1024, 0] - ref).abs() <= LSE_ATOL * (1.0 + ref.abs())).all()
