"""Attention of 2^24 and more query rows over their own keys, few rows a sequence and a block of them: the rotation takes a
workgroup of 256 threads a row, 2^32 threads and more in all.  A sequence's first row stands at position 0 and sees one key: its
output is that key's value, exactly, and its logsumexp their logit."""
import pytest
import torch

import paper_2502_14317_amd as pc
from helpers import LSE_ATOL

pytestmark = pytest.mark.gpu

B, D = 1 << 20, 64


@pytest.mark.parametrize("n_q", [16, 17], ids=["few_rows", "block"])
def test_2_24_query_rows(n_q):
    print("many query rows", n_q, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n_q)
    q, k, v = (torch.randn((B, n_q, 1, D), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    out = torch.full((B, n_q, 1, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, 1, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, n_q, 0, 1, 1, 1, D, True))
    ws.fill_(0xFF)                                          # NaN wherever nothing was written
    pc.pc_parallel_attn(q, None, None, None, k, v, B, n_q, 0, 1, 1, 1, D, 0, 1.0e4, 0.0, out, lse, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(lse).all()
    assert torch.equal(out[:, 0], v[:, 0])
    ref = (q[:, 0, 0].float() * k[:, 0, 0].float()).sum(dim=-1) / 8.0
    assert ((lse[:, 0, 0] - ref).abs() <= LSE_ATOL * (1.0 + ref.abs())).all()
