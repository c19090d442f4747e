"""A layer's selections in one launch or apart, on either side of the line that chunks and block sums draw (with the
gather of small segments and without): the launches that ran, and the bits of the separate calls."""
import pytest
import torch

import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import ParallelCompLayer

pytestmark = pytest.mark.gpu


# C, w, w_q, heads, D, keep chunks, keep tokens, one launch
@pytest.mark.parametrize("C,w,wq,H,D,kc,kt,one", [
    (44, 200, 20, 8, 128, 3, 150, True),         # 44 x (8 + 400)
    (45, 200, 20, 8, 128, 3, 150, False),
    (64, 40, 20, 68, 64, 2, 33, True),           # with the gather: 64 x (68 + 400)
    (64, 40, 20, 69, 64, 2, 33, False),
])
def test_selections_in_one_launch_or_apart(C, w, wq, H, D, kc, kt, one):
    print("selection route", C, w, wq, H, D, kc, kt, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(C + H)
    q, k, v = (torch.randn((C, w + wq, H, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    a, b = (ParallelCompLayer(C, w, wq, H, H, D, 8, 1.0e4, kc, kt) for _ in range(2))
    for layer in (a, b):
        layer.tok_idx.fill_(-9); layer.kc.fill_(3); layer.vc.fill_(3)
    a.ws.fill_(0xFF)
    pc.pc_profile_begin()
    try:
        a.forward(q, k, v)
        torch.cuda.synchronize()
    finally:
        pc.pc_profile_end()
    names = [name for name, _ in pc.pc_profile_records()]
    assert names.count("select_chunks_kernel") == names.count("chunk_score_kernel") == int(not one)
    assert names.count("gather_kv_kernel") == int(not (one and 4 * D * kt <= 65536))
    b.chunk_prefill(q, k, v)
    b.evict_and_attend(q, v)
    torch.cuda.synchronize()
    for name in ("tok_score", "chunk_score", "chunk_idx", "chunk_top", "tok_idx", "kc", "vc"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
