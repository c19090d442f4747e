"""Score calls of 2^24 and more (chunk, KV head) pairs, whose workgroups pass the 2^32 threads of a grid dimension.
Chunks of one context row and one query row, which votes: the key's probability is a sigmoid."""
import pytest
import torch

import paper_2502_14317_amd as pc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,D", [(1 << 20, 16, 128), (1 << 20, 17, 64)])
def test_scores_of_more_than_2_24_groups(C, H, D):
    print("score groups", C, H, D, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(D)
    mk = lambda: torch.randn((C, 2, H, D), generator=gen, device="cuda", dtype=torch.bfloat16)
    q, k = mk(), mk()
    shape = pc.make_shape(C, 1, 1, H, H, D, 1, 1.0e4)
    tok = torch.full((C, H, 1), float("nan"), device="cuda")
    chunk = torch.full((C,), float("nan"), device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
    pc.pc_chunk_query_scores(shape, q, k, tok, chunk, ws)
    torch.cuda.synchronize()
    theta = 1.0e4 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device="cuda") / D)
    cs, sn = theta.cos(), theta.sin()                                     # position 1
    for c0 in range(0, C, 1 << 16):
        x = q[c0:c0 + (1 << 16), 1].double()
        a, b = x[..., :D // 2], x[..., D // 2:]
        rot = torch.cat([a * cs - b * sn, b * cs + a * sn], dim=-1)
        # the query and the key of one position keep their product under its rotation
        y0, y1 = (rot * k[c0:c0 + (1 << 16), 0].double()).sum(-1), (x * k[c0:c0 + (1 << 16), 1].double()).sum(-1)
        p = torch.sigmoid((y0 - y1) / D ** 0.5)
        got = tok[c0:c0 + (1 << 16), :, 0].double()
        assert ((got - p).abs() <= 1e-3 * p).all(), c0                   # the scores' tolerance
        assert ((chunk[c0:c0 + (1 << 16)].double() - p.sum(-1)).abs() <= 1e-3 * p.sum(-1)).all(), c0
