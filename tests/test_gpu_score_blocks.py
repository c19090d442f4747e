"""Scores with few voting columns where pass 2 takes other key blocks than pass 1: up to 1024 keys, against the
oracle on some of the chunks."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc

from helpers import S_ATOL, S_RTOL, assert_close

pytestmark = pytest.mark.gpu

# C, w, w_q, H_q, H_kv, D, voting rows, ragged
CASES = [
    (64, 1300, 40, 4, 4, 64, 32, False),      # one column block: 512 keys in pass 1, 1024 in pass 2
    (64, 2049, 33, 4, 4, 64, 8, True),        # 8 columns, 3 x 1024, one key in the last, ragged and empty chunks
    (128, 1025, 40, 2, 2, 128, 32, False),    # 1024 + 1: angles read anew behind 512 keys
    (128, 2048, 64, 2, 2, 128, 48, False),    # two column blocks, the voting rows inside the query block: 2 x 1024
    (32, 1500, 36, 32, 8, 128, 32, True),     # four column blocks, keys in tiles of 64
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(int(x)) for x in c))
def test_score_blocks(case):
    C, w, wq, Hq, Hkv, D, obs, ragged = case
    print("score blocks", case, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(C + w)
    q, k = (torch.randn((C, w + wq, h, D), generator=gen, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv))
    lens = np.full(C, w, dtype=np.int32)
    if ragged:
        lens[:] = np.random.default_rng(w).integers(0, w + 1, size=C)
        lens[:5] = 0, 1, w, 1024, 1025
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, obs, 1.0e4)
    tok = torch.full((C, Hkv, w), float("nan"), dtype=torch.float32, device="cuda")
    chunk = torch.full((C,), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
    ws.fill_(0xFF)
    pc.pc_chunk_query_scores(shape, q, k, tok, chunk, ws, chunk_lens=torch.from_numpy(lens).cuda() if ragged else None)
    torch.cuda.synchronize()
    assert torch.isfinite(tok).all() and torch.isfinite(chunk).all()
    for c in (0, 1, 2, 3, 4, C - 1):
        n = int(lens[c])
        pos = np.arange(n + wq)
        qr = oracle.rope(q[c, :n + wq].double().cpu().numpy(), pos, 1.0e4)
        kr = oracle.rope(k[c, :n + wq].double().cpu().numpy(), pos, 1.0e4)
        ref = np.zeros((Hkv, w))
        total = 0.0
        if n:
            ref[:, :n], total = oracle.query_scores(qr, kr, n, obs, Hkv)
        assert_close(tok[c].cpu().numpy(), ref, S_ATOL, S_RTOL, f"tok_score c={c}")
        assert_close(chunk[c].cpu().numpy(), total, S_ATOL, S_RTOL, f"chunk_score c={c}")


# Pass 1 takes 512 keys a workgroup in both calls, pass 2 1024 with all the chunks (512 workgroups of them) and 512 with some
@pytest.mark.parametrize("C,some,w,wq,H,D", [(64, 48, 1300, 40, 4, 64), (128, 100, 1025, 40, 2, 128)], ids=["d64", "d128"])
def test_blocks_of_512_and_1024_keys_give_the_same_bits(C, some, w, wq, H, D):
    print("score blocks, bits", C, some, w, D, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(D)
    q, k = (torch.randn((C, w + wq, H, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    toks = []
    for n in (C, some):
        shape = pc.make_shape(n, w, wq, H, H, D, 32, 1.0e4)
        tok = torch.full((n, H, w), float("nan"), dtype=torch.float32, device="cuda")
        ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
        pc.pc_chunk_query_scores(shape, q[:n], k[:n], tok, None, ws)
        toks.append(tok)
    torch.cuda.synchronize()
    assert torch.equal(toks[0][:some], toks[1])
