"""Scores of one long sequence with few voting columns, on either side of the 64 key blocks of 256 keys up
to which pass 2 combines the row logsumexp itself (a launch in between does beyond)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import S_ATOL, S_RTOL, assert_close, bits_to_dev

pytestmark = pytest.mark.gpu


# rows of the sequence, H_q, D, voting rows: one, two and three or four blocks of 32 columns
@pytest.mark.parametrize("L,Hq,D,obs", [(64 * 256, 2, 64, 5), (64 * 256 + 1, 2, 64, 5), (64 * 256 + 1, 3, 128, 17),
                                        (64 * 256, 4, 128, 32), (70 * 256, 4, 64, 32)])
def test_long_sequence_scores(L, Hq, D, obs):
    print("long sequence", L, Hq, D, obs, flush=True)
    wq = obs + 3
    w = L - wq
    r = np.random.default_rng([77, L, Hq, D])
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((1, L, h, D)).astype(np.float32))
    q, k = mk(Hq), mk(1)
    shape = pc.make_shape(1, w, wq, Hq, 1, D, obs, 5.0e5)
    tok = torch.full((1, 1, w), float("nan"), dtype=torch.float32, device="cuda")
    chunk = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
    ws.fill_(0xFF)                                          # NaN patterns: nothing may be read before it is written
    pc.pc_profile_begin()
    try:
        pc.pc_chunk_query_scores(shape, bits_to_dev(q), bits_to_dev(k), tok, chunk, ws)
        torch.cuda.synchronize()
    finally:
        pc.pc_profile_end()
    assert [name for name, _ in pc.pc_profile_records()].count("scores_lse_kernel") == int(L > 64 * 256)
    pos = np.arange(L)
    qr, kr = (oracle.rope(bf16_bits_to_f64(x[0]), pos, 5.0e5) for x in (q, k))
    ref, total = oracle.query_scores(qr, kr, w, obs, 1)
    assert_close(tok[0].cpu().numpy(), ref, S_ATOL, S_RTOL, "tok_score")
    assert_close(chunk[0].cpu().numpy(), total, S_ATOL, S_RTOL, "chunk_score")
