"""Scores of many voting columns where the voting rows reach into the context, so that some keys are hidden from some rows:
heads of fewer rows than a block of 32 columns, of one more or one less, and of all rows, in both tile sizes, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import S_ATOL, S_RTOL, assert_close, bits_to_dev

pytestmark = pytest.mark.gpu

# C, w, w_q, H_q, H_kv, D, voting rows
CASES = [
    (2, 140, 1, 64, 1, 64, 3),         # eleven heads meet in a block of columns
    (2, 131, 0, 150, 1, 128, 1),       # a row a head, no query rows: only the last key is hidden from nobody
    (2, 200, 5, 16, 1, 128, 31),
    (2, 200, 5, 8, 1, 64, 33),
    (1, 97, 7, 3, 1, 64, 64),          # a head ends with a block
    (90, 129, 130, 1, 1, 128, 259),    # every row votes; 270 workgroups: 128-key tiles, the last of one context key
    (130, 140, 20, 4, 1, 64, 100),
    (130, 130, 9, 20, 1, 128, 17),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_voting_rows_among_the_context(case):
    C, w, wq, Hq, Hkv, D, obs = case
    print("masked columns", case, flush=True)
    r = np.random.default_rng([71, C, w, wq, Hq, D])
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((C, w + wq, h, D)).astype(np.float32))
    q, k = mk(Hq), mk(Hkv)
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, obs, 1.0e4)
    tok = torch.full((C, Hkv, w), float("nan"), dtype=torch.float32, device="cuda")
    chunk = torch.full((C,), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
    ws.fill_(0xFF)                                          # NaN patterns: nothing may be read before it is written
    pc.pc_chunk_query_scores(shape, bits_to_dev(q), bits_to_dev(k), tok, chunk, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(tok).all()
    pos = np.arange(w + wq)
    for c in {0, 1, C // 2, C - 1} & set(range(C)):
        qr = oracle.rope(bf16_bits_to_f64(q[c]), pos, 1.0e4)
        kr = oracle.rope(bf16_bits_to_f64(k[c]), pos, 1.0e4)
        ref, total = oracle.query_scores(qr, kr, w, obs, Hkv)
        assert_close(tok[c].cpu().numpy(), ref, S_ATOL, S_RTOL, f"tok_score c={c}")
        assert_close(chunk[c].cpu().numpy(), total, S_ATOL, S_RTOL, f"chunk_score c={c}")
