"""Scores with more than four blocks of 32 (voting row, head) columns: block and tile edges of the
kernel that keeps the keys in LDS, both of its tile sizes, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import S_ATOL, S_RTOL, assert_close, bits_to_dev

pytestmark = pytest.mark.gpu

# C, w, w_q, H_q, H_kv, D, voting rows, ragged
CASES = [
    (2, 63, 65, 8, 2, 64, 33, False),       # 132 columns: the fifth block holds 4; few workgroups, 64-key tiles
    (1, 129, 40, 3, 1, 128, 53, False),     # 159 columns, voting rows reach into the context (masked keys)
    (1, 128, 300, 1, 1, 128, 288, False),   # 288 columns: nine blocks, a wavefront has three
    (65, 127, 40, 8, 2, 64, 40, True),      # 160 columns, 260 workgroups: 128-key tiles, ragged and empty chunks
    (43, 257, 41, 12, 3, 128, 41, False),   # 164 columns, 387 workgroups: a tile of one context key
    (70, 100, 140, 2, 2, 64, 200, False),   # 200 columns, 280 workgroups: masked 128-key tiles
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(int(x)) for x in c))
def test_scores_many_columns(case):
    C, w, wq, Hq, Hkv, D, obs, ragged = case
    print("many columns", case, flush=True)
    r = np.random.default_rng([62, C, w, wq, Hq, D])
    lens = np.full(C, w, dtype=np.int32)
    if ragged:
        lens = r.integers(0, w + 1, size=C).astype(np.int32)
        lens[:3] = 0, w, 1
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((C, w + wq, h, D)).astype(np.float32))
    q, k = mk(Hq), mk(Hkv)
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, obs, 1.0e4)
    tok = torch.full((C, Hkv, w), float("nan"), dtype=torch.float32, device="cuda")
    chunk = torch.full((C,), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
    ws.fill_(0xFF)                                          # NaN patterns: nothing may be read before it is written
    pc.pc_chunk_query_scores(shape, bits_to_dev(q), bits_to_dev(k), tok, chunk, ws,
                             chunk_lens=torch.from_numpy(lens).cuda() if ragged else None)
    torch.cuda.synchronize()
    for c in range(C):
        n = int(lens[c])
        pos = np.arange(n + wq)
        qr = oracle.rope(bf16_bits_to_f64(q[c])[:n + wq], pos, 1.0e4)
        kr = oracle.rope(bf16_bits_to_f64(k[c])[:n + wq], pos, 1.0e4)
        ref = np.zeros((Hkv, w))
        total = 0.0
        if n:
            ref[:, :n], total = oracle.query_scores(qr, kr, n, obs, Hkv)
        assert_close(tok[c].cpu().numpy(), ref, S_ATOL, S_RTOL, f"tok_score c={c}")
        assert_close(chunk[c].cpu().numpy(), total, S_ATOL, S_RTOL, f"chunk_score c={c}")
