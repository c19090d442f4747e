"""Scores with many voting columns where the last tile of a ragged chunk (of 128 keys or, with few workgroups, 64) holds any
number of keys that count and the rows behind the chunk are NaN: the products run over whole tiles or, with up to 64 keys
in one of 128, over its first half; what lies behind the keys has to drop out."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import S_ATOL, S_RTOL, assert_close, bits_to_dev

pytestmark = pytest.mark.gpu

# C, w, w_q, H_q, D, voting rows: 5 column blocks (a wavefront has two), 8 (two each), 17 (the first has five).
# 86 chunks of up to 384 rows are 258 workgroups of 128 keys, 24 fewer than 256: 64 keys.
CASES = [(86, 300, 33, 5, 128, 32), (86, 257, 52, 5, 64, 50), (86, 190, 68, 8, 128, 66),
         (24, 300, 33, 5, 128, 32), (24, 190, 68, 8, 64, 66)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_many_columns_nan_behind_chunks(case):
    C, w, wq, Hq, D, obs = case
    Hkv = 1
    print("many columns, padding", case, flush=True)
    r = np.random.default_rng([67, w, wq, Hq, D])
    lens = r.integers(1, w + 1, size=C).astype(np.int32)
    edge = [0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 127, 128, 129, 160, 192, w]          # the context ends there
    edge += [e - wq for e in (64, 65, 128, 129, 192, 193, 256, 257)]                   # the sequence does
    lens[:len(edge)] = np.clip(edge, 0, w)
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((C, w + wq, h, D)).astype(np.float32))
    q, k = mk(Hq), mk(Hkv)
    for c in range(C):
        q[c, lens[c] + wq:] = k[c, lens[c] + wq:] = 0x7FC0
    shape = pc.make_shape(C, w, wq, Hq, Hkv, D, obs, 1.0e4)
    tok = torch.full((C, Hkv, w), float("nan"), dtype=torch.float32, device="cuda")
    chunk = torch.full((C,), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_chunk_query_scores_workspace_bytes(shape))
    ws.fill_(0xFF)
    pc.pc_chunk_query_scores(shape, bits_to_dev(q), bits_to_dev(k), tok, chunk, ws, chunk_lens=torch.from_numpy(lens).cuda())
    torch.cuda.synchronize()
    for c in range(len(edge)):
        n = int(lens[c])
        pos = np.arange(n + wq)
        qr = oracle.rope(bf16_bits_to_f64(q[c])[:n + wq], pos, 1.0e4)
        kr = oracle.rope(bf16_bits_to_f64(k[c])[:n + wq], pos, 1.0e4)
        ref = np.zeros((Hkv, w))
        total = 0.0
        if n:
            ref[:, :n], total = oracle.query_scores(qr, kr, n, obs, Hkv)
        assert_close(tok[c].cpu().numpy(), ref, S_ATOL, S_RTOL, f"tok_score c={c} n={n}")
        assert_close(chunk[c].cpu().numpy(), total, S_ATOL, S_RTOL, f"chunk_score c={c} n={n}")
