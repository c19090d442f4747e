"""Scores with many voting columns where the last 128-key tile of a ragged chunk holds 1 to 128 keys that count and the
rows behind the chunk are NaN: the products run over whole tiles, what lies behind the keys has to drop out."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import S_ATOL, S_RTOL, assert_close, bits_to_dev

pytestmark = pytest.mark.gpu

# w, w_q, H_q, D, voting rows: 5 column blocks (a wavefront has two), 8 (two each), 17 (the first has five)
CASES = [(300, 33, 5, 128, 32), (257, 52, 5, 64, 50), (190, 68, 8, 128, 66)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_many_columns_nan_behind_chunks(case):
    w, wq, Hq, D, obs = case
    C, Hkv = 86, 1                                          # 3 (2) tiles a chunk: at least 256 workgroups at 128 keys
    if C * ((w + wq + 127) // 128) < 256:
        C = 128
    print("many columns, padding", case, C, flush=True)
    r = np.random.default_rng([67, w, wq, Hq, D])
    lens = r.integers(1, w + 1, size=C).astype(np.int32)
    edge = [0, 1, 31, 32, 33, 64, 95, 96, 127, 128, 129, 160, w]
    lens[:len(edge)] = [min(e, w) for e in edge]
    lens[len(edge):len(edge) + 4] = [max(0, 128 - wq), max(1, 129 - wq), 256 - wq, min(w, 257 - wq)]     # the sequence ends at a tile
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
    for c in range(20):
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
