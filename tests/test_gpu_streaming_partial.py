"""Streaming with many voting columns and a short last batch: the workspace sized for a full batch
serves it (128 chunks take 128-key score blocks, the last 127 take 64-key ones)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_14317_amd.layer import StreamingParallelComp
from workloads import bf16_bits_to_f64, f32_to_bf16_bits

from helpers import S_ATOL, S_RTOL, assert_close, bits_to_dev

pytestmark = pytest.mark.gpu


def test_short_last_batch_with_many_voting_columns():
    C, bc, w, wq, Hq, Hkv, D, keep, kt = 255, 128, 100, 28, 16, 2, 64, 4, 20
    print("streaming, short last batch", flush=True)
    r = np.random.default_rng(72)
    mk = lambda h: f32_to_bf16_bits(r.standard_normal((C, w + wq, h, D)).astype(np.float32))
    q, k, v = mk(Hq), mk(Hkv), mk(Hkv)
    st = StreamingParallelComp(C, bc, w, wq, Hq, Hkv, D, wq, 1.0e4, keep, kt)
    st.forward(bits_to_dev(q), bits_to_dev(k), bits_to_dev(v))
    torch.cuda.synchronize()
    got = st.chunk_score.cpu().numpy()
    pos = np.arange(w + wq)
    for c in range(C):
        qr, kr = (oracle.rope(bf16_bits_to_f64(x[c]), pos, 1.0e4) for x in (q, k))
        tok, total = oracle.query_scores(qr, kr, w, wq, Hkv)
        assert_close(got[c], total, S_ATOL, S_RTOL, f"chunk_score c={c}")
        if c >= bc:
            assert_close(st.tok_score[c - bc].cpu().numpy(), tok, S_ATOL, S_RTOL, f"tok_score c={c}")
    order = sorted(range(C), key=lambda c: (-got[c], c))[:keep]
    assert st.queue_id.cpu().tolist() == order
    assert torch.isfinite(st.global_o.float()).all()
