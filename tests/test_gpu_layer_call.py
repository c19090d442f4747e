"""pc_layer_forward (ParallelCompLayer.forward) against the separate calls (chunk_prefill, evict_and_attend): the
same bits everywhere but in the global attention, whose keys may be cut into other parts, so that its
probabilities round to bf16 against other references (2^-9 relative each; outputs within the outputs'
tolerance).  Shapes on either side of the rules: more than 64 chunks or 2048 block sums a chunk (selection in
launches of its own), segments of 64 KiB and more (gather in a launch of its own), few query columns (no tile path), global attention cut into parts, a global workgroup
count that is no multiple of 8, ragged chunks, calibration; and 64 query rows a wavefront next to the global attention."""
import numpy as np
import pytest
import torch

from paper_2502_14317_amd.layer import ParallelCompLayer
from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close

pytestmark = pytest.mark.gpu

# C, w, w_q, H_q, H_kv, D, obs, keep chunks, keep tokens, ragged, calibration
CASES = [
    (1, 1, 17, 1, 1, 64, 1, 1, 1, False, None),
    (3, 130, 33, 6, 2, 128, 33, 2, 50, False, (0.05, 0, 20)),
    (4, 200, 64, 8, 8, 64, 32, 4, 200, True, None),
    (64, 65, 5, 4, 1, 64, 5, 9, 33, False, None),
    (65, 40, 20, 2, 1, 128, 8, 64, 13, False, None),         # 65 chunks
    (2, 300, 4, 4, 1, 128, 4, 1, 77, True, (0.01, 10, 90)),  # 16 columns: the few-row path
    (2, 4500, 40, 32, 32, 64, 40, 2, 900, False, None),      # 71 x 32 block sums a chunk
    (1, 600, 19, 40, 8, 64, 19, 1, 580, False, None),
    (2, 3000, 300, 4, 4, 128, 20, 2, 2900, False, None),     # cut into parts
    (3, 300, 20, 4, 2, 64, 20, 2, 256, False, None),         # 64 KiB a segment: gathered by the selection
    (3, 300, 20, 4, 2, 64, 20, 2, 257, True, None),          # above
    (3, 1300, 40, 4, 2, 128, 20, 3, 128, True, (0.0, 0, 1290)),   # heads without 128 candidates: zero rows
]
# 64 query rows a wavefront: 4, 2, 8 heads and one a workgroup, (sequence, KV head) groups beyond a multiple of 8
WIDE = [
    (6, 1220, 61, 12, 3, 128, 61, 2, 300, True, None),
    (5, 3030, 58, 12, 2, 128, 32, 3, 700, False, (0.05, 0, 20)),
    (9, 1250, 31, 8, 1, 128, 31, 9, 620, True, None),
    (2, 7700, 57, 7, 7, 128, 57, 2, 7000, False, None),      # global attention cut into parts, here and in the case above
]


@pytest.mark.parametrize("case", CASES + WIDE, ids=lambda c: "x".join(map(str, c[:9])))
def test_layer_call_is_the_separate_calls(case):
    C, w, wq, Hq, Hkv, D, obs, kc, kt, ragged, cal = case
    print("layer call", case, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(w * 100 + C)
    mk = lambda h, s=1.0: (torch.randn((C, w + wq, h, D), generator=gen, device="cuda") * s).to(torch.bfloat16)
    q, k, v = mk(Hq, 1.5), mk(Hkv), mk(Hkv)
    lens, first = None, None
    if ragged:
        host = [w - (c * 37) % max(1, w // 2) for c in range(C)]
        lens, first = torch.tensor(host, dtype=torch.int32, device="cuda"), host[0]
    a, b = (ParallelCompLayer(C, w, wq, Hq, Hkv, D, obs, 1.0e4, kc, kt, calibration=cal) for _ in range(2))
    for layer in (a, b):
        layer.o.fill_(7); layer.tok_idx.fill_(-9); layer.kc.fill_(3); layer.tok_cnt.fill_(0)
    a.ws.fill_(0xFF)
    a.forward(q, k, v, chunk_lens=lens, first_len=first)
    b.chunk_prefill(q, k, v, chunk_lens=lens, first_len=first)
    b.evict_and_attend(q, v)
    torch.cuda.synchronize()
    for name in ("tok_score", "chunk_score", "chunk_idx", "chunk_top", "tok_idx", "tok_cnt", "kc", "vc"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    rows = [w + wq] * C if lens is None else [n + wq for n in lens.tolist()]
    for c, n in enumerate(rows):
        assert torch.equal(a.o[c, :n], b.o[c, :n]) and torch.equal(a.lse[c, :, :n], b.lse[c, :, :n]), c
        assert torch.equal(a.k_rope[c, :n], b.k_rope[c, :n]), c
    assert_close(a.global_o.double().cpu().numpy(), b.global_o.double().cpu().numpy(), O_ATOL, O_RTOL, "global o")
    assert_close(a.global_lse.cpu().numpy(), b.global_lse.cpu().numpy(), LSE_ATOL, 1e-3, "global lse")
