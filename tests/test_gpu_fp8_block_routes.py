"""A block of query rows over the 8-bit cache, widened to tile images or to rows (with the tail and the self segment
read where they lie): on either side of the rule, at the edges of tiles and blocks, the same bits as the 16-bit call
over the widened segments and the tail as one more segment, with NaN behind every length."""
import pytest
import torch

import paper_2502_14317_amd as pc
from helpers import fp8_from_rows

pytestmark = pytest.mark.gpu

# B, n_q, S, k_t (tail capacity too: the same tiles), H_q, H_kv, D, tail, self, per-head lengths, images
CASES = [
    (4, 100, 11, 97, 128, 16, 128, True, True, True, True),
    (4, 100, 33, 31, 128, 16, 128, True, True, False, True),
    (4, 101, 31, 33, 128, 16, 64, True, False, True, True),
    (4, 100, 16, 64, 128, 16, 128, False, True, False, True),
    (4, 100, 9, 130, 128, 16, 64, True, True, True, True),
    (4, 129, 9, 127, 128, 16, 64, False, False, False, True),
    (4, 100, 2, 97, 128, 16, 128, True, True, True, False),
    (4, 3, 11, 97, 128, 16, 128, True, True, False, False),
    (2, 40, 0, 65, 8, 2, 64, True, True, False, False),
    (1, 33, 3, 31, 8, 2, 128, True, False, True, False),
    (1, 1, 5, 161, 40, 2, 64, True, False, True, False),
    (2, 65, 4, 33, 6, 2, 128, False, True, False, False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_both_routes_are_the_16_bit_call(case):
    B, n_q, S, kt, Hq, Hkv, D, has_tail, has_self, per_head, images = case
    print("fp8 route", case, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B * 100 + kt)
    mk = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    q = mk(B, n_q, Hq, D)
    slf = [mk(B, n_q, Hkv, D) for _ in range(2)] if has_self else [None, None]
    T = S + int(has_tail)
    lens = torch.randint(0, kt + 1, (B, T, Hkv) if per_head else (B, T), generator=gen, device="cuda", dtype=torch.int32)
    lens.view(-1)[0] = kt
    if has_tail and per_head:
        lens[:, S] = lens[:, S, :1]                        # a tail has one length for all heads
    per = lens if per_head else lens[:, :, None].expand(B, T, Hkv)
    dead = torch.arange(kt, device="cuda") >= per[..., None]
    rows, dev, scales = [], [], []
    for w in "kv":
        codes = (torch.randint(0, 0x48, (B, S, Hkv, kt, D), generator=gen, device="cuda")
                 + 0x80 * torch.randint(0, 2, (B, S, Hkv, kt, D), generator=gen, device="cuda")).to(torch.uint8)
        scale = torch.rand((B, S, Hkv), generator=gen, device="cuda") * 0.7 + 0.2
        wide = (codes.view(torch.float8_e4m3fn).float() * scale[..., None, None]).to(torch.bfloat16)
        wide = torch.cat([wide, mk(B, 1, Hkv, kt, D)], dim=1) if has_tail else wide
        wide[dead] = float("nan")
        codes[dead[:, :S]] = 0x7f                          # NaN
        rows.append(wide.contiguous()); scales.append(scale)
        dev.append(fp8_from_rows(w, codes) if S else torch.zeros((1,), dtype=torch.uint8, device="cuda").expand(64).contiguous())
    out = [torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    lse = [torch.full((B, Hq, n_q), float("nan"), device="cuda") for _ in range(2)]
    ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, n_q, T, kt, Hq, Hkv, D, has_self))
    pc.pc_parallel_attn(q, *rows, lens, *slf, B, n_q, T, kt, Hq, Hkv, D, 50, 1.0e4, 0.0, out[0], lse[0], ws, int(per_head))
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, n_q, S, kt, kt if has_tail else 0, Hq, Hkv, D, has_self))
    ws.view(torch.uint8).fill_(0xff)                       # NaN wherever nothing was written
    tail = [x[:, S:].contiguous() for x in rows] if has_tail else [None, None]
    tail_len = (per[:, S, :1].contiguous() if has_tail else None)
    pc.pc_profile_begin()
    try:
        pc.pc_parallel_attn_fp8(q, *dev, *scales, lens[:, :S].contiguous() if S else None, *tail, tail_len, kt if has_tail else 0,
                                B, n_q, S, kt, Hq, Hkv, D, 50, 1.0e4, 0.0, out[1], lse[1], ws, seg_len_per_head=int(per_head),
                                k_self=slf[0], v_self=slf[1])
        torch.cuda.synchronize()
    finally:
        pc.pc_profile_end()
    names = [name for name, _ in pc.pc_profile_records()]
    assert names.count("fp8_images_kernel") == int(images) and names.count("fp8_rows_kernel") == int(S > 0 and not images)
    assert torch.equal(lse[0], lse[1])
    seen = torch.isfinite(lse[0]).transpose(1, 2)          # (a row without any key has the same output, zeros)
    assert torch.equal(out[0], out[1]) and torch.isfinite(out[1].float()[seen]).all()
