"""A block of query rows over the 8-bit cache with 64 packed rows a wavefront (runs of 32 tiles and more, workgroups that fill
the CUs; test_wide_routes_host.py checks that every case gets it): edges of tiles, blocks and parts, lengths of zero, with NaN behind every length, against 64 bits."""
import pytest
import torch

import paper_2502_14317_amd as pc
from helpers import LSE_ATOL, O_ATOL, O_RTOL, fp8_from_rows

pytestmark = pytest.mark.gpu

# B, n_q, S, k_t (tail capacity too), H_q, H_kv, tail, self, per-head lengths
CASES = [
    (4, 125, 33, 97, 128, 16, True, True, True),            # 1000 packed rows: the last block of a workgroup is cut off; one part
    (4, 17, 70, 97, 128, 16, True, True, False),            # 136 rows, several parts
    (4, 130, 64, 64, 64, 64, False, False, False),          # one head a group, tiles full
    (4, 65, 70, 63, 192, 64, True, False, True),            # groups of 3; more segments than lanes, every tile masked
    (8, 512, 5, 900, 16, 16, False, True, False),           # the causal diagonal over 8 tiles, 4 of them a workgroup's own
]


@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_block_attention_over_images(case, zero):
    B, n_q, S, kt, Hq, Hkv, has_tail, has_self, per_head = case
    D, G, pos0 = 128, Hq // Hkv, 50
    print("wide images", case, zero, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B * 100 + kt)
    mk = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    q = mk(B, n_q, Hq, D)
    slf = [mk(B, n_q, Hkv, D) for _ in range(2)] if has_self else [None, None]
    T = S + int(has_tail)
    lens = torch.randint(0, kt + 1, (B, T, Hkv) if per_head else (B, T), generator=gen, device="cuda", dtype=torch.int32)
    lens.view(-1)[0] = kt
    if zero:
        lens[-1] = 0
    if has_tail and per_head:
        lens[:, S] = lens[:, S, :1]                        # a tail has one length for all heads
    per = lens if per_head else lens[:, :, None].expand(B, T, Hkv)
    dead = torch.arange(kt, device="cuda") >= per[..., None]
    rows, dev, scales = [], [], []
    for w in "kv":
        codes = (torch.randint(0, 0x48, (B, S, Hkv, kt, D), generator=gen, device="cuda")
                 + 0x80 * torch.randint(0, 2, (B, S, Hkv, kt, D), generator=gen, device="cuda")).to(torch.uint8)
        scale = torch.rand((B, S, Hkv), generator=gen, device="cuda") * 0.3 + 0.1
        wide = (codes.view(torch.float8_e4m3fn).float() * scale[..., None, None]).to(torch.bfloat16)
        wide = torch.cat([wide, mk(B, 1, Hkv, kt, D)], dim=1) if has_tail else wide
        wide[dead] = float("nan")
        codes[dead[:, :S]] = 0x7f                          # NaN
        rows.append(wide); scales.append(scale); dev.append(fp8_from_rows(w, codes))
    out = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, n_q, S, kt, kt if has_tail else 0, Hq, Hkv, D, has_self))
    ws.view(torch.uint8).fill_(0xff)                       # NaN wherever nothing was written
    tail = [x[:, S:].contiguous() for x in rows] if has_tail else [None, None]
    pc.pc_profile_begin()
    try:
        pc.pc_parallel_attn_fp8(q, *dev, *scales, lens[:, :S].contiguous(), *tail, per[:, S, :1].contiguous() if has_tail else None,
                                kt if has_tail else 0, B, n_q, S, kt, Hq, Hkv, D, pos0, 1.0e4, 0.0, out, lse, ws,
                                seg_len_per_head=int(per_head), k_self=slf[0], v_self=slf[1])
        torch.cuda.synchronize()
    finally:
        pc.pc_profile_end()
    assert [name for name, _ in pc.pc_profile_records()].count("fp8_images_kernel") == 1
    f64 = torch.float64
    theta = 1.0e4 ** (-2.0 * torch.arange(D // 2, dtype=f64, device="cuda") / D)
    ang = (pos0 + torch.arange(n_q, device="cuda", dtype=f64))[:, None] * theta
    x, y = q.to(f64)[..., :D // 2], q.to(f64)[..., D // 2:]
    c, s = ang.cos()[None, :, None], ang.sin()[None, :, None]
    qr = torch.cat([x * c - y * s, y * c + x * s], dim=-1)
    causal = torch.arange(n_q, device="cuda")[None, :] > torch.arange(n_q, device="cuda")[:, None]
    for b in range(B):
        for g in range(Hkv):
            ks, vs = (torch.cat([r[b, t, g, :int(per[b, t, g])].to(f64) for t in range(T)]
                                + ([z[b, :, g].to(f64)] if has_self else [])) for r, z in zip(rows, slf))
            for h in range(g * G, (g + 1) * G):
                if ks.shape[0] == 0:                       # no key at all: zeros and -inf
                    assert (out[b, :, h] == 0).all() and torch.isneginf(lse[b, h]).all()
                    continue
                sc = (qr[b, :, h] @ ks.t().contiguous()) / D ** 0.5
                if has_self:
                    sc[:, -n_q:].masked_fill_(causal, float("-inf"))
                ref, ref_lse = torch.softmax(sc, dim=1) @ vs, torch.logsumexp(sc, dim=1)
                err = (out[b, :, h].to(f64) - ref).abs() - O_RTOL * ref.abs()
                assert torch.isfinite(out[b, :, h].float()).all() and float(err.max()) <= O_ATOL, (b, h, float(err.max()))
                assert float((lse[b, h].to(f64) - ref_lse).abs().max()) <= LSE_ATOL, (b, h)
