"""Few query rows and decoding steps with NaN in every cache row behind the lengths (and behind the row that a step
stores): rows behind a segment's end are asked for with the block that holds its last ones, and must arrive as zeros.
Lengths on either side of the 16- and 32-key edges, one a segment and one a head, against one softmax in fp32."""
import pytest
import torch

import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc
from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close

pytestmark = pytest.mark.gpu

LENS = [1, 15, 16, 17, 31, 33, 32, 47, 48, 49, 63, 65, 0, 64]


def _reference(q, keys, vals, dead):
    """q [B, n_q, Hq, D], keys, vals [B, S, Hkv, k_t, D], dead [B, S, Hkv, k_t]: one softmax over the live rows."""
    B, n_q, Hq, D = q.shape
    Hkv = keys.shape[2]
    flat = lambda x: x.transpose(1, 2).reshape(B, Hkv, 1, 1, -1, *x.shape[4:])
    live = ~flat(dead)
    k, v = (torch.where(live[..., None], flat(x.float()), 0.0) for x in (keys, vals))
    s = (q.float().transpose(1, 2).reshape(B, Hkv, Hq // Hkv, n_q, 1, D) * k).sum(-1) / D ** 0.5
    s = torch.where(live, s, float("-inf"))
    o = (torch.softmax(s, -1)[..., None] * v).sum(-2)
    return o.reshape(B, Hq, n_q, D).transpose(1, 2), torch.logsumexp(s, -1).reshape(B, Hq, n_q)


def _check(out, lse, ref):
    assert_close(out.float().cpu().numpy(), ref[0].cpu().numpy(), O_ATOL, O_RTOL, "out")
    assert_close(lse.cpu().numpy(), ref[1].cpu().numpy(), LSE_ATOL, 1e-3, "lse")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("per_head", [False, True])
@pytest.mark.parametrize("call", ["attention", "step", "step 8 bit"])
@pytest.mark.parametrize("shift", range(7))
def test_rows_behind_the_lengths(call, per_head, D, shift):
    B, S, Hq, Hkv, kt = 2, 4, 6, 2, 70
    n_q = 3 if call == "attention" else 1
    print("NaN rows", call, per_head, D, shift, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(100 * D + shift)
    mk = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    q, k, v = mk(B, n_q, Hq, D), mk(B, 1, Hkv, D), mk(B, 1, Hkv, D)
    n = B * S * (Hkv if per_head else 1)
    lens = torch.tensor([LENS[(2 * i + shift) % len(LENS)] for i in range(n)], dtype=torch.int32, device="cuda")
    lens = lens.view((B, S, Hkv) if per_head else (B, S))
    if call == "step 8 bit" and per_head:
        lens[:, -1] = lens[:, -1, :1]                      # the tail has one length for all heads
    per = lens if per_head else lens[:, :, None].expand(B, S, Hkv)
    row = torch.arange(kt, device="cuda")
    kc, vc = mk(B, S, Hkv, kt, D), mk(B, S, Hkv, kt, D)
    dead = row >= per[..., None]
    kc[dead] = float("nan"); vc[dead] = float("nan")
    out = torch.full((B, n_q, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, n_q), float("nan"), device="cuda")
    if call == "attention":
        ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, n_q, S, kt, Hq, Hkv, D, False))
        ws.view(torch.uint8).fill_(0xff)
        pc.pc_parallel_attn(q, kc, vc, lens, None, None, B, n_q, S, kt, Hq, Hkv, D, -1, 1.0e4, 0.0, out, lse, ws, int(per_head))
        torch.cuda.synchronize()
        return _check(out, lse, _reference(q, kc, vc, dead))
    # the step: the new row behind the last segment's, everything behind it NaN still
    new = row == per[:, -1, :, None]
    after = dead.clone()
    after[:, -1] &= ~new
    keys, vals = kc.clone(), vc.clone()
    keys[:, -1] = torch.where(new[..., None], k.transpose(1, 2), keys[:, -1])
    vals[:, -1] = torch.where(new[..., None], v.transpose(1, 2), vals[:, -1])
    if call == "step":
        ws = pc.alloc_workspace(pc.pc_decode_step_workspace_bytes(B, S, kt, Hq, Hkv, D))
        ws.view(torch.uint8).fill_(0xff)
        pc.pc_decode_step(q, k, v, B, S, kt, Hq, Hkv, D, -1, 1.0e4, 0.0, kc, vc, lens, out, lse, ws, int(per_head))
        torch.cuda.synchronize()
        assert torch.equal(kc.view(torch.int16), keys.view(torch.int16)) and torch.equal(vc.view(torch.int16), vals.view(torch.int16))
        return _check(out, lse, _reference(q, keys, vals, after))
    codes = [fp8_alloc(B, S - 1, Hkv, kt, D) for _ in range(2)]
    scales = [torch.empty((B, S - 1, Hkv), device="cuda") for _ in range(2)]
    sl = lens[:, :-1].contiguous()
    pc.pc_kv_quantize_fp8(kc[:, :-1].contiguous(), vc[:, :-1].contiguous(), sl, B, S - 1, kt, Hkv, D, *codes, *scales, int(per_head))
    tail = [x[:, -1:].contiguous() for x in (kc, vc)]
    tail_len = per[:, -1, :1].to(torch.int32).contiguous()
    ws = pc.alloc_workspace(pc.pc_decode_step_fp8_workspace_bytes(B, S - 1, kt, kt, Hq, Hkv, D))
    ws.view(torch.uint8).fill_(0xff)
    pc.pc_decode_step_fp8(q, k, v, *codes, *scales, sl, *tail, tail_len, kt, B, S - 1, kt, Hq, Hkv, D, -1, 1.0e4, 0.0, out, lse, ws,
                          int(per_head))
    torch.cuda.synchronize()
    assert torch.equal(tail[0][:, 0].view(torch.int16), keys[:, -1].view(torch.int16))
    assert torch.equal(tail[1][:, 0].view(torch.int16), vals[:, -1].view(torch.int16))
    for x, s in zip((keys, vals), scales):
        sc = s[..., None, None]
        x[:, :-1] = ((x[:, :-1].float() / sc).to(torch.float8_e4m3fn).float() * sc).to(torch.bfloat16)
    _check(out, lse, _reference(q, keys, vals, after))
