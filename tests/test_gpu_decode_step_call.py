"""pc_decode_step and pc_decode_step_fp8 at their edges against pc_kv_append followed by the attention call: an
empty tail, a full one (the token is dropped), rows that arrive rotated, a length per head, the query
rotated in front (more than 512 workgroups), more than 16 heads a group (the tile path).

Cache rows and lengths are the same bits.  Outputs differ by the new key's probability, which the two
calls round to bf16 and the step does not: at most 2^-9 of |v| - |out|, half of a bf16 step of the
values, so the tolerance of the outputs covers it (values of standard deviation 1)."""
import pytest
import torch

import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc
from helpers import LSE_ATOL, O_ATOL, O_RTOL, assert_close

pytestmark = pytest.mark.gpu

# B, S (with the tail), k_t, H_q, H_kv, D, tail length, per-head lengths, pos
CASES = [
    (2, 3, 70, 8, 2, 128, 0, 0, 5),
    (1, 2, 64, 4, 1, 64, 64, 0, 900),        # full: dropped
    (3, 2, 33, 6, 6, 128, 32, 1, 0),         # the last row
    (2, 4, 40, 12, 4, 64, 7, 1, -1),         # rows arrive rotated
    (1, 1, 100, 16, 1, 128, 31, 0, 70000),   # the tail alone; 16 columns
    (513, 2, 32, 2, 1, 64, 3, 0, 17),        # rotated in front
    (1, 2, 96, 40, 2, 64, 20, 0, 33),        # 20 heads a group
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("eight_bit", [False, True], ids=["16bit", "8bit"])
def test_step_is_append_then_attention(case, eight_bit):
    B, S, kt, Hq, Hkv, D, n, per_head, pos = case
    print("decode step", case, eight_bit, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B * 1000 + kt)
    mk = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    q, k, v = mk(B, 1, Hq, D), mk(B, 1, Hkv, D), mk(B, 1, Hkv, D)
    S8 = S - 1
    lens = torch.randint(1, kt + 1, (B, S, Hkv) if per_head else (B, S), generator=gen, device="cuda", dtype=torch.int32)
    lens[:, S - 1] = n
    if per_head:
        lens[:, S - 1, 1:] = max(n - 1, 0)                 # the heads' tails differ
    both = []
    kc, vc = mk(B, S, Hkv, kt, D), mk(B, S, Hkv, kt, D)
    for step in (False, True):
        out = torch.full((B, 1, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((B, Hq, 1), float("nan"), dtype=torch.float32, device="cuda")
        if not eight_bit:
            kk, vv, sl = kc.clone(), vc.clone(), lens.clone()
            if step:
                ws = pc.alloc_workspace(pc.pc_decode_step_workspace_bytes(B, S, kt, Hq, Hkv, D))
                pc.pc_decode_step(q, k, v, B, S, kt, Hq, Hkv, D, pos, 1.0e4, 0.0, kk, vv, sl, out, lse, ws, per_head)
            else:
                ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, 1, S, kt, Hq, Hkv, D, False))
                pc.pc_kv_append(k, v, B, 1, S, S - 1, kt, Hkv, D, pos, 1.0e4, kk, vv, sl, per_head)
                pc.pc_parallel_attn(q, kk, vv, sl, None, None, B, 1, S, kt, Hq, Hkv, D, pos, 1.0e4, 0.0, out, lse, ws, per_head)
        else:
            k8, v8 = fp8_alloc(B, max(S8, 1), Hkv, kt, D), fp8_alloc(B, max(S8, 1), Hkv, kt, D)
            ks = torch.ones((B, max(S8, 1), Hkv), dtype=torch.float32, device="cuda")
            vs = torch.ones_like(ks)
            sl8 = lens[:, :S8].contiguous()
            if S8:
                pc.pc_kv_quantize_fp8(kc[:, :S8].contiguous(), vc[:, :S8].contiguous(), sl8, B, S8, kt, Hkv, D, k8, v8, ks, vs, per_head)
            kk, vv = kc[:, S8:].clone(), vc[:, S8:].clone()
            sl = torch.full((B, 1), n, dtype=torch.int32, device="cuda")
            tail = (kk, vv, sl, kt)
            if step:
                ws = pc.alloc_workspace(pc.pc_decode_step_fp8_workspace_bytes(B, S8, kt, kt, Hq, Hkv, D))
                pc.pc_decode_step_fp8(q, k, v, k8, v8, ks, vs, sl8, *tail, B, S8, kt, Hq, Hkv, D, pos, 1.0e4, 0.0, out, lse, ws, per_head)
            else:
                ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, 1, S8, kt, kt, Hq, Hkv, D))
                pc.pc_kv_append(k, v, B, 1, 1, 0, kt, Hkv, D, pos, 1.0e4, kk, vv, sl)
                pc.pc_parallel_attn_fp8(q, k8, v8, ks, vs, sl8, *tail, B, 1, S8, kt, Hq, Hkv, D, pos, 1.0e4, 0.0, out, lse, ws, per_head)
        torch.cuda.synchronize()
        both.append((kk, vv, sl, out, lse))
    (k0, v0, s0, o0, l0), (k1, v1, s1, o1, l1) = both
    assert torch.equal(k0, k1) and torch.equal(v0, v1) and torch.equal(s0, s1)
    assert_close(o1.double().cpu().numpy(), o0.double().cpu().numpy(), O_ATOL, O_RTOL, "out")
    assert_close(l1.double().cpu().numpy(), l0.double().cpu().numpy(), LSE_ATOL, 1e-3, "lse")


@pytest.mark.parametrize("B,S,kt,cap", [(33, 4, 256, 96), (72, 2, 700, 40), (2, 8, 2048, 512), (1, 1, 33, 31)])
def test_parts_of_either_rule_attend_to_the_same_keys(B, S, kt, cap):
    """Shapes where the split cuts into fewer parts than the workspace has room for: the 8-bit segments and
    their tail, and both precisions of the same cache, against one softmax in fp32."""
    Hq, Hkv, D, pos = 8, 4, 64, 12
    print("parts", B, S, kt, cap, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B + kt)
    mk = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    q, kc, vc = mk(B, 1, Hq, D), mk(B, S, Hkv, kt, D), mk(B, S, Hkv, kt, D)
    k_tail, v_tail = mk(B, 1, Hkv, cap, D), mk(B, 1, Hkv, cap, D)
    n_tail = torch.full((B, 1), cap, dtype=torch.int32, device="cuda")

    def reference(keys, vals):                             # [B, Hkv, n, D] fp32; q arrives rotated
        s = (q.float().view(B, Hkv, Hq // Hkv, 1, D) * keys[:, :, None]).sum(-1) / D ** 0.5
        return (torch.softmax(s, -1)[..., None] * vals[:, :, None]).sum(-2).reshape(B, 1, Hq, D), torch.logsumexp(s, -1).reshape(B, Hq, 1)

    flat = lambda x: x.float().transpose(1, 2).reshape(B, Hkv, -1, D)
    out = torch.full((B, 1, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, 1), float("nan"), dtype=torch.float32, device="cuda")
    ws = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, 1, S, kt, Hq, Hkv, D, False))
    pc.pc_parallel_attn(q, kc, vc, None, None, None, B, 1, S, kt, Hq, Hkv, D, -1, 1.0e4, 0.0, out, lse, ws)
    ro, rl = reference(flat(kc), flat(vc))
    assert_close(out.float().cpu().numpy(), ro.cpu().numpy(), O_ATOL, O_RTOL, "out")
    assert_close(lse.cpu().numpy(), rl.cpu().numpy(), LSE_ATOL, 1e-3, "lse")
    k8, v8 = fp8_alloc(B, S, Hkv, kt, D), fp8_alloc(B, S, Hkv, kt, D)
    ks = torch.empty((B, S, Hkv), dtype=torch.float32, device="cuda")
    vs = torch.empty_like(ks)
    pc.pc_kv_quantize_fp8(kc, vc, None, B, S, kt, Hkv, D, k8, v8, ks, vs)
    ws = pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, 1, S, kt, cap, Hq, Hkv, D))
    pc.pc_parallel_attn_fp8(q, k8, v8, ks, vs, None, k_tail, v_tail, n_tail, cap, B, 1, S, kt, Hq, Hkv, D, -1, 1.0e4,
                            0.0, out, lse, ws)
    deq = lambda x, sc: ((x.float() / sc[..., None, None]).to(torch.float8_e4m3fn).float() * sc[..., None, None])
    cat = lambda x, sc, t: torch.cat([flat(deq(x, sc)), t[:, 0].float()], dim=2)
    ro, rl = reference(cat(kc, ks, k_tail), cat(vc, vs, v_tail))
    assert_close(out.float().cpu().numpy(), ro.cpu().numpy(), O_ATOL, O_RTOL, "out, 8 bit")
    assert_close(lse.cpu().numpy(), rl.cpu().numpy(), LSE_ATOL, 1e-3, "lse, 8 bit")
