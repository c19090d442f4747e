"""A workspace sized for a batch of query blocks serves every smaller one, with the results of a
workspace of its own."""
import pytest
import torch

import paper_2502_14317_amd as pc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_self", [False, True], ids=["segments", "with self"])
def test_batch_workspace_serves_smaller_batches_and_blocks(with_self):
    B, n_q, S, kt, Hq, Hkv, D = 8, 512, 8, 2048, 32, 8, 128
    g = torch.Generator(device="cuda").manual_seed(73)
    mk = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)
    q, kc, vc, ks, vs = mk(B, n_q, Hq, D), mk(B, S, Hkv, kt, D), mk(B, S, Hkv, kt, D), mk(B, n_q, Hkv, D), mk(B, n_q, Hkv, D)
    big = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(B, n_q, S, kt, Hq, Hkv, D, with_self))

    def run(b, n, ws):
        print("workspace reuse", with_self, b, n, flush=True)
        out = torch.full((b, n, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((b, Hq, n), float("nan"), dtype=torch.float32, device="cuda")
        self_k, self_v = (ks[:b, :n].contiguous(), vs[:b, :n].contiguous()) if with_self else (None, None)
        ws.fill_(0xFF)
        pc.pc_parallel_attn(q[:b, :n].contiguous(), kc[:b], vc[:b], None, self_k, self_v, b, n, S, kt, Hq, Hkv, D, 900,
                            1.0e4, 0.0, out, lse, ws)
        torch.cuda.synchronize()
        assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
        return out, lse

    for b in range(B, 0, -1):
        for n in (n_q, 224):
            own = pc.alloc_workspace(pc.pc_parallel_attn_workspace_bytes(b, n, S, kt, Hq, Hkv, D, with_self))
            got, ref = run(b, n, big), run(b, n, own)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
