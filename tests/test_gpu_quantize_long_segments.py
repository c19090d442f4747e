"""8-bit codes of segments whose bytes pass 2^31: every unit is written, from the first to the last.  The rows
repeat every 4096, so the codes of all repetitions are those of a short segment with the same maxima, bit for bit."""
import pytest
import torch

import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import fp8_alloc

pytestmark = pytest.mark.gpu

PERIOD = 4096


@pytest.mark.parametrize("with_max", [False, True])
@pytest.mark.parametrize("k_t,D", [(1 << 24, 128), ((1 << 25) + 32, 64), ((1 << 24) + PERIOD, 64)])
def test_every_unit_of_a_long_segment(k_t, D, with_max):
    print("quantize long", k_t, D, with_max, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(k_t % 1000 + D)
    short = [torch.randn((1, 1, 1, PERIOD, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2)]
    amax = [x.abs().amax(dim=(3, 4)).float() for x in short]

    def run(x, rows):
        c = [fp8_alloc(1, 1, 1, rows, D).fill_(0x55) for _ in range(2)]
        s = [torch.empty((1, 1, 1), device="cuda") for _ in range(2)]
        if with_max:
            pc.pc_kv_quantize_fp8_amax(*x, *amax, None, 1, 1, rows, 1, D, *c, *s)
        else:
            pc.pc_kv_quantize_fp8(*x, None, 1, 1, rows, 1, D, *c, *s)
        torch.cuda.synchronize()
        return c, s

    want, want_s = run(short, PERIOD)
    whole, rest = k_t // PERIOD, k_t % PERIOD
    got, got_s = run([torch.cat([x.expand(1, 1, whole, PERIOD, D).reshape(1, 1, 1, -1, D), x[:, :, :, :rest]], dim=3) for x in short], k_t)
    for w, g in zip(want + want_s, got + got_s):
        w, g = w.view(-1), g.view(-1)
        if w.numel() == 1:
            assert torch.equal(w, g)
            continue
        n = w.numel()
        for i in range(0, whole, 512):
            part = g[i * n:min(i + 512, whole) * n].view(-1, n)
            assert (part == w).all(), i
        assert torch.equal(g[whole * n:], w[:rest * D])
