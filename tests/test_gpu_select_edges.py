"""Token selection at the edges of its size classes and of its binning: exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_14317_amd as pc

pytestmark = pytest.mark.gpu


def _scores(kind, n, r):
    x = r.standard_normal(n).astype(np.float32)
    if kind == "equal":
        x[:] = 0.25
    elif kind == "two values one bit apart":
        x[:] = np.float32(1.0)
        x[r.random(n) < 0.5] = np.nextafter(np.float32(1.0), np.float32(2.0))
    elif kind == "whole range":                  # every exponent, both signs, both zeros and infinities, NaN
        x = r.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32).view(np.float32).copy()
        x[: min(n, 6)] = [np.inf, -np.inf, 0.0, -0.0, np.nan, np.finfo(np.float32).max][: min(n, 6)]
    elif kind == "one far above":
        x *= np.float32(1e-3)
        x[n // 2] = np.float32(1e30)
    return x


@pytest.mark.parametrize("kind", ["normal", "equal", "two values one bit apart", "whole range", "one far above"])
@pytest.mark.parametrize("n", [1, 63, 512, 513, 1024, 1025, 2049, 4096, 4097, 8193, 16385, 32768])
def test_select_tokens_edges(n, kind):
    print("select", n, kind, flush=True)
    r = np.random.default_rng([65, n, len(kind)])
    score = np.stack([_scores(kind, n, r) for _ in range(2)])
    dev = torch.from_numpy(score).cuda()
    for k in sorted({1, (n + 1) // 2, n}):
        out = torch.full((1, 2, k), -7, dtype=torch.int32, device="cuda")
        pc.pc_select_tokens_topk(dev, None, 1, 2, n, k, out)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out[0].cpu().numpy(), oracle.select_tokens(score, k))
