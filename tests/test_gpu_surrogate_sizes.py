"""Gradient of the surrogate at the edges of its split: a workgroup takes 64
samples, a wave 16 of them; the reduction takes 32 partials per wave and 256 per
round (2048 and 16384 samples).

Against the oracle with the same BF16 roundings.  The tolerance is one BF16
rounding: where FP32 and FP64 round a hidden value differently, one operand
element changes by 2^-8 of itself, which no block's norm can follow by more.
"""
import numpy as np
import pytest

import fspb_inputs as fi

pytestmark = pytest.mark.gpu

BLOCKS = [(0, 256), (256, 320), (320, 4416), (4416, 4480), (4480, 4544), (4544, 4545)]


@pytest.mark.parametrize("n", [1, 16, 17, 65, 2048, 2049, 16384, 16385])
def test_gradient_at_split_edges(oracle_lib, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Surrogate
    rng = np.random.default_rng(n)
    p = fi.surrogate_init(4)
    p[256:320] = rng.normal(0, 0.2, 64)
    p[4416:4480] = rng.normal(0, 0.2, 64)
    sur = Surrogate(fi.default_kernel(3), p, max_batch=32768)
    x = rng.uniform(-1, 1, (n, 4)).astype(np.float32)
    t = rng.uniform(0, 1, n).astype(np.float32)
    xg, tg = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(t).to("cuda:0")
    g, loss = sur.gradient(xg, tg)
    ref_loss, ref = oracle_lib.mlp_loss_grad(p.astype(np.float64), x.astype(np.float64), t.astype(np.float64),
                                             bf16=True)
    g1 = g.cpu().numpy()
    assert abs(loss - ref_loss) <= 2.0 ** -7 * ref_loss
    for a, b in BLOCKS:
        r = np.linalg.norm(g1[a:b].astype(np.float64) - ref[a:b]) / np.linalg.norm(ref[a:b])
        assert r <= 2.0 ** -8, (n, a, r)
    g2, loss2 = sur.gradient(xg, tg)                       # a fixed order of summation
    assert loss2 == loss
    np.testing.assert_array_equal(g2.cpu().numpy(), g1)
