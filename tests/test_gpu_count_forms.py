"""VOI counts by a workgroup and by a wave per beamlet give the same matrix: a plan on its own
against the same plan in a batch (always a wave per beamlet), on both sides of the beamlet
count and of the row count that decide, and with rows of the block that hold no member."""
import numpy as np
import pytest

import fspb_inputs as fi

pytestmark = pytest.mark.gpu


def _water(n, s, hole=None):
    g = fi.water_phantom(n, s)
    if hole is not None:
        g.density[hole] = 0.0
    return g


def _cases():
    yield "many", _water((20, 20, 20), (0.5, 0.5, 0.5)), fi.coplanar_beams(1, (0.0, 0.0, 0.0), 100.0, 0.06, 0.06, 96, 86)
    yield "edge", _water((20, 20, 20), (0.5, 0.5, 0.5)), fi.coplanar_beams(2, (0.0, 0.0, 0.0), 100.0, 0.1, 0.1, 64, 64)
    yield "tall", _water((2, 740, 740), (0.3, 0.005, 0.005)), fi.coplanar_beams(4, (0.0, 0.0, 0.0), 100.0, 1.0, 1.0, 1, 1)
    yield "holes", _water((40, 37, 35), (0.3, 0.3, 0.3), np.s_[:, ::3, 5:30]), fi.coplanar_beams(3, (0.1, 0.2, 0.0), 100.0, 0.5, 0.5, 5, 4)
    yield "sparse", _water((40, 65, 41), (0.3, 0.3, 0.3), np.s_[4:, 3:, :]), fi.coplanar_beams(2, (0.1, 0.2, 0.0), 100.0, 0.5, 0.5, 5, 4)


@pytest.mark.parametrize("case", ["many", "edge", "tall", "holes", "sparse"])
def test_single_plan_equals_batch(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Batch, Plan
    g, beams = next((g, b) for name, g, b in _cases() if name == case)
    prob = fi.Problem(case, g, beams, fi.default_kernel(3))
    batch = Batch([Plan(prob, "cuda:0")])
    batch.run()
    torch.cuda.synchronize()
    assert batch.check() == 0
    want = batch.outputs()[0]
    plan = Plan(prob, "cuda:0")
    for _ in range(2):
        c = plan.compute()
        assert c.nnz == batch.nnz[0] and c.nnz > 0
        assert torch.equal(c.indptr, want.indptr) and torch.equal(c.indices, want.indices)
        assert torch.equal(c.values.view(torch.int32), want.values.view(torch.int32))
