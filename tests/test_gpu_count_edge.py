"""VOI counts on both sides of the beamlet count that decides between a workgroup and a wave per
beamlet: the same matrix as the plan's in a batch, which always counts by waves."""
import pytest

import fspb_inputs as fi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beams,nu,nv", [(2, 32, 32), (1, 3, 683), (1, 23, 89)])
def test_single_plan_equals_batch(beams, nu, nv):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Batch, Plan
    g = fi.water_phantom((24, 21, 22), (0.5, 0.5, 0.5))
    prob = fi.Problem("edge", g, fi.coplanar_beams(beams, (0.0, 0.0, 0.0), 100.0, 0.1, 0.02, nu, nv), fi.default_kernel(3))
    batch = Batch([Plan(prob, "cuda:0")])
    batch.run()
    torch.cuda.synchronize()
    want = batch.outputs()[0]
    c = Plan(prob, "cuda:0").compute()
    assert c.nnz > 0
    assert torch.equal(c.indptr, want.indptr) and torch.equal(c.indices, want.indices)
    assert torch.equal(c.values.view(torch.int32), want.values.view(torch.int32))
