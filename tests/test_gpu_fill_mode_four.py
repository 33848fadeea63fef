"""The fill with one reciprocal for all terms runs where the terms' sigmas are multiples of the first's,
and only there: a kernel whose FP32 parameters are the same but whose slopes miss the ratio by 1e-10
takes a reciprocal per term, so some entries differ in the last bits; both follow the oracle."""
import os
import sys

import numpy as np
import pytest

import fspb_inputs as fi

sys.path.insert(0, os.path.dirname(__file__))
from parity import compare_plan  # noqa: E402

pytestmark = pytest.mark.gpu

LAWS = {   # sigma0 and slope of each term
    "two": ([0.2, 0.4], [0.4 / 30, 0.8 / 30]),
    "three": ([0.2, 0.3, 0.7], [0.01, 0.015, 0.035]),
}


def _problem(law, miss):
    k = fi.default_kernel(71)
    k.sigma0, slope = list(LAWS[law][0]), LAWS[law][1]
    k.sigma_slope = [s * (1.0 + miss * i) for i, s in enumerate(slope)]
    n = len(slope)
    k.weight, k.width_scale = [0.9, 0.08, 0.02][:n], [1.0] * n
    g = fi.slab_phantom(71, n=(44, 40, 24), spacing=(0.5, 0.45, 0.55), lung_side=(2, 6), bone_side=(1, 3))
    return fi.Problem(law, g, fi.coplanar_beams(2, (0.13, -0.07, 0.05), 100.0, 0.6, 0.6, 3, 2, start_deg=7.0), k)


@pytest.mark.parametrize("law", LAWS)
def test_the_mode_follows_the_sigma_law(law, oracle_lib):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Plan
    values = []
    for miss in (0.0, 1e-14, 1e-10):     # a ratio, one within rounding, none
        prob = _problem(law, miss)
        assert np.array_equal(np.float32(prob.kernel.sigma_slope), np.float32(_problem(law, 0.0).kernel.sigma_slope))
        plan = Plan(prob, "cuda:0", erf_form="mirrored")
        assert plan.desc.fill_erf_mode == 3
        csr = plan.compute()
        compare_plan(oracle_lib.OraclePlan(prob), csr)
        values.append(csr.values.cpu().numpy().view(np.int32))
    assert np.array_equal(values[0], values[1])
    assert np.any(values[0] != values[2])
