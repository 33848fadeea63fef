"""Density masks of grid rows at the edges of the mask pass's steps (64 voxels, four of them
together): the matrix against the FP64 oracle, members and values, with voxels left out."""
import os
import sys

import numpy as np
import pytest

import fspb_inputs as fi

sys.path.insert(0, os.path.dirname(__file__))
from parity import compare_plan  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [63, 64, 65, 255, 256, 257, 321, 513])
def test_masked_rows_against_the_oracle(oracle_lib, nx):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Plan
    g = fi.water_phantom((nx, 9, 40), (20.0 / nx, 0.7, 0.45))
    rng = np.random.default_rng(nx)
    g.density[rng.uniform(size=g.density.shape) < 0.1] = 0.0
    g.density[:, 2, -1] = 1.0
    g.density[:, 3, :] = 0.0
    prob = fi.Problem("rows", g, fi.coplanar_beams(2, (0.1, 0.0, 0.05), 100.0, 1.0, 1.0, 2, 2), fi.default_kernel(3))
    plan = Plan(prob, "cuda:0")
    r = compare_plan(oracle_lib.OraclePlan(prob), plan.compute())
    assert r["rows"] == 8 and r["n"] > 0
