"""The fill's sigma laws (fixed multiples of the first term's, or not; one to four terms) and its
workgroups per beamlet (one beamlet to many, few tiles to many), each against the oracle, and the
batch's fill bit-identical to the plan's own."""
import os
import sys

import numpy as np
import pytest

import fspb_inputs as fi

sys.path.insert(0, os.path.dirname(__file__))
from parity import compare_plan  # noqa: E402

pytestmark = pytest.mark.gpu

KERNELS = {   # weight, sigma0, slope, width scale
    "one": ([1.0], [0.25], [0.012], [1.0]),
    "twofold": ([0.9, 0.1], [0.2, 0.4], [0.4 / 30, 0.8 / 30], [1.0, 1.0]),
    "narrower_second": ([0.7, 0.3], [0.5, 0.25], [0.02, 0.01], [1.0, 1.1]),
    "threefold": ([0.8, 0.15, 0.05], [0.2, 0.3, 0.7], [0.01, 0.015, 0.035], [1.0, 0.9, 1.2]),
    "constant": ([0.6, 0.2, 0.1, 0.1], [0.3, 0.4, 0.5, 0.6], [0.0] * 4, [1.0] * 4),
    "apart": ([0.9, 0.1], [0.2, 0.4], [0.4 / 30, 0.1 / 30], [1.0, 1.0]),
}


def _problem(kernel, n, spacing, nb, nu, nv, phantom="slab"):
    k = fi.default_kernel(61)
    k.weight, k.sigma0, k.sigma_slope, k.width_scale = (list(x) for x in KERNELS[kernel])
    if phantom == "slab":
        g = fi.slab_phantom(61, n=n, spacing=spacing, lung_side=(2, 6), bone_side=(1, 3))
    else:
        g = fi.pelvis_phantom(61, n=n, spacing=spacing)
    return fi.Problem(kernel, g, fi.coplanar_beams(nb, (0.13, -0.07, 0.05), 100.0, 0.6, 0.6, nu, nv, start_deg=7.0), k)


CASES = [(k, (41, 37, 23), (0.5, 0.45, 0.55), 3, 3, 2, "slab") for k in KERNELS] + [
    ("twofold", (9, 7, 1), (0.5, 0.5, 0.5), 1, 1, 1, "slab"),
    ("twofold", (150, 160, 40), (0.2, 0.2, 0.3), 1, 1, 1, "slab"),
    ("twofold", (90, 96, 30), (0.5, 0.4, 0.6), 2, 2, 3, "pelvis"),
    ("twofold", (20, 20, 18), (1.0, 1.0, 1.0), 9, 24, 24, "slab"),   # every axis meets the grid
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1][0]}x{c[1][1]}x{c[1][2]}-{c[3] * c[4] * c[5]}")
def test_fill_against_the_oracle(case, oracle_lib):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Batch, Plan
    prob = _problem(*case)
    plan = Plan(prob, "cuda:0")
    csr = plan.compute()
    compare_plan(oracle_lib.OraclePlan(prob), csr)
    batch = Batch([Plan(prob, "cuda:0"), Plan(_problem("threefold", (20, 20, 10), (1.0, 1.0, 1.0), 1, 2, 2), "cuda:0")])
    batch.run()
    got = batch.outputs()[0]
    torch.cuda.synchronize()
    assert torch.equal(got.indices, csr.indices)
    assert torch.equal(got.values.view(torch.int32), csr.values.view(torch.int32))
