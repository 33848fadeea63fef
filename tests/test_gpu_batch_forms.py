"""Batches of plans with the compact erf table, with the mirrored one and with both, up to the LDS that
a plan may have: each plan's matrix has the bits of the plan's own, in every launch shape."""
import pytest

import fspb_inputs as fi

pytestmark = pytest.mark.gpu


def _problem(seed, sz):
    """A water phantom whose depth tables are as long as its slices are thin."""
    g = fi.water_phantom((36, 33, 9), (0.5, 0.45, sz), rho=1.0 + 0.01 * seed)
    return fi.Problem("thin", g, fi.coplanar_beams(2, (0.1, -0.1, 0.0), 100.0, 0.5, 0.4, 3, 1, start_deg=5.0 + seed),
                      fi.default_kernel(seed))


FORMS = {   # erf table form and slice spacing of each plan
    "compact": [("compact", 0.05), ("compact", 0.3), ("compact", 0.2)],
    "mirrored": [("mirrored", 0.3), ("mirrored", 0.05), ("mirrored", 0.2)],
    "both": [("compact", 0.02), ("mirrored", 0.3), ("compact", 0.1), ("mirrored", 0.04)],
    "largest": [("compact", 0.00455), ("mirrored", 0.5)],
    "largest_alone": [("compact", 0.00455)],
}


@pytest.mark.parametrize("form", FORMS)
def test_batch_has_the_plans_bits(form):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import Batch, Plan
    make = lambda: [Plan(_problem(k, sz), "cuda:0", erf_form=f) for k, (f, sz) in enumerate(FORMS[form])]
    alone, together = make(), make()
    if form.startswith("largest"):
        assert 63 * 1024 < alone[0].desc.fill_lds_bytes <= 64 * 1024
    want = [p.compute() for p in alone]
    batch = Batch(together)
    for shape in [(4, 4, 0, 64, 1), (2, 8, 1, 128, 2), (8, 2, 0, 256, 4)]:
        batch.set_config(*shape)
        for _ in range(2):
            for out in batch.outputs():
                out.values.zero_()
                out.indices.zero_()
            batch.run()
            torch.cuda.synchronize()
            assert batch.check() == 0
            for out, w in zip(batch.outputs(), want):
                assert w.nnz > 0 and torch.equal(out.indptr, w.indptr) and torch.equal(out.indices, w.indices)
                assert torch.equal(out.values.view(torch.int32), w.values.view(torch.int32))
