"""Calls whose time follows from another call's of the same work: a shape must not cost a multiple of it."""
import pytest

pytestmark = pytest.mark.gpu


def _us(call, n=100):
    import torch
    call()
    best = float("inf")
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


def _rows(rows, length, n):
    """Rows of consecutive columns, their starts spread evenly over n columns."""
    import torch
    from paper_0908_4417_amd import CSR
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    start = torch.linspace(0, n - length, rows, device="cuda").long()[:, None]
    idx = (start + torch.arange(length, device="cuda")).int().reshape(-1)
    ip = torch.arange(rows + 1, dtype=torch.int64, device="cuda") * length
    return CSR(ip, idx, torch.rand(rows * length, device="cuda"), n)


def test_gradient_of_many_short_rows():
    """9000 rows of 50 entries take what 2000 of 225 take (7.6 and 7.5 us; 20.5 with 1024 threads a row)."""
    import torch
    n = 100000
    many, few = _rows(9000, 50, n), _rows(2000, 225, n)
    r = torch.rand(n, device="cuda")
    assert _us(lambda: many.gradient(r)) < 1.8 * _us(lambda: few.gradient(r))


def test_dose_of_rows_of_a_thousand_entries():
    """2000 rows of 1000 entries: 13.6 us, where 2000 rows of 100 take 10 (29.8 in shares too short for windows)."""
    import torch
    n = 100000
    rows, short = _rows(2000, 1000, n), _rows(2000, 100, n)
    w = torch.rand(2000, device="cuda")
    assert _us(lambda: rows.dose(w)) < 2.0 * _us(lambda: short.dose(w))


def test_voxel_dose_of_short_rows():
    """Voxel rows of three entries: 8100 beamlets take what 100 take (7.6 us; 13.5 with w copied to LDS)."""
    import torch
    from paper_0908_4417_amd import VoxelCSR
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 64 ** 3
    ip = torch.arange(n + 1, dtype=torch.int64, device="cuda") * 3
    val = torch.rand(3 * n, device="cuda")
    t = {}
    for beamlets in (100, 8100):
        idx = (torch.arange(3 * n, device="cuda") * beamlets // (3 * n)).int()
        T, w = VoxelCSR(ip, idx, val, beamlets), torch.rand(beamlets, device="cuda")
        t[beamlets] = _us(lambda: T.dose(w))
    assert t[8100] < 1.35 * t[100]


def test_transpose_of_rows_without_gaps():
    """18 runs to a bucket of 576 entries (0.39 ms) take less than twice their half (0.26 ms; 0.57 with four waves a bucket)."""
    n = 2000000
    D, half = _rows(9000, 4000, n), _rows(4500, 4000, n)
    assert _us(D.transpose, 10) < 1.8 * _us(half.transpose, 10)


def test_counts_of_many_beamlets():
    """Mask, counts and tables: 8100 beamlets take less than 8370 (125 and 129 us; 156 with a workgroup a beamlet)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import fspb_inputs as fi
    from paper_0908_4417_amd import Plan
    g = fi.slab_phantom(3, n=(128, 128, 128), spacing=(0.25, 0.25, 0.25))
    t = {}
    for nv in (30, 31):
        beams = fi.coplanar_beams(9, (0.13, -0.07, 0.05), 100.0, 0.5, 0.5, 30, nv)
        plan = Plan(fi.Problem("counts", g, beams, fi.default_kernel(3)), "cuda:0")
        t[nv] = _us(plan.raytrace, 30)
    assert t[30] < 1.08 * t[31]


def test_batch_of_both_erf_forms():
    """Six plans with the compact erf table and 46 KB of LDS beside six with the mirrored one and 25 take less than the two
    batches apart (2.69 ms and 1.95 + 0.90): room for the mirrored table in both leaves two workgroups per CU instead of
    three (3.57 ms)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import fspb_inputs as fi
    from paper_0908_4417_amd import Batch, Plan
    thin = fi.water_phantom((96, 96, 100), (0.4, 0.4, 0.023))
    body = fi.pelvis_phantom(3)
    iso = (0.13, -0.07, 0.05)
    plans = lambda form: [Plan(fi.Problem("thin", thin, fi.coplanar_beams(3, iso, 100.0, 0.5, 0.5, 8, 2, start_deg=5.0),
                                          fi.default_kernel(k)), "cuda:0", erf_form=form) for k in range(6)]
    other = lambda form: [Plan(fi.Problem("body", body, fi.coplanar_beams(2, iso, 100.0, 0.25, 0.25, 24, 24, start_deg=5.0),
                                          fi.default_kernel(k)), "cuda:0", erf_form=form) for k in range(6)]
    t = []
    for ps in (plans("compact") + other("mirrored"), other("mirrored"), plans("compact")):
        batch = Batch(ps)
        batch.set_config(4, 4, 0)
        t.append(_us(batch.run, 10))
    assert t[0] < 1.1 * (t[1] + t[2])
