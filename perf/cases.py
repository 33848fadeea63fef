"""Performance cases of the FSPB dose engine: what a treatment-planning program has it do.

A planning program computes the dose-deposition matrix D of a plan (again whenever the density
changes), then iterates on the beamlet weights with Eq. 1 and its adjoint, on the beamlet rows or,
for repeated products, on the voxel rows after one transpose.  Many small plans are computed as a
batch, and a learned kernel can stand in for the analytic one.  Geometry belongs to the case;
densities, depth dose, weights, residuals and network parameters are drawn from the seed.

``exact`` evaluates the same quantities in plain FP64 torch: sorted Siddon crossings, a dense VOI
test of every voxel, ``erf`` itself.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_0908_4417_amd import Batch, Plan, Surrogate

DEVICE = "cuda:0"
F64 = torch.float64
SAD = 100.0
ISO = (0.13, -0.07, 0.05)      # off the voxel planes, as a clinical isocentre is
PDD_STEP = 0.1
HIDDEN = 64
D_MAX, UV_MAX = 30.0, 3.0      # the surrogate's training box

# sizes of the repository's own workloads
WATER = dict(phantom="water", nx=64, ny=64, nz=64, sx=0.4, sy=0.4, sz=0.4,
             beams=1, start=0.0, nu=10, nv=10, side=1.0, cutoff=3.0)
SLAB = dict(phantom="slab", nx=128, ny=128, nz=128, sx=0.25, sy=0.25, sz=0.25,
            beams=9, start=0.0, nu=30, nv=30, side=0.5, cutoff=3.0)
PELVIS = dict(phantom="body", nx=256, ny=256, nz=100, sx=0.2, sy=0.2, sz=0.3,
              beams=9, start=0.0, nu=24, nv=24, side=0.25, cutoff=3.0)


def listed():
    return [
        # one open field on a small water phantom: a dose check, all latency
        dict(name="plan_water", kind="plan", **WATER),
        # nine-field plan on a heterogeneous 128^3 grid: the benchmark workload
        dict(name="plan_slab", kind="plan", **SLAB),
        # nine-field prostate-sized plan with narrow beamlets and air around the body
        dict(name="plan_pelvis", kind="plan", **PELVIS),
        # fitted beam data (depth-tabulated three-term kernel, off-axis A) with the trilinear-sampled
        # depth table, on a ragged cropped grid
        dict(name="plan_tables", kind="tables", phantom="slab", nx=117, ny=93, nz=75, sx=0.3, sy=0.3, sz=0.3,
             beams=5, start=11.0, nu=13, nv=11, side=0.5, cutoff=3.0),
        # a clinic's queue of uneven plans computed by one graph launch
        dict(name="batch_uneven", kind="batch", plans=8, mix=3, nnz=4.0e8),
        # one optimiser iteration on a small D: dose, residual, gradient; launches count
        dict(name="iterate_water", kind="iterate", **WATER),
        # Eq. 1 on the beamlet rows of a full plan
        dict(name="dose_slab", kind="dose", **SLAB),
        # its adjoint
        dict(name="gradient_slab", kind="gradient", **SLAB),
        # the voxel-row form, made once per plan before an optimisation
        dict(name="transpose_slab", kind="transpose", **SLAB),
        # Eq. 1 on the voxel rows, the reproducible product of an optimisation loop
        dict(name="voxel_dose_slab", kind="voxel_dose", **SLAB),
        # the learned kernel inside the fill, on the patient-sized plan
        dict(name="surrogate_pelvis", kind="surrogate", **PELVIS),
        # one training gradient of the learned kernel at its training batch
        dict(name="surrogate_gradient", kind="mlp_gradient", samples=16384),
    ]


def _est_nnz(c):
    """Entries of D by VOI volume (an upper estimate)."""
    depth = min(c["nx"] * c["sx"], c["ny"] * c["sy"])
    ext = [2 * c["cutoff"], min(2 * c["cutoff"], c["nz"] * c["sz"])]
    return c["beams"] * c["nu"] * c["nv"] * ext[0] * ext[1] * depth / (c["sx"] * c["sy"] * c["sz"])


def _geometry(rng, most):
    log = lambda a, b: math.exp(rng.uniform(math.log(a), math.log(b)))
    c = dict(phantom=rng.choice(["water", "slab", "body", "arms"]), nx=int(log(40, 257)), ny=int(log(40, 257)),
             nz=int(log(24, 129)))
    s = round(rng.uniform(25.0, 45.0) / max(c["nx"], c["ny"]), 3)
    c.update(sx=s, sy=s, sz=round(min(0.5, rng.uniform(12.0, 30.0) / c["nz"]), 3))
    side = rng.choice([0.25, 0.5, 1.0, round(log(0.2, 1.0), 2)])
    c.update(beams=rng.randint(1, 9), start=round(rng.uniform(0.0, 40.0), 1), nu=rng.randint(4, 30),
             nv=rng.randint(4, 30), side=side, cutoff=3.0)
    want = log(2e6, most)
    for _ in range(60):
        if _est_nnz(c) <= want:
            break
        k = max(("beams", "nu", "nv"), key=lambda q: c[q])
        c[k] = max(1, int(c[k] * 0.8))
    return c


def draw(rng):
    kind = rng.choice(["plan", "plan", "plan", "tables", "batch", "iterate", "dose", "gradient", "transpose",
                       "transpose", "voxel_dose", "surrogate", "mlp_gradient"])
    if kind == "mlp_gradient":
        return dict(kind=kind, samples=int(math.exp(rng.uniform(math.log(100), math.log(16384)))))
    if kind == "batch":
        return dict(kind=kind, plans=rng.randint(2, 12), mix=rng.randint(10, 10 ** 6), nnz=round(rng.uniform(5e7, 4e8)))
    return dict(kind=kind, **_geometry(rng, {"surrogate": 1.5e8, "tables": 3e8}.get(kind, 6e8)))


# ------------------------------------------------------------------ inputs

def _coords(c):
    n, s = (c["nx"], c["ny"], c["nz"]), (c["sx"], c["sy"], c["sz"])
    origin = tuple(-0.5 * (n[k] - 1) * s[k] for k in range(3))
    return origin, [origin[k] + s[k] * torch.arange(n[k], dtype=F64, device=DEVICE) for k in range(3)]


def _density(c, seed):
    """[nz, ny, nx] float32: which voxels are air outside the body is the case's, the densities the seed's."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed))
    origin, (x, y, z) = _coords(c)
    d = torch.ones((c["nz"], c["ny"], c["nx"]), device=DEVICE)
    X, Y, Z = x[None, None, :], y[None, :, None], z[:, None, None]
    half = [-0.5 * c["s" + k] * c["n" + k] for k in "xyz"]
    if c["phantom"] in ("water", "slab"):
        d += 0.01 * torch.rand(d.shape, generator=gen, device=DEVICE)
    if c["phantom"] == "slab":
        for k in range(8):
            side = rng.uniform(4.0, 10.0, 3) if k < 4 else rng.uniform(1.0, 3.0, 3)
            cen = [half[a] * rng.uniform(-1.0, 1.0) for a in range(3)]
            box = ((X - cen[0]).abs() <= side[0] / 2) & ((Y - cen[1]).abs() <= side[1] / 2) & ((Z - cen[2]).abs() <= side[2] / 2)
            d[box] = 0.25 if k < 4 else 1.8
    if c["phantom"] in ("body", "arms"):
        ax, ay = 0.66 * -half[0], 0.43 * -half[1]
        d = 0.95 + 0.1 * torch.rand(d.shape, generator=gen, device=DEVICE)
        el = lambda a, b, x0=0.0, y0=0.0: (((X - x0) / a) ** 2 + ((Y - y0) / b) ** 2 <= 1.0).expand(d.shape)
        body = el(ax, ay)
        ring = el(0.76 * ax, 0.73 * ay) & ~el(0.70 * ax, 0.63 * ay)
        d[ring] = float(rng.uniform(1.5, 1.9))
        d[el(rng.uniform(0.8, 1.2) * 0.12 * ax, 0.18 * ay, 0.0, 0.32 * ay)] = 0.001
        if c["phantom"] == "arms":          # air between body and arms: holes inside a grid row
            r = 0.12 * -half[0]
            body = body | el(r, 1.3 * r, 0.85 * -half[0]) | el(r, 1.3 * r, 0.85 * half[0])
        d[~body] = 0.0
    return origin, d.float().contiguous()


def _pdd(seed):
    rng = np.random.default_rng(seed + 977)
    d = np.arange(601) * PDD_STEP
    p = (0.25 + 0.75 * (1 - np.exp(-2.498 * d))) * np.exp(-0.045 * d)
    p = p * (1.0 + sum(rng.uniform(-0.002, 0.002) * np.cos(2 * np.pi * d / rng.uniform(8, 25) + rng.uniform(0, 6.28))
                       for _ in range(3)))
    return (p / p.max()).astype(np.float32)


def _tables(seed, pdd):
    rng = np.random.default_rng(seed + 71)
    d = np.arange(81) * 0.5
    c1 = np.array([[0.8], [0.15], [0.05]]) * (1.0 + rng.uniform(-0.15, 0.15, (3, 1)) * np.tanh(d / 10.0))
    c2 = 1.0 + rng.uniform(-0.03, 0.05, (3, 1)) * d / 40.0
    c3 = (np.array([[0.15], [0.4], [1.2]]) + np.array([[0.012], [0.03], [0.08]]) * d
          + rng.uniform(0.0, 1e-4, (3, 1)) * d ** 2)
    th, ad = np.arange(9) * 0.025, np.arange(len(pdd)) * PDD_STEP
    A = pdd[None, :] * (1.0 + 0.8 * th[:, None] ** 2 * np.exp(-ad / 15.0))
    f = lambda v: np.ascontiguousarray(v, dtype=np.float32)
    return SimpleNamespace(c1=f(c1), c2=f(c2), c3=f(c3), depth_step=0.5, A=f(A), theta_step=0.025, adepth_step=PDD_STEP)


def _kernel(c, seed):
    pdd = _pdd(seed)
    tables = _tables(seed, pdd) if c["kind"] == "tables" else None
    return SimpleNamespace(weight=[0.9, 0.1], sigma0=[0.2, 0.4], sigma_slope=[0.4 / 30, 0.8 / 30], width_scale=[1.0, 1.0],
                           n_terms=3 if tables else 2, pdd=pdd, pdd_step=PDD_STEP, cutoff_u=c["cutoff"], cutoff_v=c["cutoff"],
                           table_step=0.0, rho_min=0.0, depth="trilinear" if tables else "siddon", tables=tables)


def _problem(c, seed):
    origin, dens = _density(c, seed)
    beams = [SimpleNamespace(gantry_deg=c["start"] + k * 360.0 / c["beams"], isocenter=ISO, sad=SAD, beamlet_a=c["side"],
                             beamlet_b=c["side"], nu=c["nu"], nv=c["nv"], u0=-0.5 * (c["nu"] - 1) * c["side"],
                             v0=-0.5 * (c["nv"] - 1) * c["side"]) for k in range(c["beams"])]
    grid = SimpleNamespace(density=dens, spacing=(c["sx"], c["sy"], c["sz"]), origin=origin)
    return SimpleNamespace(grid=grid, beams=beams, kernel=_kernel(c, seed))


def _batch_cases(c):
    """The uneven plans of a batch: 64..256 points an axis, 5-9 beams, beamlets of 0.25, 0.5 or 1 cm over 6 x 6 cm."""
    rng = np.random.default_rng(c["mix"])
    out = []
    for k in range(c["plans"]):
        n = [int(v) for v in (rng.integers(64, 257), rng.integers(64, 257), rng.integers(64, 129))]
        side = float(rng.choice([0.25, 0.5, 1.0]))
        ext = rng.uniform(25.0, 51.0)
        s = round(ext / max(n[0], n[1]), 3)
        q = dict(kind="plan", phantom=str(rng.choice(["slab", "body"])), nx=n[0], ny=n[1], nz=n[2], sx=s, sy=s,
                 sz=round(min(0.5, ext * 0.6 / n[2]), 3), beams=int(rng.integers(5, 10)), start=round(rng.uniform(0, 40), 1),
                 nu=int(round(6.0 / side)), nv=int(round(6.0 / side)), side=side, cutoff=3.0)
        while _est_nnz(q) > c["nnz"] / c["plans"] and q["nv"] > 2:      # a shorter field
            q["nv"] -= 1
        out.append(q)
    return out


def _network(seed):
    rng = np.random.default_rng(seed + 5)
    lim = lambda a, b: math.sqrt(6.0 / (a + b))
    w1 = rng.uniform(-lim(4, HIDDEN), lim(4, HIDDEN), HIDDEN * 4)
    w2 = rng.uniform(-lim(HIDDEN, HIDDEN), lim(HIDDEN, HIDDEN), HIDDEN * HIDDEN)
    w3 = rng.uniform(-lim(HIDDEN, 1), lim(HIDDEN, 1), HIDDEN)
    b = rng.uniform(-0.1, 0.1, 2 * HIDDEN + 1)
    return np.concatenate([w1, b[:HIDDEN], w2, b[HIDDEN:2 * HIDDEN], w3, b[2 * HIDDEN:]]).astype(np.float32)


def _samples(c, seed):
    """Training points (d, |u|, |v|, a): dense near the beam axis and the surface, a tenth at zero depth."""
    rng = np.random.default_rng(seed + 55)
    n = c["samples"]
    s = np.empty((n, 4))
    s[:, :3] = np.array([D_MAX, UV_MAX, UV_MAX]) * rng.uniform(0, 1, (n, 3)) ** 2
    s[rng.uniform(size=n) < 0.1, 0] = 0.0
    s[:, 3] = np.exp(rng.uniform(math.log(0.25), 0.0, n))
    return s.astype(np.float32)


# ------------------------------------------------------------------ the framework

def prepare(case, seed):
    kind = case["kind"]
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed) + 1)
    if kind == "mlp_gradient":
        sur = Surrogate(_kernel(dict(kind=kind, cutoff=3.0), seed), _network(seed), max_batch=16384, device=DEVICE)
        feats, targets = sur.targets(torch.from_numpy(_samples(case, seed)).to(DEVICE))
        return SimpleNamespace(kind=kind, sur=sur, feats=feats, targets=targets)
    if kind == "batch":
        batch = Batch([Plan(p, DEVICE, density=p.grid.density) for p in (_problem(q, seed + i) for i, q in enumerate(_batch_cases(case)))])
        return SimpleNamespace(kind=kind, batch=batch)
    prob = _problem(case, seed)
    plan = Plan(prob, DEVICE, density=prob.grid.density)
    if kind in ("plan", "tables"):
        return SimpleNamespace(kind=kind, plan=plan)
    if kind == "surrogate":
        sur = Surrogate(prob.kernel, _network(seed), device=DEVICE)
        plan.set_surrogate(sur)
        return SimpleNamespace(kind=kind, plan=plan, sur=sur)
    D = plan.compute()
    st = SimpleNamespace(kind=kind, D=D, w=torch.rand(plan.n_beamlets, generator=gen, device=DEVICE))
    if kind == "gradient":
        st.r = torch.randn(plan.n_voxels, generator=gen, device=DEVICE)
    if kind == "iterate":
        st.goal = 30.0 * torch.rand(plan.n_voxels, generator=gen, device=DEVICE)
    if kind == "voxel_dose":
        st.D = D.transpose()
    return st


def run(st):
    if st.kind in ("plan", "tables", "surrogate"):
        D = st.plan.compute()
        return D.indptr, D.indices, D.values
    if st.kind == "batch":
        st.batch.run()
        return [(D.indptr, D.indices, D.values) for D in st.batch.outputs()]
    if st.kind in ("dose", "voxel_dose"):
        return st.D.dose(st.w)
    if st.kind == "gradient":
        return st.D.gradient(st.r)
    if st.kind == "iterate":
        dose = st.D.dose(st.w)
        return dose, st.D.gradient(dose - st.goal)
    if st.kind == "transpose":
        T = st.D.transpose()
        return T.indptr, T.indices, T.values
    return st.sur.gradient(st.feats, st.targets)


# ------------------------------------------------------------------ work

def _count(c):
    """Entries of D: the VOI members of every eleventh beamlet, scaled up."""
    prob = _problem(c, 0)
    G = _frames(c, prob)
    take = torch.arange(0, G.n, 11)
    n = sum(int(len(vox)) for _, vox in _members(c, prob, G, take))
    return n * G.n / len(take)


def work(case):
    kind = case["kind"]
    if kind == "mlp_gradient":
        n = case["samples"]
        return {"bytes": 20.0 * n + 8.0 * 4545, "flops": 3 * 2.0 * 4545 * n}
    if kind == "batch":
        w = [work(q) for q in _batch_cases(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    vox, nnz = case["nx"] * case["ny"] * case["nz"], _count(case)
    rows = case["beams"] * case["nu"] * case["nv"]
    if kind in ("plan", "tables", "surrogate"):
        # density in, pointers, columns and values out; an erf counted as ten operations
        return {"bytes": 4.0 * vox + 8.0 * rows + 8.0 * nnz,
                "flops": nnz * {"plan": 120.0, "tables": 190.0, "surrogate": 2.0 * 4545}[kind]}
    if kind == "transpose":
        return {"bytes": 16.0 * nnz + 8.0 * rows + 8.0 * vox, "flops": 0.0}
    if kind == "iterate":
        return {"bytes": 16.0 * nnz + 8.0 * rows + 12.0 * vox, "flops": 4.0 * nnz}
    ptr = 8.0 * (vox if kind == "voxel_dose" else rows)
    return {"bytes": 8.0 * nnz + ptr + 4.0 * rows + 4.0 * vox, "flops": 2.0 * nnz}


# ------------------------------------------------------------------ FP64 reference

def _frames(c, prob):
    """Beamlet frames (source, axis, lateral axes), entry and exit, table points: FP64 tensors, one row a beamlet."""
    S, e, x1, th = [], [], [], []
    for b in prob.beams:
        g = math.radians(b.gantry_deg)
        iso = torch.tensor(b.isocenter, dtype=F64)
        src = iso + SAD * torch.tensor([math.sin(g), -math.cos(g), 0.0], dtype=F64)
        eu, ev = torch.tensor([math.cos(g), math.sin(g), 0.0], dtype=F64), torch.tensor([0.0, 0.0, 1.0], dtype=F64)
        iu, iv = torch.arange(b.nu, dtype=F64), torch.arange(b.nv, dtype=F64)
        p = iso + (b.v0 + iv * b.beamlet_b)[:, None, None] * ev + (b.u0 + iu * b.beamlet_a)[None, :, None] * eu
        ax = (p - src).reshape(-1, 3)
        ax = ax / ax.norm(dim=1, keepdim=True)
        xx = eu - (ax @ eu)[:, None] * ax
        S.append(src.expand_as(ax))
        e.append(ax)
        x1.append(xx / xx.norm(dim=1, keepdim=True))
        th.append(torch.acos((ax @ ((iso - src) / SAD)).clamp(-1, 1)))
    G = SimpleNamespace(S=torch.cat(S).to(DEVICE), e=torch.cat(e).to(DEVICE), eu=torch.cat(x1).to(DEVICE), theta=torch.cat(th).to(DEVICE))
    G.ev = torch.linalg.cross(G.eu, G.e)
    G.n = len(G.e)
    sp = torch.tensor(prob.grid.spacing, dtype=F64, device=DEVICE)
    lo = torch.tensor(prob.grid.origin, dtype=F64, device=DEVICE) - 0.5 * sp
    hi = lo + sp * torch.tensor([c["nx"], c["ny"], c["nz"]], dtype=F64, device=DEVICE)
    t1, t2 = (lo - G.S) / G.e, (hi - G.S) / G.e
    big = torch.full_like(t1, 1e300)
    flat = G.e == 0
    G.tA = torch.where(flat, -big, torch.minimum(t1, t2)).amax(1)
    G.tB = torch.where(flat, big, torch.maximum(t1, t2)).amin(1)
    outside = (flat & ((G.S < lo) | (G.S >= hi))).any(1)
    G.hit = (G.tB > G.tA) & ~outside
    G.m = torch.ceil((G.tB - G.tA) / (0.5 * min(prob.grid.spacing)) - 1e-9).clamp(min=1).long()
    G.m = torch.where(G.hit, G.m, torch.ones_like(G.m))
    G.step = (G.tB - G.tA) / G.m
    G.lo, G.sp = lo, sp
    return G


def _depth_tables(c, prob, G, js):
    """Depth at the table points of beamlets js, [len(js), longest]: exact path integral, or trilinear samples and trapezoids."""
    rho, n = prob.grid.density.double(), (c["nx"], c["ny"], c["nz"])
    S, e, tA, tB, m = G.S[js], G.e[js], G.tA[js], G.tB[js], G.m[js]
    k = torch.arange(int(m.max()) + 1, device=DEVICE)
    t = torch.where(k >= m[:, None], tB[:, None], tA[:, None] + k * G.step[js][:, None])
    if prob.kernel.depth == "trilinear":
        org = torch.tensor(prob.grid.origin, dtype=F64, device=DEVICE)
        P = (S[:, None] + t[..., None] * e[:, None] - org) / G.sp
        val, f, i0 = torch.zeros_like(t), [], []
        for a in range(3):
            q = P[..., a].clamp(0, n[a] - 1)
            i = q.floor().long().clamp(max=max(n[a] - 2, 0))
            f.append(q - i)
            i0.append(i)
        for corner in range(8):
            b = [(corner >> a) & 1 for a in range(3)]
            w = torch.ones_like(t)
            for a in range(3):
                w = w * (f[a] if b[a] else 1 - f[a])
            i = [(i0[a] + b[a]).clamp(max=n[a] - 1) for a in range(3)]
            val += w * rho[i[2], i[1], i[0]]
        inc = 0.5 * (val[:, 1:] + val[:, :-1]) * (t[:, 1:] - t[:, :-1])
        return torch.cat([torch.zeros_like(tA)[:, None], inc.cumsum(1)], 1)
    cross = [tA[:, None], tB[:, None]]
    for a in range(3):
        plane = G.lo[a] + G.sp[a] * torch.arange(n[a] + 1, dtype=F64, device=DEVICE)
        q = (plane - S[:, a:a + 1]) / e[:, a:a + 1]
        cross.append(torch.where(torch.isfinite(q), q, tA[:, None]))
    cut = torch.minimum(torch.maximum(torch.cat(cross, 1), tA[:, None]), tB[:, None]).sort(1).values
    mid = S[:, None] + (0.5 * (cut[:, 1:] + cut[:, :-1]))[..., None] * e[:, None]
    i = [((mid[..., a] - G.lo[a]) / G.sp[a]).floor().long().clamp(0, n[a] - 1) for a in range(3)]
    seg = rho[i[2], i[1], i[0]]
    cum = torch.cat([torch.zeros_like(tA)[:, None], (seg * (cut[:, 1:] - cut[:, :-1])).cumsum(1)], 1)
    at = (torch.searchsorted(cut, t.contiguous(), right=True) - 1).clamp(0, seg.shape[1] - 1)
    return cum.gather(1, at) + seg.gather(1, at) * (t - cut.gather(1, at))


def _members(c, prob, G, js):
    """(beamlet, flat voxel) of the VOI members of beamlets js, in row order: pieces, from a dense test of every voxel."""
    _, (x, y, z) = _coords(c)
    inside = prob.grid.density > prob.kernel.rho_min
    cut = c["cutoff"] / SAD
    per = max(1, int(1.5e8 // inside.numel()))
    js = js.to(DEVICE)
    for j in js.split(per):
        aff = lambda ax: (((z[None] - G.S[j, 2:]) * ax[j, 2:])[:, :, None, None] + ((y[None] - G.S[j, 1:2]) * ax[j, 1:2])[:, None, :, None]
                          + ((x[None] - G.S[j, :1]) * ax[j, :1])[:, None, None, :])
        t = aff(G.e) * cut
        ok = (aff(G.eu).abs() <= t) & (aff(G.ev).abs() <= t) & inside & G.hit[j][:, None, None, None]
        at = ok.reshape(len(j), -1).nonzero()
        yield j[at[:, 0]], at[:, 1]


def _lin(tab, x):
    """Linear interpolation of a table at table coordinate x, held at its ends."""
    x = x.clamp(0, tab.shape[-1] - 1)
    k = x.floor().long().clamp(max=tab.shape[-1] - 2)
    f = x - k
    return tab[..., k] * (1 - f) + tab[..., k + 1] * f


def _bracket(u, h, s):
    q = 1.0 / (math.sqrt(2.0) * s)
    return torch.special.erf((h - u) * q) + torch.special.erf((h + u) * q)


def _profile(K, d, u, v, a):
    L = 0.0
    for w, s0, s1, c2 in zip(K.weight, K.sigma0, K.sigma_slope, K.width_scale):
        s = s0 + s1 * d
        L = L + w / 4 * _bracket(u, c2 * a / 2, s) * _bracket(v, c2 * a / 2, s)
    return L


def _features(d, u, v, a):
    return torch.stack([2 * (d.clamp(min=0) / D_MAX).sqrt() - 1, 2 * (u.abs() / UV_MAX).sqrt() - 1,
                        2 * (v.abs() / UV_MAX).sqrt() - 1, (a - 0.625) / 0.375], -1)


def _unpack(p):
    H, o, out = HIDDEN, 0, []
    for shape in ((H, 4), (H,), (H, H), (H,), (H,), ()):
        k = int(np.prod(shape)) if shape else 1
        out.append(p[o:o + k].reshape(shape))
        o += k
    return out


def _net(p, x):
    w1, b1, w2, b2, w3, b3 = _unpack(p)
    silu = torch.nn.functional.silu
    return silu(silu(x @ w1.T + b1) @ w2.T + b2) @ w3 + b3


def _rows(c, seed):
    """FP64 D: row pointers, columns, values."""
    prob = _problem(c, seed)
    G, K = _frames(c, prob), prob.kernel
    _, (x, y, z) = _coords(c)
    pdd = torch.from_numpy(K.pdd).double().to(DEVICE)
    T = {k: torch.from_numpy(getattr(K.tables, k)).double().to(DEVICE) for k in ("c1", "c2", "c3", "A")} if K.tables else None
    net = torch.from_numpy(_network(seed)).double().to(DEVICE) if c["kind"] == "surrogate" else None
    every = torch.arange(G.n)
    tab = torch.zeros((G.n, int(G.m.max()) + 1), dtype=F64, device=DEVICE)
    for js in every.split(256):
        t = _depth_tables(c, prob, G, js.to(DEVICE))
        tab[js.to(DEVICE), :t.shape[1]] = t
    count = torch.zeros(G.n, dtype=torch.int64, device=DEVICE)
    cols, vals = [], []
    for j, vox in _members(c, prob, G, every):
        count += torch.bincount(j, minlength=G.n)
        out = []
        for jj, vv in zip(j.split(1 << 22), vox.split(1 << 22)):
            P = torch.stack([x[vv % c["nx"]], y[vv // c["nx"] % c["ny"]], z[vv // (c["nx"] * c["ny"])]], 1) - G.S[jj]
            t = (P * G.e[jj]).sum(1)
            r = SAD / t
            u, v = (P * G.eu[jj]).sum(1) * r, (P * G.ev[jj]).sum(1) * r
            tau = torch.minimum(((t - G.tA[jj]) / G.step[jj]).clamp(min=0), G.m[jj].double())
            k = torch.minimum(tau.floor().long(), G.m[jj] - 1)
            d = tab[jj, k] * (1 - (tau - k)) + tab[jj, k + 1] * (tau - k)
            if T:
                th = (G.theta[jj] / K.tables.theta_step).clamp(0, T["A"].shape[0] - 1)
                i = th.floor().long().clamp(max=T["A"].shape[0] - 2)
                xa = (d / K.tables.adepth_step).clamp(0, T["A"].shape[1] - 1)
                q = xa.floor().long().clamp(max=T["A"].shape[1] - 2)
                lin = lambda row: T["A"][row, q] * (1 - (xa - q)) + T["A"][row, q + 1] * (xa - q)
                A, L = lin(i) * (1 - (th - i)) + lin(i + 1) * (th - i), 0.0
                for n in range(3):
                    c1, c2, c3 = (_lin(T[name][n], d / K.tables.depth_step) for name in ("c1", "c2", "c3"))
                    L = L + c1 / 4 * _bracket(u, c2 * c["side"] / 2, c3) * _bracket(v, c2 * c["side"] / 2, c3)
                val = A * L
            else:
                val = _lin(pdd, d / PDD_STEP) * _profile(K, d, u, v, c["side"])
            if net is not None and 0.25 <= c["side"] <= 1.0:
                box = (d <= D_MAX) & (u.abs() <= UV_MAX) & (v.abs() <= UV_MAX)
                val = torch.where(box, _net(net, _features(d, u, v, torch.full_like(d, c["side"]))), val)
            out.append(val * r * r)
        cols.append(vox.int())
        vals += out
    ptr = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEVICE), count.cumsum(0)])
    return ptr, torch.cat(cols), torch.cat(vals)


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp_gradient":
        s = torch.from_numpy(_samples(case, seed)).double().to(DEVICE)
        K = _kernel(dict(kind=kind, cutoff=3.0), seed)
        d, u, v, a = s.unbind(1)
        y = _lin(torch.from_numpy(K.pdd).double().to(DEVICE), d / PDD_STEP) * _profile(K, d, u, v, a)
        p = torch.from_numpy(_network(seed)).double().to(DEVICE).requires_grad_()
        loss = (_net(p, _features(d, u, v, a)) - y).square().mean()
        loss.backward()
        return p.grad, float(loss.detach())
    if kind == "batch":
        out = []
        for i, q in enumerate(_batch_cases(case)):
            out.append((None, None, _rows(q, seed + i)[2]))
        return out
    if kind == "transpose" and _est_nnz(case) > 1.2e9:
        return None
    ptr, col, val = _rows(case, seed)
    if kind in ("plan", "tables", "surrogate"):
        return None, None, val
    if kind == "transpose":
        order = col.sort(stable=True).indices
        return None, None, val[order]
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed) + 1)
    vox, n = case["nx"] * case["ny"] * case["nz"], len(ptr) - 1
    w = torch.rand(n, generator=gen, device=DEVICE).double()
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE), ptr.diff())
    product = lambda: torch.zeros(vox, dtype=F64, device=DEVICE).index_add_(0, col, val * w[row])
    adjoint = lambda r: torch.zeros(n, dtype=F64, device=DEVICE).index_add_(0, row, val * r[col.long()])
    if kind in ("dose", "voxel_dose"):
        return product()
    if kind == "gradient":
        return adjoint(torch.randn(vox, generator=gen, device=DEVICE).double())
    goal = 30.0 * torch.rand(vox, generator=gen, device=DEVICE)
    dose = product()
    return dose, adjoint(dose - goal.double())
