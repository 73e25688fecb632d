"""Performance cases of the HVOX transforms: what a user's program runs through
the package's public entry points (``Plan``, ``autograd``, ``RadioPlan``), from
a 0.04 ms call to the full SKA-like transform.

``listed()`` names the cases, ``draw(rng)`` makes another of the same ranges,
``prepare`` builds what a program holds before its calls (coordinates, plan,
data on the GPU), ``run`` is one call, ``work`` the bytes and operations a call
cannot do without and ``exact`` its result in float64 from plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2306_06007_amd import Plan, autograd, workloads
from paper_2306_06007_amd.radio import RadioPlan

SPEED_OF_LIGHT = 299_792_458.0   # m/s
# terms of the double sum above which exact() gives no value (about 15 s)
EXACT_TERMS = 1.5e11
# stations of the telescope-radius ladder's rungs are fixed by its visibility counts
RUNGS = {0.1: (273, 80), 0.3: (13_113, 160), 1.0: (94_878, 360), 3.0: (148_365, 900), 100.0: (393_984, 13_500)}


def listed():
    return [
        # the smallest calls: a compact array's snapshot, where launches and latency count
        dict(name="compact-f32-synthesis", kind="disk", n_vis=2000, n_pix=3072, dtype="f32", eps=1e-4,
             direction="synthesis"),
        dict(name="compact-f64-analysis", kind="disk", n_vis=2000, n_pix=3072, dtype="f64", eps=1e-6,
             direction="analysis"),
        # direction-dependent calibration: a few patches of pixels seen by a 100 km array
        dict(name="sparse-calibrators-f32", kind="sparse", radius_km=100.0, regions=5, side=10, dtype="f32", eps=1e-4,
             direction="synthesis"),
        # a request of the serving loop (deterministic plans) on wide-field baselines, uneven sizes
        dict(name="serving-wide-field-f32", kind="serving", layout="lofar", n_vis=70_001, n_pix=90_007, dtype="f32",
             eps=1e-4, direction="analysis"),
        # four polarisations and four channels through the radio front end's adjoint
        dict(name="radio-4pol-4chan-f32", kind="radio", n_ant=60, n_times=12, n_chan=4, n_pol=4, side=300,
             dtype="f32", eps=1e-4, direction="analysis"),
        # time-variable primary beams: three gain terms through the DDE entry point
        dict(name="primary-beams-f32", kind="dde", n_ant=130, n_times=9, terms=3, n_pix=50_021, dtype="f32", eps=1e-4,
             direction="synthesis"),
        # double precision at the accuracy an imaging loop asks of it
        dict(name="ska-like-f64", kind="ska", n_ant=75, n_times=50, n_pix=150_000, dtype="f64", eps=1e-9,
             direction="synthesis"),
        # an imaging iteration: forward model, residual, gradient
        dict(name="imaging-gradient-f32", kind="gradient", n_ant=100, n_times=50, n_pix=200_000, dtype="f32",
             eps=1e-4, direction="both"),
        # a dense direction-cosine image, sub-problems split between NUFFT and direct sums
        dict(name="dense-3km-f32", kind="dense", radius_km=3.0, dtype="f32", eps=1e-4, direction="synthesis",
             nufft=False),
        # every sub-problem through the NUFFT grids, both precisions
        dict(name="dense-3km-all-nufft-f32", kind="dense", radius_km=3.0, dtype="f32", eps=1e-4,
             direction="analysis", nufft=True),
        dict(name="dense-1km-all-nufft-f64", kind="dense", radius_km=1.0, dtype="f64", eps=1e-9,
             direction="synthesis", nufft=True),
        # the headline workload, one direction
        dict(name="ska-like-full-f32", kind="ska", n_ant=200, n_times=50, n_pix=1_000_000, dtype="f32", eps=1e-4,
             direction="synthesis"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["disk", "sparse", "serving", "radio", "dde", "ska", "gradient", "dense", "ska"])
    dtype = rng.choice(["f32", "f32", "f64"])
    eps = rng.choice([1e-3, 1e-4, 1e-5] if dtype == "f32" else [1e-6, 1e-7, 1e-9])
    direction = rng.choice(["synthesis", "analysis"])
    c = dict(kind=kind, dtype=dtype, eps=eps, direction=direction)
    if kind == "disk":
        c.update(n_vis=_log(rng, 300, 20_000), n_pix=_log(rng, 300, 20_000))
    elif kind == "sparse":
        c.update(radius_km=rng.choice([1.0, 3.0, 100.0]), regions=rng.randint(3, 9), side=rng.randint(7, 14))
    elif kind == "serving":
        c.update(layout=rng.choice(["ska", "lofar"]), n_vis=_log(rng, 10_000, 400_000),
                 n_pix=_log(rng, 10_000, 400_000), dtype="f32", eps=1e-4)
    elif kind == "radio":
        c.update(n_ant=rng.randint(20, 80), n_times=rng.randint(4, 20), n_chan=rng.randint(1, 4),
                 n_pol=rng.randint(1, 4), side=_log(rng, 64, 400), dtype="f32", eps=rng.choice([1e-3, 1e-4]))
    elif kind == "dde":
        c.update(n_ant=rng.randint(40, 150), n_times=9, terms=rng.choice([2, 3, 5]), n_pix=_log(rng, 5000, 120_000))
        c["n_times"] = 3 * c["terms"]
    elif kind == "gradient":
        c.update(n_ant=rng.randint(30, 130), n_times=rng.randint(20, 50), n_pix=_log(rng, 10_000, 300_000),
                 direction="both")
    elif kind == "dense":
        c.update(radius_km=rng.choice([0.1, 0.3, 1.0, 3.0]), nufft=rng.choice([False, True]))
        # an odd image side: every rung's own side is even
        c["side"] = RUNGS[c["radius_km"]][1] - rng.randrange(1, 40, 2)
    else:
        big = dtype == "f32"
        c.update(n_ant=rng.randint(40, 190 if big else 110), n_times=rng.randint(20, 50),
                 n_pix=_log(rng, 10_000, 900_000 if big else 300_000))
    return c


def _sizes(case):
    """(visibilities, pixels, data rows) of a case."""
    kind = case["kind"]
    if kind in ("disk", "serving"):
        return case["n_vis"], case["n_pix"], 1
    if kind == "sparse":
        return RUNGS[case["radius_km"]][0], case["regions"] * case["side"] ** 2, 1
    if kind == "dense":
        return RUNGS[case["radius_km"]][0], case.get("side", RUNGS[case["radius_km"]][1]) ** 2, 1
    pairs = case["n_ant"] * (case["n_ant"] - 1) // 2 * case["n_times"]
    if kind == "radio":
        return pairs * case["n_chan"], case["side"] ** 2, case["n_pol"]
    return pairs, case["n_pix"], case["terms"] if kind == "dde" else 1


_LAYOUT = {}


def _lofar_uvw():
    """The wide-field layout's 5 M baselines (its hour-angle span takes seconds to fit): requests sample them."""
    if "lofar" not in _LAYOUT:
        _LAYOUT["lofar"] = workloads.lofar_like_uvw()
    return _LAYOUT["lofar"]


def _geometry(case, seed):
    """uvw in wavelengths (n_vis, 3), sky points (n_pix, 3) and, for the radio front end, its own arguments."""
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    if kind == "disk":
        return workloads.uvw_disk(case["n_vis"], 1000.0, 50.0, rng), workloads.fibonacci_cap(case["n_pix"], 5.0), None
    if kind == "sparse":
        w = workloads.sparse_dcos(case["radius_km"], seed=seed, n_regions=case["regions"], side=case["side"])
        return w.uvw, w.xyz, None
    if kind == "dense":
        uvw, _ = workloads.ladder_uvw(case["radius_km"], rng)
        return uvw, workloads.dcos_grid(case.get("side", RUNGS[case["radius_km"]][1]), 30.0), None
    if kind == "serving":
        if case["layout"] == "lofar":
            base, cap = _lofar_uvw(), 60.0
        else:
            base, cap = workloads.ska_like_uvw(seed), 10.0
        idx = np.sort(rng.choice(base.shape[0], size=case["n_vis"], replace=False))
        return base[idx], workloads.fibonacci_cap(case["n_pix"], cap), None
    if kind == "radio":
        enu = workloads.gaussian_layout(case["n_ant"], 1500.0, rng)
        hours = np.radians(np.linspace(-30.0, 30.0, case["n_times"]))
        uvw_m = workloads.earth_rotation_uvw(enu, -30.0, -30.0, hours, [1.0])
        freqs = 150e6 + 1e6 * np.arange(case["n_chan"])
        xyz = workloads.dcos_grid(case["side"], 10.0)
        l, m = xyz[:, 0], xyz[:, 1]
        r2 = l * l + m * m
        xyz = np.stack([l, m, -r2 / (1.0 + np.sqrt(1.0 - r2))], axis=1)
        uvw = (uvw_m[:, None, :] * (freqs / SPEED_OF_LIGHT)[None, :, None]).reshape(-1, 3)
        return uvw, xyz, (uvw_m, freqs, l, m)
    uvw = workloads.ska_like_uvw(seed, n_ant=case["n_ant"], n_times=case["n_times"])
    return uvw, workloads.fibonacci_cap(case["n_pix"], 10.0), None


def _data(case, seed, xyz):
    """Complex128 / float64 data of a case on the GPU: intensities U[0, 1], visibilities CN(0, 1), beams."""
    n_vis, n_pix, rows = _sizes(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    cn = lambda *s: torch.complex(*(torch.randn(*s, generator=g, device="cuda", dtype=torch.float64) * math.sqrt(0.5)  # noqa: E731
                                    for _ in range(2)))
    kind = case["kind"]
    d = {}
    if kind == "gradient":
        d["x"] = rand(n_pix)
        d["y"] = cn(n_vis) * math.sqrt(n_pix / 3.0)
        return d
    lead = (rows,) if kind == "radio" else ()
    if case["direction"] == "synthesis":
        s = rand(*lead, n_pix)
        d["in"] = torch.complex(s, torch.zeros_like(s))
    else:
        d["in"] = cn(*lead, n_vis)
    if kind == "dde":
        a, b = workloads.snapshot_beams(n_vis, rows, xyz)
        d["a"], d["b"] = torch.as_tensor(a, device="cuda"), torch.as_tensor(b, device="cuda")
    return d


def _rounded(case, d):
    """The data in the case's precision."""
    cd, rd = (torch.complex128, torch.float64) if case["dtype"] == "f64" else (torch.complex64, torch.float32)
    return {k: v.to(cd if v.is_complex() else rd) for k, v in d.items()}


def prepare(case, seed):
    uvw, xyz, radio = _geometry(case, seed)
    state = _rounded(case, _data(case, seed, xyz))
    rows = _sizes(case)[2]
    opts = {}
    if case["kind"] == "serving":
        opts["deterministic"] = True
    if case["kind"] == "dense" and case["nufft"]:
        opts["direct_threshold"] = 0.0
    if rows > 1:
        opts["ntrans_hint"] = rows
    if radio is not None:
        uvw_m, freqs, l, m = radio
        state["plan"] = RadioPlan(uvw_m, freqs, l, m, case["eps"], case["dtype"], **opts)
        if case["direction"] == "analysis":
            state["in"] = state["in"].reshape(rows, uvw_m.shape[0], freqs.size)
    else:
        state["plan"] = Plan(uvw, xyz, case["eps"], case["dtype"], **opts)
    state["kind"], state["direction"] = case["kind"], case["direction"]
    return state


def run(state):
    plan, kind, synthesis = state["plan"], state["kind"], state["direction"] == "synthesis"
    if kind == "gradient":
        x = state["x"].detach().requires_grad_()
        vis = autograd.synthesis(x, plan)
        r = torch.view_as_real(vis - state["y"])
        (0.5 * (r * r).sum()).backward()
        return {"vis": vis.detach(), "grad": x.grad}
    if kind == "radio":
        return plan.dirty2vis(state["in"]) if synthesis else plan.vis2dirty(state["in"])
    if kind == "dde":
        f = plan.synthesis_dde if synthesis else plan.analysis_dde
        return f(state["in"], state["a"], state["b"])
    return plan.synthesis(state["in"]) if synthesis else plan.analysis(state["in"])


def work(case):
    """Coordinates (float64) and data in and out once.  Operations of the double sum, 30 a term and row (phase 6,
    its reduction 2, sine and cosine 14, multiply-add 8; a further row adds the 8); of a case whose sub-problems
    are all NUFFTs, those of one type-3 transform: spreading and interpolation of every point over 7^3 cells and,
    for every grid cell of the Heisenberg box, the FFT."""
    n_vis, n_pix, rows = _sizes(case)
    item = 16.0 if case["dtype"] == "f64" else 8.0
    data = rows * (n_vis + n_pix) * item
    if case["kind"] == "dde":
        data += (n_vis + n_pix) * item
    ways = 2.0 if case["kind"] == "gradient" else 1.0
    if case["kind"] == "dense" and case["nufft"]:
        # aperture diameter (2 m wavelength) x field of view per axis: the cells of an unpadded grid
        cells = max(1.0, case["radius_km"] * 1e3 * 0.52) ** 2 * max(1.0, case["radius_km"] * 1e3 * 0.5 * 0.035)
        flops = (n_vis + n_pix) * 343.0 * 4.0 + cells * 5.0 * math.log2(cells + 2.0)
    else:
        flops = float(n_vis) * n_pix * (22.0 + 8.0 * rows)
    return {"bytes": ways * ((n_vis + n_pix) * 24.0 + data), "flops": ways * flops}


def _split(a):
    """a as the sum of a part of at most 26 bits and the rest (float64)."""
    t = a * 134217729.0
    hi = t - (t - a)
    return hi, a - hi


def _double_sum(tgt, src, rows, sign):
    """out[r, k] = sum_n rows[r, n] exp(sign 2 pi i <tgt_k, src_n>) in float64: the products of the coordinates'
    high parts are exact and reduced to a fraction of a turn before the small cross terms are added."""
    th, tl = _split(tgt)
    sh, sl = _split(src)
    small = (torch.cat([th, tl, tl], 1), torch.cat([sl, sh, sl], 1).T.contiguous())
    out = torch.empty(rows.shape[0], tgt.shape[0], dtype=torch.complex128, device=tgt.device)
    step = max(1, int(1.2e8) // max(1, src.shape[0]))
    cre, cim = rows.real.T.contiguous(), rows.imag.T.contiguous()
    for k in range(0, tgt.shape[0], step):
        f = small[0][k:k + step] @ small[1]
        for d in range(3):
            p = th[k:k + step, d, None] * sh[None, :, d]
            f += p.sub_(p.round())
        f *= 2.0 * math.pi
        c, s = torch.cos(f), f.sin_().mul_(sign)
        out[:, k:k + step] = torch.complex(c @ cre - s @ cim, c @ cim + s @ cre).T
    return out


def exact(case, seed):
    n_vis, n_pix, rows = _sizes(case)
    if float(n_vis) * n_pix * (2.0 if case["kind"] == "gradient" else 1.0) > EXACT_TERMS:
        return None
    uvw, xyz, radio = _geometry(case, seed)
    d = _rounded(case, _data(case, seed, xyz))
    d = {k: v.to(torch.complex128 if v.is_complex() else torch.float64) for k, v in d.items()}
    p, r = torch.as_tensor(uvw, device="cuda"), torch.as_tensor(np.ascontiguousarray(xyz), device="cuda")
    if case["kind"] == "gradient":
        x = torch.complex(d["x"], torch.zeros_like(d["x"]))
        vis = _double_sum(p, r, x[None], -1.0)[0]
        return {"vis": vis, "grad": _double_sum(r, p, (vis - d["y"])[None], 1.0)[0].real.contiguous()}
    synthesis = case["direction"] == "synthesis"
    if case["kind"] == "dde":
        a, b = d["a"], d["b"]
        if synthesis:
            return (a * _double_sum(p, r, b * d["in"], -1.0)).sum(0)
        return (b.conj() * _double_sum(r, p, a.conj() * d["in"], 1.0)).sum(0)
    x = d["in"].reshape(-1, d["in"].shape[-1])
    out = _double_sum(p, r, x, -1.0) if synthesis else _double_sum(r, p, x, 1.0)
    if radio is not None:
        lead = (rows,)
        return out.reshape(lead + (radio[0].shape[0], radio[1].size)) if synthesis else out.reshape(lead + (n_pix,))
    return out[0]
