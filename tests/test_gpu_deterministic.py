"""Deterministic plans add the direct sum up in one order (HVOX Sect. 3.1, last
bullet; include/hvox.h, HVOX_DETERMINISTIC): a row's bits depend neither on the
rows that share its call, nor on the rows the plan was made for, nor on the
entry point and how much of its scratch the stored layers find."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2306_06007_amd as hv  # noqa: E402
from paper_2306_06007_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _noalloc(plan, direction, x):
    out = torch.empty((x.shape[0], plan.n_vis if direction == 0 else plan.n_pix), dtype=x.dtype, device="cuda")
    rc = hv.load_library().hvox_transform_noalloc(
        plan._plan, direction, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(out.data_ptr()), x.shape[0],
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, hv.load_library().hvox_last_error()
    return out


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n_vis,n_pix", [(5, 1), (1, 5), (250, 200)])
def test_row_alone_and_among_others(dtype, n_vis, n_pix):
    """A row's bits are the same whichever kernel instance (rows per launch) computes it."""
    cd = torch.complex64 if dtype == "f32" else torch.complex128
    rng = np.random.default_rng(21)
    uvw, xyz = W.uvw_disk(n_vis, 1000.0, 50.0, rng), W.fibonacci_cap(n_pix, 5.0)
    sky = torch.as_tensor(W.complex_normal(4, n_pix, rng)).to("cuda", cd)
    sky[0] = sky[0].real.to(cd)   # alone it takes the loop for real values, among the others the complex one
    vis = torch.as_tensor(W.complex_normal(4, n_vis, rng)).to("cuda", cd)
    with hv.Plan(uvw, xyz, 0.0, dtype, deterministic=True) as p:
        V, I = p.synthesis(sky), p.analysis(vis)
        for rows in (1, 2, 3):
            assert torch.equal(p.synthesis(sky[:rows]), V[:rows]) and torch.equal(p.analysis(vis[:rows]), I[:rows])


# (2,000, 3,072): some 24 layers in the plan's slabs and the static buffer; (200,000, 160,000): 20 layers of 200,000
# targets, which the plan's slabs hold (2^22 values) and the 64 MiB static buffer does not; (3, 60,000) and (500, 40,001):
# hundreds of layers of few targets, whose loads several lanes share
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n_vis,n_pix", [(2_000, 3_072), (200_000, 160_000), (3, 60_000), (500, 40_001)])
def test_direct_sum_keeps_its_order(dtype, n_vis, n_pix):
    cd = torch.complex64 if dtype == "f32" else torch.complex128
    rng = np.random.default_rng(21)
    uvw, xyz = W.uvw_disk(n_vis, 1000.0, 50.0, rng), W.fibonacci_cap(n_pix, 5.0)
    sky = torch.as_tensor(W.complex_normal(4, n_pix, rng)).to("cuda", cd)
    sky[0] = sky[0].real.to(cd)   # alone it takes the loop for real values, among the others the complex one
    vis = torch.as_tensor(W.complex_normal(4, n_vis, rng)).to("cuda", cd)
    ref = None
    for hint in (1, 4):
        with hv.Plan(uvw, xyz, 0.0, dtype, deterministic=True, ntrans_hint=hint) as p:
            V, I = p.synthesis(sky), p.analysis(vis)
            if ref is None:
                ref = (V, I)
            assert torch.equal(V, ref[0]) and torch.equal(I, ref[1])
            for t in (0, 3):
                assert torch.equal(p.synthesis(sky[t]), V[t]) and torch.equal(p.analysis(vis[t]), I[t])
            for rows in (slice(0, 4), slice(2, 3)):
                assert torch.equal(_noalloc(p, 0, sky[rows]), V[rows])
                assert torch.equal(_noalloc(p, 1, vis[rows]), I[rows])


def _launches(plan, sky):
    plan.reset_stats()
    plan.set_timing(True)
    plan.synthesis(sky)
    torch.cuda.synchronize()
    st = plan.stats()
    plan.set_timing(False)
    return st["direct"]["launches"], st["finalize"]["launches"]


def test_every_launch_of_the_direct_sum_is_timed():
    """600,000 targets: the slabs (2^22 values) hold 6 of 10 layers, so the first launch's layers go to the accumulator."""
    rng = np.random.default_rng(22)
    uvw, xyz = W.uvw_disk(600_000, 1000.0, 50.0, rng), W.fibonacci_cap(80_000, 5.0)
    sky = torch.as_tensor(W.complex_normal(4, 80_000, rng)).to("cuda", torch.complex64)
    with hv.Plan(uvw, xyz, 0.0, "f32", deterministic=True) as p:
        direct, final = _launches(p, sky[0])
        assert direct == p.info()["n_direct_layers"] > 1
        assert final == direct   # all but the last launch's layers by k_add_layers, those by the epilogue


def test_a_single_layer_that_fits_is_added_in_place():
    """Four rows on a plan made for one: its slabs hold one of 10 layers of four rows, so items add into the accumulator."""
    rng = np.random.default_rng(22)
    uvw, xyz = W.uvw_disk(600_000, 1000.0, 50.0, rng), W.fibonacci_cap(80_000, 5.0)
    sky = torch.as_tensor(W.complex_normal(4, 80_000, rng)).to("cuda", torch.complex64)
    with hv.Plan(uvw, xyz, 0.0, "f32", deterministic=True) as p:
        direct, final = _launches(p, sky)
        assert direct == 10 and final == 1
        assert torch.equal(p.synthesis(sky)[2], p.synthesis(sky[2]))
