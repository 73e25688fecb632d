"""How well float32 plans hold a phase in the direct sum (HVOX Sect. 3.1, last
bullet): sums of so few terms that the error of a term is the error of the
result, against the FP64 oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

import paper_2306_06007_amd as hv  # noqa: E402
from paper_2306_06007_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _run(direction, n_src, n_tgt, rows, scale):
    rng = np.random.default_rng(41)
    src, tgt = W.random_cap(n_src, 5.0, rng), W.uvw_disk(n_tgt, 1000.0, 50.0, rng) * scale
    data = W.complex_normal(rows, n_src, rng).astype(np.complex64)
    if direction == "synthesis":
        uvw, xyz, ref = tgt, src, oracle.synthesis(tgt, src, data.astype(np.complex128))
    else:
        uvw, xyz, ref = src, tgt, oracle.analysis(src, tgt, data.astype(np.complex128))
    with hv.Plan(uvw, xyz, 0.0, "f32") as p:
        out = getattr(p, direction)(torch.as_tensor(data).cuda()).cpu().numpy()
    return out, ref, np.abs(data).sum(-1, keepdims=True)


# targets of narrow items, of wide ones (four work items per CU of 512 targets), and phases beyond 2^18 turns
@pytest.mark.parametrize("direction", ["synthesis", "analysis"])
@pytest.mark.parametrize("n_src", [1, 2])
@pytest.mark.parametrize("n_tgt,rows,scale", [(300, 1, 1.0), (130, 4, 1.0), (600_000, 1, 1.0), (300, 3, 1e4)])
def test_one_or_two_sources_carry_a_rounding(direction, n_src, n_tgt, rows, scale):
    """A float64 sum rounded once: 2^-24 of the value, and the phase's own float64 rounding (turns 2^-50)."""
    out, ref, weight = _run(direction, n_src, n_tgt, rows, scale)
    turns = 1000.0 * scale
    assert (np.abs(out - ref) <= 2.0 ** -24 * np.abs(ref) + 2.0 * np.pi * turns * 2.0 ** -50 * weight).all()


@pytest.mark.parametrize("direction", ["synthesis", "analysis"])
@pytest.mark.parametrize("n_src", [3, 10, 30])
def test_few_sources(direction, n_src):
    """Per term the fraction of a turn, a float in [-1/2, 1/2], is off by 4e-8 rad (root mean square, 2^-26 turns at
    most), and the running sum is rounded a few times: two float32 roundings, 2^-23, bound them and
    the hardware sine.  A fraction cut to 2^-24 turns is off by 2.2e-7 rad by itself."""
    out, ref, _ = _run(direction, n_src, 3000, 1, 1.0)
    assert np.linalg.norm(out - ref) <= 2.0 ** -23 * np.linalg.norm(ref)


@pytest.mark.parametrize("scale", [1.0, 1e3])
def test_many_positive_intensities(scale):
    """A million positive intensities add up what sine and cosine average over a turn: 5e-10 a term would be 4e-7 of
    the result.  Without it the independent errors of the terms and of the runs remain, 2^-22 at most."""
    rng = np.random.default_rng(43)
    uvw, xyz = W.ska_like_uvw(7), W.fibonacci_cap(1_000_000, 10.0)
    # baselines that resolve the cap; beyond 2^18 turns: the float64 fraction
    uvw = scale * rng.permutation(uvw[np.linalg.norm(uvw, axis=1) > 500.0])[:256]
    sky = rng.random((1, 1_000_000)).astype(np.float32).astype(np.complex128)
    with hv.Plan(uvw, xyz, 0.0, "f32") as p:
        out = p.synthesis(torch.as_tensor(sky).to("cuda", torch.complex64)).cpu().numpy()
    ref = oracle.synthesis(uvw, xyz, sky)
    print(np.linalg.norm(out - ref) / np.linalg.norm(ref), flush=True)
    assert np.linalg.norm(out - ref) <= 2.0 ** -22 * np.linalg.norm(ref)
