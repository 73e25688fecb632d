"""Tensors that carry a lazy conjugation or negation (torch's conj(), _neg_view)
through the transforms and their gradients: the kernels read raw storage, so the
binding resolves such views first."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2306_06007_amd as hv  # noqa: E402
from paper_2306_06007_amd import autograd  # noqa: E402
from paper_2306_06007_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    rng = np.random.default_rng(31)
    uvw, xyz = W.uvw_disk(70, 1000.0, 50.0, rng), W.fibonacci_cap(90, 5.0)
    data = [torch.as_tensor(W.complex_normal(2, n, rng)).to("cuda", torch.complex64) for n in (90, 70, 90, 70)]
    # deterministic: equal inputs give equal bits
    with hv.Plan(uvw, xyz, 0.0, "f32", deterministic=True) as p:
        yield p, data


@pytest.mark.parametrize("lazy", [torch.Tensor.conj, torch._neg_view])
@pytest.mark.parametrize("rows", [None, 2])
def test_inputs(setup, lazy, rows):
    p, (sky, vis, b, a) = setup
    x, v = (sky[0], vis[0]) if rows is None else (sky, vis)
    for f, d in ((p.synthesis, x), (p.analysis, v), (p._analysis_real, v)):
        y = lazy(d)
        assert y.is_conj() or y.is_neg()
        assert torch.equal(f(y), f(y.resolve_conj().resolve_neg().clone()))
    for f, d in ((p.synthesis_dde, x), (p.analysis_dde, v)):
        assert torch.equal(f(lazy(d), lazy(a), lazy(b)),
                           f(*(lazy(t).resolve_conj().resolve_neg().clone() for t in (d, a, b))))


@pytest.mark.parametrize("lazy", [torch.Tensor.conj, torch._neg_view])
def test_outputs(setup, lazy):
    p, (sky, _, b, a) = setup
    stream = torch.cuda.Stream()
    ref, dde = p.synthesis(sky), p.synthesis_dde(sky, a, b)
    for st in (None, stream, stream.cuda_stream, 0):
        out, out2 = lazy(torch.zeros_like(ref)), lazy(torch.zeros_like(ref))
        torch.cuda.synchronize()
        assert p.synthesis(sky, out=out, stream=st) is out and p.synthesis_dde(sky, a, b, out=out2, stream=st) is out2
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(out2, dde)


def test_gradient_that_arrives_conjugated(setup):
    """loss = Re sum w conj(V): the gradient of V reaches the backward call as a lazy conjugate."""
    p, (sky, w, _, _) = setup
    for x in (sky.clone().requires_grad_(), sky.real.clone().requires_grad_()):
        autograd.synthesis(x, p).backward(w.conj())
        ref = p.analysis(w.conj().resolve_conj())
        assert torch.equal(x.grad, ref if x.is_complex() else ref.real)
    v = w.clone().requires_grad_()
    autograd.analysis(v, p).backward(sky.conj())
    assert torch.equal(v.grad, p.synthesis(sky.conj().resolve_conj()))
