"""Interpolation out of the kept FFT window (HVOX type-3 NUFFT, step 3) in float32: odd and
even kernel widths, one to four data rows, a z axis kept as a window (its cells are read two
at a time) and one kept whole (periodic, read one at a time), against the FP64 oracle."""
import math

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

import paper_2306_06007_amd as hv  # noqa: E402
from paper_2306_06007_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


# the requested accuracy is the bound; kernel widths from 3 upwards
@pytest.mark.parametrize("eps", [5e-1, 1e-1, 3e-2, 1e-2, 1e-3, 1e-4, 3e-5])
@pytest.mark.parametrize("w_half", [0.5, 900.0])
@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5])
def test_windows_and_widths(eps, w_half, rows):
    rng = np.random.default_rng(17)
    uvw = rng.uniform(-1.0, 1.0, (517, 3)) * (40.0, 25.0, w_half)
    xyz = W.random_cap(391, 20.0, rng)
    sky = W.complex_normal(rows, 391, rng)
    vis = W.complex_normal(rows, 517, rng)
    with hv.Plan(uvw, xyz, eps, "f32", direct_threshold=0.0, max_fft_bytes=math.inf, ntrans_hint=rows) as p:
        assert p.info()["n_pairs_nufft"] == 1
        got_v = p.synthesis(torch.as_tensor(sky).to("cuda", torch.complex64)).cpu().numpy()
        got_s = p.analysis(torch.as_tensor(vis).to("cuda", torch.complex64)).cpu().numpy()
        w = p.info()["w"]
    ev, es = oracle.rel_l2(got_v, oracle.synthesis(uvw, xyz, sky)), oracle.rel_l2(got_s, oracle.analysis(uvw, xyz, vis))
    print(eps, w, ev, es, flush=True)
    assert ev <= eps and es <= eps
