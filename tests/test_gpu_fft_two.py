"""The two-factor x and y FFT passes against the DFT written out, for every
factor of the kernel's list, pruned and full inputs and windows, line counts that do
not fill a workgroup or a block of columns (test entry of include/hvox_testing.h)."""
import ctypes

import numpy as np
import pytest

import paper_2306_06007_amd as hv
from test_gpu_fft import reference

pytestmark = pytest.mark.gpu


def _run(dtype, x_axis, y_axis, nz, sign, rc_only=False):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = hv.load_library().hvox_test_fft_two
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int32, ctypes.POINTER(ctypes.c_int32), ctypes.c_int32, ctypes.c_int32] + 3 * [ctypes.c_void_p]
    cd = torch.complex128 if dtype == "f64" else torch.complex64
    rng = np.random.default_rng(5)
    x = rng.normal(size=(nz, y_axis[1], x_axis[1])) + 1j * rng.normal(size=(nz, y_axis[1], x_axis[1]))
    xin = torch.as_tensor(x).to("cuda", cd).contiguous()
    out = torch.zeros((nz, x_axis[3], y_axis[3]), dtype=cd, device="cuda")
    rc = f(1 if dtype == "f64" else 0, (ctypes.c_int32 * 8)(*x_axis, *y_axis), nz, sign, xin.data_ptr(), out.data_ptr(),
           torch.cuda.current_stream().cuda_stream)
    if rc_only:
        return rc
    assert rc == 0
    x = xin.cpu().numpy().astype(np.complex128)
    ref = np.stack([reference(np.ascontiguousarray(reference(p, x_axis[0], x_axis[2], x_axis[3], sign).T), y_axis[0],
                              y_axis[2], y_axis[3], sign) for p in x])
    got = out.cpu().numpy().astype(np.complex128)
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def _axis(n, kind):
    r = n // 3 + 1
    return (n, n, 0, n) if kind == "full" else (n, max(2, n * 2 // 3 // 2 * 2), -r, 2 * r + 1)


# every factor appears in x and in y; twice the bound of one pass of the general kernel's test
@pytest.mark.parametrize("dtype,tol,lengths", [
    ("f32", 4e-6, [12, 18, 24, 30, 72, 90, 108, 150, 180, 216, 300, 324, 432, 486, 500, 648, 810, 864, 1000, 1200, 1296, 1440]),
    ("f64", 2e-13, [12, 18, 24, 30, 72, 90, 108, 150, 180, 216, 300, 324, 432, 486, 500, 600, 648])])
@pytest.mark.parametrize("sign", [-1, 1])
def test_every_factor(dtype, tol, lengths, sign):
    for i, n in enumerate(lengths):
        m = lengths[(i * 7 + 3) % len(lengths)]
        for kinds, nz in ((("pruned", "full"), 2), (("full", "pruned"), 1)):
            if kinds[0] == "full" and n > 1024:
                continue
            err = _run(dtype, _axis(n, kinds[0]), _axis(m, kinds[1]), nz, sign)
            print(dtype, n, m, kinds, err, flush=True)
            assert err < tol, (n, m, kinds, err)


def test_lengths_without_two_factors_are_refused():
    ok = _axis(48, "pruned")
    assert _run("f32", _axis(1250, "pruned"), ok, 1, 1, rc_only=True) == -1
    assert _run("f64", ok, _axis(720, "pruned"), 1, 1, rc_only=True) == -1
    assert _run("f32", (48, 32, -3, 9), ok, 1, 1, rc_only=True) == -1
