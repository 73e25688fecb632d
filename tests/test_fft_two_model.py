"""CPU check of the two-factor FFT passes' addressing and algebra
(tests/fft_two_model.cpp, a host model of the kernel's index arithmetic built
against the planner): every access of every length they take stays inside its
buffer, every output is written once, and the passes are the padded DFT."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2306_06007_amd", "csrc")


@pytest.mark.parametrize("dtype,longest", [(0, 1600), (1, 648)], ids=["f32", "f64"])
def test_every_two_factor_length(tmp_path, dtype, longest):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path / "fft_two_model")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "fft_two_model.cpp"), os.path.join(CSRC, "planner.cpp"), "-o", exe, "-lpthread"],
                   check=True)
    r = subprocess.run([exe, str(dtype)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert int(r.stdout.split()[1]) > 30 and int(r.stdout.split()[3]) == longest, r.stdout
