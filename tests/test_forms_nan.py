"""The host checks of the device arithmetic (``forms_check.cpp``, ``recon_forms_check.cpp``,
``adjoint_check.cpp``) with maxima that keep a NaN: a form that returns NaN anywhere on their data, the
zero collision times included, shows as a deviation of NaN and not as none.  Bounds are those of the
checks' own tests."""
import math
import os
import subprocess

import pytest

from test_recon_forms import BOUNDS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
TESTS = os.path.join(ROOT, "tests")


def _run(tmp_path, name):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / name)
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-x", "hip", "--offload-arch=gfx950", "-include",
                    os.path.join(TESTS, "sticky_nan.hpp"), os.path.join(TESTS, name + ".cpp"), "-o", exe], check=True,
                   capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    return {ln.split()[0]: float(ln.split()[1]) for ln in out}


def test_forms_are_finite(tmp_path):
    worst = _run(tmp_path, "forms_check")
    assert len(worst) == 9
    for name, e in worst.items():
        assert e < (1e-10 if name.startswith("omega") else 1e-12), worst  # false for NaN


def test_reconstruction_forms_are_finite(tmp_path):
    worst = _run(tmp_path, "recon_forms_check")
    assert sorted(worst) == sorted(BOUNDS)
    for name, e in worst.items():
        assert e < BOUNDS[name], worst


def test_adjoints_are_finite(tmp_path):
    worst = _run(tmp_path, "adjoint_check")
    for name, e in worst.items():
        assert math.isfinite(e) and e < 1e-6, (name, e)
