"""The forms of reconstruction and fluxes that the FP64 kernels run against the candidate forms
that the FP32 kernels run, both in FP64 on the host (``tests/forms_check.cpp``).

Tolerance: both forms evaluate the same polynomial from the same averages; with sound speeds of
order one to ten the projections amplify a rounding of the data (1.1e-16 of its maximum) by up to
about 1e3, so 1e-12 of the data.  The limiter weight is compared where the indicators stand clear
of rounding (jumps and independent states).  Fluxes are compared relative to the largest of their
values at the point, where the moments' cancellations cost about the same."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def worst(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("forms") / "forms_check")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-x", "hip", "--offload-arch=gfx950",
                    os.path.join(ROOT, "tests", "forms_check.cpp"), "-o", exe], check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    return {ln.split()[0]: float(ln.split()[1]) for ln in out}


@pytest.mark.parametrize("name", [a + b for a in ("normal", "omega", "tangential") for b in ("_char", "_comp")] +
                         ["flux_lf", "flux_gks", "flux_df"])
def test_fp64_forms_equal_candidate_forms(worst, name):
    assert worst[name] < (1e-10 if name.startswith("omega") else 1e-12), worst
