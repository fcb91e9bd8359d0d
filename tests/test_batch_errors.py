"""Error exits of batches that run to a final time (``tests/batch_errors_check.cpp``): the library's host code
against a runtime on the CPU in which one call fails.  Whichever call it is, nothing is left running when
the error is returned, the next call starts afresh, and the plan gives back what it took."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def violations(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("batch_errors")
    flags = [HIPCC, "-std=c++17", "-O0", "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-c"]
    subprocess.run(flags + [os.path.join(ROOT, "paper_2402_10914_amd", "csrc", "dfw_step.hip"), "-o", str(d / "step.o")],
                   check=True, capture_output=True)
    subprocess.run(flags + [os.path.join(ROOT, "tests", "batch_errors_check.cpp"), "-o", str(d / "check.o")], check=True,
                   capture_output=True)
    # the host object refers to its device code by a symbol of its own, which nothing here reads
    names = subprocess.run(["nm", "-u", str(d / "step.o")], check=True, capture_output=True, text=True).stdout.split()
    defs = [f"-Wl,--defsym={n}=0" for n in names if n.startswith("__hip_fatbin")]
    subprocess.run(["g++", "-no-pie", str(d / "step.o"), str(d / "check.o"), "-o", str(d / "check")] + defs, check=True,
                   capture_output=True)
    out = subprocess.run([str(d / "check")], check=True, capture_output=True, text=True).stdout.splitlines()
    return {ln.split()[0]: int(ln.split()[1]) for ln in out}


@pytest.mark.parametrize("fault", ["none_graph", "none_direct", "hipEventCreateWithFlags_graph",
                                   "hipEventCreateWithFlags_direct", "hipHostMalloc_graph", "hipHostMalloc_direct",
                                   "hipStreamEndCapture_graph", "hipGraphInstantiate_graph", "hipGraphLaunch_graph",
                                   "hipEventRecord_graph", "hipEventRecord_direct", "hipEventSynchronize_graph",
                                   "hipEventSynchronize_direct", "hipMemcpyAsync_graph", "hipMemcpyAsync_direct"])
def test_error_exit(violations, fault):
    assert violations[fault] == 0, violations
