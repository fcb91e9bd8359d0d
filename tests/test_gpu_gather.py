"""Window sums of the adjoint's gather: grids of odd and even width whose cells lie in three or four
windows, in the first and the last (partly empty) window of a line, and have one or several ghost cells
that fold back to them.  The whole gradient, entry by entry, against the oracle's forward mode, within
the 1e-10 (relative L1) that rounding through two FP64 steps leaves with room to spare."""
import pytest

torch = pytest.importorskip("torch")
from paper_2402_10914_amd import workloads as WL  # noqa: E402
from test_gpu_adjoint import (_dt_of, _gpu_grad, _oracle_full_grad, _random_states, _rel_l1,  # noqa: E402
                              _seeds)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["periodic", "transmissive", "mixed"])
@pytest.mark.parametrize("nx,ny", [(3, 4), (4, 3), (8, 5), (5, 8), (9, 7)])
def test_gradient_entries_on_every_window_position(nx, ny, bc):
    pr = _random_states(nx, ny, 21)
    pr.bc_x = WL.BC_PERIODIC if bc == "periodic" else WL.BC_TRANSMISSIVE
    pr.bc_y = WL.BC_TRANSMISSIVE if bc == "transmissive" else WL.BC_PERIODIC
    dt = _dt_of(pr, 0.2)
    gW, gA = _seeds(pr, 22)
    gW0, gA0, _, _ = _gpu_grad(pr, WL.FLUX_LF, dt, 2, 2, gW, gA)
    oW, oA = _oracle_full_grad(pr, WL.FLUX_LF, dt, 2, gW, gA)
    assert _rel_l1(gW0, oW) <= 1e-10
    assert _rel_l1(gA0, oA) <= 1e-10
