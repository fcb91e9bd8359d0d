"""The tile shape that the library chooses for tile index 0 changes no bit: grid sizes on both sides of
every line of the choice (a tile per compute unit, four per unit, 24 per unit with and without 4 %
fewer tall tiles), single grids, a batch, the operator and a gradient, against an explicit shape."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2402_10914_amd import workloads as WL  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = [(1, 9), (64, 63), (128, 136), (160, 170), (300, 310), (333, 487), (1001, 750), (1024, 1000)]


def _run(nx, ny, dtype, tile, flux=0):
    from paper_2402_10914_amd import api
    pr = WL.riemann4(nx, ny, seed=3, flux=flux)
    st = api.Stepper.for_problem(pr, api.Params(flux=flux, cfl=0.4, tile=tile), dtype)
    W = torch.tensor(pr.W, dtype=dtype, device="cuda")
    A = torch.tensor(pr.alpha, dtype=dtype, device="cuda")
    t, fs = st.run(W, A, 2)
    L = st.rhs(W, A, 1e-4, want_alpha=True)
    return [x.cpu().numpy() for x in (W, A, *L)] + [np.array([t, fs])]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_default_tile_equals_explicit_tile(nx, ny, dtype):
    for a, b in zip(_run(nx, ny, dtype, 0), _run(nx, ny, dtype, 1)):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("sizes", [[(20, 30)] * 3, [(40, 100)] * 40, [(300, 250)] * 12])
def test_default_tile_of_a_batch(sizes):
    from paper_2402_10914_amd import api
    probs = [WL.density_wave(nx, ny) for nx, ny in sizes]
    out = []
    for tile in (0, 1):
        b = api.Batch([(p.nx, p.ny, p.dx, p.dy, p.bc_x, p.bc_y) for p in probs], api.Params(cfl=0.4, tile=tile))
        W, A = b.pack([p.W for p in probs], [p.alpha for p in probs])
        b.run(W, A, 2)
        out.append((W.cpu().numpy(), A.cpu().numpy()))
    assert all(np.array_equal(x, y) for x, y in zip(*out))


def test_default_tile_of_a_gradient():
    from paper_2402_10914_amd import api
    pr = WL.bumps(48)
    g = []
    for tile in (0, 1):
        adj = api.Adjoint(api.Stepper.for_problem(pr, api.Params(cfl=0.5, tile=tile)), 4, 2)
        W = torch.tensor(pr.W, device="cuda")
        A = torch.tensor(pr.alpha, device="cuda")
        adj.forward(W, A)
        g.append([x.cpu().numpy() for x in adj.backward(torch.ones_like(W) * 1e-3)])
    assert all(np.array_equal(x, y) for x, y in zip(*g))
