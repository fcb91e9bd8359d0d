"""Uniform flow: the DF of every cell is 1 and the state stays as it is, exactly, for any ratio of specific
heats.  (The gas-kinetic kernels form the DF as gamma^2 / (gamma^2 + (gamma D)^2), which a reciprocal of
gamma^2 rounds off 1 for some gamma, 5/3 among them.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("gamma", [1.2, 1.4, 5.0 / 3.0, 2.0])
def test_df_is_one_in_uniform_flow(gamma, dtype):
    from paper_2402_10914_amd import api
    nx, ny, rho, u, v, p = 24, 20, 1.125, 0.25, -0.5, 0.75
    W0 = np.empty((4, ny, nx))
    W0[0], W0[1], W0[2], W0[3] = rho, rho * u, rho * v, p / (gamma - 1) + 0.5 * rho * (u * u + v * v)
    for kw in (dict(flux=0), dict(flux=1), dict(flux=1, time_limiter=1), dict(flux=1, df_stage=1), dict(flux=0, time_scheme=1)):
        st = api.Stepper(nx, ny, 0.1, 0.1, 0, None, api.Params(gamma=gamma, cfl=0.4, **kw), dtype)
        W = torch.tensor(W0, dtype=dtype, device="cuda")
        A = torch.ones(ny, nx, dtype=dtype, device="cuda")
        start = W.clone()
        st.run(W, A, 2)
        assert bool((A == 1).all()), (kw, (A - 1).abs().max().item())
        assert torch.equal(W, start), kw
