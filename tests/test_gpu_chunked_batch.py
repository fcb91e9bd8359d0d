"""Batches that run to a final time go in chunks of steps and end when no grid is left to advance: the
states, times, failing steps and recorded time steps are those of single runs, bit for bit, for step
counts around the chunk (16), runs that end in different chunks, runs that the step count cuts off, a
grid that fails at once, with and without the captured graphs, and when the plan is run again."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2402_10914_amd import workloads as WL  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsteps", [0, 15, 16, 17, 33, 200])
@pytest.mark.parametrize("graph", [True, False])
def test_chunked_batch_equals_single_runs(nsteps, graph):
    from paper_2402_10914_amd import api
    probs = [WL.problem_123(m, n=n) for m, n in ((1.2, 100), (1.5, 40), (1.1, 16))] + [WL.riemann4(24, 20, seed=5)]
    bad = WL.density_wave(12)
    bad.W[3, 0, 0] = -1.0  # non-physical input: fails before the first step
    probs.append(bad)
    params = api.Params(flux=api.FLUX_LF, cfl=0.5, time_scheme=api.TIME_SSPRK3, switch_rule=2, t_end=0.05)
    b = api.Batch([(p.nx, p.ny, p.dx, p.dy, p.bc_x, p.bc_y) for p in probs], params)
    W0, A0 = b.pack([p.W for p in probs], [p.alpha for p in probs])
    W, A = W0.clone(), A0.clone()
    dth = torch.empty(len(probs) * max(nsteps, 1), dtype=torch.float64, device="cuda")
    for _ in range(2):
        W.copy_(W0)
        A.copy_(A0)
        dth.fill_(-1.0)
        ts, fs = b.run(W, A, nsteps, use_graph=graph, dt_hist=dth)
        got = dth[:len(probs) * nsteps].view(len(probs), nsteps) if nsteps else None
        for g, (p, (w, a)) in enumerate(zip(probs, b.unpack(W, A))):
            st = api.Stepper.for_problem(p, params)
            w1 = torch.tensor(p.W, device="cuda")
            a1 = torch.tensor(p.alpha, device="cuda")
            d1 = torch.full((max(nsteps, 1),), -1.0, dtype=torch.float64, device="cuda")
            t, f = st.run(w1, a1, nsteps, dt_hist=d1)
            assert (t, f) == (ts[g], fs[g])
            assert np.array_equal(w.cpu().numpy(), w1.cpu().numpy(), equal_nan=True)
            assert np.array_equal(a.cpu().numpy(), a1.cpu().numpy(), equal_nan=True)
            if nsteps:
                assert torch.equal(got[g], d1)
