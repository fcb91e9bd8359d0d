"""The shape that the library chooses for tile index 0 changes no bit in any form of the interface kernel:
grids on both sides of the lines of the choice (tiles per compute unit with 8x28, 4x60 and 16x12 tiles), with
the GKS flux, SSP-RK3, the time limiter, the switch rules, component-wise reconstruction and the DF of the
first stage, in both element types, against every explicit shape."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2402_10914_amd import workloads as WL  # noqa: E402

pytestmark = pytest.mark.gpu

# 8x28 (one tile per unit), 4x60 (four against three), 16x12 (two against one), 8x28 (six each)
SIZES = [(160, 160), (300, 300), (1500, 9), (400, 390)]
FORMS = {"gks": dict(flux=1), "rk3": dict(time_scheme=1), "limiter": dict(flux=1, time_limiter=1), "min": dict(switch_rule=1),
         "own": dict(flux=1, switch_rule=2), "componentwise": dict(componentwise=1), "df_stage": dict(df_stage=1)}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("nx,ny", SIZES)
def test_chosen_shape_equals_every_explicit_shape(nx, ny, form, dtype):
    from paper_2402_10914_amd import api
    pr = WL.riemann4(nx, ny, seed=[4, nx])
    ref = None
    for tile in range(len(api.tile_shapes())):
        st = api.Stepper.for_problem(pr, api.Params(cfl=0.4, tile=tile, **FORMS[form]), dtype)
        W = torch.tensor(pr.W, dtype=dtype, device="cuda")
        A = torch.tensor(pr.alpha, dtype=dtype, device="cuda")
        t, fs = st.run(W, A, 2)
        L = st.rhs(W, A, 1e-4, want_alpha=True) if "time_scheme" not in FORMS[form] else ()
        out = [x.cpu().numpy() for x in (W, A, *L)] + [np.array([t, fs])]
        if ref is None:
            ref = out
        assert all(np.array_equal(x, y, equal_nan=True) for x, y in zip(out, ref)), tile
