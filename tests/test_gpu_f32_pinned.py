"""FP32 runs bit for bit: states, DF and times of small runs and operators in every form of the kernels, against
hashes recorded from the FP32 kernels as they first were (``golden/f32_runs.json``, written by running this
file as a script).  Callers read FP32 times in double and follow them step by step, so a last bit that moves
in a state moves every later time step; the compiler chooses which products of a sum to fuse, and this is what
holds that choice.  Inputs are made with additions, multiplications and divisions only, the same bits
everywhere."""
import hashlib
import json
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "f32_runs.json")
FORMS = {"lf": {}, "lf_limiter": dict(time_limiter=1), "rk3": dict(time_scheme=1), "lf_comp": dict(componentwise=1),
         "lf_min": dict(switch_rule=1), "lf_own": dict(switch_rule=2), "lf_df1": dict(df_stage=1),
         "gks": dict(flux=1), "gks_limiter": dict(flux=1, time_limiter=1), "gks_comp": dict(flux=1, componentwise=1),
         "gks_own": dict(flux=1, switch_rule=2), "gks_df1": dict(flux=1, df_stage=1)}
# name: cells, boundary (0 periodic, 1 transmissive)
GRIDS = {"smooth": (53, 41, 0), "jumps": (48, 64, 1), "strip": (90, 3, 0), "rest": (33, 20, 1)}


def _state(name):
    """W [4, ny, nx] and alpha [ny, nx] in FP64."""
    nx, ny, bc = GRIDS[name]
    x = (np.arange(nx) + 0.5)[None, :] / nx + np.zeros((ny, 1))
    y = (np.arange(ny) + 0.5)[:, None] / ny + np.zeros((1, nx))
    b = 16 * x * (1 - x) * y * (1 - y)  # one smooth bump, zero on the border
    rho, u, v, p = 1 + 0.25 * b, 0.5 - 0.125 * b, 0.25 * b, 1 + 0.5 * b * b
    if name == "jumps":
        q = (x < 0.55).astype(float) + 2 * (y < 0.45)
        rho, u = 0.5 + 0.375 * q, 0.75 - 0.5 * (q == 1)
        v, p = 0.25 * (q == 2) - 0.5 * (q == 3), 0.25 + 0.625 * q * q
    if name == "rest":
        u = v = 0 * x
        rho, p = 1 + 0 * x, np.where(x < 0.5, 1.0, 0.1)
    W = np.stack([rho, rho * u, rho * v, p / 0.4 + 0.5 * rho * (u * u + v * v)])
    return W, 1 - 0.75 * (((np.arange(nx)[None, :] * 7 + np.arange(ny)[:, None] * 3) % 11) < 2)


def _hash(*tensors):
    """Of the bits, every NaN the same."""
    parts = [torch.where(torch.isnan(t), torch.full_like(t, float("nan")), t) for t in tensors]
    return hashlib.sha1(b"".join(t.cpu().numpy().tobytes() for t in parts)).hexdigest()[:16]


def _run(grid, form):
    from paper_2402_10914_amd import api
    nx, ny, bc = GRIDS[grid]
    W0, A0 = _state(grid)
    st = api.Stepper(nx, ny, 1.0 / nx, 1.0 / ny, bc, None, api.Params(cfl=0.4, **FORMS[form]), torch.float32)
    W = torch.tensor(W0, dtype=torch.float32, device="cuda")
    A = torch.tensor(A0, dtype=torch.float32, device="cuda")
    out = [] if "time_scheme" in FORMS[form] else [_hash(*st.rhs(W, A, 1e-3, want_alpha=True))]
    t, fail = st.run(W, A, 6)
    return out + [_hash(W, A), float(t).hex(), fail]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("grid", GRIDS)
def test_bits(grid, form):
    with open(GOLDEN) as f:
        assert _run(grid, form) == json.load(f)[f"{grid}/{form}"]


if __name__ == "__main__":
    import sys
    with open(sys.argv[1], "w") as f:
        f.write("{\n" + ",\n".join(json.dumps(f"{g}/{m}") + ": " + json.dumps(_run(g, m)) for g in GRIDS for m in FORMS) + "\n}\n")
