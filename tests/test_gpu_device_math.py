"""The device sequences that stand for IEEE divisions and square roots, against the IEEE results.

FP64 (``rcp_any``, ``sqrt_inv``): an estimate refined to a relative error far below the unit u = 2^-53 and
rounded by one fused operation, so 1/x and the root lie within one unit in the last place, and the root's
reciprocal, refined from the same estimate (its own final rounding, then the root's), within two; zero,
infinite, NaN and negative operands give the IEEE results, which the failing states of a run rely on.

FP64 quotient of a positive number (``quotient_any``): corrected by its residual, so within one unit too, and
exactly 1 for n / n; the same special operands.

FP32 (``cand::recip``, ``cand::root``): bit for bit the IEEE results for every argument, among them those
whose reciprocal or root the estimates alone miss (1/x subnormal or overflowing, roots of numbers below
2^-102, subnormal and negative subnormal ones)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import device_math  # noqa: E402

pytestmark = pytest.mark.gpu


def _arguments(dtype):
    """Ordinary operands over the exponents, both signs, and the values beside powers of two."""
    rng = np.random.default_rng(17)
    top = 1000 if dtype == np.float64 else 120
    x = np.ldexp(rng.uniform(1, 2, 200000), rng.integers(-top, top, 200000)).astype(dtype)
    p = np.ldexp(dtype(1), np.arange(-top, top)).astype(dtype)
    return np.concatenate([x, p, np.nextafter(p, dtype(0)), np.nextafter(p, dtype(np.inf))])


def _call(name, x, n_out):
    d = torch.from_numpy(x).cuda()
    out = [torch.empty_like(d) for _ in range(n_out)]
    torch.cuda.synchronize()
    assert getattr(device_math.load(), name)(d.data_ptr(), *[o.data_ptr() for o in out], d.numel()) == 0
    return [o.cpu().numpy() for o in out]


def _ulps(got, want):
    return np.max(np.abs(got - want) / np.spacing(np.abs(want)))


def test_f64_ordinary_operands():
    x = _arguments(np.float64)
    r, _, _ = _call("dm_f64", np.concatenate([x, -x]), 3)
    assert _ulps(r, 1.0 / np.concatenate([x, -x])) <= 1
    _, s, i = _call("dm_f64", x, 3)
    assert _ulps(s, np.sqrt(x)) <= 1
    assert _ulps(i, 1.0 / np.sqrt(x)) <= 2


SPECIAL = [0.0, -0.0, np.inf, -np.inf, np.nan]


def test_f64_special_operands():
    x = np.array(SPECIAL + [-1.0, -1e-300, -1e300])
    r, s, i = _call("dm_f64", x, 3)
    with np.errstate(all="ignore"):
        want = 1.0 / x, np.sqrt(x), 1.0 / np.sqrt(x)
    assert np.array_equal(r[:5], want[0][:5], equal_nan=True) and np.array_equal(np.signbit(r[:2]), np.signbit(want[0][:2]))
    assert _ulps(r[5:], want[0][5:]) <= 1
    assert np.array_equal(s, want[1], equal_nan=True)
    assert np.array_equal(i, want[2], equal_nan=True)


def test_f64_ends_of_the_range():
    # 1/x subnormal or overflowing, and the root of subnormal numbers: within the spacing there, or the
    # infinity that 1/x of the smallest numbers is
    x = np.array([5e-324, 1e-310, 2.0**-1030, 2.0**-1024, 2.0**-1023, 2.0**-1022, 2.0**1022, 2.0**1023, 1.7e308])
    r, s, i = _call("dm_f64", x, 3)
    with np.errstate(all="ignore"):
        want = 1.0 / x, np.sqrt(x), 1.0 / np.sqrt(x)
    fin = np.isfinite(want[0])
    assert np.array_equal(r[~fin], want[0][~fin])
    assert _ulps(r[fin], want[0][fin]) <= 1
    assert _ulps(s, want[1]) <= 1 and _ulps(i, want[2]) <= 2


@pytest.mark.parametrize("n", [1.0, 1.2**2, 1.4**2, (5.0 / 3.0) ** 2, 4.0])
def test_f64_quotient(n):
    x = np.concatenate([_arguments(np.float64), [n], SPECIAL])
    d = torch.from_numpy(x).cuda()
    q = torch.empty_like(d)
    torch.cuda.synchronize()
    assert device_math.load().dm_quotient(d.data_ptr(), q.data_ptr(), n, d.numel()) == 0
    q = q.cpu().numpy()
    k = len(x) - len(SPECIAL)
    assert q[k - 1] == 1.0
    assert _ulps(q[:k], n / x[:k]) <= 1
    with np.errstate(all="ignore"):
        assert np.array_equal(q[k:], n / x[k:], equal_nan=True)


def test_f32_special_operands():
    x = np.array(SPECIAL + [-1.0, -1e-30, -1e30], dtype=np.float32)
    r, s = _call("dm_f32", x, 2)
    with np.errstate(all="ignore"):
        assert np.array_equal(r, np.float32(1) / x, equal_nan=True)
        assert np.array_equal(np.signbit(r[:4]), np.signbit(x[:4]))
        assert np.array_equal(s, np.sqrt(x), equal_nan=True)


def test_f32_every_argument():
    bad = torch.zeros(2, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    assert device_math.load().dm_all_f32(bad.data_ptr()) == 0
    assert bad.tolist() == [0, 0]
