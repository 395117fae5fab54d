"""The warm start's two-body solve over its range: eccentricities up to 0.98, steps from zero
over many revolutions forward and backward, against Kepler's equation solved by bisection in
long double.  The bar follows from the arithmetic: the anomaly change is off by a few ulp of the
angle n dt, and the state by that times its velocity along the orbit, largest at perihelion
(|v| r0 / r_p ~ 2 / (1 - e) of the mean)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _reference(y0, dt):
    """States after dt (mu = 1) in long double."""
    ld = np.longdouble
    y0, dt = y0.astype(ld), dt.astype(ld)
    r, v = y0[:, :3], y0[:, 3:]
    r0 = np.sqrt((r * r).sum(1))
    al = 2 / r0 - (v * v).sum(1)
    a = 1 / al
    n = al * np.sqrt(al)
    sig = (r * v).sum(1)
    ec, es = 1 - r0 * al, sig / np.sqrt(a)
    lo, hi = n * dt - 2, n * dt + 2          # F rises and |x - n dt| <= 2e
    for _ in range(90):
        x = (lo + hi) / 2
        up = x - ec * np.sin(x) + es * (1 - np.cos(x)) - n * dt > 0
        hi, lo = np.where(up, x, hi), np.where(up, lo, x)
    s, c = np.sin(x), np.cos(x)
    rn = a + (r0 - a) * c + sig * np.sqrt(a) * s
    f, g = 1 - a / r0 * (1 - c), dt - (x - s) / n
    fd, gd = -np.sqrt(a) * s / (rn * r0), 1 - a / rn * (1 - c)
    return np.concatenate([f[:, None] * r + g[:, None] * v, fd[:, None] * r + gd[:, None] * v], axis=1)


@pytest.mark.parametrize("e_max", [0.0, 0.3, 0.8, 0.98])
@pytest.mark.parametrize("dt_max", [1e-3, 0.5, 6.0, 60.0])
def test_kepler_step_over_its_range(e_max, dt_max):
    from paper_2301_03989_amd import build, pcprop
    from paper_2301_03989_amd import workloads as W
    build.ensure_built()
    rng = np.random.default_rng([int(100 * e_max), int(1000 * dt_max)])
    n = 700
    a, e = rng.uniform(0.3, 3.0, n), e_max * rng.uniform(0.9, 1.0, n)
    y0 = W.elements_to_states(a, e, *(rng.uniform(0.0, 2 * np.pi, n) for _ in range(4)))
    dt = rng.uniform(-dt_max, dt_max, n)
    y, ok = pcprop.Context(0).eval_kepler(torch.tensor(y0.T.copy(), device="cuda"), torch.tensor(dt, device="cuda"))
    assert ok.cpu().numpy().all()
    ref = _reference(y0, dt)
    d = np.abs(y.cpu().numpy().T - ref.astype(np.float64))
    rp = a * (1.0 - e)
    angle = 1.0 + np.abs(dt) * a ** -1.5      # rounding of n dt and of x
    bar = 64 * 2.2e-16 * angle / (1.0 - e) ** 2
    assert (d[:, :3].max(1) <= bar * a * (1 + e)).all(), (d[:, :3].max(1) / (bar * a)).max()
    assert (d[:, 3:].max(1) <= bar * np.sqrt(2.0 / rp)).all(), (d[:, 3:].max(1) / (bar * np.sqrt(2.0 / rp))).max()


@pytest.mark.parametrize("dt_max", [1e4, 3e7])
def test_kepler_step_over_many_revolutions(dt_max):
    test_kepler_step_over_its_range(0.6, dt_max)
