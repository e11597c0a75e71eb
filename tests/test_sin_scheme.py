"""The sin and cos used by the HIP kernels, evaluated step by step in float32
(double for the reduction of large arguments), stay within 1.5 ulp of the
exact values over the whole float range."""
from fractions import Fraction as F

import numpy as np
import pytest

f32, f64 = np.float32, np.float64
PIECES = [0xa2f9836, 0xe4e4415, 0x29fc275, 0x7d1f534, 0xddc0db6, 0x295993c, 0x439041f, 0xe5163ab]
HALF_PI = [float.fromhex(h) for h in ("0x1.921fb6p+0", "-0x1.777a5cp-25", "-0x1.ee59dap-50")]


def pi_fraction(bits=500):
    one = 1 << bits

    def arctan_inv(n):
        t = one // n
        s, k, sign = t, 1, -1
        while t:
            t //= n * n
            k += 2
            s += sign * (t // k)
            sign = -sign
        return s
    return F(4 * (4 * arctan_inv(5) - arctan_inv(239)), one)


def fma(a, b, c):
    return (a.astype(f64) * f64(b) + f64(c)).astype(f32)


def polynomials(r, k):
    u = (r * r).astype(f32)
    p = np.full_like(r, f32(2.7557319223985893e-6))
    for c in (-1.9841269841269841e-4, 8.3333333333333333e-3, -1.6666666666666667e-1):
        p = (u.astype(f64) * p + f64(f32(c))).astype(f32)
    s = ((r * u).astype(f32).astype(f64) * p + r).astype(f32)
    q = np.full_like(r, f32(-2.7557319223985888e-7))
    for c in (2.4801587301587302e-5, -1.3888888888888889e-3, 4.1666666666666667e-2, -0.5, 1.0):
        q = (u.astype(f64) * q + f64(f32(c))).astype(f32)
    a, b = np.where(k & 1, q, s), np.where(k & 1, s, q)
    return np.where(k & 2, -a, a), np.where((k + 1) & 2, -b, b)


def sincos_small(x):
    k = np.rint((x * f32(0.63661977236758134)).astype(f32))
    r = x
    for c in HALF_PI:
        r = fma(-k, c, r)
    return polynomials(r, k.astype(np.int64))


def sincos_large(x):
    p = np.zeros(x.shape, f64)
    for i, c in enumerate(PIECES):
        t = x.astype(f64) * (c * 2.0 ** (-28 * (i + 1)))
        p += t - 4 * np.rint(t * 0.25)
    k = np.rint(p)
    return polynomials(((p - k) * 1.5707963267948966).astype(f32), k.astype(np.int64))


def test_constants_are_those_of_pi():
    pi = pi_fraction()
    rest = pi / 2
    for c in HALF_PI:
        assert f32(float(rest)) == f32(c)
        rest -= F(c)
    rest = 2 / pi
    for i, c in enumerate(PIECES):
        assert c == int(rest * (1 << 28 * (i + 1)))
        rest -= F(c, 1 << 28 * (i + 1))


def ulps(got, ref):
    return np.abs(got.astype(f64) - ref) / np.spacing(np.abs(ref).astype(f32)).astype(f64)


def test_within_1_5_ulp_below_65536():
    rng = np.random.default_rng(3)
    for lim in (1e-3, 0.8, 1.6, 7.0, 300.0, 65536.0):
        x = rng.uniform(-lim, lim, 400_000).astype(f32)
        s, c = sincos_small(x)
        assert ulps(s, np.sin(x.astype(f64))).max() < 1.5
        assert ulps(c, np.cos(x.astype(f64))).max() < 1.5


def test_large_arguments():
    pi = pi_fraction()
    rng = np.random.default_rng(4)
    x = (10.0 ** rng.uniform(4.82, 38.5, 4000)).astype(f32)
    x[::2] *= -1
    s, c = sincos_large(x)
    red = [F(float(v)) - 2 * pi * round(F(float(v)) / (2 * pi)) for v in x]
    red = np.array([float(v) for v in red])
    assert ulps(s, np.sin(red)).max() < 1.5
    assert ulps(c, np.cos(red)).max() < 1.5


@pytest.mark.gpu
def test_kernels_follow_the_scheme_over_the_float_range():
    """One hidden layer of two neurons that pass x and y on: the query returns
    sin of the coordinates themselves."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    import workloads as wl
    print("sin over the float range", flush=True)
    pb = wl.tiny(dim=2, width=2, depth=1, n_pde=16, n_obs=4, n_gh=0, n_anc=1, seed=1)
    pb.activation = "sin"
    pb.subs[0].theta[:] = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 1, 0, 0, 0, 0, 0], f32)
    rng = np.random.default_rng(6)
    x = np.zeros((2000, 3), f32)
    x[:, 0] = rng.uniform(-100, 100, 2000)
    x[:, 1] = 10.0 ** rng.uniform(-6, 38, 2000)
    pi = pi_fraction()
    red = np.array([float(F(float(v)) - 2 * pi * round(F(float(v)) / (2 * pi))) for v in x[:, 1]])
    ctx = P.context_from_problem(pb, device="cuda")
    try:
        got = ctx.query(torch.from_numpy(x).cuda(), sub=0, what="value").cpu().numpy()
    finally:
        ctx.close()
    assert ulps(got[:, 0], np.sin(x[:, 0].astype(f64))).max() < 1.5
    assert ulps(got[:, 1], np.sin(red)).max() < 1.5
