"""The step's double-precision functions on the device (ems_math.hpp): errors
against long double over the ranges the transport uses, square roots and
quotients against the correctly rounded ones; the largest errors are printed.

Bounds.  Logarithm, exponential, sine and cosine: those of the host check of
the same polynomials (half a unit for the last rounding and a third for the
terms before it; the same and the rounding of 1 + r over half a binade; one
rounding each of the angle and the polynomial).  Square root: correctly rounded
while the residual of its last correction is exact, that is from 2^-968 (106
bits above the smallest number); below, the residual's rounding (half of
2^-1074, over twice the root) adds at most half a unit down to the smallest
normal number.  Quotients: correctly rounded while residual, quotient and
reciprocal stay normal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 1 << 20


@pytest.fixture(scope="module")
def E():
    import paper_2209_15445_amd as E
    return E


def on_device(E, function, a, b=None):
    import torch
    d = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()
    e = None if b is None else torch.from_numpy(np.ascontiguousarray(b, dtype=np.float64)).cuda()
    return E.debug_device_math(function, d, e).cpu().numpy()


def worst(got, exact):
    """largest error in units in the last place of the exact value"""
    unit = np.spacing(np.abs(exact.astype(np.float64)))
    return float(np.max(np.abs((got - exact).astype(np.float64)) / unit))


def powers(g, n, lo, hi):
    """random fractions times 2^lo .. 2^hi, and every power of two between"""
    v = np.ldexp(1.0 + g.random(n), g.integers(lo, hi, n))
    return np.concatenate([v, np.ldexp(1.0, np.arange(lo, hi + 1))])


def test_logarithm(E):
    g = np.random.default_rng(1)
    draws = np.concatenate([g.random(N), [2.0**-53, 1 - 2.0**-53, 0.5]])
    x = np.concatenate([np.exp(g.random(N) * 40 - 14), draws[draws > 0], powers(g, N, -1022, 1023),
                        1 + (g.random(N) - 0.5) * 2.0 ** (-40 * g.random(N))])
    exact = np.log(x.astype(np.longdouble))
    got = on_device(E, "log", x)
    one = exact == 0
    assert np.all(got[one] == 0)
    w = worst(got[~one], exact[~one])
    print(f"log of {len(x)} numbers: {w:.3f} units", flush=True)
    assert w < 0.84


def test_exponential(E):
    g = np.random.default_rng(2)
    x = np.concatenate([(g.random(N) - 0.5) * 60, -8 * g.random(N), (g.random(N) - 0.5) * 1400, [0.0, -0.0, 709.0]])
    w = worst(on_device(E, "exp", x), np.exp(x.astype(np.longdouble)))
    print(f"exp of {len(x)} numbers: {w:.3f} units", flush=True)
    assert w < 0.9
    assert np.array_equal(on_device(E, "exp", [-1e6, -800.0]), [0.0, 0.0])


def test_sine_and_cosine_of_a_turn(E):
    g = np.random.default_rng(3)
    u = np.concatenate([g.random(2 * N), np.arange(0, 65) / 64.0, [2.0**-53, 1 - 2.0**-53]])
    t = 2 * np.arccos(np.longdouble(-1)) * u.astype(np.longdouble)
    w = max(float(np.abs(on_device(E, "sin_turn", u) - np.sin(t)).max()),
            float(np.abs(on_device(E, "cos_turn", u) - np.cos(t)).max()))
    print(f"sine and cosine of {len(u)} turns: {w:.3g}", flush=True)
    assert w < 2.3e-16


def test_square_root(E):
    g = np.random.default_rng(4)
    v = np.concatenate([powers(g, 2 * N, -968, 1023), 1 - g.random(N) * 2.0**-20, [0.0]])
    assert np.array_equal(on_device(E, "sqrt", v), np.sqrt(v))
    low = powers(g, N, -1022, -968)
    w = worst(on_device(E, "sqrt", low), np.sqrt(low.astype(np.longdouble)))
    print(f"square roots below 2^-968: {w:.3f} units", flush=True)
    assert w <= 1.0
    # (below the normal numbers some bits remain)
    tiny = powers(g, N, -1074, -1022)
    r = on_device(E, "sqrt", tiny) / np.sqrt(tiny) - 1
    print(f"square roots of subnormal numbers: {np.abs(r).max():.3g} relative", flush=True)
    assert np.all(np.abs(r) < 2.0**-40)
    assert np.array_equal(on_device(E, "sqrt", [np.inf]), [np.inf])
    assert np.isnan(on_device(E, "sqrt", [-1.0, np.nan])).all()


def test_quotients(E):
    g = np.random.default_rng(5)
    a, b = powers(g, 2 * N, -400, 400), powers(g, 2 * N, -400, 400)
    a *= np.where(g.random(len(a)) < 0.5, -1, 1)
    assert np.array_equal(on_device(E, "quotient", a, b), a / b)
    assert np.array_equal(on_device(E, "quotient", np.zeros(4), [1.0, 3.0, 1e-30, 1e30]), np.zeros(4))
    f, h = powers(g, 2 * N, -50, 50).astype(np.float32), powers(g, 2 * N, -50, 50).astype(np.float32)
    assert np.array_equal(on_device(E, "quotient_f32", f, h), (f / h).astype(np.float64))
