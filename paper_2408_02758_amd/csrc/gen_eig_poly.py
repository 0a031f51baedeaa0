"""Coefficients of the 3x3 eigenvalue steps in ftle_device_math.h.

The largest eigenvalue of a symmetric 3x3 tensor is q + 2 p c, where c is
the largest root of 4 c^3 - 3 c = r, i.e. c = cos(acos(r) / 3) (the
trigonometric solution of the characteristic cubic).  With s = sqrt((1+r)/2)
this is c(s) = cos((2/3) acos(s)), an analytic function on [0, 1] (c(0) = 1/2,
c(1) = 1).  This script fits it by least squares in the Chebyshev basis on
[0, 1] (degree 7, 400001 samples) and prints the monomial coefficients for a
Horner evaluation in float32 (max error about 1.2e-7 in c).

For float64 (coefficients64) the polynomial is the Chebyshev economisation of
c's Taylor series about s = 1/2, in powers of u = s - S0 (whose coefficients
shrink, unlike those of powers of s), in rational arithmetic.  S0 lies next to
1/2 where the first two coefficients happen to be doubles to 1/100 of a rounding
(at 1/2 theirs biased c by 2.8e-17).  c satisfies
(1 - s^2) c'' - s c' + (4/9) c = 0, which gives the series from c(1/2) =
cos 40 deg (a root of 8 x^3 - 6 x + 1) and c'(1/2) = (2/3) sin 40 deg / sin 60 deg.
"""
from fractions import Fraction as Fr

import numpy as np

S0 = Fr(32768 - 278, 65536)


def coefficients(deg: int = 7):
    s = np.linspace(0.0, 1.0, 400001)
    c = np.cos(2.0 / 3.0 * np.arccos(s))
    fit = np.polynomial.chebyshev.Chebyshev.fit(s, c, deg, domain=[0, 1])
    poly = fit.convert(kind=np.polynomial.Polynomial, domain=[0, 1], window=[0, 1])
    return poly.coef, float(np.max(np.abs(poly(s) - c)))


def _round(x, bits=400):
    return Fr(round(x * (1 << bits)), 1 << bits)


def _newton(f, df, x):
    for _ in range(12):
        x = _round(x - f(x) / df(x))
    return x


def coefficients64(n: int = 20, terms: int = 60):
    """(coefficients of (s - S0)^0 .. (s - S0)^(n-1), sum of the dropped Chebyshev coefficients)."""
    c0 = _newton(lambda x: 8 * x ** 3 - 6 * x + 1, lambda x: 24 * x * x - 6, Fr(766, 1000))
    s0 = _newton(lambda x: x * x - (1 - c0 * c0), lambda x: 2 * x, Fr(643, 1000))
    sin60 = _newton(lambda x: x * x - Fr(3, 4), lambda x: 2 * x, Fr(866, 1000))
    a = [c0, Fr(2, 3) * s0 / sin60]
    for k in range(terms):      # the equation at s = 1/2 + u, power u^k
        v = ((k + 1) * k + Fr(1, 2) * (k + 1)) * a[k + 1] + (k * (k - 1) + k - Fr(4, 9)) * a[k]
        a.append(_round(v / (Fr(3, 4) * (k + 2) * (k + 1))))
    t = [[Fr(1)], [Fr(0), Fr(1)]]                  # Chebyshev polynomials of 2 u
    while len(t) < terms:
        c = [Fr(0)] + [2 * v for v in t[-1]]
        for i, v in enumerate(t[-2]):
            c[i] -= v
        t.append(c)
    p, cheb = [a[k] / 2 ** k for k in range(terms)], [Fr(0)] * terms
    for k in range(terms - 1, -1, -1):
        cheb[k] = p[k] / t[k][k]
        for i, v in enumerate(t[k]):
            p[i] -= cheb[k] * v
    out = [Fr(0)] * n
    for k in range(n):
        for i, v in enumerate(t[k]):
            out[i] += cheb[k] * v
    out = [v * 2 ** k for k, v in enumerate(out)]
    for i in range(n):                             # powers of s - 1/2 to powers of s - S0
        for k in range(n - 2, i - 1, -1):
            out[k] += (S0 - Fr(1, 2)) * out[k + 1]
    return [float(v) for v in out], float(sum(abs(v) for v in cheb[n:]))


if __name__ == "__main__":
    coef, err = coefficients64()
    print(f"// float64, powers of s - {float(S0)!r}; dropped terms {err:.1e}")
    for k, a in enumerate(coef):
        print(f"// u^{k}: {a!r}")
    coef, err = coefficients()
    print(f"// max |error| in float64: {err:.2e}")
    for k, a in enumerate(coef):
        print(f"constexpr float kEigC{k} = {a:.9e}f;")
