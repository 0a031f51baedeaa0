"""Coefficients of the sine and cosine polynomials in ftle_advect.hip.

Lanczos' Chebyshev economisation, in exact rational arithmetic: the Taylor
series of each function in z (argument squared), truncated far below double
precision, is written in Chebyshev polynomials shifted to [0, zmax], cut after
n terms and written back in powers of z.  The printed bound is the sum of the
dropped Chebyshev coefficients' magnitudes.

  sin(pi r) / pi = r + r^3 P(r^2),  |r| <= 1/2     (8 terms)
  sin(r) = r + r^3 P(r^2),  |r| <= pi/4              (6 terms)
  cos(r) = 1 - r^2/2 + r^4 P(r^2),  |r| <= pi/4      (6 terms)
"""
from fractions import Fraction as Fr
from math import factorial

PI = Fr(31415926535897932384626433832795028841971693993751058209749445923078164062862090, 10 ** 79)
TERMS = 24


def shifted_chebyshev(n, zmax):
    """T_0..T_{n-1}(2 z / zmax - 1) as lists of powers of z."""
    u = [Fr(-1), Fr(2) / zmax]
    t = [[Fr(1)], u]
    while len(t) < n:
        a, b = t[-1], t[-2]
        c = [Fr(0)] * (len(a) + 1)
        for i, v in enumerate(a):
            c[i] += 2 * u[0] * v
            c[i + 1] += 2 * u[1] * v
        for i, v in enumerate(b):
            c[i] -= v
        t.append(c)
    return t


def economise(taylor, zmax, n):
    t = shifted_chebyshev(len(taylor), zmax)
    p, cheb = list(taylor), [Fr(0)] * len(taylor)
    for k in range(len(taylor) - 1, -1, -1):       # highest power first
        cheb[k] = p[k] / t[k][k]
        for i, v in enumerate(t[k]):
            p[i] -= cheb[k] * v
    out = [Fr(0)] * n
    for k in range(n):
        for i, v in enumerate(t[k]):
            out[i] += cheb[k] * v
    return out, sum(abs(c) for c in cheb[n:])


def main():
    eighth2 = (PI / 4) ** 2
    for name, taylor, zmax, n in (
            ("(sin(pi r) / (pi r) - 1) / r^2",
             [(-1) ** (k + 1) * PI ** (2 * k + 2) / factorial(2 * k + 3) for k in range(TERMS)], Fr(1, 4), 8),
            ("(sin(r) / r - 1) / r^2", [Fr((-1) ** (k + 1), factorial(2 * k + 3)) for k in range(TERMS)], eighth2, 6),
            ("(cos(r) - 1 + r^2/2) / r^4", [Fr((-1) ** k, factorial(2 * k + 4)) for k in range(TERMS)], eighth2, 6)):
        c, bound = economise(taylor, zmax, n)
        print(f"{name}: dropped terms <= {float(bound):.1e}")
        for k, v in enumerate(c):
            print(f"  z^{k}: {float(v)!r}")


if __name__ == "__main__":
    main()
