"""Writes expint_consts.h: E_3(x) for 0 < x <= 1 by its power series and for
x > 1 as e^{-x} / x g(1/x), g by a polynomial on each octave of x.

The polynomials interpolate g at Chebyshev nodes; g itself is the continued
fraction x / (x + 3 - 3 / (x + 5 - 8 / (x + 7 - ...))), i (i + 2) in the i-th
numerator, evaluated backwards in 80-bit arithmetic.

Run:  python gen_expint_consts.py > expint_consts.h
"""
import math

import numpy as np

LD = np.longdouble
DEGREE, OCTAVES = 18, 5          # [1, 2), [2, 4), [4, 8), [8, 16), [16, inf)


def g(y):
    """x e^x E_3(x) at x = 1/y (1 at y = 0)."""
    if y == 0:
        return LD(1)
    x, n = LD(1) / y, 1200
    b = x + LD(3 + 2 * n)
    for i in range(n, 0, -1):
        b = x + LD(3 + 2 * (i - 1)) - LD(i * (i + 2)) / b
    return x / b


def octave(o):
    """Monomial coefficients in t = 2 (y - lo) / (hi - lo) - 1, lowest first."""
    hi = LD(0.5) ** o
    lo = LD(0) if o == OCTAVES - 1 else hi / 2
    n = DEGREE + 1
    k = np.arange(n)
    t = np.cos(LD('3.14159265358979323846264338327950288') * (2 * k + 1).astype(LD) / LD(2 * n))
    f = np.array([g(lo + (hi - lo) * (v + 1) / 2) for v in t], dtype=LD)
    c = [LD(2) / n * np.sum(f * np.cos(j * np.arccos(t))) for j in range(n)]
    c[0] /= 2
    mono, a, b = np.zeros(n, LD), np.zeros(n, LD), np.zeros(n, LD)      # T_j by its recurrence
    a[0] = 1
    mono += c[0] * a
    b[1] = 1
    mono += c[1] * b
    for j in range(2, n):
        r = -a
        r[1:] += 2 * b[:-1]
        a, b = b, r
        mono += c[j] * b
    return mono


def main():
    print("// Generated by gen_expint_consts.py: constants of E_3(x).\n#pragma once\n")
    print("// x <= 1: E_3 = 1/2 - x + x^2/2 (3/2 - gamma - ln x) + x^3 (c_0 + c_1 x + ...)")
    s = [-((-1.0) ** k) / ((k - 2) * math.factorial(k)) for k in range(3, 19)]
    print("#define PZ_E3_PSI %s" % repr(1.5 - 0.57721566490153286061))
    print("#define PZ_E3_SERIES_N %d\n#define PZ_E3_SERIES \\\n    %s\n" % (len(s), ", ".join(repr(v) for v in s)))
    print("// x > 1: rows of %d monomials, octave 0 first" % (DEGREE + 1))
    print("#define PZ_E3_OCTAVES %d\n#define PZ_E3_DEGREE %d\n#define PZ_E3_TABLE \\" % (OCTAVES, DEGREE))
    for o in range(OCTAVES):
        print("    %s%s" % (", ".join(repr(float(v)) for v in octave(o)), ", \\" if o + 1 < OCTAVES else ""))


if __name__ == "__main__":
    main()
