"""Coefficients of the cutoff polynomials used by the kernels.

fc(t) = (1 + cos(pi sqrt(t))) / 2 on t = r^2 / rc^2 in [0, 1], interpolated at
the Chebyshev points and converted to powers:
  FP32  degree 6 in t: max error 5.5e-9 in fc and 5.4e-7 in dfc/dt (FP32
        rounding 6e-8);
  FP64  degree 10 in t - 1/2, from long double: within 9e-17 in fc and 6e-15 in
        dfc/dt.  The nearest doubles of the coefficients leave fc too large by 6e-17
        of its mean over a sphere of neighbours, most of it from the constant term,
        which a sum of many terms shows; the first four are therefore rounded
        together, to leave the least mean (1.2e-17).  (Powers of t from double
        precision had 1.4e-15 and 1.7e-13, and a mean error of -2e-16.)
Prints the C++ initialisers pasted into common.h (FcPoly<float>, FcPoly<double>).

    python paper_2002_00054_amd/csrc/gen_cutoff.py
"""
import itertools

import numpy as np
from numpy.polynomial import chebyshev as C, polynomial as P

L = np.longdouble
PI = L("3.14159265358979323846264338327950288")


def fc(t):
    return (1 + np.cos(PI * np.sqrt(t))) / 2


def fit(deg):
    """Powers of t, in double precision."""
    ch = C.Chebyshev.interpolate(lambda x: 0.5 * (1 + np.cos(np.pi * np.sqrt(x))), deg, domain=[0, 1])
    return ch.convert(kind=P.Polynomial, domain=[0, 1], window=[0, 1]).coef


def fit_centred(deg):
    """Powers of t - 1/2, by Newton's divided differences in long double."""
    n = deg + 1
    u = np.cos(PI * (np.arange(n, dtype=L) + L(0.5)) / n) / 2
    d = fc(u + L(0.5))
    for k in range(1, n):
        d[k:] = (d[k:] - d[k - 1:-1]) / (u[k:] - u[:-k])
    p = np.zeros(n, dtype=L)
    p[0] = d[-1]
    for i in range(n - 2, -1, -1):
        q = np.roll(p, 1)
        q[0] = 0
        p = q - p * u[i]
        p[0] += d[i]
    return p.astype(np.float64)


def least_mean(c):
    """The first four coefficients one or two ulp away from the nearest doubles, so that
    the error's mean relative to fc's is least, the worst of several weights: points
    of a sphere (r^2 dr), less and more of them far out (e^{-b t})."""
    t = (np.arange(20000, dtype=L) + L(0.5)) / 20000
    u, f = t - L(0.5), fc(t)
    w = [np.sqrt(t) * np.exp(-L(b) * t) for b in (0, 0.4, 1.1, 2.5)]

    def mean(e):
        return np.array([float((x * e).sum() / (x * f).sum()) for x in w])

    base = mean(P.polyval(u, c.astype(L)) - f)
    ulp = np.spacing(np.abs(c[:4]))
    step = [mean(L(ulp[i]) * u ** i) for i in range(4)]
    k = min(itertools.product((-1, 0, 1), (-1, 0, 1), range(-2, 3), range(-2, 3)),
            key=lambda k: np.max(np.abs(base + sum(k[i] * step[i] for i in range(4)))))
    c = c.copy()
    c[:4] += k * ulp
    return c


def main():
    t = np.linspace(0, 1, 100001).astype(L)
    df = np.where(t > 0, -PI * np.sin(PI * np.sqrt(t)) / (4 * np.sqrt(np.maximum(t, L(1e-30)))), -PI ** 2 / 4)
    for name, c, u in (("float", fit(6), t), ("double", least_mean(fit_centred(10)), t - L(0.5))):
        f = P.polyval(u, c.astype(L))
        g = P.polyval(u, P.polyder(c.astype(L)))
        print("// FcPoly<%s>: degree %d, max |error| %.2e, of the derivative %.2e"
              % (name, len(c) - 1, np.max(np.abs(f - fc(t))), np.max(np.abs(g - df))))
        print("{" + ", ".join("%.17g" % x for x in c) + "}")


if __name__ == "__main__":
    main()
