"""Derive the constants of trig.h: the argument reduction from pi itself, and
the polynomial coefficients by Remez's exchange method.

pi is computed to 120 decimal digits with Machin's formula in integer
arithmetic; pi/2 is the sum of three doubles, each the nearest one to what the
ones before it leave.  The polynomials minimise the largest error of the function they
stand for over their interval (E. Ya. Remez, 1934): with f given by its
rational Taylor series, each round solves w(x_i) (P(x_i) - f(x_i)) =
(-1)^i E at the current points exactly, and moves the points to the extrema
of the weighted error.  Prints C++ hex-float literals and each fit's error.
"""
from fractions import Fraction
from math import factorial


def arctan_inv(x, digits):
    """arctan(1/x) * 10^digits, integer arithmetic."""
    scale = 10 ** (digits + 10)
    total, term, n, sign = 0, scale // x, 1, 1
    while term:
        total += sign * (term // n)
        term //= x * x
        n += 2
        sign = -sign
    return total // 10 ** 10


def pi_fraction(digits=120):
    return Fraction(16 * arctan_inv(5, digits) - 4 * arctan_inv(239, digits), 10 ** digits)


def evaluate(coeffs, x):
    v = Fraction(0)
    for c in reversed(coeffs):
        v = v * x + c
    return v


def solve(a, b):
    """Gaussian elimination over the rationals."""
    n = len(b)
    m = [row[:] + [v] for row, v in zip(a, b)]
    for i in range(n):
        p = next(r for r in range(i, n) if m[r][i] != 0)
        m[i], m[p] = m[p], m[i]
        for r in range(i + 1, n):
            f = m[r][i] / m[i][i]
            if f:
                m[r] = [u - f * v for u, v in zip(m[r], m[i])]
    x = [Fraction(0)] * n
    for i in reversed(range(n)):
        x[i] = (m[i][n] - sum(m[i][j] * x[j] for j in range(i + 1, n))) / m[i][i]
    return x


def dyadic(x, bits=60):
    return Fraction(round(x * 2 ** bits), 2 ** bits)


def remez(f, weight, top, terms, rounds=8, grid=400):
    """Coefficients c[0..terms) minimising max |weight (P - f)| on (0, top], and
    that maximum; f and weight map a rational to a rational."""
    import math
    pts = [dyadic(Fraction(top) * Fraction(0.5 - 0.5 * math.cos(math.pi * (i + 0.5) / (terms + 1))))
           for i in range(terms + 1)]
    xs = [dyadic(Fraction(top) * Fraction(i, grid), 40) for i in range(1, grid + 1)]
    fx, wx = [f(x) for x in xs], [weight(x) for x in xs]
    for _ in range(rounds):
        a, b = [], []
        for i, x in enumerate(pts):
            w = weight(x)
            a.append([w * x ** j for j in range(terms)] + [Fraction(-1) ** (i + 1)])
            b.append(w * f(x))
        c = [dyadic(v, 160) for v in solve(a, b)[:terms]]
        err = [float(w * (evaluate(c, x) - v)) for x, v, w in zip(xs, fx, wx)]
        runs, k = [], 0  # the largest error of every run of one sign
        for i in range(1, len(err) + 1):
            if i == len(err) or (err[i] > 0) != (err[k] > 0):
                runs.append(max(range(k, i), key=lambda j: abs(err[j])))
                k = i
        while len(runs) > terms + 1:
            runs.pop(min(range(len(runs)), key=lambda j: abs(err[runs[j]])))
        if len(runs) < terms + 1:
            break
        pts = [xs[j] for j in runs]
    return c, max(abs(e) for e in err)


def series(coeff, terms=14):
    cs = [coeff(n) for n in range(terms)]
    return lambda x: evaluate(cs, x)


def tan_coeffs(n):
    """Taylor coefficients of tan x in odd powers: t[k] of x^(2k+1)."""
    s = [Fraction((-1) ** k, factorial(2 * k + 1)) for k in range(n)]
    c = [Fraction((-1) ** k, factorial(2 * k)) for k in range(n)]
    t = []
    for k in range(n):
        t.append(s[k] - sum(t[j] * c[k - j] for j in range(k)))
    return t


def show(prefix, coeffs, err, first=1):
    for i, c in enumerate(coeffs):
        v = float(c)
        print(f"constexpr double {prefix}{i + first} = {v.hex()};  // {v!r}")
    print(f"// {prefix}: largest error {err:.3g}")


def main():
    pi = pi_fraction()
    half_pi = pi / 2
    hi = Fraction(float(half_pi))
    lo = Fraction(float(half_pi - hi))
    tail = float(half_pi - hi - lo)
    for name, v in (("kPio2Hi", float(hi)), ("kPio2Lo", float(lo)), ("kPio2Tail", tail),
                    ("kTwoOverPi", float(1 / half_pi))):
        print(f"constexpr double {name} = {v.hex()};  // {v!r}")
    # sin r = r + r w P(w), cos r = 1 - w/2 + w^2 Q(w), w = r^2, |r| <= pi/4
    # (a little more for the rounding of the quadrant): relative and absolute
    quarter = dyadic((pi / 4 * (1 + Fraction(1, 2 ** 20))) ** 2, 40)
    sin_f = series(lambda n: Fraction((-1) ** (n + 1), factorial(2 * n + 3)))
    cos_f = series(lambda n: Fraction((-1) ** n, factorial(2 * n + 4)))
    show("S", *remez(sin_f, lambda w: w, quarter, 6))
    show("C", *remez(cos_f, lambda w: w * w, quarter, 6))
    # sin d = d (1 + w P(w)), tan(d/2) = d (1/2 + w Q(w)): absolute errors
    # over |d| <= top, d weighted by its largest value there
    t = tan_coeffs(16)
    tan_f = series(lambda n: t[n + 1] / 2 ** (2 * n + 3))
    for top, terms, names in ((Fraction(1, 64), 2, ("T", "U")), (Fraction(1, 8), 4, ("V", "W"))):
        wt = lambda w, top=top: w * top  # noqa: E731
        show(names[0], *remez(sin_f, wt, top * top, terms))
        show(names[1], *remez(tan_f, wt, top * top, terms))


if __name__ == "__main__":
    main()
