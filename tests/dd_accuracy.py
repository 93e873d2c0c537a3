"""Arguments and bars for the double-double operations of ddmath.hpp, shared by the tests of their
host and device builds.

Bars, u = 2^-53, in units of u^2 of the result: a sum or product rounds by up to 3.
 * a/b: the remainder's low part two roundings of at most 1, the last sum 1: 3; 4 asked.
 * sqrt: one correction of a root from a reciprocal root within 3.5 u leaves 3.5^2 / 2 = 6 and its own
   rounding 4 x 3.5 = 14: 20 (two corrections leave less).
 * log: two sums (6), and of atanh t, a quotient (4) and a sum (3), what it is of the whole, at most
   all of it once: 13; 14 asked.  On top the error of the table entry and of e ln 2 as double pairs, which
   just below 1 (e = -1, table entry near ln 2) are large against the result.
 * atan(a/b): the quotient's numerator and denominator (two products, two sums: 12) and itself (4)
   scale t, at most half of the result or all of it; two sums (6) and pi/2: 24."""
import mpmath as mp
import numpy as np

U2 = mp.mpf(2) ** -106


def _pairs(x, rng, rel):
    lo = x * rng.uniform(-rel, rel, len(x))
    hi = x + lo
    return np.stack([hi, lo - (hi - x)], axis=1)


def arguments():
    """{name: (fn, (n, 4) array of a and b)}; fn as in pic_devcheck_dd."""
    rng = np.random.default_rng(3)
    n = 1500

    def logu(lo, hi, m=n):
        return np.exp(rng.uniform(np.log(lo), np.log(hi), m))

    steps = (rng.integers(0, 1024, n) + 0.5) / 1024
    one = np.ones(n)
    raw = {
        "log": (0, logu(1e-8, 1e8), one),
        "log at half steps": (0, 1 + steps, one),
        "log just below 1": (0, 1 - logu(2.0 ** -12, 2.0 ** -9), one),
        "log nearer below 1": (0, 1 - logu(1e-14, 2.0 ** -12), one),
        "log just above 1": (0, 1 + logu(1e-14, 2.0 ** -9), one),
        "atan": (1, logu(1e-12, 1e12), logu(1e-8, 1e4)),
        "atan at half steps": (1, steps * 0.75, 0.75 * one),
        "atan near 0": (1, logu(2.0 ** -13, 2.0 ** -9), one),
        "atan near 1": (1, 1 + rng.uniform(-1e-3, 1e-3, n), one),
        "sqrt": (2, logu(1e-16, 1e8), one),
        "quotient": (3, logu(1e-8, 1e8, 10 * n), logu(1e-8, 1e8, 10 * n)),
    }
    return {k: (fn, np.ascontiguousarray(np.concatenate([_pairs(a, rng, 5e-17),
                                                         _pairs(b, rng, 5e-17)], axis=1)))
            for k, (fn, a, b) in raw.items()}


def _pair_error(v):
    hi = mp.mpf(float(v))
    return abs(v - hi - mp.mpf(float(v - hi)))


def _log_tables(a):
    e = int(mp.floor(mp.log(a, 2)))
    c = 1 + mp.mpf(int(round((float(a * mp.mpf(2) ** -e) - 1) * 1024))) / 1024
    return _pair_error(mp.log(c)) + abs(e) * _pair_error(mp.log(2)) + (
        abs(e) > 1) * abs(e) * mp.mpf(2) ** -108  # e ln 2 is exact for e = 0 and -1


def worst(fn, arg, out):
    """The largest error over its bar."""
    mp.mp.dps = 60
    w = mp.mpf(0)
    for row, o in zip(arg, out):
        a, b = mp.mpf(row[0]) + mp.mpf(row[1]), mp.mpf(row[2]) + mp.mpf(row[3])
        ref = (mp.log(a), mp.atan(a / b), mp.sqrt(a), a / b)[fn]
        bar = (14, 24, 20, 4)[fn] * U2 * abs(ref) + (_log_tables(a) if fn == 0 else 0)
        w = max(w, abs(mp.mpf(o[0]) + mp.mpf(o[1]) - ref) / bar)
    return float(w)
