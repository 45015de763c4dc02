"""Derives the polynomial coefficients of the device exp2 and log2 (lbm_device.hpp).

Both are Chebyshev interpolation fits computed here in 60-digit arithmetic
(mpmath.chebyfit), rounded to double, then checked on a dense grid:

  exp2: R(f) ~ (2^f - 1) / f on |f| <= 1/2, so 2^f = 1 + f R(f), R of
        degree 10.
  log2: Q(w) ~ (2 atanh(z) / (z ln 2) - 2 / ln 2) / w with w = z^2 on
        [0, 0.02944] (z = (m - 1)/(m + 1) for m between the double with high
        word 0x3fe6a09e, just below sqrt(1/2), and twice it), so
        log2 m = z (c0 + w Q(w)) with c0 = 2 / ln 2 rounded to double, Q of
        degree 6.

Prints the C++ initialisers and the worst relative error of each
approximation with the double coefficients (evaluated exactly), which must
stay far below one ulp (1.1e-16).  Run: python3 gen_poly.py
"""
import struct

import mpmath as mp

mp.mp.dps = 60


def fit(f, a, b, deg):
    coef, _ = mp.chebyfit(f, [a, b], deg + 1, error=True)
    return [float(c) for c in coef]  # highest degree first


def horner(c, x):
    acc = mp.mpf(c[0])
    for k in c[1:]:
        acc = acc * x + mp.mpf(k)
    return acc


def worst(full, approx, a, b, n=20001):
    w = mp.mpf(0)
    for i in range(n):
        x = a + (b - a) * mp.mpf(i) / (n - 1)
        ref = full(x)
        w = max(w, abs(approx(x) - ref) / abs(ref))
    return w


def main():
    ln2 = mp.log(2)
    A = mp.mpf("0.5000001")

    def R(f):
        return (mp.power(2, f) - 1) / f if f != 0 else ln2

    ce = fit(R, -A, A, 10)
    err_e = worst(lambda f: mp.power(2, f), lambda f: 1 + f * horner(ce, f),
                  -A, A)

    lo = mp.mpf(struct.unpack(">d", bytes.fromhex("3fe6a09e00000000"))[0])
    zmax = max(abs((m - 1) / (m + 1)) for m in (lo, 2 * lo))
    W = zmax**2 * (1 + mp.mpf("1e-9"))
    c0 = float(2 / ln2)

    def Q(w):
        if w == 0:
            return 2 / ln2 / 3
        z = mp.sqrt(w)
        return (2 * mp.atanh(z) / ln2 / z - 2 / ln2) / w

    cl = fit(Q, mp.mpf(0), W, 6)

    def log2_approx(z):
        w = z * z
        return z * (mp.mpf(c0) + w * horner(cl, w))

    err_l = worst(lambda z: 2 * mp.atanh(z) / ln2, log2_approx,
                  mp.mpf("1e-8"), zmax)

    print("// exp2: R(f), degree 10, highest first; worst rel. error %.2e" % err_e)
    for c in ce:
        print("  %s," % float(c).hex())
    print("// log2: Q(w), degree 6, highest first, then c0; worst rel. error %.2e"
          % err_l)
    for c in cl + [c0]:
        print("  %s," % float(c).hex())


if __name__ == "__main__":
    main()
