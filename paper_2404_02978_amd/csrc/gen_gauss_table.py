"""Writes kGaussTab, the tables of the binary64 Gaussian generator (qrfs_f64.hip).

Entry i of 64:
  r, L   L = 2 ln r for the uniforms whose mantissa f in [1/2, 1) lies around
         c = 1/2 + (i + 1/2) / 128, with r close to 1/c.  L is a multiple of
         2^-44, so that it adds exactly to a multiple of the high part of
         2 ln 2 (one of 2^-44 too): of the multiples next to 2 ln(1/c) the one
         is taken whose e^(L/2) lies closest to a binary64 number, r.  r = 1
         and L = 0 in the last entry, so that uniforms next to 1 cancel
         nothing.
  s, c, s', c'   sin and cos of 2 pi (i + 1/2) / 64, each with the part that
         its rounding to binary64 left over.
mpmath at 60 digits.  Run:
    python gen_gauss_table.py      (prints the C++ constants)
"""
import mpmath as mp

mp.mp.dps = 60
GRID = 44
TRIES = 16384  # leaves |L - 2 ln r| below 2^-62


def log_entry(i):
    if i == 63:
        return 1.0, 0.0
    c = mp.mpf(1) / 2 + (i + mp.mpf(1) / 2) / 128
    n0 = int(mp.nint(mp.ldexp(-2 * mp.log(c), GRID)))
    step = mp.exp(mp.ldexp(1, -GRID - 1))
    x = mp.exp(mp.ldexp(n0 - TRIES // 2, -GRID - 1))
    best = None
    for n in range(n0 - TRIES // 2, n0 + TRIES // 2):
        r = float(x)
        err = abs(mp.mpf(r) / x - 1)
        if best is None or err < best[0]:
            best = (err, r, n)
        x *= step
    return best[1], float(mp.ldexp(best[2], -GRID))


def pair(x):
    hi = float(x)
    return hi, float(x - mp.mpf(hi))


if __name__ == "__main__":
    for i in range(64):
        r, L = log_entry(i)
        a = 2 * mp.pi * (i + mp.mpf(1) / 2) / 64
        s, sl = pair(mp.sin(a))
        c, cl = pair(mp.cos(a))
        print("    {%r, %r, %r, %r,\n     %r, %r}," % (r, L, s, c, sl, cl))
    l2 = 2 * mp.log(2)
    hi = mp.ldexp(mp.nint(mp.ldexp(l2, GRID)), -GRID)
    print("2 ln 2 = %r + %r" % (float(hi), float(l2 - hi)))
    print("2 pi = %r + %r" % pair(2 * mp.pi))
