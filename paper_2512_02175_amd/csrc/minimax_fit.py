"""Fits the FP64 Box-Muller polynomials of mg_kernels.hip (neg2log_unit and
sincos_turn) by the Remez exchange algorithm, in 60-digit arithmetic
(mpmath), prints their coefficients, highest degree first, as the kernels
hold them, and writes their tables, mg_bm64.inc.  A development tool: nothing
imports it.

* logarithm: log1p(z) = z + z^2 q(z) on [-2^-8, 2^-7], q of degree 5, minimax
  for the relative error of log1p (weight z^2 / log1p(z) on q's error);
* sine on |x| <= pi/128: sin x = x + x^3 s(x^2), s of degree 2, weight x^2;
* cosine: cos x - 1 = x^2 c(x^2), c of degree 2, weight x^2;
* the logarithm's table: for interval i of 128 of the mantissa ([45/64 +
  i/256, + 1/256) below 1, steps of 1/128 from 1, i = 76, on) the double c
  near the reciprocal of its middle whose logarithm lies closest to a
  multiple of 2^-48, of the 20000 nearest (c = 1 for the intervals at 1), and
  that multiple of -2 log(1/c): its sum with k ln 2's first part, a multiple
  of 2^-32 below 32, is then exact.  In the seven intervals before those at 1,
  where -2 log u is smallest beside the constant and z, 200000 doubles 70001
  ulps apart are tried (the logarithms of neighbours, of c near 1, fall on few
  fractions of 2^-48), and in the last of them they lie just below the c that
  makes z = 2^-9 at its upper end, so that z passes 2^-9, where its rounding
  error doubles, only where -2 log u has passed 2^-6;
* the angle's table: for i of 128 the angle a near i/128 turns, a multiple
  of 2^-50, whose cosine and sine both lie within 2^-62 of a double (the
  nearest such a; a = 0 for i = 0), with those doubles.

The exchange runs on a dense Chebyshev grid: solve for the coefficients and
the levelled error E on n + 2 reference points, move the references to the
alternating extrema of the weighted error, repeat until the largest error
matches |E|.

    python minimax_fit.py
"""
import math
import os

import mpmath as mp

mp.mp.dps = 60


def remez(f, w, a, b, n, iters=40, grid=8000):
    xs = [a + (b - a) * (1 - mp.cos(mp.pi * i / (grid - 1))) / 2 for i in range(grid)]
    fx = [f(x) for x in xs]
    wx = [w(x) for x in xs]
    m = n + 2
    ref = [a + (b - a) * (1 - mp.cos(mp.pi * i / (m - 1))) / 2 for i in range(m)]
    coef, worst = None, None
    for _ in range(iters):
        A = mp.matrix(m, m)
        rhs = mp.matrix(m, 1)
        for i, x in enumerate(ref):
            for k in range(n + 1):
                A[i, k] = x ** k
            A[i, n + 1] = (-1) ** i / w(x)
            rhs[i] = f(x)
        sol = mp.lu_solve(A, rhs)
        coef, lev = [sol[k] for k in range(n + 1)], sol[n + 1]
        err = [wx[i] * (fx[i] - mp.polyval(coef[::-1], xs[i])) for i in range(grid)]
        worst = max(abs(e) for e in err)
        if abs(worst - abs(lev)) <= worst * mp.mpf("1e-8"):
            break
        ext = [i for i in range(grid)
               if i in (0, grid - 1) or (err[i] - err[i - 1]) * (err[i + 1] - err[i]) <= 0]
        alt = []
        for i in ext:
            if alt and mp.sign(err[i]) == mp.sign(err[alt[-1]]):
                if abs(err[i]) > abs(err[alt[-1]]):
                    alt[-1] = i
            else:
                alt.append(i)
        while len(alt) > m:
            alt.pop(0 if abs(err[alt[0]]) < abs(err[alt[-1]]) else -1)
        if len(alt) < m:
            break
        ref = [xs[i] for i in alt]
    return coef, worst


def log_table():
    rows = []
    for i in range(128):
        lo = 45 / 64 + i / 256 if i < 76 else 1 + (i - 76) / 128
        hi = lo + (1 / 256 if i < 76 else 1 / 128)
        best = (1.0, 0.0)
        if i not in (75, 76):
            mid, err = float(2 / (mp.mpf(lo) + mp.mpf(hi))), mp.inf
            if i == 74:
                mid = float((1 + mp.mpf(2) ** -9) / mp.mpf(hi) * (1 - mp.mpf("2e-6")))
            near1 = 68 <= i < 76
            step = math.ulp(mid) * (70001 if near1 else 1)
            for k in range(200000 if near1 else 20000):
                v = mid + (k + 1) // 2 * (1 if k % 2 else -1) * step
                scaled = -mp.ldexp(mp.log(mp.mpf(v)), 48)
                e = abs(scaled - mp.nint(scaled))
                if e < err:
                    err, best = e, (v, -2.0 * float(mp.ldexp(mp.nint(scaled), -48)))
        rows.append(best)
    return rows


def turn_table():
    one = 1 << 100                       # fixed point of the search
    rows = [(1.0, 0.0, 0.0)]

    def off(v):                          # distance of v / one from a double
        lsb = 1 << max(abs(v).bit_length() - 53, 0)
        return abs((v + lsb // 2) % lsb - lsb // 2)

    for i in range(1, 129):
        a0 = int(mp.nint(mp.ldexp(2 * mp.pi * i / 128, 50)))
        base = mp.ldexp(mp.mpf(a0), -50)
        c0, s0 = (int(mp.nint(v * one)) for v in (mp.cos(base), mp.sin(base)))
        for k in range(1 << 22):
            d = (k + 1) // 2 * (1 if k % 2 else -1)          # delta = d 2^-50
            q = d * d >> 1
            c = c0 - (s0 * d >> 50) - (c0 * q >> 100)
            n = s0 + (c0 * d >> 50) - (s0 * q >> 100)
            if off(c) < one >> 62 and off(n) < one >> 62:
                break
        a = mp.ldexp(mp.mpf(a0 + d), -50)
        rows.append((float(mp.cos(a)), float(mp.sin(a)), float(a)))
    return rows


HEAD = {
    "kLogTab": """// {c, -2 log(1/c)}: c close to the reciprocal of the middle of interval i of
// the mantissa, [45/64 + i/256, + 1/256) below 1 and steps of 1/128 from 1 (i
// = 76) on; c is the one among the nearest 20000 doubles whose logarithm is
// closest to a multiple of 2^-48 (for i = 68 .. 74 of others, minimax_fit.py),
// and 1 for the two intervals at 1.
""",
    "kTurnTab": """// {cos a, sin a, a}: a close to i/128 turns, such that its cosine and sine
// are within 2^-62 of doubles.
""",
}


def write_tables(path):
    with open(path, "w") as f:
        f.write("// mg_bm64.inc -- tables of the FP64 Box-Muller (neg2log_unit and "
                "sincos_turn\n// in mg_kernels.hip), printed by minimax_fit.py.\n")
        for name, rows in (("kLogTab", log_table()), ("kTurnTab", turn_table())):
            n, m = len(rows), len(rows[0])
            f.write(HEAD[name] + f"static __device__ const double {name}[{n}][{m}] = {{\n")
            for r in rows:
                f.write("    {" + ", ".join(float(v).hex() for v in r) + "},\n")
            f.write("};\n")


def main():
    tiny = mp.mpf("1e-40")
    half, X = mp.mpf(1) / 2, (mp.pi / 128) ** 2
    fits = {
        "logarithm q": (lambda z: (mp.log1p(z) - z) / z ** 2 if abs(z) > tiny else -half,
                        lambda z: z ** 2 / mp.log1p(z) if z != 0 else tiny,
                        -mp.mpf(2) ** -8, mp.mpf(2) ** -7, 5),
        "sine s": (lambda x: (mp.sin(mp.sqrt(x)) - mp.sqrt(x)) / (mp.sqrt(x) * x)
                   if x > 0 else -mp.mpf(1) / 6, lambda x: x if x > 0 else tiny, mp.mpf(0), X, 2),
        "cosine c": (lambda x: (mp.cos(mp.sqrt(x)) - 1) / x if x > 0 else -half,
                     lambda x: x if x > 0 else tiny, mp.mpf(0), X, 2),
    }
    for name, (f, w, a, b, n) in fits.items():
        coef, worst = remez(f, w, a, b, n)
        print(f"{name}: weighted error {mp.nstr(worst, 4)} (2^{mp.nstr(mp.log(worst, 2), 4)})")
        for c in coef[::-1]:
            print(f"  {float(c)!r}")
    write_tables(os.path.join(os.path.dirname(os.path.abspath(__file__)), "mg_bm64.inc"))


if __name__ == "__main__":
    main()
