"""Writes bk_cheb.inc: cos(n pi (j + 1/2) / M) and the monomial coefficients of the
Chebyshev polynomials T_n, n < M, for M = 5 and 9 (40 digits, rounded to double)."""
import os

import mpmath as mp

mp.mp.dps = 40


def monomials(M):
    T = [[1], [0, 1]]
    while len(T) < M:
        a = [0] + [2 * v for v in T[-1]]
        T.append([x - (T[-2][i] if i < len(T[-2]) else 0) for i, x in enumerate(a)])
    return [[t[k] if k < len(t) else 0 for k in range(M)] for t in T]


def rows(vals):
    return "{" + ",\n ".join("{" + ", ".join(r) + "}" for r in vals) + "}"


def main():
    out = ["// made by gen_cheb.py"]
    for M in (5, 9):
        cosn = [["%r" % float(mp.cos(n * mp.pi * (j + mp.mpf(1) / 2) / M)) if 2 * j + 1 != M or n % 2 == 0 else "0.0"
                 for j in range(M)] for n in range(M)]
        mono = [["%d.0" % v for v in r] for r in monomials(M)]
        out.append("static __constant__ const ChebTab<%d> kCheb%d = {\n%s,\n%s};" % (M, M, rows(cosn), rows(mono)))
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "bk_cheb.inc"), "w") as f:
        f.write("\n".join(out) + "\n")


if __name__ == "__main__":
    main()
