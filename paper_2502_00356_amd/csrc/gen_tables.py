"""Writes bk_tables.inc: the constant tables of libbesselk as device constants,
so that no call has to set anything up on the GPU.

  kRuleTab   strip half-widths a_k = (pi/2) 2^(-k/2) and (pi/2)(1 - 2^(-k/2)),
             k = 1..8 (15 distinct values), with 1 - cos a_k and log sec a_k
             (node-count rule); 2^(j/64), j = 0..63 (table-driven exponential);
             log(1 + j/64) and 1 / (1 + j/64), j = 0..64 (table-driven log1p).
  kTemmeTab  Taylor coefficients, in mu^2, of Temme's
             Gamma1(mu) = (1/Gamma(1 - mu) - 1/Gamma(1 + mu)) / (2 mu) and
             Gamma2(mu) = (1/Gamma(1 - mu) + 1/Gamma(1 + mu)) / 2 (both even in mu);
             ten terms leave below 4e-18 at |mu| = 1/2.

Every value is computed in mpmath at 60 digits and rounded to the nearest double.
Run: python gen_tables.py (rewrites bk_tables.inc beside this file).
"""
import os

import mpmath as mp

mp.mp.dps = 60
HERE = os.path.dirname(os.path.abspath(__file__))
RULE_CAND = 15
TEMME_TERMS = 10


def dbl(v):
    return float.hex(float(mp.mpf(v)))


def half_widths():
    vals = []
    for k in range(1, 9):
        f = mp.power(2, -mp.mpf(k) / 2)
        for c in (mp.pi / 2 * f, mp.pi / 2 * (1 - f)):
            if all(abs(c - v) > mp.mpf("1e-15") for v in vals):
                vals.append(c)
    assert len(vals) == RULE_CAND, len(vals)
    return vals


def temme_taylor():
    """Coefficients of mu^(2k), k < TEMME_TERMS: 1/Gamma(1 + mu) = sum_n c_n mu^n gives
    Gamma1 = -sum c_(2k+1) mu^(2k) and Gamma2 = sum c_(2k) mu^(2k)."""
    c = mp.taylor(lambda z: mp.rgamma(1 + z), 0, 2 * TEMME_TERMS)
    return [-c[2 * k + 1] for k in range(TEMME_TERMS)], [c[2 * k] for k in range(TEMME_TERMS)]


def fmt(vals, per_line=4):
    items = [dbl(v) for v in vals]
    lines = [", ".join(items[i:i + per_line]) for i in range(0, len(items), per_line)]
    return "{\n        " + ",\n        ".join(lines) + "}"


def main():
    a = half_widths()
    omc = [1 - mp.cos(v) for v in a]
    lsec = [-mp.log(mp.cos(v)) for v in a]
    tab = [mp.power(2, mp.mpf(j) / 64) for j in range(64)]
    tab += [mp.log1p(mp.mpf(j) / 64) for j in range(65)]
    tab += [1 / (1 + mp.mpf(j) / 64) for j in range(65)]
    g1, g2 = temme_taylor()
    text = ("// Generated by gen_tables.py (mpmath, 60 digits, rounded to double); do not edit.\n"
            "// Constant tables of the device code; see gen_tables.py for their definitions.\n"
            "static __constant__ RuleTable kRuleTab = {\n"
            "    " + fmt(a) + ",\n    " + fmt(omc) + ",\n    " + fmt(lsec) + ",\n    " + fmt(tab) + "};\n\n"
            "static __constant__ TemmeCoef kTemmeTab = {\n"
            "    " + fmt(g1) + ",\n    " + fmt(g2) + "};\n")
    with open(os.path.join(HERE, "bk_tables.inc"), "w") as f:
        f.write(text)


if __name__ == "__main__":
    main()
