"""Generate pt_crtables.h: constants of the correctly rounded log1p / expm1 / log.

Every value is computed in 90-digit decimal arithmetic and split into a
double-double (hi = the nearest double, lo = the nearest double to the rest),
printed as exact hexadecimal floating-point literals.

  log:  m in [sqrt(1/2), sqrt(2)] is reduced by c_j = RN(256/j), j = round(256 m);
        LOG_C[j-181] = c_j and LOG_L[j-181] = -ln(c_j) (double-double, of the exact c_j).
  exp:  EXP_T[j] = 2^(j/128), j = 0..127 (double-double).
  LN2 (double-double); ln2/128 = C1 + C2 + C3 with C1 holding 33 significant bits so
  that K*C1 is exact for |K| < 2^20; INV = RN(128/ln2).
  INVK[k] = 1/k and INVF[k] = 1/k! (double-double) for the polynomial steps.

  First phase (lean): LEAN_LOG[i] = {c, Lh, Ll} for the 256 cells of [0x1.6ap-1, 0x1.6ap0) that share the
  leading eight mantissa bits: c = RN(1/centre) -- 1 in the two cells next to 1 -- and -ln(c) =
  Lh + Ll with Lh a multiple of 2^-42, so that k LN2_42 + Lh is exact; LN2_42 is ln2 rounded to
  2^-42, LN2_42L the rest.  LOG_V / EXP_V: the polynomials V of log1p(r) = r + r^2 V(r) and
  e^r - 1 = r + r^2 V(r), interpolated at the Chebyshev nodes of the reduced range.

Run:  python paper_2302_13590_amd/csrc/gen_crtables.py
"""
import decimal
import math
import os
import struct

D = decimal.Decimal
decimal.getcontext().prec = 90

LOG_J0, LOG_J1 = 181, 362       # round(256*sqrt(1/2)) .. round(256*sqrt(2))


def dd(v: decimal.Decimal):
    h = float(v)                 # correctly rounded
    lo = float(v - D(h))
    return h, lo


def hx(x: float) -> str:
    if x == 0.0:
        return "0x0p+0"
    return float.hex(x)


def trunc_bits(x: float, keep: int) -> float:
    """x with only its `keep` leading significant bits."""
    b = struct.unpack("<Q", struct.pack("<d", x))[0]
    drop = 52 - (keep - 1)
    b &= ~((1 << drop) - 1)
    return struct.unpack("<d", struct.pack("<Q", b))[0]


def split42(v: decimal.Decimal):
    """v as a multiple of 2^-42 (a double) and the double nearest to the rest."""
    h = float((v * D(2) ** 42).to_integral_value()) * 2.0 ** -42
    return h, float(v - D(h))


def cheb_poly(f, lo: float, hi: float, deg: int):
    """Coefficients (lowest first, rounded to double) of the polynomial of degree deg that
    interpolates f at the Chebyshev nodes of [lo, hi]."""
    n = deg + 1
    x = [D((lo + hi) / 2 + (hi - lo) / 2 * math.cos(math.pi * (2 * i + 1) / (2 * n))) for i in range(n)]
    m = [[x[i] ** j for j in range(n)] + [f(x[i])] for i in range(n)]
    for i in range(n):
        for r in range(n):
            if r != i:
                q = m[r][i] / m[i][i]
                m[r] = [a - q * b for a, b in zip(m[r], m[i])]
    return [float(m[i][n] / m[i][i]) for i in range(n)]


def log_v(r: decimal.Decimal):
    """(log1p(r) - r) / r^2 by its series (|r| <= 2^-7)."""
    return sum((D(-1) ** (k + 1) / k) * r ** (k - 2) for k in range(2, 60))


def exp_v(r: decimal.Decimal):
    """(e^r - 1 - r) / r^2 by its series."""
    return sum(r ** (k - 2) / D(math.factorial(k)) for k in range(2, 40))


def main():
    ln2 = D(2).ln()
    lines = ["// Generated by gen_crtables.py -- do not edit.",
             "// Constants of the correctly rounded log1p / expm1 / log (double-double hi, lo).",
             "#pragma once", ""]
    lines.append("#define PT_CR_LOG_J0 %d" % LOG_J0)
    lines.append("#define PT_CR_LOG_J1 %d" % LOG_J1)
    c_vals, l_vals = [], []
    for j in range(LOG_J0, LOG_J1 + 1):
        c = 256.0 / j                                    # correctly rounded double of 256/j
        c_vals.append(c)
        l_vals.append(dd(-(D(c).ln())))
    lines.append("PT_CR_TABLE double PT_CR_LOG_C[%d] = {" % len(c_vals))
    lines += ["    %s," % hx(c) for c in c_vals]
    lines.append("};")
    lines.append("PT_CR_TABLE double PT_CR_LOG_L[%d][2] = {" % len(l_vals))
    lines += ["    {%s, %s}," % (hx(h), hx(lo)) for h, lo in l_vals]
    lines.append("};")
    lines.append("PT_CR_TABLE double PT_CR_EXP_T[128][2] = {")
    for j in range(128):
        h, lo = dd((ln2 * j / 128).exp())
        lines.append("    {%s, %s}," % (hx(h), hx(lo)))
    lines.append("};")
    h, lo = dd(ln2)
    lines.append("#define PT_CR_LN2_H %s" % hx(h))
    lines.append("#define PT_CR_LN2_L %s" % hx(lo))
    q = ln2 / 128
    c1 = trunc_bits(float(q), 33)
    c2 = float(q - D(c1))
    c3 = float(q - D(c1) - D(c2))
    lines.append("#define PT_CR_LN2_128_1 %s" % hx(c1))
    lines.append("#define PT_CR_LN2_128_2 %s" % hx(c2))
    lines.append("#define PT_CR_LN2_128_3 %s" % hx(c3))
    lines.append("#define PT_CR_INV_LN2_128 %s" % hx(float(128 / ln2)))
    lines.append("#define PT_CR_SQRT2 %s" % hx(math.sqrt(2.0)))
    n = 24
    lines.append("PT_CR_TABLE double PT_CR_INVK[%d][2] = {" % n)
    lines.append("    {0x0p+0, 0x0p+0},")
    for k in range(1, n):
        a, b = dd(D(1) / k)
        lines.append("    {%s, %s}," % (hx(a), hx(b)))
    lines.append("};")
    lines.append("PT_CR_TABLE double PT_CR_INVF[%d][2] = {" % n)
    for k in range(n):
        a, b = dd(D(1) / math.factorial(k))
        lines.append("    {%s, %s}," % (hx(a), hx(b)))
    lines.append("};")
    lines.append("#define PT_CR_LEAN_OFF 0x3fe6a000   // high word of 0x1.6ap-1")
    lines.append("PT_CR_TABLE double PT_CR_LEAN_LOG[256][3] = {")
    for i in range(256):
        bits = 0x3fe6a000 + (i << 12)
        lo = struct.unpack("<d", struct.pack("<Q", bits << 32))[0]
        hi = struct.unpack("<d", struct.pack("<Q", (bits + 0x1000) << 32))[0]
        c = 1.0 if lo == 1.0 or hi == 1.0 else 1.0 / ((lo + hi) / 2)
        h, lw = split42(-(D(c).ln()))
        lines.append("    {%s, %s, %s}," % (hx(c), hx(h), hx(lw)))
    lines.append("};")
    h, lw = split42(ln2)
    lines.append("#define PT_CR_LN2_42 %s" % hx(h))
    lines.append("#define PT_CR_LN2_42L %s" % hx(lw))
    for name, f, lo, hi, deg in (("LOG_V", log_v, -1.02 * 2.0 ** -9, 1.02 * 2.0 ** -8, 5),
                                 ("EXP_V", exp_v, -float(ln2) / 256 * 1.001, float(ln2) / 256 * 1.001, 4)):
        for k, v in enumerate(cheb_poly(f, lo, hi, deg)):
            lines.append("#define PT_CR_%s%d %s" % (name, k, hx(v)))
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "pt_crtables.h")
    with open(path, "w") as f:
        f.write("\n".join(lines) + "\n")
    print(path)


if __name__ == "__main__":
    main()
