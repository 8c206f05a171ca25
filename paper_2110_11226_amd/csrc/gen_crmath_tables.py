"""Writes gp_crmath_tables.h: the constant tables of the correctly rounded
float32 sin, cos and log in gp_crmath.h, computed with mpmath at 200 bits.

  * kSinCosTab: sin and cos of k pi/128, k = 0..255, rounded to double (the
    sine of 0 is -0, so that sin(-0) = -0 comes out of the same operations);
  * kLogTab: 256 entries indexed by the top 8 bits of a float's mantissa m in
    [1, 2): c (1 / the bucket's centre rounded to float, 1 for the first
    bucket and 1/2 for the last; held as a double, exactly) and L = -log(c)
    for buckets below sqrt(2), -log(2c) from there on (the mantissa is then
    halved and the exponent raised by one), rounded to double;
  * NUDGE below: entries moved by an ulp of the double, each because one
    input's double evaluation otherwise falls on the wrong side of a float
    rounding boundary (crmath_check.cpp, run over every float, finds such
    inputs and shows that the moved tables have none left);
  * kSinExc, kCosExc, kLogExc: the inputs (float bits of |x|, or of x for
    log) whose double evaluation rounds to the wrong float, with their
    correctly rounded results.  They are found by crmath_check.cpp, which runs
    the header's functions over every float; `python gen_crmath_tables.py
    exceptions.txt` folds its list in (one "op bits result" line each).

Run from this directory: python gen_crmath_tables.py [exceptions.txt]
"""
import math
import struct
import sys

import mpmath as mp

mp.mp.prec = 200


def f32(v):
    return struct.unpack("f", struct.pack("f", float(v)))[0]


# (table, entry, column) -> ulps.  (These inputs have large exponents, where an
# ulp of the sum is many of L; near E = 0 such an L is still within 2^-45 of
# -log c, and the exhaustive check finds no input of the bucket rounded wrongly.)
NUDGE = {
    ("log", 130, 1): 8,     # 0x3c413d3a
    ("log", 186, 1): 128,     # 0x4c5d65a5
    ("log", 177, 1): 192,     # 0x65d890d3
    ("log", 99, 1): 128,     # 0x6f31a8ec
}


def nudged(table, i, col, v):
    for _ in range(abs(NUDGE.get((table, i, col), 0))):
        v = math.nextafter(v, math.inf if NUDGE[table, i, col] > 0 else -math.inf)
    return v


def log_table():
    rows = []
    for i in range(256):
        centre = 1 + (i + mp.mpf(0.5)) / 256
        if i == 0:
            c = mp.mpf(1)
        elif i == 255:
            c = mp.mpf(0.5)
        else:
            c = mp.mpf(f32(1 / centre))
        L = -mp.log(2 * c) if i >= 106 else -mp.log(c)
        rows.append((float(c), nudged("log", i, 1, float(L))))
    return rows


def sincos_table():
    rows = []
    for k in range(256):
        a = k * mp.pi / 128
        s, c = (0.0 if k % 128 == z else float(f(a)) for f, z in ((mp.sin, 0), (mp.cos, 64)))
        rows.append((-0.0 if k == 0 else nudged("sincos", k, 0, s), nudged("sincos", k, 1, c)))
    return rows


def main():
    exc = {"sin": [], "cos": [], "log": []}
    if len(sys.argv) > 1:
        for line in open(sys.argv[1]):
            parts = line.split()
            if len(parts) == 3 and parts[0] in exc:
                exc[parts[0]].append((int(parts[1], 0), int(parts[2], 0)))
    out = ["// Generated by gen_crmath_tables.py (mpmath, 200 bits); do not edit.",
           "#pragma once", "", "#include <cstdint>", "", "namespace gp {", "namespace crm {", "",
           "struct alignas(16) LogEntry {", "    double c;     // 1 / bucket centre (a float value)",
           "    double hi;    // L = -log(c) or -log(2c), rounded", "};", ""]
    out.append("struct alignas(16) SinCosEntry {")
    out.append("    double s;     // sin(k pi/128), rounded")
    out.append("    double c;     // cos(k pi/128), rounded")
    out.append("};")
    out.append("")
    out.append("GP_CRTAB SinCosEntry kSinCosTab[256] = {")
    for sv, cv in sincos_table():
        out.append("    {%s, %s}," % (sv.hex(), cv.hex()))
    out.append("};")
    out.append("")
    out.append("GP_CRTAB LogEntry kLogTab[256] = {")
    for c, hi in log_table():
        out.append("    {%s, %s}," % (c.hex(), hi.hex()))
    out.append("};")
    for name in ("sin", "cos", "log"):
        rows = sorted(set(exc[name]))
        out.append("")
        out.append(f"constexpr int k{name.capitalize()}ExcN = {len(rows)};")
        out.append(f"GP_CRTAB uint32_t k{name.capitalize()}Exc[{max(len(rows), 1)}][2] = {{")
        for a, b in rows:
            out.append("    {0x%08xu, 0x%08xu}," % (a, b))
        if not rows:
            out.append("    {0xffffffffu, 0u},")
        out.append("};")
    out += ["", "}  // namespace crm", "}  // namespace gp", ""]
    with open("gp_crmath_tables.h", "w") as f:
        f.write("\n".join(out))


if __name__ == "__main__":
    main()
