"""Writes kashin_tables.h: cos/sin of 2*pi*m/R for the radices other than powers of two that the
FFT kernels use, and
the orthonormal DCT-II matrices of the odd lengths the incoherence rotation uses.

Run: python gen_tables.py > kashin_tables.h   (values are correctly rounded to float)
"""
import math

RADICES = (3, 5, 7, 25, 43)
OUTER = (16, 20, 24, 32)  # outer radices with e^{i pi q / R} tables (compact eps factors)


def fmt(v):
    """%.9e of v, with the values that are exactly zero (cos and sin at odd multiples of pi/2,
    which the double-precision library returns as about 1e-16) written as 0, so that the kernels'
    compile-time tests for zero constants skip them."""
    return "%.9ef" % (0.0 if abs(v) < 1e-12 else v)


print("// Generated by gen_tables.py: cos/sin(2*pi*m/R), m in [0, R), rounded to float.")
print("#pragma once")
print("namespace kashin {")
print("template <int R> struct CisTab;")
for r in RADICES:
    c = ", ".join(fmt(math.cos(2 * math.pi * m / r)) for m in range(r))
    s = ", ".join(fmt(math.sin(2 * math.pi * m / r)) for m in range(r))
    print("template <> struct CisTab<%d> {" % r)
    print("  static constexpr float c[%d] = {%s};" % (r, c))
    print("  static constexpr float s[%d] = {%s};" % (r, s))
    print("};")
# orthonormal DCT-II of odd length B, row-major [k][j]:
# sqrt(2/B) * (1/sqrt(2) if k == 0 else 1) * cos(pi (2j+1) k / (2B))
print("template <int B> struct DctTab;")
for b in (3, 43):
    vals = []
    for k in range(b):
        for j in range(b):
            v = math.sqrt(2.0 / b) * math.cos(math.pi * (2 * j + 1) * k / (2 * b))
            if k == 0:
                v /= math.sqrt(2.0)
            vals.append(fmt(v))
    print("template <> struct DctTab<%d> {" % b)
    print("  static constexpr float m[%d] = {%s};" % (b * b, ", ".join(vals)))
    print("};")
print("// cos/sin(pi q / R), q in [0, R)")
print("template <int R> struct HalfTab;")
for r in OUTER:
    c = ", ".join(fmt(math.cos(math.pi * q / r)) for q in range(r))
    s = ", ".join(fmt(math.sin(math.pi * q / r)) for q in range(r))
    print("template <> struct HalfTab<%d> {" % r)
    print("  static constexpr float c[%d] = {%s};" % (r, c))
    print("  static constexpr float s[%d] = {%s};" % (r, s))
    print("};")
print("}  // namespace kashin")
