"""Writes csrc/fp64_tables.hpp: the tables of the double-precision Box-Muller
map (fp64_math.hpp).  Run once by hand; the library build reads only the
header.

LOG_TABLE: 256 cells of z in [0.70801, 1.41602), cut on the high word of its
double, (hi - LOG_OFFSET) >> 12; a cell holds (1/c, -2 ln c), 1/c a double next
to the inverse of the cell's centre, chosen among 600 neighbours so that
-2 ln c lies within about a thousandth of an ulp of a double (the accurate
tables of S. Gal and B. Bachelis, ACM TOMS 17(1), 1991).  LOG_OFFSET puts 1.0
in the middle of a cell whose c is exactly 1, so that ln z keeps its relative
precision as z -> 1.
TRIG_TABLE: (cos, sin) of 2 pi i / 256.

Usage: python -m paper_2309_10477_amd.gen_fp64_tables
"""
from __future__ import annotations

import math
import os
import struct
from decimal import Decimal, getcontext

getcontext().prec = 40
HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "csrc", "fp64_tables.hpp")
LOG_OFFSET = 0x3FE6A800
PI = Decimal("3.14159265358979323846264338327950288419716939937510582097494459")


def from_high_word(hi: int) -> float:
    """The double with high word hi and a zero low word."""
    return struct.unpack(">d", struct.pack(">II", hi, 0))[0]


def log_row(i: int):
    lo = from_high_word(LOG_OFFSET + (i << 12))
    hi = from_high_word(LOG_OFFSET + ((i + 1) << 12))
    if lo < 1.0 < hi:
        return 1.0, 0.0
    centre, best = 2.0 / (lo + hi), None
    for k in range(600):
        inv = centre * (1.0 + k * 2.0 ** -40)
        exact = 2 * Decimal(inv).ln()
        off = abs(Decimal(float(exact)) - exact) / Decimal(math.ulp(float(exact)))
        if best is None or off < best[0]:
            best = (off, inv, float(exact))
    return best[1:]


def cos_sin(i: int):
    """(cos, sin) of 2 pi i / 256, exact at the quadrants, by Taylor series in one octant."""
    q, r = divmod(i, 64)
    x = PI * r / 128

    def series(first):
        term, total, k = (Decimal(1), Decimal(1), 0) if first == 0 else (x, x, 1)
        for _ in range(40):
            term = -term * x * x / ((k + 1) * (k + 2))
            total += term
            k += 2
        return total

    c, s = (Decimal(1), Decimal(0)) if r == 0 else (series(0), series(1))
    c, s = [(c, s), (-s, c), (-c, -s), (s, -c)][q]
    return float(c) + 0.0, float(s) + 0.0


def table(name: str, rows) -> str:
    body = "".join("    {%s, %s},\n" % tuple(float(v).hex() for v in row) for row in rows)
    return f"__device__ const double {name}[256][2] = {{\n{body}}};\n"


def main():
    text = ("// Generated by gen_fp64_tables.py.\n#pragma once\n\nnamespace heston {\n\n"
            f"constexpr uint32_t LOG_OFFSET = {LOG_OFFSET:#010x}u;\n"
            + table("LOG_TABLE", [log_row(i) for i in range(256)])
            + table("TRIG_TABLE", [cos_sin(i) for i in range(256)])
            + "\n} // namespace heston\n")
    with open(OUT, "w") as f:
        f.write(text)


if __name__ == "__main__":
    main()
