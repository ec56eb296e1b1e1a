"""The double-precision Box-Muller map of the path kernels: its generated
tables, and the map evaluated from them on the CPU as the kernels do (the same
cells, series and order, an FMA rounded twice), against numpy's long double at
the uniforms where it can go wrong: both edges of every table cell in every
binade, the smallest and the largest uniform, the neighbours of 1 and of the
zeros of the cosine and sine."""
import os
import re

import numpy as np
import pytest

HDR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2309_10477_amd", "csrc", "fp64_tables.hpp")
M_MAX = (1 << 23) - 1  # a uniform is (m + 1/2) 2^-23, m the top 23 bits of a word


def table(name):
    body = re.search(name + r"\[256\]\[2\] = \{(.*?)\n\};", open(HDR).read(), re.S).group(1)
    v = [float.fromhex(x) for x in re.findall(r"-?0x[0-9a-f.]+p[+-]\d+", body)]
    return np.array(v).reshape(256, 2)


def offset():
    return int(re.search(r"LOG_OFFSET = (0x[0-9a-f]+)u", open(HDR).read()).group(1), 16)


def neg2_log(m):
    d = ((m.astype(np.uint64) << np.uint64(1)) | np.uint64(1)).astype(np.float64)
    bits = d.view(np.uint64)
    t = (bits >> np.uint64(32)).astype(np.int64) - offset()
    row = table("LOG_TABLE")[(t >> 12) & 255]
    hi = ((t & 0xFFFFF) + offset()).astype(np.uint64)
    z = ((hi << np.uint64(32)) | (bits & np.uint64(0xFFFFFFFF))).view(np.float64)
    L = np.longdouble  # the two FMAs whose single rounding matters
    r = (L(z) * row[:, 0] - 1).astype(np.float64)
    h = (L(24 - (t >> 20)) * 1.38629436111989061883 + row[:, 1]).astype(np.float64)
    p = r * (1.0 / 3.0) - 0.4
    for c in (0.5, -2.0 / 3.0, 1.0, -2.0):
        p = r * p + c
    assert np.abs(r).max() < 2.0 ** -8.9
    return r * p + h


def cos_sin(m):
    row = table("TRIG_TABLE")[((m + (1 << 14)) >> 15) & 255]
    low = ((m & 0x7FFF) ^ 0x4000) - 0x4000
    d = (low + 0.5) * (2 * np.pi * 2.0 ** -23)
    q = d * d
    sd = d + d * q * (-1 / 6 + q * (1 / 120 - q / 5040))
    cd = q * (-0.5 + q * (1 / 24 - q / 720))
    C, S = row[:, 0], row[:, 1]
    return C + (C * cd - S * sd), S + (S * cd + C * sd)


def log_points():
    edges = []
    for i in range(257):
        z = np.array([offset() + (i << 12)], np.uint64) << np.uint64(32)
        for k in range(25):
            e = int(np.floor(z.view(np.float64)[0] * 2.0 ** k)) // 2
            edges += [e - 1, e, e + 1]
    m = np.array(edges + list(range(64)) + [M_MAX - k for k in range(64)])
    return np.unique(m[(m >= 0) & (m <= M_MAX)])


def test_radius():
    m = log_points()
    u = (m.astype(np.longdouble) + np.longdouble(0.5)) * np.longdouble(2) ** -23
    want = -2 * np.log(u)
    rel = np.abs(neg2_log(m) - want) / want
    # three roundings of the sum and its parts, the constant and the second FMA rounding
    assert rel.max() < 4 * 2.0 ** -52


@pytest.mark.parametrize("half", [0, 1])
def test_angle(half):
    i = np.arange(256)[:, None] * (1 << 15) + (half << 14) + np.arange(-8, 9)
    m = np.unique(i.ravel() % (1 << 23))
    c, s = cos_sin(m)
    # octant-reduced reference, exact quarter turns
    L = np.longdouble
    u = (m.astype(L) + L(0.5)) * L(2) ** -23
    quarter = np.floor(4 * u + L(0.5))
    y = 2 * np.arccos(L(-1)) * (u - quarter / 4)
    k = quarter.astype(int) % 4
    cy, sy = np.cos(y), np.sin(y)
    want_c = np.choose(k, [cy, -sy, -cy, sy])
    want_s = np.choose(k, [sy, cy, -sy, -cy])
    assert np.abs(c - want_c).max() < 2 * 2.0 ** -52
    assert np.abs(s - want_s).max() < 2 * 2.0 ** -52
    # next to their zeros the values keep their relative precision
    near = np.abs(want_c) < 1e-5
    if half == 0:
        assert near.any() and (np.abs(c - want_c)[near] < 8 * 2.0 ** -52 * np.abs(want_c)[near]).all()
