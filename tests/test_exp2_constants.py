"""Host checks of the constants behind the line passes' 2^r (k_common.h): the polynomial of
2^r - 1 over r, and c2 / ln 2 in two parts, against mpmath."""
import os
import re

import mpmath as mp

HDR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2609_17273_amd", "csrc", "k_common.h")
NUM = r"(-?[0-9][0-9.e+-]*)"


def _body(name):
    text = open(HDR).read()
    start = text.index(name)
    return text[start:text.index("\n}\n", start)]


def test_exp2_polynomial():
    """12 Chebyshev points on [-1/2, 1/2] leave 2^r at most 4.3e-18 (ln 2^12 sqrt 2 / 2^23 12!), a
    constant term of 1 in place of theirs as much again; coefficients in 53 bits at most
    2^-53 sum c_k 2^-k = 2^-53 (sqrt 2 - 1) = 4.6e-17."""
    body = _body("double exp2m1_over(double r)")
    c = [mp.mpf(float(v)) for v in re.findall(r"double p = " + NUM, body) + re.findall(r"fma\(p, r, " + NUM, body)]
    assert len(c) == 11
    with mp.workdps(40):
        for i in range(-500, 501):
            r = mp.mpf(i) / 1000
            p = mp.polyval(c, r)
            assert abs(1 + r * p - mp.power(2, r)) <= mp.mpf(4.3e-18) * 2 + mp.mpf(2) ** -53 * (mp.sqrt(2) - 1), i


def test_c2_over_ln2_parts():
    """The high and the low part together are the library's c2 (64 bits, kH kC / kKB) over ln 2, to the
    low part's own rounding."""
    text = open(os.path.join(os.path.dirname(HDR), "xsec_internal.h")).read()
    k = {n: float(re.search(n + " = " + NUM + ";", text).group(1)) for n in ("kH", "kC", "kKB", "kLN2")}
    assert "kC2 = kH * kC / kKB;" in text
    body = _body("void two_part_rate(")
    assert "ch = kC2 / kLN2;" in body
    low = float(re.search("cl = " + NUM + ";", body).group(1))
    c2 = k["kH"] * k["kC"] / k["kKB"]
    with mp.workdps(50):
        assert abs(mp.mpf(c2) / mp.log(2) - (mp.mpf(c2 / k["kLN2"]) + low)) <= abs(low) * mp.mpf(2) ** -53
