"""The fitted forms of csrc/bmds.hip's near_tail, read from the source and
compared with 30-digit values: the upper normal tail (z + 3) q(z) / e(z),
e = exp(-z^2 / 2), as a polynomial in u = z / (z + 3) (interpolated in the
Chebyshev nodes of z in [0, 7]), and log(1 - q) = -(2 s + s^3 a(s^2)),
s = q / (2 - q)."""
import pathlib
import re

import mpmath as mp
import pytest

SRC = (pathlib.Path(__file__).parent.parent / "paper_2010_02994_amd" / "csrc" / "bmds.hip").read_text()


def _fits():
    body = SRC[SRC.index("void near_tail("):]
    c = [mp.mpf(float(v)) for v in re.findall(r"in_place\((-?[0-9.e+-]+)\)", body[:body.index("\n}\n")])]
    assert len(c) == 21 + 10
    return c[:21], c[21:]


def _tail(z):
    u = z / (z + 3)
    return mp.polyval(_fits()[0], u) * mp.exp(-z * z / 2) / (z + 3)


@pytest.mark.parametrize("lo,hi,tol", [(0.0, 4.0, 4e-16), (4.0, 7.0, 1e-15), (7.0, 9.0, 5e-13)])
def test_tail_fit(lo, hi, tol):
    with mp.workdps(30):
        for k in range(401):
            z = mp.mpf(lo) + (mp.mpf(hi) - lo) * k / 400
            q = mp.erfc(z / mp.sqrt(2)) / 2
            assert abs(_tail(z) / q - 1) <= tol, float(z)


def test_log_fit():
    with mp.workdps(30):
        for k in range(1, 401):
            q = mp.mpf(k) / 800   # up to 1/2
            s = q / (2 - q)
            lphi = -(s ** 3 * mp.polyval(_fits()[1], s * s) + 2 * s)
            assert abs(lphi / mp.log(1 - q) - 1) <= 2e-16
