"""The tables of the FP64 Box-Muller (csrc/mg_bm64.inc) hold what the kernel's
error bounds rest on: checked against 50-digit values."""
import os
import re

import mpmath as mp
import pytest

INC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2512_02175_amd", "csrc", "mg_bm64.inc")


def _table(name):
    text = open(INC).read()
    body = text[text.index(name + "["):]
    body = body[:body.index("};")]
    return [tuple(float.fromhex(v) for v in row.split(","))
            for row in re.findall(r"\{(-?0x[^{}]+)\}", body)]


@pytest.mark.parametrize("i", [0, 1, 31, 74, 75, 76, 77, 100, 127])
def test_log_table(i):
    """z = m c - 1 lies in [-2^-8, 2^-7) on the interval, the constant is a
    multiple of 2^-47 within 2^-59 of -2 log(1/c), zero around 1."""
    rows = _table("kLogTab")
    assert len(rows) == 128
    lo = 45 / 64 + i / 256 if i < 76 else 1 + (i - 76) / 128
    hi = lo + (1 / 256 if i < 76 else 1 / 128)
    c, k = rows[i]
    with mp.workdps(50):
        assert -mp.mpf(2) ** -8 <= mp.mpf(lo) * c - 1
        assert mp.mpf(hi) * c - 1 <= mp.mpf(2) ** -7
        assert abs(k - 2 * mp.log(mp.mpf(c))) < mp.mpf(2) ** -59
        assert float(k * 2.0 ** 47).is_integer()
    if i in (75, 76):
        assert (c, k) == (1.0, 0.0)


@pytest.mark.parametrize("i", [0, 1, 2, 31, 32, 33, 63, 64, 96, 127, 128])
def test_turn_table(i):
    """a is a multiple of 2^-50 within 2^-29 of i/128 turns; cosine and sine
    are within 2^-62 of its own."""
    rows = _table("kTurnTab")
    assert len(rows) == 129
    c, s, a = rows[i]
    assert float(a * 2.0 ** 50).is_integer()
    with mp.workdps(50):
        assert abs(a - 2 * mp.pi * i / 128) < mp.mpf(2) ** -29
        assert abs(c - mp.cos(mp.mpf(a))) < mp.mpf(2) ** -62
        assert abs(s - mp.sin(mp.mpf(a))) < mp.mpf(2) ** -62
