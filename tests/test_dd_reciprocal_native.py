"""The complex double-double reciprocal of the pivot steps (csrc/dd.h compiled for the host) in exact rational
arithmetic, beside the same by three quotients per component."""
import math
import os
import random
import subprocess
from fractions import Fraction as F

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"   # (address spaces of the header)


def _number(rng):
    hi = rng.choice([rng.uniform(-1, 1), rng.gauss(0, 1), 2.0 ** rng.randint(-60, 60) * rng.uniform(-2, 2)])
    return hi, rng.uniform(-0.5, 0.5) * math.ulp(hi)


@pytest.mark.skipif(not os.path.exists(CLANG), reason="no clang++")
def test_reciprocal_no_less_accurate_than_quotients(tmp_path):
    exe = str(tmp_path / "driver")
    subprocess.run([CLANG, "-std=c++17", "-O1", "-I", os.path.join(HERE, "native", "host_hip"), "-o", exe,
                    os.path.join(HERE, "native", "dd_driver.cpp")], check=True)
    rng = random.Random(17)
    pts = []
    for k in range(8000):
        re, im = _number(rng), _number(rng)
        if k % 5 == 0:
            im = (0.0, 0.0)
        elif k % 5 == 1:
            im = (re[0] * 1e-9, 0.0)
        elif k % 5 == 2:
            re, im = (re[0] * 2.0 ** 700, re[1] * 2.0 ** 700), (im[0] * 2.0 ** 700, im[1] * 2.0 ** 700)
        pts.append(re + im)
    text = "\n".join(" ".join(v.hex() for v in p) for p in pts)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.strip().split("\n")
    total, worst = [0.0, 0.0], [0.0, 0.0]
    for p, line in zip(pts, out):
        v = [F(float.fromhex(x)) for x in line.split()]
        re, im = F(p[0]) + F(p[1]), F(p[2]) + F(p[3])
        d = re * re + im * im
        for w in (0, 1):
            # in units of 2^-106 |1 / a|
            e2 = max(abs(v[4 * w] + v[4 * w + 1] - re / d), abs(v[4 * w + 2] + v[4 * w + 3] + im / d)) ** 2 * d
            e = math.sqrt(float(e2 * 2 ** 212))
            total[w] += e / len(pts)
            worst[w] = max(worst[w], e)
    print("mean and worst, in 2^-106 of |1/a|:", total, worst)
    # the mean error of some 8000 is known to a few percent; no step may cost a whole bit over the quotients
    assert total[0] <= 1.05 * total[1]
    assert worst[0] <= 2.0 * worst[1]
