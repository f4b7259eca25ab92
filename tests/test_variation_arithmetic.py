"""The arithmetic of crossover and mutation (rvea_variation.h) compiled for the
host: the spread factor against the power in long double, the distance between
mutation sites against the quotient."""
import math
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2404_01159_amd", "csrc")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    out = str(tmp_path_factory.mktemp("variation") / "probe")
    subprocess.run([cxx, "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(HERE, "golden", "variation_probe.cpp"), "-o", out], check=True)
    return out


# The product for t has n - 1 roundings of half an ulp (2^-53), of which the
# correction leaves the n-th part, and the last fused multiply-add has one more;
# the terms left out and the coefficients' own rounding are far smaller.
@pytest.mark.parametrize("n", list(range(1, 65)))
def test_error_is_below_two_half_ulps(probe, n):
    step = 61 if n in (1, 2, 21, 32, 33, 63, 64) else 1009
    r = subprocess.run([probe, "spread", str(n), str(step)], capture_output=True, text=True, check=True)
    assert float(r.stdout) <= 2.0, r.stdout


def test_gap_is_the_quotients_floor(probe):
    """Quotients that are whole numbers (the logarithm a rounded multiple of
    log(1-p)) or next to one, and the ends: certain mutation, U = 1 and a rate
    that is nearly 0."""
    rng = random.Random(5)
    rows = [(0.0, -0.5, 9), (-0.5, -math.inf, 9), (0.0, -math.inf, 9), (-36.7, -1e-310, 9),
            (-1e-16, -1e-310, 9), (0.0, -1e-310, 9)]
    for _ in range(20000):
        lq = math.log1p(-1.0 / rng.randint(2, 5000))
        logu = rng.randint(1, 400) * lq
        rows.append((rng.choice([logu, math.nextafter(logu, 0.0), math.nextafter(logu, -99.0)]), lq,
                     rng.choice([300, 5000])))
    text = "".join(f"{a.hex()} {b.hex()} {d}\n" for a, b, d in rows)
    r = subprocess.run([probe, "gap"], input=text, capture_output=True, text=True, check=True)
    got = [int(x) for x in r.stdout.split()]
    want = [d if a / b >= d else int(a / b) for a, b, d in rows]
    assert got == want
