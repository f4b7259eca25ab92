"""The spread factor's arithmetic (rvea_spread.h) compiled for the host, against
the power in long double."""
import os
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
    out = str(tmp_path_factory.mktemp("spread") / "probe")
    subprocess.run([cxx, "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(HERE, "golden", "spread_error.cpp"), "-o", out], check=True)
    return out


# The product for t has n - 1 roundings of half an ulp (2^-53), of which the
# correction leaves the n-th part, and the last fused multiply-add has one more;
# the terms left out and the coefficients' own rounding are far smaller.
@pytest.mark.parametrize("n", list(range(1, 65)))
def test_error_is_below_two_half_ulps(probe, n):
    step = 61 if n in (1, 2, 21, 32, 33, 63, 64) else 1009
    r = subprocess.run([probe, str(n), str(step)], capture_output=True, text=True, check=True)
    assert float(r.stdout) <= 2.0, r.stdout
