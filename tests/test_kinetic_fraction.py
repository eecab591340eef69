"""The force model's kinetic fraction 1/2 erfc(-x) as k_plane<double> forms it, on the host (the same
source), against the long double erfc.  It is a fraction of particles: the small ones keep their
digits.  Tolerances: one unit (2^-52) where it is formed from the polynomial, whose sum is at least
1/4; five units beyond, the host C library's bound for its erfc."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
def test_small_fractions_keep_their_digits(tmp_path):
    exe = str(tmp_path / "kinetic_fraction")
    csrc = os.path.join(ROOT, "paper_2306_04467_amd", "csrc")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-I", csrc,
                    os.path.join(ROOT, "tests", "host", "kinetic_fraction.hip"), "-o", exe], check=True, timeout=300)
    rows = [[float(x) for x in line.split()] for line in
            subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120).stdout.splitlines()]
    assert len(rows) == 7
    for lo, hi, worst in rows:
        assert worst <= (2.0 ** -52 if lo >= -0.5 and hi <= 1.0 else 5 * 2.0 ** -52), (lo, hi, worst)
