"""The training export holds its right-hand sides in registers (no scratch memory)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
def test_features_do_not_spill():
    from paper_2306_04467_amd import build

    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    asm = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-o", "-", "-I", build.CSRC,
                          os.path.join(ROOT, "tests", "host", "features.hip")],
                         check=True, capture_output=True, text=True, timeout=600).stdout
    scratch = dict(re.findall(r"\.amdhsa_kernel (\S*k_features\S*).*?\.amdhsa_private_segment_fixed_size (\d+)", asm, re.S))
    assert len(scratch) == 2 and set(scratch.values()) == {"0"}, scratch
