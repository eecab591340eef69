"""What a step leaves for the next one (ghost cells, wave speeds) and what is formed of a loaded
checkpoint come from different kernels and must round alike for a restarted run to keep the bits of the
uninterrupted one.  Hence their sums of products are written with explicit fused operations: the
compiler has nothing left to contract, and the code is the same with contraction on and off."""
import collections
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _fp64_operations(contract):
    csrc = os.path.join(ROOT, "paper_2306_04467_amd", "csrc")
    asm = subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only", "-S", "-o", "-",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", f"-ffp-contract={contract}",
                          "-I", csrc, os.path.join(ROOT, "tests", "host", "step_rounding.hip")],
                         check=True, capture_output=True, text=True, timeout=300).stdout
    ops = {}
    for name, body in re.findall(r"^(\S*k_(?:ghost_fill|speed)\S*):.*?\n(.*?)\.end_amdhsa_kernel", asm, re.S | re.M):
        found = (("fma" if "fma" in op else op) for op in re.findall(r"\bv_(fma|fmac|mul|add)_f64", body))
        ops[name] = collections.Counter(found)
    return ops


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
def test_contraction_changes_nothing():
    fast, off = _fp64_operations("fast-honor-pragmas"), _fp64_operations("off")
    assert len(fast) == 4 and fast == off, (fast, off)
