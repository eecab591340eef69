"""The reconstruction writes its records over the differences that other lanes of the wave have put in
LDS, and each edge's records over the last one's.  A block is one wave, for which a barrier is no
instruction but keeps the compiler from moving LDS accesses across it: in the code of every instance
each of the three edges' records (the last three runs of writes) lies between two barriers."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
def test_records_lie_between_barriers():
    from paper_2306_04467_amd import build

    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    asm = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-o", "-", "-I", build.CSRC,
                          os.path.join(ROOT, "tests", "host", "recon_order.hip")],
                         check=True, capture_output=True, text=True, timeout=600).stdout
    kernels = re.findall(r"^(\S*k_recon\S*):.*?\n(.*?)\.end_amdhsa_kernel", asm, re.S | re.M)
    assert len(kernels) == 6
    for name, body in kernels:
        events = re.sub(r"(.)\1+", r"\1", "".join(
            "b" if "barrier" in x else "R" if "read" in x else "W" for x in
            re.findall(r"^\s+(ds_read|ds_write|s_barrier|; wave barrier)", body, re.M)))
        tail = events[:events.rindex("W") + 2]
        assert tail.endswith("RbWbRbWbRbWb"), (name, events)
