"""CPU-only: parts of the kernel headers that run on the host as well.  The
transform multiply's passes over every size, with signed overflow trapped
(host_ntt_check.hip), and the extents of a division's buffers and products
(host_div_check.hip), each compiled for the host alone."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.parametrize("name,last", [("host_ntt_check", "114 products, 0 wrong"), ("host_div_check", "divisions")])
def test_host(tmp_path, name, last):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / name)
    r = subprocess.run([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-Wall", "-Wno-unused-function",
                        "-Xarch_host", "-fsanitize=signed-integer-overflow", "-Xarch_host",
                        "-fsanitize-trap=signed-integer-overflow", os.path.join(HERE, name + ".hip"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith(last), (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
