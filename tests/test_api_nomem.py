"""A read-out that finds no host memory for its chunk sums ends with HLB_ERR_NOMEM,
not with a C++ exception through the C entry (hlb_api.cpp, host build)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_readouts_without_host_memory(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "api_nomem")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-x", "hip",
                           os.path.join(HERE, "hostcheck", "api_nomem.cpp"), "-o", exe], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()
    hip, nomem = "-3", "-6"
    assert out == [hip, hip, nomem, nomem]
