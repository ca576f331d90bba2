"""The bfloat16 GEMM's address and dispatch rules on the CPU: a host program
(gemm_bf16_host.cpp) against the library's own header and host code."""
import os
import subprocess

import pytest

from paper_2606_28516_amd import build as hb

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(hb.HIPCC) or not os.path.exists(hb.LIB):
        pytest.skip("needs hipcc and the built library")
    out = str(tmp_path_factory.mktemp("gemm_host") / "gemm_bf16_host")
    subprocess.check_call([hb.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", f"-I{hb.INCLUDE}",
                           f"-I{hb.CSRC}", os.path.join(HERE, "gemm_bf16_host.cpp"), "-o", out,
                           f"-L{hb.HERE}", "-l:" + os.path.basename(hb.LIB), f"-Wl,-rpath,{hb.HERE}"])
    return out


@pytest.mark.parametrize("check", ["parts", "supported", "far_rows"])
def test_host_rules(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
