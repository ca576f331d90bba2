"""The bfloat16 GEMM's address and dispatch rules on the CPU: a host program
(gemm_bf16_host.cpp) against the library's own header and host code."""
import os
import subprocess

import pytest

from paper_2606_28516_amd import build as hb
from tests import test_gpu_gemm_bf16 as gpu

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


def _tiles(program, products):
    args = [str(v) for p in products for v in p]
    return subprocess.run([program, "tiles", *args], capture_output=True, text=True, check=True,
                          timeout=60).stdout.splitlines()


ALL = {"64", "128", "128 deep", "256 long", "320", "duo"}


def test_gpu_sizes_cover_every_tile(program):
    """What test_gpu_gemm_bf16.py says about its sizes."""
    fc1 = _tiles(program, [(T, H, D, 1, 0, D, D) for T, D, H in gpu.SIZES])
    fc2 = _tiles(program, [(T, D, H, 0, 0, H, H) for T, D, H in gpu.SIZES])
    assert set(fc1) == ALL and set(fc2) == ALL - {"duo"}
    # the sizes with a short last tile in rows, columns and k
    ragged = [(T, D, H) for T, D, H in gpu.SIZES if T % 64 and D % 64 and H % 64]
    assert {"320", "256 long"} <= set(_tiles(program, [(T, H, D, 1, 0, D, D) for T, D, H in ragged]))
    want = ["64", "128", "128 deep", "256 long", "320", "duo"]
    assert _tiles(program, [(M, N, K, 1, 0, K, K) for M, N, K in gpu.TILES]) == want
    assert _tiles(program, [(M, N, K, 0, 0, K, K) for M, N, K in gpu.TILES])[:5] == want[:5]
    for T, D, H, E, r, q, y, tu in gpu.GROUPED:
        pairs = E * (E - 1) // 2
        assert _tiles(program, [(T, D, r + q, 0, E, r, r + q), (T, D, r + 2 * q, 0, pairs, r, r + q)]) == [y, y]
        assert _tiles(program, [(T, r + 2 * q, H, 0, pairs, H, H)]) == [tu]
