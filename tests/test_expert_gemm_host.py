"""Arithmetic of the expert GEMM kernels that host code can run: a small program (expert_gemm_host.cpp) is compiled
from the kernels' header for the host alone and checks it against plain 64-bit arithmetic."""
import os
import subprocess

import pytest

from paper_2605_17889_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = tmp_path_factory.mktemp("host") / "expert_gemm_host"
    subprocess.run([hip_build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(hip_build.ROOT, "include"), "-I", hip_build.CSRC,
                    os.path.join(HERE, "expert_gemm_host.cpp"), "-o", str(out)], check=True)
    return str(out)


def check(program, *args):
    proc = subprocess.run([program, *map(str, args)], capture_output=True, text=True, timeout=60)
    assert proc.returncode == 0, proc.stdout[-2000:] + proc.stderr[-2000:]


@pytest.mark.parametrize("K", [256, 384, 512, 4096])
def test_store_bounds_of_wide_outputs(program, K):
    """An upper wavefront's rows times the bytes of a very wide row: 256 rows of 2^22 floats are 2^32 bytes."""
    check(program, "store_bounds", K)


def test_tiles_cover_every_row_and_empty_halves_are_no_tiles(program):
    """A lower half without rows is named so: a workgroup that takes it for a tile multiplies over all of the reduction
    for outputs that are never stored."""
    check(program, "tiles")
