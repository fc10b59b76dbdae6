"""The host side of the tiled GEMM (gemm_tile_plan.h), compiled with g++: where its kernels'
loads read. CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="session")
def tile_model(tmp_path_factory):
    """Runs tests/host/tile_model.cpp with one argument and a standard input: its lines."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("tile") / "tile_model")
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "tile_model.cpp"),
                    "-o", exe], check=True)

    def run(what, text=""):
        return subprocess.run([exe, what], input=text, capture_output=True, text=True, check=True,
                              timeout=300).stdout.splitlines()
    return run


def test_tile_loads_stay_in_their_buffers(tile_model):
    """Every load of activations, codes and tables that the range check lets through reads
    inside its buffer, whether the check leaves the scalar offset out or takes it from the
    size: partial tiles of every number of rows, last super-rounds of one chunk."""
    lines = tile_model("reads")
    assert len(lines) > 100
    bad = [line for line in lines if line.split()[5:] != ["0", "0", "0"]]
    assert not bad, (len(bad), bad[:8])
