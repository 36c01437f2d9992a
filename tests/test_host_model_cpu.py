"""CPU: error paths of the C ABI's host code over a model of the device (host_model.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_model(tmp_path_factory):
    from paper_1210_3450_amd import build
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC)))
    exe = str(tmp_path_factory.mktemp("host_model") / "host_model")
    subprocess.check_call([
        os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-O1", "-g", "-Wno-everything",
        "-D__HIP_PLATFORM_AMD__", "-D__align__(x)=__attribute__((aligned(x)))", "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
        "-I", os.path.join(ROOT, "paper_1210_3450_amd", "csrc"), os.path.join(ROOT, "tests", "host_model.cpp"),
        "-o", exe])
    return exe


@pytest.mark.parametrize("scenario", ["plain", "lost_decision", "out_of_memory", "tile_arrays",
                                      "autotune_without_tiles", "rescale_in_place", "autotune_ensemble", "tile_capacity"])
def test_host_model(host_model, scenario, tmp_path):
    r = subprocess.run([host_model, scenario], capture_output=True, text=True, timeout=120, cwd=tmp_path)
    assert r.returncode == 0, (r.returncode, r.stderr[-4000:])
