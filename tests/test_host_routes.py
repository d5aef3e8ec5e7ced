"""Which route the host code takes where one GPU cannot show it, with a stand-in for the HIP runtime (no GPU):
tests/c/host_routes.cpp, linked against the built library."""
import os
import shutil
import subprocess

import pytest

import paper_2104_07857_amd as zi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_07857_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    rocm = "/opt/rocm/include"
    if shutil.which("g++") is None or not os.path.exists(os.path.join(rocm, "hip", "hip_runtime_api.h")):
        pytest.skip("no host compiler or no HIP headers")
    out = str(tmp_path_factory.mktemp("routes") / "host_routes")
    libdir = os.path.dirname(zi.LIB_PATH)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-isystem", rocm, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "c", "host_routes.cpp"), "-o", out, "-L", libdir, "-lzi",
                        "-Wl,-rpath," + libdir, "-Wl,--allow-shlib-undefined"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


@pytest.mark.parametrize("check", ["peer", "sizes", "capture", "replays", "skipped", "earlier_work", "one_tensor_kernels", "uploads", "loads", "offload", "spanning", "link_tiles"])
def test_route(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-2000:]
