"""The library's host code on a stand-in HIP runtime (host_runtime_test.cpp):
devices, stream order after errors, launch limits and memory; no GPU."""
import os
import shutil
import subprocess

import pytest

import paper_2410_14462_amd as lv

HERE = os.path.dirname(os.path.abspath(__file__))
TESTS = ["destroy_on_other_device", "order_after_failed_diffusion", "edge_weight_launches",
         "graph_order_launches", "uplift_launches", "diffusion_memory", "graph_scratch"]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(lv.LIB_PATH):
        from paper_2410_14462_amd import build
        build.build()
    out = str(tmp_path_factory.mktemp("host_runtime") / "host_runtime_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-I", os.path.join(os.path.dirname(HERE), "include"),
                    os.path.join(HERE, "host_runtime_test.cpp"), lv.LIB_PATH, "-Wl,-rpath," + os.path.dirname(lv.LIB_PATH),
                    "-Wl,-rpath-link,/opt/rocm/lib", "-o", out], check=True)
    return out


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("name", TESTS)
def test_host(exe, name):
    r = subprocess.run([exe, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr[-2000:]
