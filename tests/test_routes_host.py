"""What the entry points ask of the GPU, checked on the CPU with a stand-in for the HIP runtime.

tests/native/route_check.cpp links the built libsv.so and supplies the runtime's functions itself
(tests/native/host_runtime.h): kernels are recorded by name, copies by size, host allocations are
counted and a chosen launch fails.  So which kernels a call launches, when, and what it packs for
them is checked through the public C interface at any state size.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2608_16940_amd")


@pytest.fixture(scope="module")
def exe():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    out = os.path.join(ROOT, "_build")
    os.makedirs(out, exist_ok=True)
    path = os.path.join(out, "route_check")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                        "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "route_check.cpp"),
                        os.path.join(PKG, "libsv.so"), "-Wl,-rpath," + PKG, "-Wl,-rpath," + os.path.join(rocm, "lib"),
                        "-Wl,--unresolved-symbols=ignore-in-shared-libs", "-rdynamic", "-o", path],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return path


@pytest.mark.parametrize("check", ["packed_once", "first_copy_early", "long_plan_bounded",
                                   "bound_bytes_cheap_and_enough", "bound_runs_what_the_plan_runs",
                                   "narrow_gates_packed_lean", "small_batch_one_copy",
                                   "failed_launch_in_a_list", "failed_launch_in_a_plan",
                                   "failed_launch_releases_its_slot"])
def test_route(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout[-4000:], r.stderr[-2000:])
    assert "route checks passed" in r.stdout
