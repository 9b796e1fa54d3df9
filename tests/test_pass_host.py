"""The fused-pass builder against gate-by-gate application, and the layout passes, on the CPU.

tests/native/pass_check.cpp replays the builder's device data in FP64 the way
the kernel reads it, for n = 1..17 qubits, random targets in any order, gates
of every width, diagonals with and without unit entries, in both precisions;
every slot, table entry and offset is range-checked.  Built with the address
and undefined-behaviour sanitizers.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_16940_amd", "csrc")


def test_passes_equal_gates_one_by_one():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = os.path.join(ROOT, "_build")
    os.makedirs(out, exist_ok=True)
    exe = os.path.join(out, "pass_check")
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "native", "pass_check.cpp"),
                        os.path.join(CSRC, "sv_pass_host.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe, "2"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-6000:])
    assert "pass checks passed" in r.stdout


def test_layout_passes_reach_the_target():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = os.path.join(ROOT, "_build")
    os.makedirs(out, exist_ok=True)
    exe = os.path.join(out, "perm_check")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", CSRC, os.path.join(ROOT, "tests", "native", "perm_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-6000:])
    assert "permutation checks passed" in r.stdout


def test_programs_equal_gates_one_by_one():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = os.path.join(ROOT, "_build")
    os.makedirs(out, exist_ok=True)
    exe = os.path.join(out, "prog_check")
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "native", "prog_check.cpp"),
                        os.path.join(CSRC, "sv_prog_host.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-6000:])
    assert "program checks passed" in r.stdout


def test_chains_equal_gates_one_by_one():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = os.path.join(ROOT, "_build")
    os.makedirs(out, exist_ok=True)
    exe = os.path.join(out, "chain_check")
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "native", "chain_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-6000:])
    assert "chain checks passed" in r.stdout
