"""The matrix-core form's host plan driven by a C++ model of the kernel's data
flow (lane by lane: operands, record writes and reads, the neighbour tiles'
blocks), against neighbour counts taken cell by cell, for both stencils, over
the named fractals and 300 random ones at every tile level, under
AddressSanitizer and UndefinedBehaviorSanitizer (CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2110_12952_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_matrix_plan_model(tmp_path):
    exe = str(tmp_path / "matrix_model")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I", CSRC, os.path.join(ROOT, "tests", "sanitize", "matrix_model.cpp"),
                        os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "matrix_plan.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    if r.returncode != 0 and "sanitize" in r.stderr:
        pytest.skip("sanitizer build unavailable: " + r.stderr[-400:])
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0 and "runtime error" not in r.stderr, r.stdout[-2000:] + r.stderr[-2000:]
    assert int(r.stdout.split()[-1]) > 300


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_sparse_fractals_within_time_and_memory(tmp_path):
    # a square of s^(m - q) blocks a side must not be held whole: up to the
    # largest r, 1 GiB of address space and half a second for each descriptor
    exe = str(tmp_path / "sparse_plans")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, os.path.join(ROOT, "tests", "sanitize", "sparse_plans.cpp"),
                        os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "matrix_plan.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    made, longest = r.stdout.split()
    assert int(made) > 100 and float(longest) < 0.5


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_occupancy_is_asked_once_per_launch_shape(tmp_path):
    exe = str(tmp_path / "occupancy_cache")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC,
                        os.path.join(ROOT, "tests", "sanitize", "occupancy_cache.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
