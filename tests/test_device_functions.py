"""Device functions of the library, run on the host (tests/devcheck): each program
includes the kernels' own header, built by the host compiler with stand-ins for
the few instructions it uses, and exits non-zero where a function breaks its
contract."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "devcheck")
INCLUDES = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2508_07476_amd", "csrc"), HERE, "/opt/rocm/include"]


def _run(name, tmp_path, *extra):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are not installed")
    exe = str(tmp_path / name)
    cmd = [gxx, "-std=c++20", "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", *extra,
           *(f"-I{d}" for d in INCLUDES), os.path.join(HERE, name + ".cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-1000:]
    assert "devcheck: OK" in r.stdout


def test_ties_between_equal_cross_products(tmp_path):
    _run("eigen_ties", tmp_path)


def test_e3_is_of_unit_length_in_float64(tmp_path):
    _run("eigen_unit", tmp_path)


def test_integration_pieces_load_each_sample_once(tmp_path):
    _run("strided_loads", tmp_path)


def test_runs_of_marked_cells(tmp_path):
    _run("cell_runs", tmp_path, "-pthread")


def test_head_products_read_the_waves_own_rows(tmp_path):
    _run("head_places", tmp_path)
