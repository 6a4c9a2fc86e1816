"""What the host code plans, checked on a machine without a GPU
(tests/hostcheck/plans.cpp): the library's host translation units under
AddressSanitizer and UBSan, linked against the stand-in runtime and the stand-in
launch functions, with further checks wrapped around the launches of the tensor
path, the surrogate's layers and the re-angling call."""

import concurrent.futures as cf
import os
import re
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "tests", "hostcheck"))

WRAPPED = re.compile(r"\bT (_ZN2st\d+launch_(?:grad_fused|grad_fused_grouped|strided|sg_conv|angles)E\w+)")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc is not installed")
    import build as hc
    out = str(tmp_path_factory.mktemp("plans"))
    srcs = [os.path.join(hc.CSRC, u) for u in hc.LIB_UNITS]
    srcs += [os.path.join(hc.HERE, u) for u in ("hip_stub.cpp", "stub_kernels.cpp", "plans.cpp")]
    objs = [os.path.join(out, os.path.splitext(os.path.basename(s))[0] + ".o") for s in srcs]
    with cf.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        list(ex.map(hc._compile, srcs, objs))
    undefined = "".join(subprocess.run([hc.tool("nm"), "-u", o], capture_output=True, text=True, check=True).stdout
                        for o in objs)
    blobs = os.path.join(out, "blobs.c")
    with open(blobs, "w") as fh:
        fh.write("".join(f"const char {n}[16] = {{0}};\n" for n in sorted(set(re.findall(r"__hip_fatbin_\w+", undefined)))))
    subprocess.run([hc.tool("clang"), "-c", blobs, "-o", blobs[:-2] + ".o"], check=True, capture_output=True)
    stubs = subprocess.run([hc.tool("nm"), os.path.join(out, "stub_kernels.o")], capture_output=True, text=True, check=True)
    wraps = [f"-Wl,--wrap={s}" for s in WRAPPED.findall(stubs.stdout)]
    assert len(wraps) == 5
    exe = os.path.join(out, "plans")
    r = subprocess.run([hc.tool("clang++"), "-fsanitize=address,undefined", *wraps, *objs, blobs[:-2] + ".o", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _run(exe, group):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe, group], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    assert "plans: OK" in r.stdout
    assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr


def test_mask_cells_from_four_million_voxels(plans):
    _run(plans, "threshold")


def test_surrogate_mask_cells_from_one_million_voxels(plans):
    _run(plans, "surrogate_threshold")


def test_gradient_split_targets(plans):
    _run(plans, "split")


def test_mask_cells_stay_in_their_buffers(plans):
    _run(plans, "cells")


def test_wide_accesses_of_the_reangling_call(plans):
    _run(plans, "angles")
