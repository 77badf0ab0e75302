"""Copies to the host that fail half way (tests/abi_copy_failure.cpp): the
library's sources linked against definitions of the HIP calls they make, so
that no device is needed.  CPU only."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_13839_amd", "csrc")
OUT = os.path.join(ROOT, "paper_2410_13839_amd", "_build", "copy_failure")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-std=c++17", "-O1", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src):
    obj = os.path.join(OUT, os.path.basename(src) + ".o")
    r = subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return obj


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not available")
def test_no_copy_is_in_flight_after_a_failed_one():
    os.makedirs(OUT, exist_ok=True)
    build = __import__("paper_2410_13839_amd.build", fromlist=["SOURCES"])
    srcs = [os.path.join(CSRC, s) for s in build.SOURCES] + [os.path.join(ROOT, "tests", "abi_copy_failure.cpp")]
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(_compile, srcs))
    exe = os.path.join(OUT, "abi_copy_failure")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", *objs, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "copy failure ok" in r.stdout, (r.stdout[-2000:], r.stderr[-4000:])
