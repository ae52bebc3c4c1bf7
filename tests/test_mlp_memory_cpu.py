"""The surrogate network's host side when device or pinned memory runs out, on
the CPU (AddressSanitizer / UndefinedBehaviorSanitizer build against host
memory in place of the device's): every allocation of a growing batch fails
once, and batches that fitted before are then evaluated from whole buffers."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1801_03039_amd", "csrc")
ROCM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")

pytestmark = pytest.mark.skipif(
    shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")),
    reason="needs g++ and the HIP headers")


def test_failed_allocations(tmp_path):
    exe = str(tmp_path / "mlp_driver")
    subprocess.run(["g++", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=undefined", "-g", "-O1", "-D__HIP_PLATFORM_AMD__",
                    "-isystem", ROCM, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(HERE, "sanitize", "mlp_driver.cpp"),
                    os.path.join(CSRC, "ebic_mlp.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=600)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    assert "mlp driver ok" in r.stdout
