"""The library's memory pool (csrc/memory.hip) on the CPU, with a stand-in for
the HIP runtime (pool_harness.cpp): its bookkeeping, bounds and threads."""
import os
import shutil
import subprocess

import pytest

pytestmark = pytest.mark.cpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1505_07630_amd", "csrc")
SCENARIOS = ["reuse", "wait_in_alloc", "wait_in_free", "full", "threads", "no_host_memory", "bounds", "no_info"]


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("pool") / "pool")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", CSRC, "-x", "c++", os.path.join(CSRC, "memory.hip"),
                    os.path.join(ROOT, "tests", "pool_harness.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("scenario", SCENARIOS)
def test_pool(harness, scenario):
    r = subprocess.run([harness, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
