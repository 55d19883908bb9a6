"""Launch sequences of the host side of the library (``lbm_ch_api.cpp``) on a CPU device
(``tests/host/device_double.cpp``): which buffers a call reads and writes, what it leaves
when a launch fails, and which launches a call is made of.  Built with AddressSanitizer and
UndefinedBehaviorSanitizer; needs no GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_1805_00007_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")
pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang not installed")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launches") / "driver")
    r = subprocess.run([CLANG, "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        "-I", os.path.join(ROCM, "include"),
                        os.path.join(HERE, "device_double.cpp"), os.path.join(HERE, "launch_driver.cpp"),
                        os.path.join(CSRC, "lbm_ch_api.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("check", ["failed_launch", "failed_batch_and_load", "readout_beside_a_step",
                                   "autotune", "batch_autotune", "load_routes"])
def test_launches(driver, check):
    r = subprocess.run([driver, check], capture_output=True, text=True, timeout=300)
    print(r.stdout, r.stderr[-4000:])
    assert r.returncode == 0
