"""The host runtime (hs_runtime.cpp) on the CPU, against stand-ins of the HIP calls that count what is
alive and can be told to fail (host_runtime_driver.cpp): what cannot be provoked on a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("g++ or the HIP headers not available")
    exe = str(tmp_path_factory.mktemp("host") / "host_runtime_driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        os.path.join(ROOT, "tests", "host_runtime_driver.cpp"),
                        os.path.join(ROOT, "paper_2506_23917_amd", "csrc", "hs_runtime.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("name", ["side_stream", "other_device", "first_read", "no_memory", "no_arrays"])
def test_host_runtime(driver, name):
    r = subprocess.run([driver, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
