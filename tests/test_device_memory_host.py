"""The device buffers and the blocks kept between setups, on the host: device_memory_host.cpp
builds the library's header over a model of the HIP memory calls and checks one scenario a run."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs a host C++ compiler and the HIP headers")
    out = str(tmp_path_factory.mktemp("device_memory") / "device_memory_host")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    f"-I{ROOT}/include", os.path.join(ROOT, "tests", "device_memory_host.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("scenario", ["two_devices", "release_waits", "scopes_wait", "refused_waits",
                                      "rounds", "bound", "given_back"])
def test_scenario(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
