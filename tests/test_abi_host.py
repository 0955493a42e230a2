"""The ABI's own code over a stand-in for the HIP runtime (tests/abi_host_main.cpp): what the execution
calls do when an upload has failed, and what a failed parameter change leaves behind.  Host code, under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INCLUDE = "/opt/rocm/include"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP_INCLUDE), reason="g++ or the HIP headers not available")
def test_abi_over_a_stand_in_runtime(tmp_path):
    exe = str(tmp_path / "abi_host")
    csrc = os.path.join(ROOT, "paper_2409_19256_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-Wl,--wrap=_Znwm",  # operator new(size_t) can be told to fail
                    "-D__HIP_PLATFORM_AMD__", "-I", HIP_INCLUDE, "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(csrc, "planner.cpp"), os.path.join(ROOT, "tests", "abi_host_main.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
