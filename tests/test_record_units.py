"""Records of the device lists: how a workgroup finds its record, and that few workgroups have nothing to do."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_records_fit_the_pieces(tmp_path):
    exe = str(tmp_path / "record_units")
    csrc = os.path.join(ROOT, "paper_2409_19256_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "planner.cpp"),
                    os.path.join(ROOT, "tests", "record_units_main.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
