"""Failure paths of a handle, without a GPU: rqa_api.cpp is built with g++ against
the HIP runtime and the engine of tests/host/api_checks.cpp, under AddressSanitizer
and UndefinedBehaviorSanitizer, and runs that program's checks."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import ENV, HOST, REPO, SAN


def test_failed_launches_and_pinned_results(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    csrc = os.path.join(REPO, "paper_2402_16853_amd", "csrc")
    exe = str(tmp_path / "api_checks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include",
                    "-I" + os.path.join(REPO, "include"), "-I" + csrc, *SAN,
                    os.path.join(HOST, "api_checks.cpp"), os.path.join(csrc, "rqa_api.cpp"), "-o", exe],
                   check=True)
    # (streams that the handle or the checks leave are the program's end)
    env = dict(ENV, ASAN_OPTIONS=ENV["ASAN_OPTIONS"].replace("detect_leaks=1", "detect_leaks=0"))
    r = subprocess.run([exe], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
