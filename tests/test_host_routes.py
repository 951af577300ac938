"""The routes and scratch layouts of the planner, driven by the host programs under
tests/host, built with g++ under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_04559_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", ["route_check", "layout_check"])
def test_host_program(tmp_path, name):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / name)
    build = subprocess.run(
        [gxx, "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
         "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
         "-I", os.path.join(ROOT, "include"), "-I", CSRC,
         os.path.join(ROOT, "tests", "host", name + ".cpp"), os.path.join(CSRC, "plan.cpp"),
         "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0:abort_on_error=0",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    run = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=240)
    assert run.returncode == 0, (run.stdout[-2000:], run.stderr[-4000:])
    assert name + " OK" in run.stdout
