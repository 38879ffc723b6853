"""Which form a submission runs and what its kernels get of the caller's workspace: the
library's host code with stand-in launchers, under the address and undefined-behaviour
sanitizers (tests/host_runtime/forms_driver.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
H = os.path.join(ROOT, "tests", "host_runtime")
CSRC = os.path.join(ROOT, "paper_1912_08810_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = os.path.join(tmp_path_factory.mktemp("forms"), "forms_driver")
    cmd = ["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-x", "c++", "-I", H,
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "sse_runtime.hip"),
           os.path.join(CSRC, "sse_geometry.hip"), os.path.join(H, "launch_stubs.cpp"),
           os.path.join(H, "forms_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _run(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1"))
    assert r.returncode == 0 and "OK" in r.stdout, (r.stdout[-2000:], r.stderr[-3000:])


def test_batch_takes_a_workspace_of_the_direct_size(driver):
    _run(driver, "batch_in_a_direct_workspace")


def test_workspace_may_start_at_any_word(driver):
    _run(driver, "workspace_at_any_word")
