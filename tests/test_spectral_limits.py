"""Launch sizes of the spectral form at the ends of the sizes it is chosen for (host code),
under the address and undefined-behaviour sanitizers."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
H = os.path.join(ROOT, "tests", "host_runtime")
CSRC = os.path.join(ROOT, "paper_1912_08810_amd", "csrc")


def test_launches_stay_below_two_to_the_32_threads(tmp_path):
    exe = os.path.join(tmp_path, "spectral_limits_check")
    cmd = ["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-x", "c++", "-I", H,
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "sse_geometry.hip"),
           os.path.join(H, "spectral_limits_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1"))
    print(r.stdout[-1000:])
    assert r.returncode == 0 and "OK" in r.stdout, (r.stdout[-2000:], r.stderr[-3000:])
