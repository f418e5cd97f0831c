"""How the request queue groups its fused launches (a bound on a launch's work,
short requests apart from long ones, waiting requests still cancellable),
checked on the CPU with the stand-in HIP runtime of tests/fake_hip/, whose event
queries the driver holds back, under AddressSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
CSRC = os.path.join(ROOT, "paper_1708_02835_amd", "csrc")
FAKE = os.path.join(ROOT, "tests", "fake_hip")


def test_launches_are_bounded_and_short_requests_go_apart(tmp_path):
    if not os.path.exists(CLANG) and not shutil.which(CLANG):
        pytest.skip("clang++ not available")
    flags = ["-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-I", FAKE, "-I",
             os.path.join(ROOT, "include"), "-I", CSRC]
    objs = []
    for src, extra in [(os.path.join(CSRC, "serve.cpp"), ["-DhipEventQuery=gated_event_query"]),
                       (os.path.join(CSRC, "engine.cpp"), []), (os.path.join(CSRC, "batch.cpp"), []),
                       (os.path.join(FAKE, "fake_hip.cpp"), []), (os.path.join(FAKE, "fake_kernels.cpp"), []),
                       (os.path.join(FAKE, "tick_driver.cpp"), [])]:
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        subprocess.check_call([CLANG, *flags, *extra, "-c", src, "-o", objs[-1]])
    exe = tmp_path / "tick_driver"
    subprocess.check_call([CLANG, "-fsanitize=address", *objs, "-o", str(exe), "-lpthread"])
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120,
                       env={**os.environ, "ASAN_OPTIONS": "detect_leaks=1:halt_on_error=1"})
    assert p.returncode == 0 and p.stdout.strip().endswith("ok"), (p.stdout[-2000:], p.stderr[-4000:])
