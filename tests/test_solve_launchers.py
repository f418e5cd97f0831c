"""The launchers that builds without device code leave out (weak symbols): the
library has every one of them, and a build that has not refuses variances
instead of returning unsolved values."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"
CSRC = os.path.join(ROOT, "paper_1708_02835_amd", "csrc")
FAKE = os.path.join(ROOT, "tests", "fake_hip")


def weak_names():
    names = set()
    for f in os.listdir(CSRC):
        if f.endswith(".hpp"):
            text = open(os.path.join(CSRC, f)).read()
            for decl in re.findall(r"[^;{}]*__attribute__\(\(weak\)\)\s*;", text):
                names.add(re.findall(r"(\w+)\(", decl.split("__attribute__")[0])[0])
    return names


def test_library_defines_every_weak_launcher():
    lib = os.path.join(ROOT, "paper_1708_02835_amd", "libgeolik.so")
    if not os.path.exists(lib) or not shutil.which("nm"):
        pytest.skip("library not built, or no nm")
    names = weak_names()
    assert len(names) >= 8, names
    out = subprocess.check_output(["nm", "-C", lib], text=True)
    defined = {m for m in re.findall(r"^[0-9a-f]+ [TtWw] gl::(\w+)\(", out, re.M)}
    assert names <= defined, names - defined


def test_variances_are_refused_where_they_cannot_be_solved(tmp_path):
    clang = os.path.join(LLVM, "clang++")
    if not os.path.exists(clang) and not shutil.which(clang):
        pytest.skip("clang++ not available")
    srcs = [os.path.join(CSRC, f) for f in ("engine.cpp", "serve.cpp", "batch.cpp")] + \
           [os.path.join(FAKE, f) for f in ("fake_hip.cpp", "fake_kernels.cpp", "krige_driver.cpp")]
    exe = tmp_path / "krige_driver"
    subprocess.check_call([clang, "-std=c++17", "-O1", "-I", FAKE, "-I", os.path.join(ROOT, "include"), "-I", CSRC, *srcs,
                           "-o", str(exe), "-lpthread"])
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0 and int(p.stdout) < 0, p.stdout
