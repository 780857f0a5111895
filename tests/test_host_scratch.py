"""The library's host code over a runtime without a device (tests/host):
memory is freed once and used only while it lives, and none is asked for under
stream capture, nor twice where it was refused; what goes to the
device is finite where kernels take places from it."""
import os
import shutil
import subprocess

import pytest

import paper_1907_04435_amd as sa

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host") / "scratch")
    lib = os.path.dirname(sa.LIB_PATH)
    cmd = [shutil.which("g++") or "c++", "-O1", "-std=c++17", "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"),
           os.path.join(HERE, "host", "scratch.cpp"), "-o", out, "-L", lib, "-lsa",
           "-Wl,-rpath," + lib, "-Wl,-rpath-link," + os.path.join(ROCM, "lib")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return out


@pytest.mark.parametrize("scenario", ["edit_score", "capture", "short_of_memory", "sun_without_direction", "fan_masks", "many_bins"])
def test_holds(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=120)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stdout + r.stderr
