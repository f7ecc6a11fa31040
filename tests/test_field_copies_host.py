"""The host side of the field copies (fieldio.hip) on the CPU, over a stand-in
for the HIP runtime with two devices (tests/host/field_copies.cpp): what the
copies ask of the runtime, and what they do where it refuses."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "field_copies")
    csrc = os.path.join(ROOT, "paper_1812_03191_amd", "csrc")
    # host code only: the kernels' code object, which the stand-in does not load, is left out
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--cuda-host-only", "-no-hip-rt", "-O1", "-std=c++17", "-I" + csrc,
           "-I" + os.path.join(ROOT, "include"), "-x", "hip", os.path.join(csrc, "fieldio.hip"),
           os.path.join(ROOT, "tests", "host", "field_copies.cpp"), "-Wl,--unresolved-symbols=ignore-all", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    return exe


@pytest.mark.parametrize("what", ["device", "no pinned memory"])
def test_field_copies(program, what):
    res = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    print(res.stdout)
    assert res.returncode == 0, res.stdout + res.stderr
