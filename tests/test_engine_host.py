"""The engine's host side on the CPU, over a stand-in for the HIP runtime that knows
what is in flight (tests/host/engine_teardown.cpp): an engine that goes while its
last replay runs waits for it before it destroys the graph and frees the job tables,
on the null stream as on any other."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "engine_teardown")
    csrc = os.path.join(ROOT, "paper_1812_03191_amd", "csrc")
    # host code only: the kernels' code object, which the stand-in does not load, is left out
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--cuda-host-only", "-no-hip-rt", "-O1", "-std=c++17",
           "-I" + csrc, "-I" + os.path.join(ROOT, "include"), "-x", "hip"]
    cmd += [os.path.join(csrc, f) for f in ("dfk.hip", "api.hip", "fieldio.hip", "force_noalloc.hip")]
    cmd += [os.path.join(ROOT, "tests", "host", "engine_teardown.cpp"), "-Wl,--unresolved-symbols=ignore-all", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    return exe


@pytest.mark.parametrize("stream", ["null stream", "own stream"])
def test_teardown_in_flight(program, stream):
    res = subprocess.run([program, stream], capture_output=True, text=True, timeout=60)
    print(res.stdout)
    assert res.returncode == 0, res.stdout + res.stderr
