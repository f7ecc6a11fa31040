"""The host side of the engine and of the step graphs on the CPU, over a stand-in for
the HIP runtime that knows what is in flight and can refuse a launch
(tests/host/engine_host.cpp): an engine that goes while its last replay runs waits for
it before it destroys the graph and frees the job tables, on the null stream as on any
other, and a capture that a launch is missing from is reported and not kept."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "engine_host")
    csrc = os.path.join(ROOT, "paper_1812_03191_amd", "csrc")
    # host code only: the kernels' code object, which the stand-in does not load, is left out
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--cuda-host-only", "-no-hip-rt", "-O1", "-std=c++17",
           "-I" + csrc, "-I" + os.path.join(ROOT, "include"), "-x", "hip"]
    cmd += [os.path.join(csrc, f) for f in ("dfk.hip", "api.hip", "fieldio.hip", "force_noalloc.hip")]
    cmd += [os.path.join(ROOT, "tests", "host", "engine_host.cpp"), "-Wl,--unresolved-symbols=ignore-all", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    return exe


@pytest.mark.parametrize("what", ["null stream", "own stream", "launch refused in the engine",
                                  "launch refused in a step graph"])
def test_host_side(program, what):
    res = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    print(res.stdout)
    assert res.returncode == 0, res.stdout + res.stderr
