"""The alignment that the compiler is told of the fused x + y pass's loads: under
boundary mode 2 the lane past a row's last cell loads a pair of velocities one
entry early, at an odd index, so those loads may assume no more than an entry's
alignment (read from the unoptimised device IR; host only)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    csrc = os.path.join(ROOT, "paper_1812_03191_amd", "csrc")
    out = str(tmp_path_factory.mktemp("ir") / "dfk.ll")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "--cuda-device-only", "-O1",
           "-std=c++17", "-I" + csrc, "-I" + os.path.join(ROOT, "include"), "-emit-llvm", "-S", "-Xclang",
           "-disable-llvm-passes", os.path.join(csrc, "dfk.hip"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    with open(out) as fh:
        text = fh.read()
    return {m.group(1): m.group(2) for m in re.finditer(r"^define [^@]*@(\w+)\([^\n]*\{\n(.*?)^\}", text, re.S | re.M)}


@pytest.mark.parametrize("T,size", [("f", 4), ("d", 8)])
def test_pairs_past_the_row_end(functions, T, size):
    # XyOwn<T, 2, group, 4, mode 2, frontiers>::load of the momenta's groups
    loads = [b for f, b in functions.items() if re.search(rf"5XyOwnI{T}Li2ELi[123]ELi4ELi2ELi\dEE4loadEi$", f)]
    assert loads
    for body in loads:
        early = 0
        for part in body.split("10tangential")[1:]:
            called = re.search(r"@(\w*row_load\w*)\(", part).group(1)
            vector = re.findall(rf"load <2 x (?:float|double)>, .*align (\d+)", functions[called])
            assert vector and all(int(a) <= size for a in vector), (called, vector)
            early += 1
        assert early
