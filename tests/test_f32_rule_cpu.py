"""The fp32 projections' launch rule: groups of two tokens, which read the weights again for every
group, only where that measured no slower."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def tokens(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    so = str(tmp_path_factory.mktemp("f32") / "libf32_rule_probe.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "f32_rule_probe.cpp"),
                        "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return C.CDLL(so).trj_test_f32_tokens


# us of the launch with four or eight tokens per workgroup -> with two
@pytest.mark.parametrize("n_in,n_out,T,pairs", [
    (1024, 256, 15, True), (1024, 256, 32, True),        # 6.7 -> 4.7, 10.7 -> 4.9
    (4096, 1024, 16, True), (4096, 1024, 32, True),      # 20.9 -> 13.7, 35.8 -> 25.5
    (512, 512, 24, True), (512, 512, 12, False),         # 6.6 -> 4.8, 4.6 -> 4.7
    (4096, 4096, 4, True), (4096, 32000, 2, True),       # 30.2 -> 22.6, 131 -> 100
    (4096, 4096, 8, False), (4096, 4096, 32, False),     # 29.6 -> 35.5, 78.7 -> 110.6
    (1024, 4096, 16, False), (1024, 4096, 32, False),    # 11.9 -> 16.1, 21.3 -> 30.0
    (2048, 2048, 16, False), (11008, 4096, 32, False),   # 12.2 -> 15.1, 211 -> 285
    (4096, 32000, 4, False), (4096, 32000, 32, False),   # 132 -> 193, 755 -> 1424
    (256, 1024, 15, False), (1024, 256, 33, False)])
def test_groups_of_two(tokens, n_in, n_out, T, pairs):
    assert (tokens(T, n_in, n_out) == 2) == pairs
