"""Places of the attention's partial sums, compiled for the host: no two sequences of a batch
share one and none lies outside the memory, also where malformed row ranges stand between valid
ones and where the ranges are not in ascending order."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    so = str(tmp_path_factory.mktemp("parts") / "libattn_parts_probe.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-fsanitize=undefined",
                        "-fno-sanitize-recover=all", os.path.join(ROOT, "tests", "attn_parts_probe.cpp"), "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)
    lib.trj_test_parts.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, C.c_void_p]

    def wrong(node_off, T, pack, ntw):
        off = np.ascontiguousarray(node_off, np.int32)
        owner = np.zeros(len(off) * 64 + (T << pack) // 32 + 64, np.int32)
        return lib.trj_test_parts(off.ctypes.data, len(off) - 1, T, pack, ntw, 128, owner.ctypes.data)
    return wrong


def ranges(rng, ascending):
    """Row ranges of a batch: mostly valid sequences, some empty, too long or outside."""
    B = int(rng.integers(1, 12))
    sizes = [int(rng.choice([0, 1, 2, 5, 9, 20, 31, 33, 64, 100, 128, 150])) for _ in range(B)]
    off = np.concatenate([[int(rng.integers(0, 3))], sizes]).cumsum()
    T = max(int(off[-1]) + int(rng.integers(0, 3)), B)
    if not ascending:
        off = rng.permutation(off) if rng.random() < 0.5 else np.roll(off, int(rng.integers(0, B + 1)))
    return off, T


@pytest.mark.parametrize("ascending", [True, False])
def test_places_do_not_meet(places, ascending):
    rng = np.random.default_rng(int(ascending))
    for _ in range(4000):
        off, T = ranges(rng, ascending)
        for pack in (0, 1, 2, 3):
            for ntw in (1, 2, 4):
                assert places(off, T, pack, ntw) == 0, (off.tolist(), T, pack, ntw)
