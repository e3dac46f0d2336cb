"""What a kernel needs once per device (the permission for more than 64 KiB of LDS) is asked
for on every device, not once per process."""
import ctypes as C
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2406_17404_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    so = str(tmp_path_factory.mktemp("once") / "libonce.so")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-shared", "-fPIC",
                        os.path.join(ROOT, "tests", "device_once_probe.cpp"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return C.CDLL(so)


@pytest.mark.parametrize("devices,fail,calls", [
    ([0, 0, 0], 0, 1), ([0, 1, 0, 1, 7], 0, 3), ([63, 63, 0], 0, 2), ([64, 64], 0, 2), ([-1, -1], 0, 2),
    ([3, 3, 3], 1, 2), ([3, 4, 3, 4], 2, 4)])
def test_once_on_every_device(lib, devices, fail, calls):
    assert lib.trj_test_once((C.c_int * len(devices))(*devices), len(devices), fail) == calls


def test_threads(lib):
    assert lib.trj_test_once_threads() == 0


def test_every_permission_is_asked_for_per_device():
    for name in os.listdir(CSRC):
        text = open(os.path.join(CSRC, name)).read()
        assert not re.search(r"static bool \w+ *=", text), name
        assert len(re.findall(r"hipFuncSetAttribute\(", text)) <= (name == "common.h"), name
