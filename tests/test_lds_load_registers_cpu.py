"""The hand-written loads to LDS tell the compiler that they change m0, the register with the
LDS address: a load to LDS that the compiler makes behind one sets it again.  Read from the
assembly of a probe built for the device; nothing runs."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no device compiler")
def test_m0_is_set_again_behind_a_hand_written_load(tmp_path):
    out = str(tmp_path / "probe.s")
    r = subprocess.run(["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "--cuda-device-only", "-S", os.path.join(ROOT, "tests", "m0_probe.hip"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels = re.findall(r"^_Z12probe_kernel.*?:.*?s_endpgm", open(out).read(), re.S | re.M)
    assert len(kernels) == 3
    for k in kernels:
        ops = re.findall(r"s_mov_b32 (m0), \S+|(global_load_lds_dword)", k)
        assert [a or b for a, b in ops] == ["m0", "global_load_lds_dword"] * 3, ops
