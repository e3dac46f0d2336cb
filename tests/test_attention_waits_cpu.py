"""The attention's walk through registers, in the assembly of this build: the wait for a block's
first K piece leaves the other K pieces and the whole V of the block before on the way.  What the
code in front of the loop waits for decides this too, which no result shows, only the time."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_17404_amd import build

NAME = r"tree_attn_bf16_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELNS_8AttnFormE0ELb([01])E"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "attn.s")
    r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "attn_bf16.hip"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = open(out).read()
    found = {}
    for m in re.finditer(r"^(\S*" + NAME + r"\S*):", text, re.M):
        body = text[m.end():text.index(".Lfunc_end", m.end())].split("\n")
        found[tuple(int(g) for g in m.groups()[1:])] = body
    return found


def main_loop(body):
    """Lines of the loop that multiplies: from the target of the backward branch around it."""
    at = {m[1]: i for i, m in enumerate(re.match(r"(\.LBB\w+):", l) for l in body) if m}
    for i, l in enumerate(body):
        m = re.search(r"s_c?branch\w*\s+(\.LBB\w+)", l)
        if m and at.get(m[1], i) < i and sum("v_mfma" in x for x in body[at[m[1]]:i]) >= 8:
            return body[at[m[1]]:i]
    raise AssertionError("no loop")


def test_all_register_forms_are_there(kernels):
    assert {k[:2] for k in kernels} == {(128, 1), (128, 2), (128, 4), (64, 1), (64, 2)} and len(kernels) == 10


@pytest.mark.parametrize("dh,tiles", [(128, 1), (128, 2), (128, 4), (64, 1), (64, 2)])
@pytest.mark.parametrize("checks_itself", [0, 1])
def test_values_stay_on_the_way(kernels, dh, tiles, checks_itself):
    body = next(v for k, v in kernels.items() if k[0] == dh and k[1] == tiles and k[3] == checks_itself)
    first = next(re.search(r"vmcnt\((\d+)\)", l) for l in main_loop(body) if "vmcnt" in l)
    pieces = dh // 16   # of K, and as many of V
    assert int(first[1]) == 2 * pieces - 1
