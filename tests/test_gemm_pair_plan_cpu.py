"""Where the many-rows projection takes turns, on the host: only at the sizes where that measured
no slower than the kernel without turns."""
import pytest

from paper_2406_17404_amd import binding as b


def takes_turns(T, n_in, n_out):
    plan = b.trj_dev_gemm_plan(T, n_in, n_out, True)
    return plan["many_rows"] == 1 and plan["row_tiles"] == 4 and plan["k_parts"] == 2


@pytest.mark.parametrize("n_in,n_out,T,turns", [
    # short k ranges were 4 to 9 % slower with turns
    (1024, 4096, 1024, False), (1024, 4096, 640, False), (2048, 8192, 512, False), (2048, 8192, 320, False),
    (2048, 11008, 160, False), (2048, 16384, 200, False), (4032, 4096, 1024, False),
    (4096, 4096, 1024, True), (4096, 4096, 896, True), (11008, 4096, 1024, True), (8192, 2048, 2048, True),
    (4096, 22016, 1024, False), (4112, 4096, 1024, False)])   # more workgroups than units; a last phase that is not whole
def test_turns(n_in, n_out, T, turns):
    assert takes_turns(T, n_in, n_out) == turns
