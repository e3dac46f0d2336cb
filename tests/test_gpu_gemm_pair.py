"""The many-rows projection whose two groups of wavefronts take turns, at its edges: one phase of
its k range, fewer phases than buffers, odd numbers of them, row and token tiles that do not fill
the last workgroups, and k ranges beside it that another kernel takes."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, rel_err, to_dev
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_linear import run_linear

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def short_k_ranges_too():
    """By itself the plan takes turns from a k range of 4096 on (test_gemm_pair_plan_cpu.py)."""
    b.trj_set_tunable("gemm_pair_min_k", 64)
    yield
    b.trj_set_tunable("gemm_pair_min_k", 4096)


def takes_turns(T, n_in, n_out):
    plan = b.trj_dev_gemm_plan(T, n_in, n_out, True)
    return plan["many_rows"] == 1 and plan["row_tiles"] == 4 and plan["k_parts"] == 2


@pytest.mark.parametrize("n_in,turns", [(64, True), (128, True), (192, True), (256, True), (320, True), (384, True),
                                        (448, True), (1088, True), (11008, True), (80, False), (1040, False)])
@pytest.mark.parametrize("T,n_out", [(1024, 4096), (1000, 4000), (500, 8000)])
def test_edges(T, n_out, n_in, turns):
    assert takes_turns(T, n_in, n_out) == turns
    if n_in > 1088 and T != 1000:
        return   # one of the long ones is enough
    got, want = run_linear("bf16", T, n_in, n_out, 1, seed=T + n_in)
    assert np.isfinite(got).all()
    # products of bf16 values are exact in fp32; at most 11008 additions of relative error 2^-24
    # each, in sums no larger than a few times the largest result
    assert rel_err(got, want) <= 1e-5


def test_phases_behind_the_last_add_nothing():
    """An odd number of phases: the last one is requested again for the group that has no turn left;
    an infinite weight in it must appear once, and not as infinity times zero."""
    T, n_in, n_out = 1024, 320, 4096
    assert takes_turns(T, n_in, n_out)
    rng = np.random.default_rng(3)
    x = I.bf16_round(rng.standard_normal((T, n_in)).astype(np.float32))
    w = I.bf16_round((rng.standard_normal((n_out, n_in)) * 0.05).astype(np.float32))
    x[:, -1] = 1.0
    w[3, -1] = np.inf
    wd = to_dev(w, torch.bfloat16)
    wp = torch.empty_like(wd)
    b.trj_pack_weight(wp, wd, n_out, n_in, b.BF16, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(2 * T * n_in + 32 * T * n_out + 1024, dtype=torch.uint8, device=DEV)
    b.trj_linear(to_dev(x, torch.bfloat16), wp, T, n_in, n_out, b.BF16, 1, ws, y)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert np.all(np.isposinf(got[:, 3]))
    rest = [i for i in range(n_out) if i != 3][:256]
    assert rel_err(got[:, rest], x.astype(np.float64) @ w[rest].astype(np.float64).T) <= 1e-5
