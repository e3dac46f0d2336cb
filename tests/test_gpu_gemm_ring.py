"""The bf16 projection kernel at the edges of its ring of phase buffers: k ranges of one
k-step up to a few phases, fewer phases than buffers, k-steps beyond the end, row tiles and
token tiles that do not fill a workgroup, and the shapes with the widest workgroups."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, rel_err, to_dev
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_linear import run_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n_in,n_out,split_k", [
    # one pass of token tiles: one to five phases of 8, 4 or 2 k-steps with and without a rest
    (5, 16, 32, 1), (33, 144, 96, 1), (64, 256, 12288, 1), (96, 400, 12320, 1), (128, 528, 12288, 1),
    (17, 64, 22016, 1), (70, 272, 28672, 1), (128, 320, 28704, 1), (64, 80, 4096, 8), (40, 2064, 4096, 4),
    # outputs too wide for one round: 16 row tiles per workgroup, the last one not full
    (5, 16, 131072, 1), (96, 80, 130080, 1), (128, 112, 131072, 1),
    # many rows: token tiles that do not fill the last block, one phase, an odd k-step count
    (129, 256, 2048, 1), (300, 48, 12288, 1), (384, 1040, 4128, 2), (640, 16, 32032, 1), (1000, 80, 22016, 1),
    (1024, 144, 12320, 1), (1024, 1104, 4096, 4)])
def test_ring_edges(T, n_in, n_out, split_k):
    got, want = run_linear("bf16", T, n_in, n_out, split_k, seed=T + n_in)
    assert np.isfinite(got).all()
    # products of bf16 values are exact in fp32; at most 2064 additions of relative error
    # 2^-24 each, in sums no larger than a few times the largest result
    assert rel_err(got, want) <= 1e-5


@pytest.mark.parametrize("T,n_in,n_out", [(20, 144, 96), (64, 48, 131072), (300, 48, 4096)])
def test_repeated_last_k_step_adds_nothing(T, n_in, n_out):
    """k-steps past the end are read from the last real one: an infinite weight there must
    appear in its sum once (and not as infinity times zero)."""
    rng = np.random.default_rng(3)
    x = I.bf16_round(rng.standard_normal((T, n_in)).astype(np.float32))
    w = I.bf16_round((rng.standard_normal((n_out, n_in)) * 0.05).astype(np.float32))
    x[:, -1] = 1.0
    w[3, -1] = np.inf
    wd = to_dev(w, torch.bfloat16)
    wp = torch.empty_like(wd)
    b.trj_pack_weight(wp, wd, n_out, n_in, b.BF16, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(2 * 128 * ((T + 127) // 128) * n_in + 32 * T * n_out + 1024, dtype=torch.uint8, device=DEV)
    b.trj_linear(to_dev(x, torch.bfloat16), wp, T, n_in, n_out, b.BF16, 1, ws, y)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert np.all(np.isposinf(got[:, 3]))
    rest = [i for i in range(n_out) if i != 3][:256]
    assert rel_err(got[:, rest], x.astype(np.float64) @ w[rest].astype(np.float64).T) <= 1e-5
