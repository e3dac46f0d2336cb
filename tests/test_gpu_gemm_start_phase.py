"""Projections of few rows, whose workgroups start at different phases of their k range and go
round: as many phases as ring buffers, one more and one less, a range of one phase, k-splits
with a shorter last one, and both sides of the limit on the activations' size."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, rel_err, to_dev
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_linear import run_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n_in,n_out,split_k", [
    # 8 k-steps per phase: 1, 3, 4, 5 phases of 12288 outputs (192 workgroups of two row tiles)
    (7, 128, 12288, 1), (33, 384, 12288, 1), (64, 512, 12288, 1), (128, 640, 12288, 1),
    # 4 k-steps per phase, split: 7 phases in splits of 2, 2, 2, 1
    (20, 448, 4096, 4), (64, 448, 4096, 4), (100, 2048, 256, 2),
    # 2 k-steps per phase, 16 row tiles per workgroup
    (5, 32, 131072, 1), (69, 160, 131072, 1),
    # activations of exactly 2^19 elements and above
    (128, 4096, 2080, 1), (96, 5504, 2080, 1), (128, 4224, 2080, 1)])
def test_start_phase(T, n_in, n_out, split_k):
    got, want = run_linear("bf16", T, n_in, n_out, split_k, seed=T + n_in)
    assert np.isfinite(got).all()
    # products of bf16 values are exact in fp32; at most 5504 additions of relative error 2^-24
    # each, in sums no larger than a few times the largest result
    assert rel_err(got, want) <= 1e-5


def test_every_k_step_is_added_once():
    """Powers of two add exactly: output r is the sum of distinct bits, one per phase of 8 k-steps,
    so a phase left out, repeated or taken with the wrong activations changes it."""
    n_in, n_out, T = 8 * 16 * 11, 12288, 40
    x, w = np.zeros((T, n_in), np.float32), np.zeros((n_out, n_in), np.float32)
    for p in range(11):
        x[:, p * 128 + 5] = 2.0 ** p
        w[:, p * 128 + 5] = 1.0
    x[:, 6] = np.arange(T)
    w[:, 6] = 2.0 ** 11
    wd = to_dev(I.bf16_round(w), torch.bfloat16)
    wp = torch.empty_like(wd)
    b.trj_pack_weight(wp, wd, n_out, n_in, b.BF16, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(2 * 128 * n_in + 4 * T * n_out + 1024, dtype=torch.uint8, device=DEV)
    b.trj_linear(to_dev(I.bf16_round(x), torch.bfloat16), wp, T, n_in, n_out, b.BF16, 1, ws, y)
    torch.cuda.synchronize()
    want = (2.0 ** 11 - 1) + 2.0 ** 11 * np.arange(T)
    assert np.array_equal(y.cpu().numpy(), np.repeat(want[:, None], n_out, 1).astype(np.float32))
