"""The fp32 kernels at the edges of their splits: few and many granules of the k range, both
token-group sizes, inputs that are not 16-byte aligned, head widths on both sides of what a
workgroup's threads cover, prefixes that end inside a group of four slots."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, rel_err, to_dev
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from test_gpu_attention import TOL, case, run_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("T,n_in,n_out", [(1, 16, 32), (5, 272, 96), (16, 1040, 64), (17, 528, 160), (31, 256, 32)])
def test_f32_linear_edges(T, n_in, n_out, shift):
    rng = np.random.default_rng(T + n_in)
    x = rng.standard_normal((T, n_in)).astype(np.float32)
    w = (rng.standard_normal((n_out, n_in)) * 0.05).astype(np.float32)
    buf = torch.zeros(T * n_in + 1, device=DEV)
    xd = buf[shift:shift + T * n_in].view(T, n_in)   # shift 1: 4-byte aligned only
    xd.copy_(torch.from_numpy(x))
    wd = to_dev(w, torch.float32)
    wp = torch.empty_like(wd)
    b.trj_pack_weight(wp, wd, n_out, n_in, b.F32, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), device=DEV)
    ws = torch.empty(2 * 128 * n_in + 32 * T * n_out + 1024, dtype=torch.uint8, device=DEV)
    b.trj_linear(xd, wp, T, n_in, n_out, b.F32, 0, ws, y)
    torch.cuda.synchronize()
    # sums of at most 1040 fp32 products in 32 parts: 2^-24 * (33 + 32) relative to |x||w|
    assert rel_err(y.cpu().numpy(), x.astype(np.float64) @ w.astype(np.float64).T) <= 1e-5


@pytest.mark.parametrize("H,dh,L,n", [(2, 32, 0, 1), (3, 32, 510, 5), (2, 96, 61, 33), (1, 160, 3, 128),
                                      (1, 544, 30, 7), (2, 64, 1023, 2)])
def test_f32_attention_edges(H, dh, L, n):
    c = case(40 + dh + L, H, dh, L, n, "f32")
    got = run_attention("f32", H, dh, [c])[0]
    assert np.isfinite(got).all()
    assert rel_err(got, O.tree_attention(*c)) <= TOL["f32"]
