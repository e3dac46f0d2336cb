"""The fp32 kernels whose threads ask for several pieces together: k ranges one granule around
a whole batch of them with few rows on both sides of each limit, and attention whose keys end
just before, at and behind the first batch of value groups, with NaN in slots nobody sees."""
import numpy as np
import pytest

from gpu_util import rel_err
from oracle import tr_oracle as O
from test_gpu_attention import TOL, case, run_attention
from test_gpu_linear import run_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in", [256, 272, 512, 1008, 1024, 1040, 2064])
@pytest.mark.parametrize("T", [1, 2, 3, 16, 17, 32, 33])
def test_linear(T, n_in):
    got, want = run_linear("f32", T, n_in, 96, 0, seed=T + n_in)
    assert np.isfinite(got).all()
    assert rel_err(got, want) <= 1e-5   # at most (65 + 32) additions of 2^-24 relative to |x||w|


# a batch covers 5 * 4 * (512 / dh) keys: 160 with heads of 64, 80 of 128, 320 of 32, 60 of 160, 20 of 512
@pytest.mark.parametrize("H,dh,L,n", [(2, 64, 158, 1), (2, 64, 159, 1), (2, 64, 160, 1), (1, 64, 150, 30), (2, 128, 79, 5),
                                      (1, 128, 400, 20), (2, 32, 316, 9), (1, 160, 57, 4), (1, 512, 17, 6), (1, 96, 0, 1)])
def test_attention(H, dh, L, n):
    c = case(60 + dh + L, H, dh, L, n, "f32")
    got = run_attention("f32", H, dh, [c])[0]
    assert np.isfinite(got).all()
    assert rel_err(got, O.tree_attention(*c)) <= TOL["f32"]
