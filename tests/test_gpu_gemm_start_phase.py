"""Projections of few rows, whose workgroups start at different phases of their k range and go
round: as many phases as ring buffers, one more and one less, a range of one phase, k-splits
with a shorter last one, in every workgroup shape with more than one row tile, and both sides of the
limit on the activations' size."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, rel_err, to_dev
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_linear import run_linear

pytestmark = pytest.mark.gpu

# knob gemm_cfg -> (row tiles, k-parts) of a workgroup, k-steps of a phase; 0: the plan's own, which
# takes 16 row tiles only for the widest outputs
SHAPES = {1: (4, 1, 4), 2: (2, 4, 8), 3: (2, 2, 4), 4: (4, 2, 4), 6: (3, 2, 8), 0: (16, 1, 2)}


def buffers(cfg, token_tiles):
    """Phases that the ring holds: what fits 160 KiB, at most four."""
    if cfg == 2:
        return 3 if token_tiles == 4 else 4
    if cfg == 6:
        return 2 if token_tiles == 4 else 3
    return 4


@pytest.fixture
def shape():
    def put(cfg):
        b.trj_set_tunable("gemm_cfg", cfg)
    yield put
    b.trj_set_tunable("gemm_cfg", 0)


def run_counted(T, ksteps, n_out, split_k):
    """Output r is, for every token, the sum of distinct powers of two, one per k-step s with s % 4 ==
    r % 4, times a small number of the token's own: exact, and changed by a k-step left out, repeated
    or taken with another one's or another token's activations."""
    n_in, s = 16 * ksteps, np.arange(ksteps)
    own = 1.0 + np.arange(T) % 3
    x, w = np.zeros((T, n_in), np.float32), np.zeros((n_out, n_in), np.float32)
    x[:, 16 * s + 5] = own[:, None] * 2.0 ** (s // 4)
    w[:, 16 * s + 5] = (s[None, :] % 4 == np.arange(n_out)[:, None] % 4)
    assert 3 * 2 ** ((ksteps + 3) // 4) < 2 ** 24 and np.array_equal(I.bf16_round(x), x)
    wd = to_dev(w, torch.bfloat16)
    wp = torch.empty_like(wd)
    b.trj_pack_weight(wp, wd, n_out, n_in, b.BF16, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(2 * 128 * n_in + 32 * T * n_out + 1024, dtype=torch.uint8, device=DEV)
    b.trj_linear(to_dev(x, torch.bfloat16), wp, T, n_in, n_out, b.BF16, split_k, ws, y)
    torch.cuda.synchronize()
    per = np.array([sum(2.0 ** (k // 4) for k in range(ksteps) if k % 4 == r) for r in range(4)])
    want = own[:, None] * per[np.arange(n_out) % 4][None, :]
    return y.cpu().numpy(), want.astype(np.float32)


@pytest.mark.parametrize("T", [7, 33, 69, 128])
@pytest.mark.parametrize("cfg", sorted(SHAPES))
def test_every_k_step_is_added_once(shape, cfg, T):
    rows, parts, steps = SHAPES[cfg]
    shape(cfg)
    n_out = 131072 if cfg == 0 else 2080   # 65 row tiles: the last workgroup is not full
    ring = buffers(cfg, min(4, (T + 31) // 32))
    for phases in sorted({1, ring - 1, ring, ring + 1, 2 * ring + 1} - {0}):
        plan = b.trj_dev_gemm_plan(T, 16 * phases * steps, n_out, True)
        assert (plan["row_tiles"], plan["k_parts"], plan["many_rows"]) == (rows, parts, 0)
        got, want = run_counted(T, phases * steps, n_out, 1)
        assert np.array_equal(got, want), phases


@pytest.mark.parametrize("T", [20, 64, 100])
@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 6])
def test_splits_with_a_shorter_last_one(shape, cfg, T):
    shape(cfg)
    got, want = run_counted(T, 7 * SHAPES[cfg][2], 1056, 4)   # 7 phases: 2, 2, 2 and 1
    assert np.array_equal(got, want)


# 2^19 activation elements, one phase of 8 k-steps below and above
@pytest.mark.parametrize("T,n_in", [(128, 4096), (128, 3968), (128, 4224), (96, 5376), (96, 5504), (64, 8192), (64, 8320)])
def test_both_sides_of_the_activations_limit(shape, T, n_in):
    shape(2)
    assert b.trj_dev_gemm_plan(T, n_in, 2080, True)["row_tiles"] == 2
    got, want = run_linear("bf16", T, n_in, 2080, 1, seed=T + n_in)
    assert np.isfinite(got).all()
    # products of bf16 values are exact in fp32; at most 8320 additions of relative error 2^-24
    # each, in sums no larger than a few times the largest result
    assert rel_err(got, want) <= 1e-5


@pytest.mark.parametrize("T,n_in,n_out", [(7, 2048, 12288), (64, 512, 12288), (128, 640, 12288), (5, 1024, 28672),
                                          (96, 1024, 22016), (128, 1024, 22016)])
def test_shapes_of_the_plan(T, n_in, n_out):
    plan = b.trj_dev_gemm_plan(T, n_in, n_out, True)
    assert plan["row_tiles"] > 1 and plan["many_rows"] == 0
    got, want = run_linear("bf16", T, n_in, n_out, 1, seed=T + n_in)
    assert rel_err(got, want) <= 1e-5   # fewer additions than above
