"""Steps of many rows whose output and down projections write the next norm's input themselves: widths with
four row groups (sums read as few parts) and more, one that is no whole number of groups and keeps the
launch behind the projection, row counts that fill and do not fill the last block, odd numbers of phases,
reading projections of every many-rows shape, and matrices off the 16-byte grid."""
import numpy as np
import pytest

from gpu_util import device_weights
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_odd_pointers import off_the_grid
import test_gpu_step as S

pytestmark = pytest.mark.gpu
TOL = 1e-2   # bf16 storage, as for all steps


@pytest.fixture
def knobs():
    """Two row tiles per wavefront and short k ranges let small projections take turns."""
    def put(wt):
        b.trj_set_tunable("gemm_big_wt", wt)
        b.trj_set_tunable("gemm_pair_min_k", 64)
        b.trj_set_tunable("max_split_k", 1)
    yield put
    b.trj_set_tunable("gemm_big_wt", 0)
    b.trj_set_tunable("gemm_pair_min_k", 4096)
    b.trj_set_tunable("max_split_k", 8)


def takes_turns(T, n_in, n_out):
    plan = b.trj_dev_gemm_plan(T, n_in, n_out, True)
    return plan["many_rows"] == 1 and plan["row_tiles"] == 4 and plan["k_parts"] == 2


def check(shape, sizes, seed):
    w = I.gen_weights(shape, seed)
    for l in w["layers"]:   # gains of their own, exact in 16 bits
        l["g_ffn"] = (0.5 + 0.25 * (np.arange(shape.d_model) % 5)).astype(np.float32)
    rng = np.random.default_rng(seed)
    trees = [I.tree_random(n, rng) for n in sizes]
    toks = [I.gen_tokens(shape.vocab, n, seed, "tree", s) for s, n in enumerate(sizes)]
    Ls = [11 + 9 * s for s in range(len(sizes))]
    S.run_and_check(shape, w, trees, toks, Ls, [S.prefix_normal(shape, seed, s, L) for s, L in enumerate(Ls)], TOL)


@pytest.mark.parametrize("sizes", [[128, 1], [128, 100, 28], [128, 127, 2], [90, 128, 128, 38]])
@pytest.mark.parametrize("d,heads,ffn", [(512, 4, 192), (640, 5, 448), (1152, 2, 320), (576, 4, 192)])
def test_widths_and_rows(knobs, d, heads, ffn, sizes):
    knobs(2)
    assert takes_turns(sum(sizes), 64 * heads, d) and takes_turns(sum(sizes), ffn, d)
    check(I.ModelShape(2, d, heads, 64, ffn, 512, "bf16"), sizes, d + sum(sizes))


@pytest.mark.parametrize("ffn,vocab", [(5504, 512), (64, 16384), (2752, 8192)])   # wide readers: 4 x 8 and 4 x 4 tiles
def test_reading_projections(knobs, ffn, vocab):
    knobs(2)
    check(I.ModelShape(1, 640, 2, 64, ffn, vocab, "bf16"), [128, 128, 44], ffn + vocab)


def test_matrices_off_the_grid(knobs, monkeypatch):
    def moved(shape, w):
        desc, dw = device_weights(shape, w)
        keep = [(a.wo, a.w_down) for a in dw._arr]
        off_the_grid(dw)
        for a, (wo, down) in zip(dw._arr, keep):   # the readers off the grid, the writers on it
            a.wo, a.w_down = wo, down
        return desc, dw
    monkeypatch.setattr(S, "device_weights", moved)
    knobs(2)
    check(I.ModelShape(2, 640, 4, 64, 192, 512, "bf16"), [128, 100], 8)
