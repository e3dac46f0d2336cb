"""Steps of many rows whose output and down projections write the next norm's input themselves: widths with
four row groups (sums read as few parts) and more, one that is no whole number of groups and keeps the
launch behind the projection, row counts that fill and do not fill the last block, odd numbers of phases,
more than four sums read by the 4 x 4 tile with and without turns, the 2 x 4, 4 x 8 and 8 x 8 tiles, and matrices
off the 16-byte grid.  Launches of the norm behind the projection are counted; rows whose sum of squares
is one part are among the cases, as 1e-2 does not see one of many equal parts missing."""
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


def check(shape, sizes, seed, norms=0, embed=None):
    """norms: launches of the norm behind a projection, in all layers."""
    w = I.gen_weights(shape, seed)
    if embed is not None:
        embed(w["embed"])
    for l in w["layers"]:   # gains of their own, exact in 16 bits
        l["g_ffn"] = (0.5 + 0.25 * (np.arange(shape.d_model) % 5)).astype(np.float32)
    rng = np.random.default_rng(seed)
    trees = [I.tree_random(n, rng) for n in sizes]
    toks = [I.gen_tokens(shape.vocab, n, seed, "tree", s) for s, n in enumerate(sizes)]
    Ls = [11 + 9 * s for s in range(len(sizes))]
    b.trj_profile_begin(5, 8)
    try:
        S.run_and_check(shape, w, trees, toks, Ls, [S.prefix_normal(shape, seed, s, L) for s, L in enumerate(Ls)], TOL)
    finally:
        launches = len(b.trj_profile_end(8))
    assert launches == norms


@pytest.mark.parametrize("sizes", [[128, 1], [128, 100, 28], [128, 127, 2], [90, 128, 128, 38]])
@pytest.mark.parametrize("d,heads,ffn", [(512, 4, 192), (640, 5, 448), (1152, 2, 320), (576, 4, 192)])
def test_widths_and_rows(knobs, d, heads, ffn, sizes):
    knobs(2)
    assert takes_turns(sum(sizes), 64 * heads, d) and takes_turns(sum(sizes), ffn, d)
    check(I.ModelShape(2, d, heads, 64, ffn, 512, "bf16"), sizes, d + sum(sizes), norms=4 if d % 128 else 0)


# 128-column parts: first and last, both sides of the sixteen that are read at a time
@pytest.mark.parametrize("d,part", [(640, 0), (640, 4), (2176, 0), (2176, 15), (2176, 16)])
def test_every_part_of_a_sum_of_squares_counts(knobs, d, part):
    knobs(2)

    def embed(e):
        cols = slice(128 * part, 128 * part + 128)
        size = 4 * (1 + np.arange(len(e)) % 5)[:, None]   # no row's factor is its neighbour's
        e[:, cols] = I.bf16_round((np.sign(e[:, cols]) * size).astype(np.float32))
    check(I.ModelShape(2, d, 2, 64, 128, 512, "bf16"), [128, 70], part, embed=embed)


def reader(T, n_in, n_out):
    p = b.trj_dev_gemm_plan(T, n_in, n_out, True)
    assert p["many_rows"] == 1
    return p["row_tiles"], p["token_tiles"], p["k_parts"]


# gate/up and LM head: 4 x 8 tiles, or 4 x 4 that take turns
@pytest.mark.parametrize("ffn,vocab,gate_up,head", [(5504, 512, (4, 8, 1), (4, 4, 2)), (64, 16384, (4, 4, 2), (4, 8, 1)),
                                                    (2752, 8192, (4, 4, 2), (4, 4, 2))])
def test_wide_readers(knobs, ffn, vocab, gate_up, head):
    knobs(2)
    assert (reader(300, 640, 2 * ffn), reader(300, 640, vocab), reader(300, 640, 384)) == (gate_up, head, (4, 4, 2))
    check(I.ModelShape(1, 640, 2, 64, ffn, vocab, "bf16"), [128, 128, 44], ffn + vocab)


def test_reader_without_turns(knobs):
    """4 x 4 tiles by gemm_ring_kernel: a k range below the least that takes turns, behind one that does."""
    knobs(2)
    b.trj_set_tunable("gemm_pair_min_k", 704)
    assert takes_turns(300, 704, 640) and reader(300, 640, 512) == reader(300, 640, 2 * 704) == (4, 4, 1)
    check(I.ModelShape(2, 640, 11, 64, 704, 512, "bf16"), [128, 128, 44], 17)


@pytest.mark.parametrize("vocab,tile", [(512, (2, 4, 4)), (8192, (4, 8, 1)), (16384, (8, 8, 1))])
def test_readers_of_other_tiles(knobs, vocab, tile):
    """Shapes as they are chosen without a knob for the tile: wide enough for the writers to take turns."""
    knobs(0)
    assert takes_turns(996, 64, 2176) and reader(996, 2176, vocab) == tile and reader(996, 2176, 192) == (2, 4, 4)
    check(I.ModelShape(1, 2176, 1, 64, 64, vocab, "bf16"), [128] * 7 + [100], vocab)


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
    assert takes_turns(228, 256, 640) and takes_turns(228, 192, 640)
    check(I.ModelShape(2, 640, 4, 64, 192, 512, "bf16"), [128, 100], 8)
