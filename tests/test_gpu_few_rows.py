"""Steps of up to eight rows, whose output and down projections add to the residual stream and write the
next norm's input in one launch: k ranges shorter than a pair of k-steps per wavefront up to several rounds
with a rest, one row, all eight and nine, several sequences, every shape of the projections that read the
many partial sums of squares, and matrices off the 16-byte grid, which keep the launches of more rows."""
import numpy as np
import pytest

from gpu_util import device_weights
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_odd_pointers import off_the_grid
import test_gpu_step as S

pytestmark = pytest.mark.gpu
TOL = 1e-2   # bf16 storage, as for all steps


def check(shape, sizes, seed, weights=None):
    w = weights or I.gen_weights(shape, seed)
    for l in w["layers"]:   # gains of their own, exact in 16 bits
        l["g_ffn"] = (0.5 + 0.25 * (np.arange(shape.d_model) % 5)).astype(np.float32)
    rng = np.random.default_rng(seed)
    trees = [I.tree_random(n, rng) for n in sizes]
    toks = [I.gen_tokens(shape.vocab, n, seed, "tree", s) for s, n in enumerate(sizes)]
    Ls = [40 + 9 * s for s in range(len(sizes))]
    S.run_and_check(shape, w, trees, toks, Ls, [S.prefix_normal(shape, seed, s, L) for s, L in enumerate(Ls)], TOL)
    return w


# d_ffn / 32 pairs of k-steps: 2 for eight wavefronts, one round of 64, a rest of a round, 129 = two rounds and one
@pytest.mark.parametrize("d,heads,ffn", [(2048, 16, 64), (2048, 8, 2048), (2112, 16, 2720), (4096, 1, 4128)])
def test_rows_and_k_ranges(d, heads, ffn):
    shape = I.ModelShape(2, d, heads, 128, ffn, 512, "bf16")
    w = None
    for sizes in ([1], [5], [8], [9], [3, 1, 4]):
        w = check(shape, sizes, 77 + ffn, w)


@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5, 6])
def test_every_shape_of_the_reading_projections(cfg):
    b.trj_set_tunable("gemm_cfg", cfg)
    try:
        check(I.ModelShape(1, 2048, 2, 64, 128, 2080, "bf16"), [7], 5)
    finally:
        b.trj_set_tunable("gemm_cfg", 0)


def test_widest_outputs():
    check(I.ModelShape(1, 2048, 2, 64, 64, 131072, "bf16"), [6], 6)   # 16 row tiles per workgroup


def test_matrices_off_the_grid(monkeypatch):
    def moved(shape, w):
        desc, dw = device_weights(shape, w)
        off_the_grid(dw)
        return desc, dw
    monkeypatch.setattr(S, "device_weights", moved)
    check(I.ModelShape(2, 2048, 4, 64, 96, 512, "bf16"), [5], 8)
