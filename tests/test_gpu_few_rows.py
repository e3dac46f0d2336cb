"""Steps of up to eight rows, whose output and down projections add to the residual stream and write the
next norm's input in one launch: k ranges shorter than a pair of k-steps per wavefront up to several rounds
with a rest, one row, all eight and nine, several sequences, every shape of the projections that read the
many partial sums of squares, and matrices off the 16-byte grid and k ranges too long for the output's
width, which keep the launches of more rows.  Launches of the split-k sum, which the steps do without,
are counted; and as 1e-2 does not see one of 128 or more equal parts missing from a sum of squares, rows
whose sum is one part are among the cases."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, Batch, device_weights, kv_heads
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_odd_pointers import off_the_grid
import test_gpu_step as S

pytestmark = pytest.mark.gpu
TOL = 1e-2   # bf16 storage, as for all steps


def check(shape, sizes, seed, weights=None, sums=0):
    """sums: launches of the split-k sum per layer; none up to eight rows."""
    w = weights or I.gen_weights(shape, seed)
    for l in w["layers"]:   # gains of their own, exact in 16 bits
        l["g_ffn"] = (0.5 + 0.25 * (np.arange(shape.d_model) % 5)).astype(np.float32)
    rng = np.random.default_rng(seed)
    trees = [I.tree_random(n, rng) for n in sizes]
    toks = [I.gen_tokens(shape.vocab, n, seed, "tree", s) for s, n in enumerate(sizes)]
    Ls = [40 + 9 * s for s in range(len(sizes))]
    b.trj_profile_begin(5, 8)
    try:
        S.run_and_check(shape, w, trees, toks, Ls, [S.prefix_normal(shape, seed, s, L) for s, L in enumerate(Ls)], TOL)
    finally:
        launches = len(b.trj_profile_end(8))
    assert launches == (sums if sum(sizes) <= 8 else 2) * shape.n_layers
    return w


# d_ffn / 32 pairs of k-steps: 2 for eight wavefronts, one round of 64, a rest of a round, 129 = two rounds and one
@pytest.mark.parametrize("d,heads,ffn", [(2048, 16, 64), (2048, 8, 2048), (2112, 16, 2720), (4096, 1, 4128)])
def test_rows_and_k_ranges(d, heads, ffn):
    shape = I.ModelShape(2, d, heads, 128, ffn, 512, "bf16")
    w = None
    for sizes in ([1], [5], [8], [9], [3, 1, 4]):
        w = check(shape, sizes, 77 + ffn, w)


# 16-column parts: first and last, both sides of what a lane reads (four parts) and of half a wavefront's
@pytest.mark.parametrize("d,part", [(2048, 0), (2048, 3), (2048, 4), (2048, 127), (2112, 128), (2112, 131), (4096, 0),
                                    (4096, 7), (4096, 124), (4096, 128), (4096, 255)])
def test_every_part_of_a_sum_of_squares_counts(d, part):
    """Rows whose residual stream is large in one part alone, and in no two rows of neighbouring ids as large:
    without the part, or with another row's, the factor is far off."""
    shape = I.ModelShape(2, d, 2, 64, 128, 512, "bf16")
    w = I.gen_weights(shape, part)
    cols = slice(16 * part, 16 * part + 16)
    size = 4 * (1 + np.arange(shape.vocab) % 5)[:, None]
    w["embed"][:, cols] = I.bf16_round((np.sign(w["embed"][:, cols]) * size).astype(np.float32))
    check(shape, [8], part, w)


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
    check(I.ModelShape(2, 2048, 4, 64, 96, 512, "bf16"), [5], 8, sums=2)


def sum_launches(shape, n):
    """Launches of the split-k sum in a step of one sequence with n rows, random weights made on the device."""
    desc = b.make_desc(shape)
    dw = b.DeviceWeights(desc)
    d, hd, kvd, f = shape.d_model, shape.n_heads * shape.head_dim, kv_heads(shape) * shape.head_dim, shape.d_ffn

    def matrix(rows, cols):
        return (torch.randn(rows, cols, device=DEV) * 0.02).to(torch.bfloat16)
    for _ in range(shape.n_layers):
        dw.add_layer(torch.ones(d, device=DEV), matrix(hd + 2 * kvd, d), matrix(d, hd), torch.ones(d, device=DEV),
                     matrix(2 * f, d), matrix(d, f))
    dw.set_globals(matrix(shape.vocab, d), torch.ones(d, device=DEV), matrix(shape.vocab, d))
    dw.finish()
    batch = Batch([I.tree_chain(n)], [0], [np.arange(n, dtype=np.int32)])
    stride = kv_heads(shape) * batch.s_pool * shape.head_dim
    kp, vp = (torch.zeros(shape.n_layers, stride, dtype=torch.bfloat16, device=DEV) for _ in "kv")
    ws = torch.empty(b.trj_workspace_bytes(desc, n, 1, batch.max_seq_slots), dtype=torch.uint8, device=DEV)
    out = [torch.zeros(n, dtype=torch.int32, device=DEV) for _ in range(6)]
    path = torch.zeros(1, b.N_MAX, dtype=torch.int32, device=DEV)
    b.trj_profile_begin(5, 8 * shape.n_layers)
    b.tr_verify_step(desc, dw.struct, kp, vp, stride, batch.s_pool, batch.tok, batch.parent, batch.node_off, batch.kv_off,
                     batch.prefix, 1, n, batch.max_seq_slots, ws, None, out[0], out[1], out[2], path, out[3], out[4], out[5])
    torch.cuda.synchronize()
    return len(b.trj_profile_end(8 * shape.n_layers))


# one layer: the sums behind the output projection (k range heads x 128) and the down projection (k range ffn)
@pytest.mark.parametrize("d,heads,ffn,sums", [
    (2048, 2, 8192, 0), (2048, 2, 8224, 1), (2496, 2, 8224, 1), (2048, 65, 64, 1), (2048, 64, 64, 0), (2560, 2, 10240, 0),
    (2560, 2, 10272, 1), (2816, 2, 12288, 0), (2816, 2, 12320, 1), (3264, 2, 12320, 1), (3328, 2, 16384, 0),
    (4096, 2, 16384, 0), (4096, 2, 16416, 1), (4096, 32, 11008, 0), (1984, 2, 64, 2), (4160, 2, 64, 2)])
def test_long_k_ranges_keep_their_splits(d, heads, ffn, sums):
    shape = I.ModelShape(1, d, heads, 128, ffn, 512, "bf16")
    assert [sum_launches(shape, n) for n in (1, 8, 9)] == [sums, sums, 2]


@pytest.mark.parametrize("shape", [I.ModelShape(2, 2048, 2, 64, 8224, 512, "bf16"),     # down projections split
                                   I.ModelShape(2, 2048, 65, 128, 64, 512, "bf16")])    # output projections split
def test_one_projection_of_a_layer_split(shape):
    check(shape, [3, 2], 3, sums=1)
