"""The one-launch prologue on both sides of the number of sequences it takes: in attention
calls the tree checks by pointer doubling, the work list and the rows without a valid sequence
(a single bf16 sequence has no prologue, the attention kernel checks it), in whole steps the
rotary table and the embedding as well."""
import numpy as np
import pytest

from gpu_util import Batch, device_weights, rel_err, run_step
from oracle import tr_oracle as O
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL, case, run_attention
from test_gpu_template import check_against_oracle, pools_for, prefix_normal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B", [1, 63, 64, 65])
def test_sequences_around_the_limit_with_deep_trees_and_malformed_ones(dtype, B):
    rng = np.random.default_rng(B)
    H, dh = 2, 64
    sizes = [int(rng.choice([1, 2, 15, 16, 17, 33, 64, 65, 128])) for _ in range(B)]
    sizes[0] = 128
    cases = []
    for s, n in enumerate(sizes):
        L = int(rng.integers(0, 100))
        # chains need every doubling round, stars one, random trees something between
        parent = [I.tree_chain(n), np.array([-1] + [0] * (n - 1), np.int32), I.tree_random(n, rng)][s % 3]
        cases.append(case(500 + s, H, dh, L, n, dtype, np.asarray(parent, np.int32)))
    bad = [s for s in (5, B - 1) if 0 < s < B]
    for s in bad:   # a parent that does not precede its child, a second root
        q, k, v, parent, L = cases[s]
        p = parent.copy()
        p[len(p) // 2] = len(p) // 2 if len(p) > 1 else 0
        cases[s] = (q, k, v, p, L)
    got = run_attention(dtype, H, dh, cases, align=32)
    for s, (g, c) in enumerate(zip(got, cases)):
        if s in bad:
            assert not g.any(), s
        else:
            assert rel_err(g, O.tree_attention(*c)) <= TOL[dtype], s


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B", [64, 65])
def test_steps_around_the_limit(dtype, B):
    shape = I.ModelShape(2, 128, 2, 64, 256, 256, dtype)
    w = I.gen_weights(shape, 340)
    rng = np.random.default_rng(B)
    sizes = [int(rng.choice([1, 2, 5, 17, 33])) for _ in range(B)]
    trees = [I.tree_random(n, rng) for n in sizes]
    sizes[9] = 5
    trees[9] = np.array([-1, 0, 3, 1, 0], np.int32)      # a parent behind its child
    Ls = [int(rng.integers(0, 60)) for _ in range(B)]
    toks = [I.gen_tokens(shape.vocab, n, 340, "tree", s) for s, n in enumerate(sizes)]
    pkvs = [prefix_normal(shape, 340, s, L) if L else None for s, L in enumerate(Ls)]
    desc, dw = device_weights(shape, w)
    batch = Batch(trees, Ls, toks)
    kp, vp = pools_for(shape, batch, Ls, pkvs)
    res = run_step(shape, desc, dw, batch, kp, vp)
    assert list(np.flatnonzero(res["status"])) == [9]
    assert res["accept_len"][9] == -1 and res["new_len"][9] == Ls[9]
    check_against_oracle(shape, w, res, batch, trees, toks, Ls, pkvs, TOL[dtype], skip=(9,))
