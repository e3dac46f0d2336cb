"""The one-launch prologue (tree checks by pointer doubling, rotary table, work list, rows
without a valid sequence, embedding) on both sides of the number of sequences it takes."""
import numpy as np
import pytest

from gpu_util import rel_err
from oracle import tr_oracle as O
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL, case, run_attention

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
