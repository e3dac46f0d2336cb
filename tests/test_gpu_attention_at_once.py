"""The bf16 attention's form that loads all of a workgroup's K/V at once, at its edges: key
streams with no, one and two blocks, a last block that holds one key, trees over one and two
query groups, and workgroups beyond it, which take another form; and trees whose
ancestor bits need one and two nodes per lane where only some streams meet the tree."""
import numpy as np
import pytest

from oracle import tr_oracle as O
from gpu_util import rel_err
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL, case, run_attention
from test_gpu_attention_ring import knobs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n", [(0, 33), (1, 64), (63, 33), (96, 64), (128, 64), (192, 64), (223, 33), (224, 33),
                                 (288, 64), (600, 40), (1025, 64), (100, 128), (513, 97)])
def test_one_and_two_sequences(knobs, L, n):
    """One sequence that the kernel checks itself (this form only with one query group), two behind
    a prologue."""
    H, dh = 3, 128
    forms = {1: set(), 2: set()}
    for tree in (I.tree_random(n, np.random.default_rng(L)), I.tree_chain(n)):
        cs = [case(5 * L + n + s, H, dh, L, n, "bf16", np.asarray(tree, np.int32)) for s in (0, 1)]
        want = [O.tree_attention(*c) for c in cs]
        for wgs in (1, 16, 64, 4096):   # from one workgroup per head and group to one block per stream
            knobs(attn_target_wgs=wgs, attn_min_bpw=1, attn_xchg_min_blocks=1 << 20)
            for B in (1, 2):
                forms[B].add(b.trj_dev_attn_launch(B, B * n, H, H, dh, L + n)["form"])
                for got, w in zip(run_attention("bf16", H, dh, cs[:B]), want):
                    assert np.isfinite(got).all() and rel_err(got, w) <= TOL["bf16"], (wgs, B)
    assert "once" in forms[2] and ("once" in forms[1]) == (n <= 64)


def test_batch(knobs):
    sizes, lens = [64, 33, 1, 50, 64, 34], [0, 200, 30, 500, 190, 96]
    cases = [case(40 + s, 2, 128, L, n, "bf16") for s, (n, L) in enumerate(zip(sizes, lens))]
    for wgs, form in ((1, "registers"), (30, "registers"), (256, "once")):
        knobs(attn_target_wgs=wgs, attn_min_bpw=1, attn_xchg_min_blocks=1 << 20)
        assert b.trj_dev_attn_launch(6, sum(sizes), 2, 2, 128, 550)["form"] == form
        for g, c in zip(run_attention("bf16", 2, 128, cases, align=32), cases):
            assert rel_err(g, O.tree_attention(*c)) <= TOL["bf16"], wgs
