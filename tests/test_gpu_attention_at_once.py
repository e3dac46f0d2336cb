"""The bf16 attention's form that loads all of a workgroup's K/V at once, at its edges: key
streams with no, one and two blocks, a last block that holds one key, trees over one and two
query groups, and workgroups one block beyond it, which take another form; and trees whose
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
def test_one_sequence(knobs, L, n):
    H, dh = 3, 128
    for tree in (I.tree_random(n, np.random.default_rng(L)), I.tree_chain(n)):
        c = case(5 * L + n, H, dh, L, n, "bf16", np.asarray(tree, np.int32))
        want = O.tree_attention(*c)
        for wgs in (1, 16, 64, 4096):   # from one workgroup per head and group to one block per stream
            knobs(attn_target_wgs=wgs, attn_min_bpw=1, attn_xchg_min_blocks=1 << 20)
            got = run_attention("bf16", H, dh, [c])[0]
            assert np.isfinite(got).all() and rel_err(got, want) <= TOL["bf16"], wgs


def test_batch(knobs):
    sizes, lens = [64, 33, 1, 50, 64, 34], [0, 200, 30, 500, 190, 96]
    cases = [case(40 + s, 2, 128, L, n, "bf16") for s, (n, L) in enumerate(zip(sizes, lens))]
    for wgs in (1, 30, 256):
        knobs(attn_target_wgs=wgs, attn_min_bpw=1, attn_xchg_min_blocks=1 << 20)
        for g, c in zip(run_attention("bf16", 2, 128, cases, align=32), cases):
            assert rel_err(g, O.tree_attention(*c)) <= TOL["bf16"], wgs
