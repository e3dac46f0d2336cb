"""One query tile whose sequence is walked by one workgroup per head: up to 24 blocks of slots, 25 are split;
a last block of one key, one row and a full tile, one sequence and two, K/V heads shared by two or four
query heads and not, heads of 64 and 128 (single heads of 64 come through rings, which have a rule of their
own)."""
import numpy as np
import pytest

from gpu_util import rel_err
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from test_gpu_attention import TOL, case, run_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,H,kv", [(128, 4, 4), (64, 2, 2), (128, 4, 2), (64, 4, 2), (64, 4, 1)])
@pytest.mark.parametrize("n", [1, 8, 32])
@pytest.mark.parametrize("slots", [512, 513, 544, 767, 768, 769])
def test_walk(slots, n, dh, H, kv):
    L, nb = slots - n, -(-slots // 32)
    cases = [case(slots + s, H, dh, L - 40 * s, n, "bf16", n_kv=0 if kv == H else kv) for s in (0, 1)]
    want = [O.tree_attention(*c) for c in cases]
    for B in (1, 2):
        plan = b.trj_dev_attn_launch(B, B * n, H, kv, dh, slots)
        if B * n <= 32 and (dh == 128 or kv < H):   # more rows may be one tree
            if nb <= 24:
                assert (plan["pack"], plan["tiles"], plan["form"], plan["splits"]) == (0, 1, "registers", 1)
            else:
                assert plan["form"] == "registers" and plan["splits"] > 1
        for got, w in zip(run_attention("bf16", H, dh, cases[:B]), want):
            assert np.isfinite(got).all() and rel_err(got, w) <= TOL["bf16"]


@pytest.mark.parametrize("B,n,heads,splits", [(1, 5, 1, 1), (3, 5, 1, 1), (6, 5, 1, 1), (8, 1, 1, 1), (12, 1, 2, 1),
                                              (2, 16, 1, 1), (2, 17, 1, 4)])   # 34 rows may be one tree: two tiles
def test_heads_worked_on_together(B, n, heads, splits):
    """Up to 24 blocks single heads are walked whole; packed only for fewer rounds of workgroups."""
    plan = b.trj_dev_attn_launch(B, B * n, 32, 8, 128, 640)
    assert (1 << plan["pack"], plan["splits"]) == (heads, splits)
