"""Batches whose row ranges do not ascend: a malformed range lies between valid ones, which keep
their answers.  Packed query heads, whose partial sums have places behind the rows in front of
them, in every form of the walk, and more sequences than the common prologue takes."""
import math

import numpy as np
import pytest
import torch

import layouts
from gpu_util import DEV, i32, rel_err, to_dev
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL, case
from test_gpu_attention_ring import knobs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture
def packing():
    def put(heads):
        b.trj_set_tunable("attn_pack", heads.bit_length())
    yield put
    b.trj_set_tunable("attn_pack", 0)


def run_out_of_order(H, Hkv, dh, sizes, lens, turn):
    """Sequences 0..turn-1 own the last rows, one with an impossible range follows, then the others
    own the first rows.  Returns (rows of a valid sequence, oracle's) for all of them."""
    n_seq = len(sizes)
    cases = [case(300 + s, H, dh, lens[s], sizes[s], "bf16", n_kv=Hkv) for s in range(n_seq)]
    head, tail = list(range(turn)), list(range(turn, n_seq))
    at_tail = sum(sizes[s] for s in tail)
    off = [at_tail]
    for s in head:
        off.append(off[-1] + sizes[s])
    off.append(0)                                   # the malformed one: from the end to the start
    for s in tail:
        off.append(off[-1] + sizes[s])
    T, order = sum(sizes), head + [None] + tail
    kv, slots = I.pool_offsets(lens, sizes, 32)
    kp, vp = np.zeros((Hkv, slots * dh), np.float32), np.zeros((Hkv, slots * dh), np.float32)
    q, parent = np.zeros((T, H, dh), np.float32), np.zeros(T, np.int32)
    for s, c in enumerate(cases):
        layouts.kv_to_pool(c[1].astype(np.float32), c[2].astype(np.float32), slots, int(kv[s]), kp, vp)
    for j, s in enumerate(order):
        if s is not None:
            q[off[j]:off[j + 1]] = cases[s][0]
            parent[off[j]:off[j + 1]] = cases[s][3]
    pick = lambda a: i32([0 if s is None else int(a[s]) for s in order])
    B, bound = len(order), max(l + n for l, n in zip(lens, sizes))
    ws = torch.empty(b.tree_attention_workspace_bytes(B, T, H, dh, bound, b.BF16), dtype=torch.uint8, device=DEV)
    out = torch.full((T, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    bf = torch.bfloat16
    b.tree_attention(to_dev(q, bf), to_dev(kp, bf), to_dev(vp, bf), i32(parent), i32(off), pick(kv), pick(lens), B, T,
                     H, dh, slots, bound, b.BF16, 1.0 / math.sqrt(dh), ws, out, n_kv_heads=Hkv)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    return [(got[off[j]:off[j + 1]], O.tree_attention(*cases[s])) for j, s in enumerate(order) if s is not None]


@pytest.mark.parametrize("H,Hkv,dh", [(8, 2, 128), (16, 1, 128), (8, 1, 64), (4, 4, 128)])
@pytest.mark.parametrize("sizes,lens,turn", [([28, 50], [1500, 1300], 1), ([20, 5, 64, 33], [900, 1600, 700, 3000], 2),
                                             ([9, 7, 3, 12, 6, 10], [1100] * 6, 3)])
def test_valid_sequences_keep_their_answers(knobs, packing, H, Hkv, dh, sizes, lens, turn):
    forms = set()
    # the plan's own, many short splits, rings
    for wgs, bpw, least in ((256, 0, 48), (4096, 1, 1 << 20), (4096, 1, 1)):
        knobs(attn_target_wgs=wgs, attn_min_bpw=bpw, attn_xchg_min_blocks=least)
        for heads in (1, 2, 4, 8):
            if (H // Hkv) % heads:
                continue
            packing(heads)
            plan = b.trj_dev_attn_launch(len(sizes) + 1, sum(sizes), H, Hkv, dh, max(map(sum, zip(sizes, lens))))
            assert 1 << plan["pack"] == heads
            forms.add((heads > 1, plan["form"], plan["splits"] > 1))
            for got, want in run_out_of_order(H, Hkv, dh, sizes, lens, turn):
                assert np.isfinite(got).all() and rel_err(got, want) <= TOL["bf16"], (wgs, least, heads)
    if (H, dh) == (8, 128):   # a batch that the plan splits, in every form
        assert {(True, "registers", True), (True, "ring", True)} <= forms and (True, "once", True) not in forms


def test_more_sequences_than_the_common_prologue_takes(knobs, packing):
    packing(4)
    rng = np.random.default_rng(4)
    sizes, lens = [int(n) for n in rng.integers(1, 20, 70)], [int(l) for l in rng.integers(500, 900, 70)]
    knobs(attn_target_wgs=4096, attn_min_bpw=1, attn_xchg_min_blocks=1 << 20)
    for got, want in run_out_of_order(4, 1, 128, sizes, lens, 30):
        assert np.isfinite(got).all() and rel_err(got, want) <= TOL["bf16"]
