"""Grouped-query attention whose query heads of a K/V head share tiles: group sizes that are, hold
and lack powers of two, trees that fill the shared tiles exactly, by one query more and less, all
forms of the walk with and without key splits, batches with ragged and malformed trees, and the
workspace sizes around which heads are packed or not."""
import math
from dataclasses import replace

import numpy as np
import pytest
import torch

import layouts
from gpu_util import DEV, Batch, rel_err, to_dev
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL, case
from test_gpu_attention_ring import knobs  # noqa: F401
from test_gpu_step import prefix_normal, run_and_check

pytestmark = pytest.mark.gpu


@pytest.fixture
def packing():
    """Works on a given number of query heads together, whatever the plan would choose by itself."""
    def put(heads):
        b.trj_set_tunable("attn_pack", heads.bit_length())
    yield put
    b.trj_set_tunable("attn_pack", 0)


def packed_sizes(share):
    return [heads for heads in (1, 2, 4, 8) if share % heads == 0]


def attention(cases, H, dh, heads, align=64):
    """tree_attention in the workspace that its own query reports; the launch works on `heads` together."""
    Hkv = cases[0][1].shape[0]
    batch = Batch([c[3] for c in cases], [c[4] for c in cases], align=align)
    plan = b.trj_dev_attn_launch(batch.B, batch.T, H, Hkv, dh, batch.max_seq_slots)
    assert 1 << plan["pack"] == heads
    ws = torch.empty(b.tree_attention_workspace_bytes(batch.B, batch.T, H, dh, batch.max_seq_slots, b.BF16),
                     dtype=torch.uint8, device=DEV)
    out = torch.full((batch.T, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    got = call(batch, *tensors(batch, cases, H, Hkv, dh), H, Hkv, dh, ws, out)
    return plan, [got[batch.rows(s)] for s in range(batch.B)]


@pytest.mark.parametrize("H,Hkv,dh", [(4, 1, 128), (8, 1, 64), (6, 2, 128), (3, 1, 128), (16, 1, 128), (12, 1, 64), (2, 1, 128)])
@pytest.mark.parametrize("L,n", [(520, 8), (700, 9), (1100, 7), (513, 69), (900, 33), (1300, 128), (2000, 1)])
def test_one_sequence(knobs, packing, H, Hkv, dh, L, n):
    forms = set()
    for tree in (I.tree_random(n, np.random.default_rng(n)), I.tree_chain(n)):
        c = case(11 * L + n, H, dh, L, n, "bf16", np.asarray(tree, np.int32), n_kv=Hkv)
        want = O.tree_attention(*c)
        for wgs, least in ((1, 1 << 20), (64, 1 << 20), (256, 48), (256, 1)):   # unsplit, split, the plan's own, rings
            knobs(attn_target_wgs=wgs, attn_xchg_min_blocks=least)
            for heads in packed_sizes(H // Hkv):
                packing(heads)
                plan, (got,) = attention([c], H, dh, heads)
                if heads > 1:
                    forms.add(("split" if plan["splits"] > 1 else "whole", plan["form"]))
                assert np.isfinite(got).all() and rel_err(got, want) <= TOL["bf16"], (wgs, least, heads)
    if H // Hkv != 3:
        assert {"split", "whole"} == {s for s, _ in forms}
    if (H // Hkv, dh) in ((4, 128), (2, 128)):   # a group in one column shares its K/V with no other workgroup
        assert ("split", "ring") in forms


@pytest.mark.parametrize("sizes,lens", [([20, 5, 33, 1, 64, 9], [900, 600, 0, 1300, 30, 777]), ([5] * 7, [600] * 7),
                                        ([128, 3, 40], [1000, 5, 700])])
def test_batch(knobs, packing, sizes, lens):
    forms = set()
    cases = [case(50 + s, 8, 128, L, n, "bf16", n_kv=2) for s, (n, L) in enumerate(zip(sizes, lens))]
    for wgs, least in ((1, 48), (100, 1 << 20), (256, 48), (256, 1)):
        knobs(attn_target_wgs=wgs, attn_xchg_min_blocks=least)
        for heads in packed_sizes(4):
            packing(heads)
            plan, got = attention(cases, 8, 128, heads, align=32)
            forms.add((heads, plan["form"]))
            for g, c in zip(got, cases):
                assert rel_err(g, O.tree_attention(*c)) <= TOL["bf16"], (wgs, least, heads)
    assert {(4, "ring"), (4, "registers"), (2, "registers")} <= forms
    assert not {(4, "once"), (2, "once")} & forms   # which does not take a sequence that must be walked whole


def call(batch, q, k, v, H, Hkv, dh, ws, out, parent=None):
    b.tree_attention(q, k, v, batch.parent if parent is None else parent, batch.node_off, batch.kv_off, batch.prefix,
                     batch.B, batch.T, H, dh, batch.s_pool, batch.max_seq_slots, b.BF16, 1.0 / math.sqrt(dh), ws, out,
                     n_kv_heads=Hkv)
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


def tensors(batch, cases, H, Hkv, dh):
    kp, vp = np.zeros((Hkv, batch.s_pool * dh), np.float32), np.zeros((Hkv, batch.s_pool * dh), np.float32)
    for s, c in enumerate(cases):
        layouts.kv_to_pool(c[1].astype(np.float32), c[2].astype(np.float32), batch.s_pool, int(batch.kv_off_h[s]), kp, vp)
    return [to_dev(a, torch.bfloat16) for a in (np.concatenate([c[0] for c in cases]).astype(np.float32), kp, vp)]


@pytest.mark.parametrize("heads", [2, 4])
@pytest.mark.parametrize("which", [0, 1, 2])
def test_malformed_tree_reads_as_zeros_in_every_head(packing, which, heads):
    packing(heads)
    sizes, lens, H, Hkv, dh = [20, 7, 33], [900, 640, 700], 8, 2, 128
    cases = [case(80 + s, H, dh, L, n, "bf16", n_kv=Hkv) for s, (n, L) in enumerate(zip(sizes, lens))]
    for subset in ([0, 1, 2], [which]):
        cs = [cases[s] for s in subset]
        batch = Batch([c[3] for c in cs], [c[4] for c in cs])
        parent = np.concatenate([c[3] for c in cs]).astype(np.int32)
        bad = subset.index(which)
        parent[int(batch.node_off.cpu()[bad]) + sizes[which] - 1] = 100   # not before its child
        ws = torch.empty(b.tree_attention_workspace_bytes(batch.B, batch.T, H, dh, batch.max_seq_slots, b.BF16),
                         dtype=torch.uint8, device=DEV)
        out = torch.full((batch.T, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
        got = call(batch, *tensors(batch, cs, H, Hkv, dh), H, Hkv, dh, ws, out, torch.from_numpy(parent).to(DEV))
        off = batch.node_off.cpu().numpy()
        for j, c in enumerate(cs):
            rows = got[off[j]:off[j + 1]]
            if j == bad:
                assert not rows.any()
            else:
                assert rel_err(rows, O.tree_attention(*c)) <= TOL["bf16"]


def test_less_workspace_still_accepted_where_single_heads_fit(packing):
    """The packed heads' partials may need more than single heads': such a call goes on with these."""
    H, Hkv, dh, n, L = 8, 1, 128, 10, 2500
    packing(8)
    cases = [case(90 + s, H, dh, L, n, "bf16", n_kv=Hkv) for s in range(3)]
    batch = Batch([c[3] for c in cases], [c[4] for c in cases])
    q, k, v = tensors(batch, cases, H, Hkv, dh)
    need = b.tree_attention_workspace_bytes(batch.B, batch.T, H, dh, batch.max_seq_slots, b.BF16)
    accepted = []
    for size in (need, need // 2, need // 4, need // 8, 4096):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        out = torch.full((batch.T, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
        try:
            got = call(batch, q, k, v, H, Hkv, dh, ws, out)
        except b.TrjError:
            accepted.append(False)
            continue
        accepted.append(True)
        for s, c in enumerate(cases):
            assert rel_err(got[s * n:(s + 1) * n], O.tree_attention(*c)) <= TOL["bf16"], size
    assert accepted[0] and not accepted[-1]


@pytest.mark.parametrize("n,L", [(16, 1000), (20, 700)])
def test_step_in_a_workspace_that_holds_single_heads_only(monkeypatch, packing, n, L):
    """Sized for a larger tree, whose heads are not packed, a workspace holds this one's single heads."""
    packing(4)
    shape = I.ModelShape(2, 256, 16, 128, 512, 512, "bf16", n_kv_heads=4)
    size, packed = (b.trj_workspace_bytes(b.make_desc(s), n, 1, L + n)
                    for s in (replace(shape, n_kv_heads=0), shape))
    assert size < packed
    monkeypatch.setattr(b, "trj_workspace_bytes", lambda *sizes: size)
    run_and_check(shape, I.gen_weights(shape, 88), [I.tree_random(n, np.random.default_rng(n))],
                  [I.gen_tokens(shape.vocab, n, 88, "tree", 0)], [L], [prefix_normal(shape, 88, 0, L)], 1e-2)
