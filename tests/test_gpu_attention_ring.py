"""The bf16 attention's two forms, K/V through rings in LDS and through registers, at their
edges: key streams with no, one and a few blocks (fewer and more than the ring holds), four
query tiles per workgroup with idle and ragged ones, batches that mix tree sizes, and operands
that do not start at a multiple of 16 bytes (which the loads straight to LDS cannot take), for
the projections too."""
import math

import numpy as np
import pytest
import torch

import layouts
from gpu_util import DEV, Batch, rel_err, to_dev
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL, case, run_attention

pytestmark = pytest.mark.gpu
KNOBS = {"attn_target_wgs": 256, "attn_min_bpw": 0, "attn_xchg_min_blocks": 48}


@pytest.fixture
def knobs():
    """Sets launch-plan knobs; the form: attn_xchg_min_blocks 1 always rings, 1 << 20 never."""
    def put(**values):
        for name, value in values.items():
            b.trj_set_tunable(name, value)
    yield put
    put(**KNOBS)



@pytest.mark.parametrize("H,dh,L,n", [
    (2, 128, 1400, 65), (1, 64, 1407, 128), (2, 128, 1536, 97), (1, 128, 2047, 69),   # four tiles (heads of 128)
    (2, 128, 1000, 33), (1, 64, 700, 64), (2, 128, 600, 17), (3, 64, 650, 20)])       # two, one
def test_streams_with_few_and_many_blocks(knobs, H, dh, L, n):
    c = case(3 * L + n, H, dh, L, n, "bf16")
    want = O.tree_attention(*c)
    for wgs, blocks in ((1, 0), (8, 1), (24, 1), (64, 1), (4096, 1), (4096, 3)):
        got = []
        for least in (1, 1 << 20):
            knobs(attn_target_wgs=wgs, attn_min_bpw=blocks, attn_xchg_min_blocks=least)
            plan = b.trj_dev_attn_plan(1, n, H, dh, False, L + n)
            assert plan["ring"] == (least == 1 and dh == 128 or n <= 32 and dh == 64)
            four = plan["ring"] and n > 64 and (wgs > H or 2 * H >= 3 * wgs)   # unsplit: not one round of workgroups
            assert plan["tiles"] == (4 if four else 1 if n <= 32 else 2)
            got.append(run_attention("bf16", H, dh, [c])[0])
            assert np.isfinite(got[-1]).all(), (wgs, blocks, least)
            assert rel_err(got[-1], want) <= TOL["bf16"], (wgs, blocks, least)
        if n <= 64:   # the same streams, in the same order: the same bits in either form
            assert np.array_equal(got[0], got[1]), (wgs, blocks)


@pytest.mark.parametrize("wgs", [8, 24, 256])   # four tiles unsplit, in two splits, two tiles
def test_batch_of_large_and_small_trees(knobs, wgs):
    sizes, lens = [128, 128, 33, 97, 1, 96], [1500, 3, 1411, 0, 900, 64]
    cases = [case(70 + s, 2, 128, L, n, "bf16") for s, (n, L) in enumerate(zip(sizes, lens))]
    assert sum(sizes) > 64 * len(sizes)
    knobs(attn_target_wgs=wgs, attn_xchg_min_blocks=1)
    plan = b.trj_dev_attn_plan(6, sum(sizes), 2, 128, False, 1628)
    assert plan["ring"] == 1 and plan["tiles"] == (4 if wgs < 256 else 2)
    for g, c in zip(run_attention("bf16", 2, 128, cases, align=32), cases):
        assert rel_err(g, O.tree_attention(*c)) <= TOL["bf16"]


def shifted(a, dtype, by):
    """The array on the device, starting `by` elements behind an allocation's start."""
    buf = torch.zeros(a.size + by, dtype=dtype, device=DEV)
    buf[by:].copy_(torch.from_numpy(np.ascontiguousarray(a, np.float32).reshape(-1)).to(dtype))
    return buf[by:]


@pytest.mark.parametrize("which", ["q", "k", "v", "workspace"])
@pytest.mark.parametrize("L,n", [(100, 20), (300, 50), (1450, 80)])
def test_attention_operands_at_any_alignment(knobs, which, L, n):
    H, dh = 2, 128
    knobs(attn_xchg_min_blocks=1)   # the plan is the ring's, with one, two and four tiles
    c = case(9 + L, H, dh, L, n, "bf16")
    batch = Batch([c[3]], [L])
    kp, vp = np.zeros((H, batch.s_pool * dh), np.float32), np.zeros((H, batch.s_pool * dh), np.float32)
    layouts.kv_to_pool(c[1].astype(np.float32), c[2].astype(np.float32), batch.s_pool, int(batch.kv_off_h[0]), kp, vp)
    q, k, v = (shifted(a, torch.bfloat16, int(which == w)) for a, w in ((c[0], "q"), (kp, "k"), (vp, "v")))
    need = b.tree_attention_workspace_bytes(1, n, H, dh, batch.max_seq_slots, b.BF16)
    ws = torch.empty(need + 8, dtype=torch.uint8, device=DEV)[8 * (which == "workspace"):]
    out = torch.full((n, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    b.tree_attention(q, k, v, batch.parent, batch.node_off, batch.kv_off, batch.prefix, 1, n, H, dh, batch.s_pool,
                     batch.max_seq_slots, b.BF16, 1.0 / math.sqrt(dh), ws, out, n_kv_heads=H)
    torch.cuda.synchronize()
    assert rel_err(out.float().cpu().numpy(), O.tree_attention(*c)) <= TOL["bf16"]


@pytest.mark.parametrize("which", ["w", "workspace"])
@pytest.mark.parametrize("T,n_in,n_out", [(20, 272, 96), (64, 1040, 4096), (300, 528, 4096)])
def test_projection_operands_at_any_alignment(which, T, n_in, n_out):
    rng = np.random.default_rng(T)
    x = I.bf16_round(rng.standard_normal((T, n_in)).astype(np.float32))
    w = I.bf16_round((rng.standard_normal((n_out, n_in)) * 0.05).astype(np.float32))
    wd = to_dev(w, torch.bfloat16)
    packed = torch.empty(n_out * n_in + 1, dtype=torch.bfloat16, device=DEV)[int(which == "w"):][:n_out * n_in]
    b.trj_pack_weight(packed, wd, n_out, n_in, b.BF16, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), dtype=torch.float32, device=DEV)
    size = 2 * 128 * ((T + 127) // 128) * n_in + 32 * T * n_out + 1024
    ws = torch.empty(size + 8, dtype=torch.uint8, device=DEV)[8 * (which == "workspace"):]
    b.trj_linear(to_dev(x, torch.bfloat16), packed, T, n_in, n_out, b.BF16, 0, ws, y)
    torch.cuda.synchronize()
    # bf16 products are exact in fp32: only the order of at most 1040 additions differs
    assert rel_err(y.cpu().numpy(), x.astype(np.float64) @ w.astype(np.float64).T) <= 1e-5


@pytest.mark.parametrize("what", ["good", "inner rows", "second root", "child before parent", "slots", "no rows",
                                  "too many rows"])
@pytest.mark.parametrize("L,n", [(40, 20), (900, 64), (1450, 128)])
@pytest.mark.parametrize("dh,least", [(64, 48), (128, 1), (128, 1 << 20)])
def test_one_sequence_checked_by_the_attention_kernel(knobs, what, L, n, dh, least):
    """A single sequence has no launch of its own for the tree's checks: rows that no valid
    sequence owns read as zeros, deep trees need every doubling round."""
    H = 2
    knobs(attn_xchg_min_blocks=least)
    for tree in (I.tree_chain(n), I.tree_random(n, np.random.default_rng(n))):
        c = case(77 + L, H, dh, L, n, "bf16", np.asarray(tree, np.int32))
        batch = Batch([c[3]], [L])
        kp, vp = np.zeros((H, batch.s_pool * dh), np.float32), np.zeros((H, batch.s_pool * dh), np.float32)
        layouts.kv_to_pool(c[1].astype(np.float32), c[2].astype(np.float32), batch.s_pool, int(batch.kv_off_h[0]),
                           kp, vp)
        before, after = (3, 4) if what == "inner rows" and n + 7 <= 128 else (0, 0)
        T = before + n + after
        parent = np.zeros(T, np.int32)
        parent[before:before + n] = c[3]
        off, prefix = [before, before + n], L
        if what == "second root":
            parent[n // 2] = -1
        elif what == "child before parent":
            parent[n - 1] = n - 1
        elif what == "slots":
            prefix = batch.s_pool
        elif what == "no rows":
            off = [n, n]
        elif what == "too many rows":
            off = [0, T + 1]
        q = np.zeros((T, H, dh), np.float32)
        q[before:before + n] = c[0]
        i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=DEV)
        out = torch.full((T, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
        ws = torch.empty(b.tree_attention_workspace_bytes(1, T, H, dh, batch.max_seq_slots, b.BF16),
                         dtype=torch.uint8, device=DEV)
        b.tree_attention(to_dev(q, torch.bfloat16), to_dev(kp, torch.bfloat16), to_dev(vp, torch.bfloat16), i32(parent),
                         i32(off), batch.kv_off, i32([prefix]), 1, T, H, dh, batch.s_pool, batch.max_seq_slots, b.BF16,
                         1.0 / math.sqrt(dh), ws, out, n_kv_heads=H)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy()
        if what in ("good", "inner rows"):
            assert rel_err(got[before:before + n], O.tree_attention(*c)) <= TOL["bf16"]
            assert not got[:before].any() and not got[before + n:].any()
        else:
            assert not got.any()
