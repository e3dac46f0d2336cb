"""bf16 operands that do not start at a multiple of 16 bytes: the projections' shapes for them,
and whole steps whose weights, pools and layers all lie off that grid."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, Batch, device_weights, kv_heads, rel_err, to_dev
from oracle import tr_oracle as O  # noqa: F401  (the checks below use it)
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_template import check_against_oracle, pools_for, prefix_normal

pytestmark = pytest.mark.gpu


def behind(t, by):
    """The tensor's values in memory that starts `by` elements behind a fresh allocation's start."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device=DEV)
    buf[by:].copy_(t.reshape(-1))
    return buf[by:]


@pytest.mark.parametrize("by", [1, 4])
@pytest.mark.parametrize("T,n_in,n_out,split_k", [
    # one to four token tiles: less than a phase, two phases, more than the buffers hold, a rest
    (5, 16, 32, 1), (20, 128, 96, 1), (33, 400, 4128, 0), (96, 1040, 4096, 0), (128, 208, 12288, 1),
    (128, 4112, 2048, 8), (160, 80, 64, 0),
    # many rows: both shapes, unsplit and split, one phase
    (300, 528, 4096, 0), (384, 1040, 4128, 2), (640, 16, 32032, 1), (1024, 1040, 12320, 1), (1000, 2064, 4096, 4)])
def test_projections(T, n_in, n_out, split_k, by):
    rng = np.random.default_rng(T + n_in)
    x = I.bf16_round(rng.standard_normal((T, n_in)).astype(np.float32))
    w = I.bf16_round((rng.standard_normal((n_out, n_in)) * 0.05).astype(np.float32))
    wd = to_dev(w, torch.bfloat16)
    wp = torch.empty_like(wd)
    b.trj_pack_weight(wp, wd, n_out, n_in, b.BF16, b.PACK_PLAIN)
    y = torch.full((T, n_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(2 * 128 * ((T + 127) // 128) * n_in + 32 * T * n_out + 1024, dtype=torch.uint8, device=DEV)
    b.trj_linear(to_dev(x, torch.bfloat16), behind(wp, by), T, n_in, n_out, b.BF16, split_k, ws, y)
    torch.cuda.synchronize()
    # products of bf16 values are exact in fp32; at most 4112 additions of relative error
    # 2^-24 each, in sums no larger than a few times the largest result
    assert rel_err(y.cpu().numpy(), x.astype(np.float64) @ w.astype(np.float64).T) <= 1e-5


def off_the_grid(dw):
    """The packed matrices moved one element on."""
    def move(p, kept):
        src = next(t for t in kept if t.data_ptr() == p)
        dw._keep.append(behind(src, 1))
        return dw._keep[-1].data_ptr()
    kept = list(dw._keep)
    for l in range(len(dw._arr)):
        for name in ("wqkv", "wo", "w_gate_up", "w_down"):
            setattr(dw._arr[l], name, move(getattr(dw._arr[l], name), kept))
    dw.struct.w_lm = move(dw.struct.w_lm, kept)


@pytest.mark.parametrize("sizes,Ls", [([20], [90]), ([64], [300]), ([128], [37]), ([90, 100, 110, 64], [64, 0, 333, 5])])
def test_step(sizes, Ls):
    shape = I.ModelShape(2, 256, 4, 64, 512, 512, "bf16")
    w = I.gen_weights(shape, 320)
    rng = np.random.default_rng(sum(sizes))
    trees = [I.tree_random(n, rng) for n in sizes]
    toks = [I.gen_tokens(shape.vocab, n, 320, "tree", s) for s, n in enumerate(sizes)]
    pkvs = [prefix_normal(shape, 320, s, L) if L else None for s, L in enumerate(Ls)]
    desc, dw = device_weights(shape, w)
    off_the_grid(dw)
    batch = Batch(trees, Ls, toks)
    planes = kv_heads(shape) * batch.s_pool * shape.head_dim
    stride = planes + 1
    host = [p.reshape(shape.n_layers, planes) for p in pools_for(shape, batch, Ls, pkvs)]
    pools = []
    for p in host:
        flat = torch.full((1 + shape.n_layers * stride,), float("nan"), dtype=torch.bfloat16, device=DEV)
        flat[1:].view(shape.n_layers, stride)[:, :planes] = to_dev(p, torch.bfloat16)
        pools.append(flat[1:])
    B, T = batch.B, batch.T
    ws = torch.empty(b.trj_workspace_bytes(desc, T, B, batch.max_seq_slots), dtype=torch.uint8, device=DEV)
    logits = torch.empty(T, shape.vocab, dtype=torch.float32, device=DEV)
    out = {k: torch.full((n,), -7, dtype=torch.int32, device=DEV)
           for k, n in dict(argmax=T, accept_len=B, best=B, bonus=B, new_len=B, status=B).items()}
    path = torch.full((B, b.N_MAX), -7, dtype=torch.int32, device=DEV)
    b.tr_verify_step(desc, dw.struct, pools[0], pools[1], stride, batch.s_pool, batch.tok, batch.parent, batch.node_off,
                     batch.kv_off, batch.prefix, B, T, batch.max_seq_slots, ws, logits, out["argmax"],
                     out["accept_len"], out["best"], path, out["bonus"], out["new_len"], out["status"])
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    res.update(path=path.cpu().numpy(), logits=logits.cpu().numpy())
    for name, p in zip(("k_pool", "v_pool"), pools):
        res[name] = p.view(shape.n_layers, stride)[:, :planes].float().cpu().numpy().reshape(
            shape.n_layers, kv_heads(shape), batch.s_pool * shape.head_dim)
    assert not res["status"].any()
    check_against_oracle(shape, w, res, batch, trees, toks, Ls, pkvs, 1e-2)
