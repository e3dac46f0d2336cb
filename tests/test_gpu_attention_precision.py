"""How close the bf16 attention is to the 64-bit result: no further off than a walk by as many
key streams as workgroups of eight wavefronts can have, written out here in 32 bits with the
weights rounded to bf16.  What differs between the two is only which keys get a weight of
exactly 1 (a stream's running maxima), so the errors are alike or the kernel's is smaller."""
import numpy as np
import pytest
import torch

from paper_2406_17404_amd import binding as b
from oracle import tr_oracle as O
from test_gpu_attention import case, run_attention

pytestmark = pytest.mark.gpu


def bf16(t):
    return t.to(torch.bfloat16).float()


def streams_walk(q, k, v, parent, L, streams, blocks):
    """Splits of `blocks` 32-slot blocks, `streams` key streams each that take every
    streams-th block: online softmax in 32 bits, weights rounded to bf16 for the product with
    V, the parts added in 32 bits."""
    q, k, v = (torch.from_numpy(np.asarray(a, np.float32)) for a in (q, k, v))
    n, H, dh = q.shape
    slots = L + n
    s = torch.einsum("nhd,hsd->hns", q, k[:, :slots]) * (1.4426950408889634 / dh ** 0.5)
    seen = torch.cat([torch.ones(n, L, dtype=torch.bool), torch.from_numpy(O.ancestor_mask(parent))], 1)
    s = s.masked_fill(~seen, -1e30)
    nb = -(-slots // 32)
    parts = []
    for b0 in range(0, nb, blocks):
        for ks in range(streams):
            m, l, o = torch.full((H, n), -1e30), torch.zeros(H, n), torch.zeros(H, n, dh)
            for blk in range(b0 + ks, min(nb, b0 + blocks), streams):
                at = slice(32 * blk, min(slots, 32 * blk + 32))
                new = torch.maximum(m, s[:, :, at].amax(2))
                p = torch.where(seen[None, :, at], torch.exp2(s[:, :, at] - new[:, :, None]), torch.zeros(()))
                f = torch.exp2(m - new)
                l = l * f + p.sum(2)
                o = o * f[:, :, None] + torch.matmul(bf16(p), v[:, at])
                m = new
            parts.append((m, l, o))
    top = torch.stack([p[0] for p in parts]).amax(0)
    w = [torch.exp2(p[0] - top) for p in parts]
    out = sum(p[2] * f[:, :, None] for p, f in zip(parts, w)) / sum(p[1] * f for p, f in zip(parts, w))[:, :, None]
    return bf16(out).permute(1, 0, 2).numpy()


def off(got, want):
    return np.sqrt(sum(((g - w) ** 2).sum() for g, w in zip(got, want)) / sum((w ** 2).sum() for w in want))


@pytest.mark.parametrize("seqs,H,dh,L,n,streams,blocks,wgs", [
    (1, 16, 128, 512, 32, 8, 8, 256),     # one query tile: eight streams, three splits
    (1, 16, 64, 2000, 32, 8, 8, 256),
    (1, 16, 128, 300, 32, 8, 8, 256),     # up to 16 blocks in one workgroup: splits of one block per stream
    (1, 16, 128, 400, 48, 4, 4, 256),
    (4, 4, 128, 1450, 69, 4, 64, 8),      # four tiles, unsplit: four streams
])
def test_error_no_larger_than_with_all_key_streams(seqs, H, dh, L, n, streams, blocks, wgs):
    cases = [case(900 + s, H, dh, L, n, "bf16") for s in range(seqs)]
    want = [O.tree_attention(*c) for c in cases]
    try:
        b.trj_set_tunable("attn_target_wgs", wgs)
        b.trj_set_tunable("attn_xchg_min_blocks", 1)
        got = run_attention("bf16", H, dh, cases)
    finally:
        b.trj_set_tunable("attn_target_wgs", 256)
        b.trj_set_tunable("attn_xchg_min_blocks", 48)
    ref = off([streams_walk(*c, streams, blocks) for c in cases], want)
    # at least 65536 outputs whose squared errors vary about as much as their mean: the ratio of
    # the two errors scatters by 0.5 / 256 * 2 = 0.4 %; half the streams cost 1.5 to 3.5 %
    assert off(got, want) <= ref * 1.008, (off(got, want), ref)
