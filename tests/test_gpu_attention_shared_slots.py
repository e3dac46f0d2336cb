"""Packed sequences whose slots overlap (the chunks of a prompt pass share one region): their
results, and the mark on their work items that keeps the streaming hint off blocks which
another sequence reads too."""
import numpy as np
import pytest
import torch

import layouts
from gpu_util import DEV, i32, rel_err, to_dev
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_attention import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks,others", [(2, 0), (8, 1), (3, 70)])   # list of up to 64 sequences, of more
@pytest.mark.parametrize("n", [20, 64])
def test_chunks_of_one_prompt(chunks, others, n):
    H, dh, L0, own = 2, 128, 96, 128
    rng = np.random.default_rng(chunks + n)
    total = -(-(L0 + chunks * n) // 64) * 64
    B, slots = chunks + others, total + others * own
    k, v = (I.bf16_round(rng.standard_normal((H, slots, dh)).astype(np.float32)) for _ in "kv")
    q = I.bf16_round(rng.standard_normal((B * n, H, dh)).astype(np.float32))
    kp, vp = (np.zeros((H, slots * dh), np.float32) for _ in "kv")
    layouts.kv_to_pool(k, v, slots, 0, kp, vp)
    kv_off = [0] * chunks + [total + own * s for s in range(others)]
    prefix = [L0 + n * c for c in range(chunks)] + [own - n] * others
    tree = np.asarray(I.tree_chain(n), np.int32)
    bound = max(p + n for p in prefix)
    ws = torch.zeros(b.tree_attention_workspace_bytes(B, B * n, H, dh, bound, b.BF16), dtype=torch.uint8, device=DEV)
    out = torch.full((B * n, H, dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    b.tree_attention(to_dev(q, torch.bfloat16), to_dev(kp, torch.bfloat16), to_dev(vp, torch.bfloat16),
                     i32(np.tile(tree, B)), i32(n * np.arange(B + 1)), i32(kv_off), i32(prefix), B, B * n, H, dh, slots,
                     bound, b.BF16, dh ** -0.5, ws, out)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    words = ws.cpu().numpy()[: ws.numel() // 4 * 4].view(np.int32)
    for s in range(B):
        at, rows = kv_off[s], slice(s * n, s * n + n)
        want = O.tree_attention(q[rows], k[:, at:at + prefix[s] + n], v[:, at:at + prefix[s] + n], tree, prefix[s])
        assert rel_err(got[rows], want) <= TOL["bf16"], s
        rec = np.array([s, 0, s * n, n, prefix[s], at // 32, 0], np.int32)   # its first item: group 0, split 0
        hits = [i for i in np.flatnonzero(words == prefix[s]) if i >= 4 and np.array_equal(words[i - 4:i + 3], rec)]
        assert len(hits) == 1 and words[hits[0] + 3] == (s < chunks), s
