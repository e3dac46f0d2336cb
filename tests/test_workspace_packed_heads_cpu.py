"""Workspace of a grouped-query step: the reported size holds the plan with packed heads and the one
without, which a smaller tree in the same workspace may take."""
from dataclasses import replace

import pytest

from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I


@pytest.mark.parametrize("slots", [400, 600, 2000, 12000])
@pytest.mark.parametrize("B,n", [(1, 1), (1, 8), (1, 16), (1, 24), (1, 32), (1, 69), (1, 128), (8, 5), (16, 20)])
def test_reported_bytes_hold_single_heads_too(B, n, slots):
    packed, single = b.make_desc(I.GQA8B), b.make_desc(replace(I.GQA8B, n_kv_heads=0))  # single heads: as many K/V heads
    assert b.trj_workspace_bytes(packed, B * n, B, slots) >= b.trj_workspace_bytes(single, B * n, B, slots)


MIB = 1 << 20


@pytest.mark.parametrize("B,T,slots,most", [
    # no number of K/V heads packs these (no tile saved, or more rounds of workgroups): single heads' need
    (1, 64, 8256, 8.2 * MIB), (1, 128, 4224, 16.3 * MIB), (8, 40, 700, 1 << 14), (8, 160, 700, 1 << 15),
    (16, 320, 4096, 1 << 15), (16, 1024, 4160, 1 << 16)])
def test_attention_alone_asks_for_no_packing_that_no_call_takes(B, T, slots, most):
    assert b.tree_attention_workspace_bytes(B, T, 32, 128, slots, b.BF16) <= most
    packs = {b.trj_dev_attn_launch(B, T, 32, kv, 128, slots)["pack"] for kv in (1, 2, 4, 8, 16, 32)}
    assert packs == {0}


def test_attention_alone_stays_within_what_the_header_states():
    limits = {1: 17, 2: 17, 3: 19, 4: 19, 5: 21, 6: 25, 7: 29}
    for B in (1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 24, 32, 64):
        for n in (1, 4, 5, 8, 12, 16, 24, 32, 33, 48, 62, 64, 69, 80, 100, 112, 128):
            for slots in (300, 542, 700, 1300, 2000, 4096, 32768, 131072):
                size = b.tree_attention_workspace_bytes(B, B * n, 32, 128, slots, b.BF16)
                assert size <= limits.get(B, 17) * MIB < b.STATIC_SCRATCH_BYTES, (B, n, slots)
