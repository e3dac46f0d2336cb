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
