"""The launch plan of the bf16 attention, on the host: it covers every row and slot of its
ranges, fits the workspace the queries report, and takes the form that measured faster."""
import itertools

import pytest

from paper_2406_17404_amd import binding as b


def plan(B, n, slots, H=32, dh=128, shared=False):
    return b.trj_dev_attn_plan(B, B * n, H, dh, shared, slots)


def test_every_plan_covers_its_rows_and_slots_and_fits_the_workspace():
    for B, n, slots, H, dh, shared in itertools.product(
            (1, 2, 3, 4, 7, 8, 12, 16, 65, 300), (1, 31, 32, 33, 64, 65, 97, 112, 128),
            (1, 31, 32, 33, 300, 512, 544, 1025, 2100, 4224, 20000, 70000), (1, 8, 32, 40, 300), (64, 128), (False, True)):
        p = plan(B, n, slots, H, dh, shared)
        nb = -(-max(slots, n) // 32)
        if slots < n:
            continue
        assert p["tiles"] in (1, 2, 4) and p["tiles"] * 32 * p["groups"] >= min(B * n, 128)
        assert 1 <= p["blocks"] <= nb and p["blocks"] * p["splits"] >= nb > p["blocks"] * (p["splits"] - 1)
        assert not (p["ring"] and shared) and (p["ring"] or p["tiles"] < 4)
        # fewer streams or splits than such a sequence could have: the reference follows every block
        assert p["lag"] == 1 or p["tiles"] == 2
        parts = B * p["groups"] * p["tiles"] * H * p["splits"] * (dh // 32 * 1024 + 64) if p["splits"] > 1 else 0
        items = 8 * B * p["groups"] * p["splits"] + 8
        assert 4 * (parts + items) <= b.tree_attention_workspace_bytes(B, B * n, H, dh, slots, b.BF16)


@pytest.mark.parametrize("B,n,slots,H,dh,shared,ring,tiles", [
    (1, 97, 1024 + 97, 32, 128, False, 0, 2), (1, 128, 512 + 128, 32, 128, False, 0, 2),
    (1, 97, 4096 + 97, 32, 128, True, 0, 2), (16, 16, 4112, 32, 128, True, 0, 2), (1, 64, 1088, 32, 128, False, 0, 2),
    (1, 5, 782, 32, 128, False, 0, 1), (1, 64, 8256, 32, 128, False, 1, 2), (16, 64, 4160, 32, 128, False, 1, 2),
    (1, 100, 8292, 32, 128, False, 1, 4), (1, 128, 4224, 32, 128, False, 1, 4), (1, 128, 2176, 32, 128, False, 0, 2), (16, 69, 2117, 32, 128, False, 1, 4), (4, 69, 2117, 32, 128, False, 1, 4),
    (3, 128, 2176, 32, 128, False, 1, 2), (4, 128, 4224, 32, 128, False, 1, 2), (8, 97, 4193, 32, 128, False, 1, 2),
    (12, 97, 4193, 16, 64, False, 0, 2), (1, 16, 528, 16, 64, False, 1, 1)])
def test_form_and_tiles(B, n, slots, H, dh, shared, ring, tiles):
    p = plan(B, n, slots, H, dh, shared)
    assert (p["ring"], p["tiles"]) == (ring, tiles)


def test_bad_arguments():
    for args in ((0, 1, 1, 64, 0, 1), (1, 129, 1, 64, 0, 1), (2, 1, 1, 64, 0, 1), (1, 1, 0, 64, 0, 1),
                 (1, 1, 1, 96, 0, 1), (1, 1, 1, 64, 0, 0)):
        with pytest.raises(b.TrjError):
            b.trj_dev_attn_plan(*args)
