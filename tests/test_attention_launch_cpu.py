"""The attention launch that really runs, on the host: with grouped-query heads too it covers every
query and slot of its ranges and fits the workspace the queries report, and with single heads it is
the plan of trj_dev_attn_plan."""
import itertools

import pytest

from paper_2406_17404_amd import binding as b


def test_every_launch_covers_its_rows_and_slots_and_fits_the_workspace():
    packed = 0
    for B, n, slots, (H, Hkv), dh in itertools.product(
            (1, 2, 3, 5, 8, 16, 40, 70), (1, 5, 9, 16, 20, 32, 33, 64, 69, 100, 128), (200, 520, 700, 1100, 3100, 12100, 33000),
            ((32, 32), (32, 16), (32, 8), (32, 4), (24, 8), (28, 4), (8, 1)), (64, 128)):
        for in_step in (False, True):
            p = b.trj_dev_attn_launch(B, B * n, H, Hkv, dh, slots, in_step)
            share, heads = H // Hkv, 1 << p["pack"]
            nb = -(-slots // 32)
            assert share % heads == 0 and (slots > 512 or heads == 1)
            assert p["tiles"] * 32 * p["groups"] >= min(B * n, 128) * heads
            assert 1 <= p["blocks"] <= nb and p["blocks"] * p["splits"] >= nb > p["blocks"] * (p["splits"] - 1)
            assert p["form"] != "ring" or share == heads          # K/V that several workgroups read come from L2
            assert p["form"] == "ring" or p["tiles"] < 4
            assert p["form"] != "once" or (p["tiles"] == 2 and dh == 128)
            assert p["lag"] == 1 or (p["tiles"] == 2 and heads == 1)
            queries = B * n * heads
            parts = (queries // 32 + B if heads > 1 else B * p["groups"] * p["tiles"]) if p["splits"] > 1 else 0
            floats = parts * (H // heads) * p["splits"] * (dh // 32 * 1024 + 64)
            items = 8 * B * p["groups"] * p["splits"] + 8
            assert 4 * (floats + items) <= b.tree_attention_workspace_bytes(B, B * n, H, dh, slots, b.BF16)
            packed += heads > 1
    assert packed > 1000


def test_single_heads_are_the_other_query_plan():
    for B, n, slots in itertools.product((1, 2, 8, 16), (1, 33, 64, 100), (100, 600, 2000, 9000)):
        p, q = b.trj_dev_attn_launch(B, B * n, 32, 32, 128, slots, True), b.trj_dev_attn_plan(B, B * n, 32, 128, False, slots)
        assert p["pack"] == 0 and all(p[k] == q[k] for k in ("tiles", "groups", "blocks", "splits", "lag"))
        assert (p["form"] == "ring") == bool(q["ring"])


# us of a call of 32 heads through registers -> at once
@pytest.mark.parametrize("n,slots,in_step,form", [
    (33, 93, False, "once"), (64, 124, False, "once"),                 # 3 and 4 blocks: 9.1 -> 9.0, 10.5 -> 9.4
    (33, 133, False, "registers"), (64, 164, True, "registers"),       # 5 and 6 blocks: 9.3 -> 11.2, 15.3 -> 16.1
    (64, 256, False, "once"), (128, 228, True, "once"),                # 8 blocks of one workgroup, two per stream: 18.2 -> 17.4
    (64, 764, False, "once"), (56, 906, True, "once"),                 # splits of 4: 23.0 -> 22.5
    (64, 1088, True, "once"), (64, 1152, True, "registers"),           # of 5, 7 of them and 8: 18.3 -> 18.0, 18.5 -> 20.6
    (64, 1248, False, "registers"), (64, 1280, True, "registers"),     # the last of 4 in 8, the last of 5
    (33, 1283, False, "registers"), (33, 1533, False, "registers"),    # of 6: 17.9 -> 21.1, 17.5 -> 20.1
    (33, 2033, False, "registers"), (48, 2048, False, "registers"),    # of 8 with one query group: 19.1 -> 21.0
    (96, 796, True, "once"), (96, 616, True, "once"),                  # with two; the last of 1 and 4 blocks: 22.8 -> 21.9
    (96, 946, True, "registers"), (80, 680, True, "registers"),        # the last of 6: 22.0 -> 23.1
    (100, 700, False, "registers"), (128, 888, False, "registers")])   # which wait for ancestor bits: 18.1 -> 20.5
def test_form_at_once(n, slots, in_step, form):
    assert b.trj_dev_attn_launch(1, n, 32, 32, 128, slots, in_step)["form"] == form


# 32 heads of 128; us of a call with 1, 2, 4, .. heads worked on together
@pytest.mark.parametrize("B,n,L,Hkv,heads", [
    (1, 5, 12000, 8, 4), (1, 16, 32000, 8, 2), (1, 20, 12000, 8, 4),    # 26.9 20.7 19.6; 48.7 35.2 36.3; 27.2 25.8 23.5
    (1, 20, 700, 8, 1), (1, 20, 1000, 8, 1), (1, 20, 1000, 4, 1),       # 12.6 14.3 14.8; 13.1 15.2 15.2
    (1, 69, 3001, 8, 4), (1, 33, 1000, 8, 4), (1, 33, 1000, 4, 1), (1, 33, 32000, 4, 8),
    (8, 16, 520, 8, 1), (8, 16, 1000, 8, 1), (8, 20, 520, 8, 1),        # 17.6 27.4 27.2; 21.5 27.4 29.2; 17.8 28.4 31.6
    (8, 1, 700, 8, 1), (8, 5, 3000, 8, 4), (8, 20, 3000, 8, 1),         # 38.7 42.7 45.6
    (16, 1, 700, 8, 2), (16, 16, 520, 8, 2), (16, 20, 520, 8, 4), (16, 20, 3000, 8, 1), (26, 17, 3205, 4, 8), (32, 1, 520, 8, 4),
    (2, 9, 700, 8, 1), (2, 33, 3000, 8, 1), (2, 69, 1000, 8, 4),        # 14.0 15.9 16.7; 24.9 30.8 28.1
    (4, 33, 520, 8, 1), (4, 69, 1000, 8, 4), (8, 33, 520, 8, 1), (8, 33, 3000, 8, 4), (16, 100, 1000, 8, 1),
    (1, 64, 3000, 8, 1), (1, 5, 500, 8, 1)])                            # no tile saved; up to 16 blocks
def test_heads_worked_on_together(B, n, L, Hkv, heads):
    assert b.trj_dev_attn_launch(B, B * n, 32, Hkv, 128, L + n)["pack"] == heads.bit_length() - 1


# heads of 64; us of a call with 1, 2, 4, .. heads worked on together
@pytest.mark.parametrize("B,n,L,H,Hkv,heads", [
    (1, 5, 520, 32, 8, 1), (1, 5, 12000, 32, 8, 4), (1, 5, 32000, 32, 8, 4),   # 17.3 14.7 14.1; 30.0 22.8 19.3
    (1, 5, 12000, 16, 4, 1), (1, 1, 32000, 16, 2, 1), (1, 100, 2000, 16, 2, 1),  # 14.4 15.1 16.7; 18.3 16.6 20.1 28.3
    (8, 16, 520, 32, 8, 1), (8, 20, 700, 32, 8, 1), (16, 20, 520, 16, 4, 1),     # 14.8 21.1 20.3; 15.4 21.1 24.5
    (2, 1, 520, 32, 8, 1), (32, 5, 1000, 32, 8, 4), (4, 69, 700, 32, 8, 4)])     # 11.2 11.3 12.2; 42.6 29.8 23.9; 26.8 17.5 17.4
def test_heads_of_64_worked_on_together(B, n, L, H, Hkv, heads):
    assert b.trj_dev_attn_launch(B, B * n, H, Hkv, 64, L + n)["pack"] == heads.bit_length() - 1


def test_bad_arguments():
    for args in ((0, 1, 1, 1, 64, 1), (1, 129, 1, 1, 64, 1), (2, 1, 1, 1, 64, 1), (1, 1, 0, 1, 64, 1), (1, 1, 4, 3, 64, 1),
                 (1, 1, 4, -1, 64, 1), (1, 1, 1, 1, 96, 1), (1, 1, 1, 1, 64, 0)):
        with pytest.raises(b.TrjError):
            b.trj_dev_attn_launch(*args)
