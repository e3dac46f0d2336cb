"""Workspace of the fp32 mode: the LM head's argmax candidates lie in buffers that the layers are done with,
so sizes are what they were without them and buffers of those sizes, once asked for, still hold a call."""
import pytest

from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I


@pytest.mark.parametrize("rows,vocab", [(1, 2048), (15, 2048), (32, 2048), (1, 16384), (128, 512), (5, 96)])
def test_a_step_needs_no_more_than_its_logits_for_the_head(rows, vocab):
    def need(v):
        return b.trj_workspace_bytes(b.make_desc(I.ModelShape(2, 256, 4, 64, 1024, v, "f32")), rows, 1, 143)

    many = 65536 * 8   # of a vocabulary whose candidates are too many for the acceptance launch
    def logits(v):
        return (rows * v * 4 + 255) // 256 * 256
    assert need(many) - need(vocab) == logits(many) - logits(vocab)


@pytest.mark.parametrize("prompt,new,size", [(1, 1, 252672), (1, 32, 260608), (32, 1, 510720), (32, 100, 536064)])
def test_a_generation_asks_for_no_more_than_it_did(prompt, new, size):
    assert b.tr_jacobi_generate_workspace_bytes(b.make_desc(I.TINY), 15, prompt, new, 512) <= size
