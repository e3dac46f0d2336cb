"""The step's argmax picked among the LM head's candidates by the acceptance launch itself: one sequence with
few candidates, up to the limit and beyond it, one candidate per row and one row, both types; rows decided
by ties within a tile and across tiles, rows with NaN logits; and a sequence whose tree is malformed."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, Batch, device_weights, fill_pool, nan_pool, run_step
from oracle import tr_oracle as O
from paper_2406_17404_amd import binding as b
from paper_2406_17404_amd import inputs as I
from test_gpu_loop import make_model

pytestmark = pytest.mark.gpu


# rows x vocabulary / 32 candidates: 2048 is the limit
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,vocab", [(1, 32), (128, 32), (5, 96), (15, 2048), (16, 4096), (17, 4096), (128, 512),
                                     (127, 544), (1, 65536), (2, 32768), (3, 21824), (33, 1984), (65, 960)])
def test_picked_argmax(dtype, n, vocab):
    shape = I.ModelShape(1, 128, 2, 64, 128, vocab, dtype)
    w = I.gen_weights(shape, n + vocab)
    v = w["w_lm"].copy()
    if vocab > 64:
        w["w_lm"][vocab // 2:] = v[:vocab - vocab // 2]      # every logit twice
    for with_nan in (False, True):
        if with_nan:
            w["w_lm"][vocab // 3] = np.nan                   # a column that never wins
        desc, dw = device_weights(shape, w)
        tree = I.tree_random(n, np.random.default_rng(n))
        batch = Batch([tree], [9], [I.gen_tokens(vocab, n, 3, "tree")])
        kp, vp = (nan_pool(1, 2, batch.s_pool, 64, dtype) for _ in range(2))
        fill_pool(kp, vp, 0, batch, 0, *I.gen_prefix_kv(shape, 3, 0, 0, 9))
        res = run_step(shape, desc, dw, batch, kp, vp)
        am = O.greedy_argmax(res["logits"])
        assert np.array_equal(res["argmax"], am)
        a, best, path, bonus = O.accept_path(am, batch_tokens(batch), tree)
        assert (res["accept_len"][0], res["best"][0], res["bonus"][0]) == (a, best, bonus)
        assert list(res["path"][0, :a + 1]) == path
        alone = run_step(shape, desc, dw, batch, kp, vp, want_logits=False)
        assert np.array_equal(alone["argmax"], am)


def batch_tokens(batch):
    return batch.tok.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_malformed_tree(dtype):
    shape = I.ModelShape(1, 128, 2, 64, 128, 256, dtype)
    w = I.gen_weights(shape, 5)
    desc, dw = device_weights(shape, w)
    tree = np.array([-1, 0, 5, 1], np.int32)
    batch = Batch([tree], [9], [I.gen_tokens(256, 4, 3, "tree")])
    kp, vp = (nan_pool(1, 2, batch.s_pool, 64, dtype) for _ in range(2))
    fill_pool(kp, vp, 0, batch, 0, *I.gen_prefix_kv(shape, 3, 0, 0, 9))
    res = run_step(shape, desc, dw, batch, kp, vp)
    assert res["status"][0] == 1 and res["accept_len"][0] == -1 and res["new_len"][0] == 9
    assert np.array_equal(res["argmax"], O.greedy_argmax(res["logits"]))


@pytest.mark.parametrize("prompt_len,size", [(1, 260608), (32, 518656)])
def test_generation_in_a_workspace_of_the_size_without_candidates(prompt_len, size):
    """Sizes that were enough before the fp32 head wrote candidates: the same tokens as with room to spare."""
    w = make_model(I.TINY, 4)
    desc, dw = device_weights(I.TINY, w)
    prompt = I.gen_tokens(I.TINY.vocab, prompt_len, 4, "prompt")
    stride = 4 * 512 * 64
    out = []
    for room in (0, 1 << 20):
        kp, vp = (torch.zeros(2, stride, device=DEV) for _ in "kv")
        ws = torch.full((size + room,), 255, dtype=torch.uint8, device=DEV)
        out.append(b.tr_jacobi_generate(desc, dw.struct, kp, vp, stride, 512, prompt, I.tree_c0(), 5, 3, 32, -1, 4, ws))
    assert out[0] == out[1] and len(out[0][0]) == 32


def argmax_launches(shape, n):
    """Launches of the argmax over logits in an fp32 step of one sequence with n rows, whose result is checked."""
    w = I.gen_weights(shape, n)
    desc, dw = device_weights(shape, w)
    batch = Batch([I.tree_random(n, np.random.default_rng(n))], [9], [I.gen_tokens(shape.vocab, n, 3, "tree")])
    kp, vp = (nan_pool(1, shape.n_heads, batch.s_pool, 64, "f32") for _ in range(2))
    fill_pool(kp, vp, 0, batch, 0, *I.gen_prefix_kv(shape, 3, 0, 0, 9))
    b.trj_profile_begin(9, 4)
    res = run_step(shape, desc, dw, batch, kp, vp)
    launches = len(b.trj_profile_end(4))
    assert np.array_equal(res["argmax"], O.greedy_argmax(res["logits"]))
    return launches


# rounds of 8 loads per thread: rows, vocabulary and whether a launch of its own takes the argmax
@pytest.mark.parametrize("n,vocab,own", [
    (5, 8192, 0), (5, 8224, 1), (5, 12992, 1), (8, 8192, 0), (16, 4096, 0), (17, 2048, 0), (17, 2080, 1), (17, 3840, 1),
    (33, 1024, 0), (33, 1056, 1), (65, 512, 0), (65, 544, 1), (128, 512, 0),          # two rounds at most
    (1, 65536, 0), (1, 65568, 1), (2, 32768, 0), (3, 21824, 0), (4, 16384, 0)])       # long rows: up to the limit
def test_rounds_of_loads(n, vocab, own):
    assert argmax_launches(I.ModelShape(1, 64, 1, 64, 4096, vocab, "f32"), n) == own


@pytest.mark.parametrize("vocab,own", [(4096, 0), (4128, 1), (65536, 1)])
def test_vocabulary_wider_than_the_layers_buffers(vocab, own):
    """Candidates lie where q, attention output and activations were: 4 x (64 + 64 + 128) bytes a row."""
    assert argmax_launches(I.ModelShape(1, 64, 1, 64, 128, vocab, "f32"), 1) == own
