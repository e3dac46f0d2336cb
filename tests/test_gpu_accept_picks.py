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
