"""A state block filled from another context's: the model in it is the other
context's, while thresholds, outputs and scratch stay this context's own."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 5])
def test_state_from_another_context(n):
    from oracle import oracle
    from paper_1907_04393_amd import fizi, scene
    dev = need_gpu()
    W, H, chunk = 320, 240, 4
    scenes = [scene.Scene(scene.SceneSpec(W, H, sigma=3.0, n_bg=6, n_hand=100, seed=(5, 5, 5, k))) for k in range(2)]
    bg, hand = [s.bg_frames(0, 6) for s in scenes], scenes[0].hand_frames(0, n)
    params = [dict(), dict(gray_S=35, min_area=60, click_fill_permille=300, bg_delta=14)]
    ctx = [fizi.Context(W, H, fizi.default_params(**p), chunk=chunk, device=dev) for p in params]
    for c, b in zip(ctx, bg):
        c.learn_background(b.to(dev))
        c.process_frames(b.to(dev))
    ctx[1].state.copy_(ctx[0].state)
    torch.cuda.synchronize()
    ctx[0].close()
    ctx[0].state.fill_(0xA5)             # nothing of the first context is read any more
    out = ctx[1].process_frames(hand.to(dev), want_hand=True)
    torch.cuda.synchronize()
    m = oracle.Model(W, H, oracle.params(**params[1]))
    m.learn(bg[0].numpy())
    got, fz, hd = (fizi.pointers_to_numpy(out["pointers"]), fizi.unpack_bits(out["fizi"], W),
                   fizi.unpack_bits(out["hand"], W))
    for k in range(n):
        ref = m.process(hand[k].numpy(), frame_index=6 + k, want_hand=True)
        assert fizi.pointer_dict(got[k]) == ref["pointer"], k
        assert np.array_equal(fz[k], ref["fizi"]) and np.array_equal(hd[k], ref["hand"]), k
        assert ctx[1].get_pointer(6 + k) == ref["pointer"], k
    ctx[1].close()
