"""The component stage in LDS (frames of at most 3072 runs; 2048 in the
persistent step) and in global memory (more) against the CPU oracle: masks
whose run counts lie on both sides of those limits, alone and in one launch,
with area ties that the first pixel decides, components that cross many bands,
and tracked frames in each path."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu

W, H = 640, 96


def _bars(n):
    """n runs in all: squares of 3 x 3 on a grid of 5 (3 runs each), then
    lines one pixel high."""
    m = np.zeros((H, W), bool)
    per_row = W // 5
    left, y = n, 0
    while left > 0 and y + 3 <= H:
        k = min(per_row, left // 3)
        for i in range(k):
            m[y:y + 3, 5 * i:5 * i + 3] = True
        left -= 3 * k
        y += 4
        if k == 0:
            for i in range(left):
                m[y, 5 * i] = True
            left = 0
    assert left == 0
    return m


def _spiral():
    m = np.zeros((H, W), bool)
    for k in range(0, 40, 8):
        m[k:k + 3, k:W - k] = True
        m[H - k - 3:H - k, k:W - k] = True
        m[k:H - k, W - k - 3:W - k] = True
        m[k + 8:H - k, k:k + 3] = True
    return m


def _frames(masks):
    f = np.full((len(masks), H, W, 3), 90, np.uint8)
    for k, m in enumerate(masks):
        f[k][m] = (200, 140, 90)
    return f


MASKS = [lambda: _bars(2047), lambda: _bars(2048), lambda: _bars(2049), lambda: _bars(3071), lambda: _bars(3072),
         lambda: _bars(3073), lambda: _bars(6000), _spiral, lambda: np.zeros((H, W), bool),
         lambda: np.random.default_rng(1).random((H, W)) < 0.1, lambda: np.random.default_rng(2).random((H, W)) < 0.4]
PARAMS = dict(gain_lo_q16=65536, gain_hi_q16=65536, open_iters=0, close_iters=0)


@pytest.mark.parametrize("track", [False, True])
@pytest.mark.parametrize("per_call", [1, 4, 11])
def test_run_counts(per_call, track):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    f = _frames([m() for m in MASKS])
    bg = np.full((2, H, W, 3), 90, np.uint8)
    ctx = fizi.Context(W, H, fizi.default_params(**PARAMS), chunk=16, device=dev)
    ctx.learn_background(torch.from_numpy(bg).to(dev))
    ctx.set_tracking(track)
    m = oracle.Model(W, H, oracle.params(**PARAMS))
    m.learn(bg)
    ref_of = oracle.Tracker(m) if track else m
    fd = torch.from_numpy(f).to(dev)
    outs = [ctx.process_frames(fd[k:k + per_call], want_hand=True) for k in range(0, len(f), per_call)]
    torch.cuda.synchronize()
    ptr = np.concatenate([fizi.pointers_to_numpy(o["pointers"]) for o in outs])
    hand = np.concatenate([fizi.unpack_bits(o["hand"], W) for o in outs])
    for k in range(len(f)):
        ref = ref_of.process(f[k], frame_index=k, want_hand=True)
        assert fizi.pointer_dict(ptr[k]) == ref["pointer"], k
        assert np.array_equal(hand[k], ref["hand"]), k
    ctx.close()


@pytest.mark.parametrize("mode", (0, 1, 2, 3, 4, 5))
def test_batch_modes(mode):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    f = _frames([m() for m in MASKS])
    bg = np.full((2, H, W, 3), 90, np.uint8)
    b = fizi.Batch([(W, H)] * len(f), fizi.default_params(**PARAMS), device=dev)
    b.set_mode(mode)
    for i in range(len(f)):
        b.learn(i, torch.from_numpy(bg).to(dev))
    m = oracle.Model(W, H, oracle.params(**PARAMS))
    m.learn(bg)
    fd = torch.from_numpy(f).to(dev)
    ptr = torch.zeros((len(f), 56), dtype=torch.uint8, device=dev)
    b.step([fd[i] for i in range(len(f))], ptr)
    b.flush()
    torch.cuda.synchronize()
    got = fizi.pointers_to_numpy(ptr)
    for i in range(len(f)):
        assert fizi.pointer_dict(got[i]) == m.process(f[i], frame_index=0)["pointer"], (mode, i)
    assert b.status() == 0
    b.close()
