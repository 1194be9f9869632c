"""Masks with more runs than the component stage holds in LDS and more joins
than the link list holds (their runs are joined by reading the mask): noise,
noise between lines of any length (runs of more columns than a window has, and
ones that start left of it) and whole frames, at frames of one word, of packed
and of wide rows, against the CPU oracle."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu

PARAMS = dict(gain_lo_q16=65536, gain_hi_q16=65536, open_iters=0, close_iters=0)
SIZES = [(64, 1100), (640, 480), (4224, 61)]


def _masks(W, H):
    rng = np.random.default_rng(W + H)
    noise = [rng.random((H, W)) < p for p in (0.2, 0.5)]
    lines = rng.random((H, W)) < 0.45
    for y in range(1, H, 3):
        x = 0
        while x < W:
            n = int(rng.integers(1, min(W, 400)))
            lines[y, x:x + n] = True
            x += n + int(rng.integers(1, 30))
    full = np.ones((H, W), bool)
    full[:, ::7] = False
    full[::5] = True
    return noise + [lines, full]


def _frames(masks, W, H):
    f = np.full((len(masks), H, W, 3), 90, np.uint8)
    for k, m in enumerate(masks):
        f[k][m] = (200, 140, 90)
    return f


@pytest.mark.parametrize("track", [False, True])
@pytest.mark.parametrize("per_call", [1, 4])
@pytest.mark.parametrize("W,H", SIZES)
def test_context(W, H, per_call, track):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    f = _frames(_masks(W, H), W, H)
    bg = np.full((2, H, W, 3), 90, np.uint8)
    ctx = fizi.Context(W, H, fizi.default_params(**PARAMS), chunk=4, device=dev)
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


@pytest.mark.parametrize("mode", (0, 2, 4))
def test_batch(mode):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    frames = {s: _frames(_masks(*s), *s) for s in SIZES}
    b = fizi.Batch(SIZES, fizi.default_params(**PARAMS), device=dev)
    b.set_mode(mode)
    models = []
    for i, (W, H) in enumerate(SIZES):
        bg = np.full((2, H, W, 3), 90, np.uint8)
        b.learn(i, torch.from_numpy(bg).to(dev))
        models.append(oracle.Model(W, H, oracle.params(**PARAMS)))
        models[-1].learn(bg)
    fd = {s: torch.from_numpy(f).to(dev) for s, f in frames.items()}
    ptrs = []
    for k in range(4):
        ptrs.append(torch.zeros((len(SIZES), 56), dtype=torch.uint8, device=dev))
        b.step([fd[s][k] for s in SIZES], ptrs[-1])
    b.flush()
    torch.cuda.synchronize()
    for k in range(4):
        got = fizi.pointers_to_numpy(ptrs[k])
        for i, s in enumerate(SIZES):
            assert fizi.pointer_dict(got[i]) == models[i].process(frames[s][k], frame_index=k)["pointer"], (mode, k, s)
    assert b.status() == 0
    b.close()
