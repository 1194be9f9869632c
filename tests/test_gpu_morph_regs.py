"""Morphology with bands held in registers, and the run pass behind it, against
the CPU oracle on masks drawn directly: a background of one gray value and
frames whose foreground is a skin colour, so that the raw mask is the drawn
one. Sizes around bands of 4, 8 and 16 rows, lane groups of 16 and 32 words and
the two-word form, borders on every side, every number of opening and closing
iterations, empty rows between full ones, noise that the opening removes, and
patterns with many runs and touching pairs (more than an LDS segment holds)."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu


def _patterns(W, H, rng):
    yield "noise", rng.random((H, W)) < 0.02
    yield "dense", rng.random((H, W)) < 0.8
    m = rng.random((H, W)) < 0.97
    yield "holes", m
    m = np.zeros((H, W), bool)
    m[:, ::7] = m[:, 1::7] = m[:, 2::7] = True            # bars: many runs a row, kept by the opening
    yield "bars", m
    c = m.copy()
    c[3::8] = True                                         # combs: bars joined and parted
    yield "combs", c
    yy, xx = np.mgrid[0:H, 0:W]
    yield "diagonals", ((xx + yy) % 11 < 4) | ((xx - yy) % 13 < 4)
    m = np.zeros((H, W), bool)
    m[:3] = m[-3:] = True
    m[:, :3] = m[:, -3:] = True
    yield "frame", m
    yield "empty", np.zeros((H, W), bool)
    yield "full", np.ones((H, W), bool)


def _check(W, H, chunk=16, short=True, frames=None, **params):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    rng = np.random.default_rng(W * 31 + H)
    masks = [m for _, m in _patterns(W, H, rng)] if frames is None else frames
    bg = np.full((2, H, W, 3), 90, np.uint8)
    f = np.full((len(masks), H, W, 3), 90, np.uint8)
    for k, m in enumerate(masks):
        f[k][m] = (200, 140, 90)
    params = dict(gain_lo_q16=65536, gain_hi_q16=65536, **params)
    ctx = fizi.Context(W, H, fizi.default_params(**params), chunk=chunk, device=dev)
    ctx.set_short_bands(short)
    ctx.learn_background(torch.from_numpy(bg).to(dev))
    out = ctx.process_frames(torch.from_numpy(f).to(dev), want_hand=True)
    torch.cuda.synchronize()
    fz, hand = fizi.unpack_bits(out["fizi"], W), fizi.unpack_bits(out["hand"], W)
    ptr = fizi.pointers_to_numpy(out["pointers"])
    m = oracle.Model(W, H, oracle.params(**params))
    m.learn(bg)
    for k in range(len(masks)):
        ref = m.process(f[k], frame_index=k, want_hand=True)
        assert np.array_equal(fz[k], ref["fizi"]), (W, H, params, k)
        assert fizi.pointer_dict(ptr[k]) == ref["pointer"], (W, H, params, k)
        assert np.array_equal(hand[k], ref["hand"]), (W, H, params, k)
    ctx.close()


@pytest.mark.parametrize("short", [True, False])
@pytest.mark.parametrize("W,H", [(64, 1), (64, 8), (128, 9), (320, 31), (1024, 17), (1088, 16), (1280, 41), (2048, 12),
                                 (2112, 9), (4096, 7), (4160, 13)])
def test_sizes(W, H, short):
    _check(W, H, short=short)


@pytest.mark.parametrize("short", [True, False])
@pytest.mark.parametrize("o,c", [(o, c) for o in range(4) for c in range(4)])
def test_iterations(o, c, short):
    _check(320, 45, short=short, open_iters=o, close_iters=c)


@pytest.mark.parametrize("o,c", [(1, 1), (2, 1)])
def test_wide_frames(o, c):
    _check(4224, 21, open_iters=o, close_iters=c)


def test_more_runs_than_a_segment():
    """No morphology: rows of up to W/2 runs, single and in stretches."""
    W, H = 1280, 40
    rng = np.random.default_rng(3)
    a = np.zeros((H, W), bool)
    a[:, ::2] = True
    b = a.copy()
    b[5::6] = False
    b[7::9] = True
    _check(W, H, open_iters=0, close_iters=0, frames=[a, b, rng.random((H, W)) < 0.5, rng.random((H, W)) < 0.1])
