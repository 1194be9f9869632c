"""Classify of several consecutive frames of one stream (the model's box held
in registers across them) against the CPU oracle, bit for bit: frame counts
around the workgroup's share, pixel counts around a wave's and a tile's, every
pixel test, every case of the hue interval, and thresholds at the ends of
their ranges. No morphology, so that I_FIZI is the AND of the three masks."""
import numpy as np
import pytest
import torch

from helpers import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu

KINDS = {"corrected": {}, "scaled": dict(brightness_mode=1), "lum": dict(lum_hi=150)}


def _frames(W, H, n, seed):
    """A background of skin and non-skin colours and frames that straddle its
    box, each at a brightness of its own; some pixels far outside."""
    rng = np.random.default_rng(seed)
    base = rng.integers(15, 235, (H, W, 3))
    base[:, : W // 2] = (rng.integers(150, 230, (H, W // 2, 1)) * np.array([1.0, 0.7, 0.45])).astype(int)
    bg = np.clip(base[None] + rng.integers(-2, 3, (3, H, W, 3)), 0, 255).astype(np.uint8)
    g = rng.uniform(0.75, 1.3, (n, 1, 1, 1))
    x = (base[None] + rng.integers(-16, 17, (n, H, W, 3))) * g
    far = rng.random((n, H, W, 1)) < 0.05
    x = np.where(far, rng.integers(0, 256, (n, H, W, 3)), x)
    return torch.from_numpy(bg), torch.from_numpy(np.clip(np.round(x), 0, 255).astype(np.uint8))


def _check(W, H, n, seed, chunk, **params):
    params = dict(open_iters=0, close_iters=0, **params)
    bg, hand = _frames(W, H, n, seed)
    g = gpu_run(bg, hand, params, chunk=chunk)
    m, outs = oracle_run(bg, hand, params)
    compare(g, m, outs, str((W, H, n, params)))


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("W,H,n", [(64, 1, 2), (64, 3, 3), (192, 5, 4), (256, 4, 5), (320, 16, 8), (64, 17, 9),
                                   (1024, 2, 15), (704, 3, 16), (128, 9, 17), (64, 33, 33)])
def test_sizes(W, H, n, kind):
    _check(W, H, n, 7 * W + H + n, chunk=40, **KINDS[kind])


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("a1,a2", [(33000, 7500), (0, 0), (1234, 1234), (2000, 20000), (9000, 8000), (30000, 15000)])
def test_hue_cases(a1, a2, kind):
    _check(192, 11, 6, a1 + a2, chunk=6, alpha1_cdeg=a1, alpha2_cdeg=a2, **KINDS[kind])


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("delta,S,lo,hi", [(0, 0, 32768, 131072), (255, 255, 32768, 131072), (3, 20, 1, 1),
                                           (10, 20, 1 << 20, 1 << 20), (0, 1, 65536, 65536)])
def test_ends_of_the_thresholds(delta, S, lo, hi, kind):
    _check(128, 13, 7, delta + S, chunk=7, bg_delta=delta, gray_S=S, gain_lo_q16=lo, gain_hi_q16=hi, **KINDS[kind])


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("W,H,chunk", [(64, 1, 8), (320, 3, 1), (704, 29, 1), (1920, 11, 8)])
def test_one_frame(W, H, chunk, kind):
    """One frame in a call, and calls cut into chunks of one frame."""
    _check(W, H, 1 if chunk > 1 else 3, W + H, chunk=chunk, **KINDS[kind])


def test_many_frames_take_the_largest_share():
    """Enough tiles that a workgroup takes 16 frames (7 workgroups per CU)."""
    _check(1920, 1080, 17, 5, chunk=17)
