"""Background learning and partial re-learning over every small number of
frames (they are taken in pairs, four in flight) and pixel count around a
wave's and a workgroup's share, from the start and on top of a model, with
masks that keep out everything, nothing or single pixels, at gains that
saturate: the model equals the CPU oracle's bit for bit."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu


def _frames(W, H, n, seed):
    rng = np.random.default_rng(seed)
    base = rng.integers(0, 256, (H, W, 3))
    g = rng.uniform(0.6, 1.6, (n, 1, 1, 1))
    return np.clip(np.round(base[None] * g + rng.integers(-9, 10, (n, H, W, 3))), 0, 255).astype(np.uint8)


def _same(ctx, m, what):
    got = [t.cpu().numpy() for t in ctx.model()[:2]]
    assert np.array_equal(got[0], m.bgmin), what
    assert np.array_equal(got[1], m.bgmax), what


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 9, 13])
@pytest.mark.parametrize("W,H", [(64, 1), (192, 5), (128, 8), (256, 17)])
def test_learn_continue_relearn(W, H, n):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    a, b, c = (_frames(W, H, n, 100 * n + W + k) for k in range(3))
    ctx, m = fizi.Context(W, H, chunk=2, device=dev), oracle.Model(W, H)
    ctx.learn_background(torch.from_numpy(a).to(dev))
    m.learn(a)
    _same(ctx, m, "learn")
    ctx.learn_background(torch.from_numpy(b).to(dev), reset=False)
    m.learn(b, reset=False)
    _same(ctx, m, "continue")
    rng = np.random.default_rng(n)
    for p in (0.5, 1.0, 0.0, 0.01):
        masks = (rng.random((n, H, W)) < p).astype(np.uint8)
        ctx.relearn_background(torch.from_numpy(c).to(dev), fizi.pack_bits(masks, device=dev))
        m.relearn(c, masks)
        _same(ctx, m, ("relearn", p))
    ctx.close()
