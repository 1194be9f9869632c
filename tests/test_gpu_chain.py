"""The tracking chain of consecutive frames against the oracle's tracker: frame
counts around the eight whose flags are read at a time and around the largest
launch, hands whose covering run starts in each of the words up to the
centroid's, before them and at the row's ends, chunks in which the hand stays,
leaves and moves between components, and more runs than LDS holds."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu

BASE = dict(open_iters=0, close_iters=0)


def _frames(masks):
    n, H, W = masks.shape
    bg = np.zeros((2, H, W, 3), np.uint8)
    bg[...] = (40, 40, 90)
    fr = np.repeat(bg[:1], n, axis=0).copy()
    fr[masks.astype(bool)] = (210, 140, 90)
    return torch.from_numpy(bg), torch.from_numpy(fr)


def _check(masks, chunk, params, calls=1):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    bg, fr = _frames(masks)
    H, W = masks.shape[1:]
    m = oracle.Model(W, H, oracle.params(**params))
    m.learn(bg.numpy())
    t = oracle.Tracker(m)
    ref = [t.process(fr[k].numpy(), frame_index=k, want_hand=True) for k in range(len(masks))]
    ctx = fizi.Context(W, H, fizi.default_params(**params), chunk=chunk, device=dev)
    ctx.learn_background(bg.to(dev))
    ctx.set_tracking(True)
    frd = fr.to(dev)
    at, per = 0, -(-len(masks) // calls)
    while at < len(masks):
        x = frd[at:at + per].contiguous()
        out = ctx.process_frames(x, want_fizi=True, want_hand=True)
        got = [fizi.pointer_dict(r) for r in fizi.pointers_to_numpy(out["pointers"])]
        hand = fizi.unpack_bits(out["hand"], W)
        for i in range(x.shape[0]):
            k = at + i
            assert got[i] == ref[k]["pointer"], (chunk, k, got[i], ref[k]["pointer"])
            assert ctx.get_pointer(k) == ref[k]["pointer"], (chunk, k)
            assert np.array_equal(hand[i], ref[k]["hand"]), (chunk, k)
        at += per
    ctx.close()
    return ref


def _wander(n, W, H, seed):
    """A square hand that mostly stays, sometimes jumps or is away, next to a
    larger rectangle that comes and goes."""
    rng = np.random.default_rng(seed)
    masks = np.zeros((n, H, W), np.uint8)
    x, y = 20, 8
    for k in range(n):
        u = rng.random()
        if u < 0.15:
            x, y = int(rng.integers(0, W - 12)), int(rng.integers(0, H // 2 - 12))
        if u < 0.9:
            masks[k, y:y + 12, x:x + 12] = 1
        if rng.random() < 0.6:
            masks[k, H // 2 + 2:H - 2, 5:45] = 1
        x = min(W - 12, x + int(rng.integers(0, 3)))
    return masks


@pytest.mark.parametrize("n,chunk,calls", [(2, 2, 1), (8, 8, 1), (9, 9, 1), (15, 16, 1), (17, 17, 1), (33, 16, 2),
                                           (64, 64, 1), (70, 64, 1)])
@pytest.mark.parametrize("radius", [24, 0])
def test_wandering_hand(n, chunk, calls, radius):
    masks = _wander(n, 192, 64, seed=n + radius)
    ref = _check(masks, chunk, dict(BASE, track_radius=radius, click_debounce=2), calls)
    areas = {r["pointer"]["area"] for r in ref}
    assert n < 9 or len(areas) > 1


@pytest.mark.parametrize("x0", [0, 1, 63, 64, 130, 200, 255, 256, 319, 320])
@pytest.mark.parametrize("x1", [330, 575, 639])
def test_covering_runs_of_many_words(x0, x1):
    """The centroid's run starts 0 to 7 words before it. The bar stays while a
    larger block joins, so the pick is the bar by the covering test alone."""
    masks = np.zeros((5, 40, 640), np.uint8)
    masks[:, 3:5, x0:x1 + 1] = 1
    masks[2:, 8:40, 0:640] = 1
    ref = _check(masks, 5, dict(BASE, track_radius=0, min_area=10))
    assert [r["pointer"]["area"] for r in ref] == [2 * (x1 + 1 - x0)] * 5


def test_forest_beyond_lds():
    """More runs than the forest's LDS holds (a dotted frame), in a chunk with
    ordinary frames."""
    masks = _wander(6, 256, 128, seed=3)
    for k in (2, 4):
        masks[k, 60:128:2, 64:256:2] = 1
        masks[k, 0:60:2, 128:256:2] = 1
    _check(masks, 6, dict(BASE, track_radius=24, min_area=20))
