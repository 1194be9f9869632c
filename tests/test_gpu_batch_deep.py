"""Batches whose streams run different openings and closings, more than four
stages among them, on frames that share a wave four or two bands at a time, have
it to themselves, or take two words per lane: every stream's masks and pointers
equal the CPU oracle's, at each band height and in short bands, launched
directly, pipelined and from graphs."""
import numpy as np
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu

NARROW = [(640, 101), (1024, 64), (1920, 75), (2560, 50)]
WIDE = NARROW + [(4224, 45), (5120, 33)]
ITERS = {8: [(1, 1), (2, 1), (2, 2), (0, 2), (1, 0), (2, 2)], 12: [(1, 1), (3, 3), (0, 2), (2, 1), (1, 1), (3, 3)]}


def _frames(W, H, seed):
    """Blobs with ragged edges and holes on a flat background, and noise."""
    rng = np.random.default_rng((W, H, seed))
    m = rng.random((H, W)) < 0.03
    for _ in range(max(4, W * H // 6000)):
        y, x, r = rng.integers(0, H), rng.integers(0, W), rng.integers(3, 16)
        yy, xx = np.ogrid[:H, :W]
        m |= (yy - y) ** 2 + (xx - x) ** 2 < r * r
    m &= rng.random((H, W)) < 0.985
    f = np.full((H, W, 3), 90, np.uint8)
    f[m] = (200, 140, 90)
    return f


@pytest.mark.parametrize("mode", (0, 1, 4))
@pytest.mark.parametrize("rows, short", [(8, 0), (16, 0), (32, 0), (16, 1)])
@pytest.mark.parametrize("ops", (8, 12))
@pytest.mark.parametrize("geoms", (NARROW, WIDE), ids=("narrow", "wide"))
def test_streams_of_different_depth(geoms, ops, rows, short, mode):
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    kw = [dict(gain_lo_q16=65536, gain_hi_q16=65536, open_iters=o, close_iters=c) for o, c in ITERS[ops][:len(geoms)]]
    b = fizi.Batch(geoms, [fizi.default_params(**k) for k in kw], device=dev)
    b.set_tuning(morph_rows=rows, short_bands=short, mode=mode)
    models = []
    for i, (W, H) in enumerate(geoms):
        bg = np.full((2, H, W, 3), 90, np.uint8)
        b.learn(i, torch.from_numpy(bg).to(dev))
        models.append(oracle.Model(W, H, oracle.params(**kw[i])))
        models[-1].learn(bg)
    steps = [[_frames(W, H, k) for W, H in geoms] for k in range(2)]
    ptrs, bits, keep = [], [], []
    for frames in steps:
        keep.append([torch.from_numpy(f).to(dev) for f in frames])
        ptrs.append(torch.zeros((len(geoms), 56), dtype=torch.uint8, device=dev))
        bits.append([torch.zeros((H, W // 64), dtype=torch.int64, device=dev) for W, H in geoms])
        b.step(keep[-1], ptrs[-1], fizi=bits[-1])
    b.flush()
    torch.cuda.synchronize()
    for k, frames in enumerate(steps):
        got = fizi.pointers_to_numpy(ptrs[k])
        for i, (W, H) in enumerate(geoms):
            ref = models[i].process(frames[i], frame_index=k)
            assert fizi.pointer_dict(got[i]) == ref["pointer"], (k, i)
            assert np.array_equal(fizi.unpack_bits(bits[k][i][None], W)[0], ref["fizi"]), (k, i)
    b.close()
