"""Learning from as many frames as one launch holds, at the largest geometry
with every row sampled: the gain sums of a workgroup pass 32 bits. Flat frames,
so that the inverse gain and the model follow from the definition."""
import pytest
import torch

from paper_1907_04393_amd import fizi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first, other", [(150, 140), (254, 253)])
def test_learn_256_frames_8192x8192(first, other):
    n, w, h = 256, 8192, 8192
    frames = torch.empty((n, h, w, 3), dtype=torch.uint8, device="cuda")
    frames.fill_(other)
    frames[0].fill_(first)
    ctx = fizi.Context(w, h, params=fizi.default_params(gain_row_stride=1), chunk=1)
    try:
        ctx.learn_background(frames)
        bgmin, bgmax, _ = ctx.model()
        # inv = round half up(2^16 ref / lum) from pixels of equal value
        inv = (2 * 65536 * first + other) // (2 * other)
        corrected = min(255, (other * inv + 32768) >> 16)
        lo, hi = min(first, corrected), max(first, corrected)
        assert (int(bgmin.amin()), int(bgmin.amax())) == (lo, lo)
        assert (int(bgmax.amin()), int(bgmax.amax())) == (hi, hi)
        # a frame of its own against that model
        out = ctx.process_frames(frames[1:2])
        assert fizi.pointers_to_numpy(out["pointers"])["inv_gain_q16"][0] == inv
    finally:
        torch.cuda.synchronize()
        ctx.close()
        del ctx, frames
        torch.cuda.empty_cache()
