"""Learning from as many frames as one launch holds, at the largest geometry
with every row sampled: the gain sums of a workgroup pass 32 bits. Flat frames,
so that the inverse gain and the model follow from the definition. And few
large frames, whose sums come from many workgroups each."""
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


@pytest.mark.parametrize("w, h, n, stride, offset", [(4160, 1999, 1, 1, 0), (4160, 1999, 2, 1, 4), (7680, 4320, 1, 2, 0),
                                                     (8192, 1023, 3, 3, 0), (3840, 2160, 4, 2, 4)])
def test_gain_of_few_large_frames(w, h, n, stride, offset):
    """More parts than a wave has lanes: gray frames of random values (no pixel
    is skin), some clipped, against 64-bit sums."""
    gen = torch.Generator(device="cuda").manual_seed(w + h + n)
    gray = torch.randint(0, 256, (n + 1, h, w), generator=gen, device="cuda", dtype=torch.int64)
    gray[1:] = torch.where(gray[1:] % 7 == 0, gray[1:], gray[1:] * 3 // 4)
    memory = torch.empty(3 * w * h * (n + 1) + 16, dtype=torch.uint8, device="cuda")
    frames = memory[offset:offset + 3 * w * h * (n + 1)].view(n + 1, h, w, 3)
    frames.copy_(gray.to(torch.uint8)[..., None])
    ctx = fizi.Context(w, h, params=fizi.default_params(gain_row_stride=stride), chunk=n)
    ctx.learn_background(frames[:1])
    out = ctx.process_frames(frames[1:])
    ref = gray[0, ::stride]
    usable = (ref > 0) & (ref < 255)
    for k in range(n):
        lum = gray[k + 1, ::stride]
        ok = usable & (lum > 0) & (lum < 255)
        num, den = 4 * int(ref[ok].sum()), 4 * int(lum[ok].sum())
        inv = min(max((num * 65536 + den // 2) // den, 32768), 131072)
        assert fizi.pointers_to_numpy(out["pointers"])["inv_gain_q16"][k] == inv, k
    ctx.close()
