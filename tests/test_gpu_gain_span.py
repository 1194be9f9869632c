"""The gain of consecutive frames of one stream (k_gain_span: sums in parts,
the inverse gain left by a frame's last workgroup, the job table written on
the device) against the CPU oracle through every pointer's inv_gain_q16 and
the learned model: sampled-row strides, sizes around an item of 16 pixels, a
workgroup and the 32 parts, frames that are only 4-byte aligned, every case
of the hue interval, clipped and skin pixels, and no usable pixel at all."""
import numpy as np
import pytest
import torch

from helpers import compare, gpu_run, need_gpu, oracle_run

pytestmark = pytest.mark.gpu


def _frames(W, H, n, seed):
    rng = np.random.default_rng(seed)
    base = rng.integers(0, 256, (H, W, 3))
    base[rng.random((H, W)) < 0.2] = (200, 140, 90)                  # skin
    base[rng.random((H, W)) < 0.1] = 77                              # gray
    out = np.clip(np.round(base[None] * rng.uniform(0.7, 1.4, (n, 1, 1, 1)) + rng.integers(-2, 3, (n, H, W, 3))),
                  0, 255).astype(np.uint8)
    out[rng.random((n, H, W)) < 0.05] = (255, 3, 0)                  # clipped
    return torch.from_numpy(out)


@pytest.mark.parametrize("W,H,rs,n", [(64, 1, 8, 1), (64, 1, 64, 2), (128, 7, 1, 3), (192, 65, 8, 16), (320, 240, 8, 1),
                                      (1024, 33, 3, 7), (640, 480, 1, 2), (64, 2048, 2, 5), (64, 5, 8, 70)])
def test_sizes(W, H, rs, n):
    bg, hand = _frames(W, H, max(2, n), 3 * W + H), _frames(W, H, n, 5 * W + H)
    params = dict(gain_row_stride=rs, gain_lo_q16=1, gain_hi_q16=1 << 20)
    g = gpu_run(bg, hand, params, chunk=80)
    m, outs = oracle_run(bg, hand, params)
    compare(g, m, outs, str((W, H, rs, n)))


@pytest.mark.parametrize("a1,a2", [(33000, 7500), (2000, 2000), (2000, 20000), (9000, 8000), (30000, 15000)])
def test_hue_cases(a1, a2):
    bg, hand = _frames(192, 40, 3, a1), _frames(192, 40, 4, a2 + 1)
    params = dict(alpha1_cdeg=a1, alpha2_cdeg=a2, gain_row_stride=1)
    g = gpu_run(bg, hand, params, chunk=4)
    m, outs = oracle_run(bg, hand, params)
    compare(g, m, outs, str((a1, a2)))


@pytest.mark.parametrize("W,H,n", [(64, 9, 1), (128, 50, 5), (320, 240, 3)])
def test_frames_only_4_byte_aligned(W, H, n):
    """Learning and processing from addresses 4 past a 16-byte boundary."""
    from oracle import oracle
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    bg, hand = _frames(W, H, 4, 1), _frames(W, H, n, 2)

    def shifted(f):
        buf = torch.empty(f.numel() + 16, dtype=torch.uint8, device=dev)
        v = buf[4:4 + f.numel()].view(f.shape)
        v.copy_(f.to(dev))
        assert v.data_ptr() % 16 == 4
        return v

    ctx = fizi.Context(W, H, chunk=8, device=dev)
    ctx.learn_background(shifted(bg))
    out = ctx.process_frames(shifted(hand))
    torch.cuda.synchronize()
    m = oracle.Model(W, H)
    m.learn(bg.numpy())
    assert np.array_equal(ctx.model()[2].cpu().numpy().view(np.uint16), m.yref)
    assert np.array_equal(ctx.model()[0].cpu().numpy(), m.bgmin)
    for k in range(n):
        ref = m.process(hand[k].numpy(), frame_index=k)
        assert fizi.pointer_dict(fizi.pointers_to_numpy(out["pointers"])[k]) == ref["pointer"], k
    ctx.close()


def test_no_usable_pixel():
    """A black first frame clips every reference: the gain is 1 throughout."""
    bg = torch.zeros((2, 24, 64, 3), dtype=torch.uint8)
    hand = _frames(64, 24, 3, 9)
    g = gpu_run(bg, hand, {}, chunk=3)
    m, outs = oracle_run(bg, hand, {})
    compare(g, m, outs, "clipped")
    assert all(p["inv_gain_q16"] == 65536 for p in g["pointers"])


def test_learning_more_frames_than_a_table_holds():
    """257 frames: the second table reads the reference the first one wrote."""
    bg, hand = _frames(64, 17, 257, 11), _frames(64, 17, 2, 12)
    g = gpu_run(bg, hand, {}, chunk=2)
    m, outs = oracle_run(bg, hand, {})
    compare(g, m, outs, "257 frames")
