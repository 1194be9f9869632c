"""The memory of a context's or batch's state block comes from the stream that
the block is initialised on (a batch's: the null stream): a block freed on another stream, which may still have
writes pending there, is not taken."""
import pytest
import torch

from helpers import need_gpu

pytestmark = pytest.mark.gpu


def test_state_block_of_the_creating_stream():
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    side = torch.cuda.Stream(dev)
    nbytes = fizi.state_bytes(640, 480, chunk=8)
    torch.cuda.empty_cache()
    freed = torch.zeros(nbytes, dtype=torch.uint8, device=dev)
    at = freed.data_ptr()
    del freed
    ctx = fizi.Context(640, 480, chunk=8, device=dev, stream=side)
    assert ctx.state.data_ptr() != at
    here = fizi.Context(640, 480, chunk=8, device=dev)
    assert here.state.data_ptr() == at
    here.close()
    ctx.close()


def test_batch_state_block_of_the_null_stream():
    from paper_1907_04393_amd import fizi
    dev = need_gpu()
    geoms = [(640, 480), (320, 240)]
    probe = fizi.Batch(geoms, device=dev)
    nbytes = probe.state.numel()
    probe.close()
    del probe
    torch.cuda.empty_cache()
    side = torch.cuda.Stream(dev)
    with torch.cuda.stream(side):
        freed = torch.zeros(nbytes, dtype=torch.uint8, device=dev)
        at = freed.data_ptr()
        del freed
        b = fizi.Batch(geoms, device=dev)
    assert b.state.data_ptr() != at
    b.close()
