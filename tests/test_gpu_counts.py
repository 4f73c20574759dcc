"""Fired counts and the channel-wise gate's mask at the edges of the counting kernels: a thread per four channels (maps of at
most 16 pixels), a wavefront per (image, word) item (64 and 256 pixels), several wavefronts per item, more items than one round
of blocks.  Counting is of whole numbers: the counts are those of the bitmap of the same call, exactly, and the channel-wise
gate keeps exactly the channels of the ungated bitmap that reach its share of the pixels."""
import math

import numpy as np
import pytest

from paper_1805_12549_amd import binding as B

pytestmark = pytest.mark.gpu

#        images, height, width, output channels
SHAPES = [(1, 1, 1, 32), (3, 1, 1, 33), (2100, 1, 1, 256), (173, 3, 5, 128), (5, 4, 4, 48),
          (5, 1, 17, 80), (40, 7, 7, 512), (2, 8, 8, 31), (3, 5, 13, 64), (9, 16, 16, 72), (7, 1, 257, 64), (3, 23, 45, 96),
          (1, 64, 64, 32), (2, 67, 81, 33), (300, 7, 6, 544)]


def _bits(bitmap, n, hw, c):
    words = bitmap.cpu().numpy().view(np.uint32).reshape(n, hw, -1)
    return ((words[:, :, np.arange(c) // 32] >> (np.arange(c) % 32).astype(np.uint32)) & 1).astype(np.int64)


@pytest.mark.parametrize("shape", SHAPES, ids=["%dx%dx%d_%d" % s for s in SHAPES])
def test_counts_are_those_of_the_bitmap(shape):
    import torch
    n, h, w, c = shape
    gen = torch.Generator(device="cuda").manual_seed(n + h + w + c)
    x = torch.randint(-8, 9, (n, h, w, 16), generator=gen, device="cuda", dtype=torch.int8)
    weights = torch.randint(-8, 9, (c, 1, 1, 16), generator=gen, device="cuda", dtype=torch.int8)
    args = dict(n_max=n, h=h, w=w, c_in=16, c_out=c, c_base=8, w_base=weights[..., :8].contiguous(),
                w_cond=weights[..., 8:].contiguous(), in_dtype=B.CG_I8, out_dtype=B.CG_I32, kh=1, kw=1, pad=0,
                gate_thr_i32=np.arange(c, dtype=np.int32) % 61 - 30)
    layer = B.GatedConv(**args)
    _, bitmap, counts = layer.forward(x)
    plain = _bits(bitmap, n, h * w, c)
    got = counts.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[2:].reshape(n, c), plain.sum(1))
    assert int(got[0]) | int(got[1]) << 32 == plain.sum()
    layer.close()

    tau = 0.5
    need = math.ceil(float(np.float32(tau)) * h * w)
    layer = B.GatedConv(tau_c=tau, **args)
    _, bitmap, counts = layer.forward(x)
    kept = plain * (plain.sum(1, keepdims=True) >= need)
    assert np.array_equal(_bits(bitmap, n, h * w, c), kept)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32)[2:].reshape(n, c), kept.sum(1))
    layer.close()
