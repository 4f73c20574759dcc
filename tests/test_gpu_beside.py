"""A layer and the 1x1 convolution beside it in one call (GatedConv.forward_beside): the bits of the two calls, whose results other tests compare with the
oracle.  The same kernels' code walks K in the same order, so no tolerance is needed."""
import numpy as np
import pytest
import torch

from paper_1805_12549_amd import binding as B

pytestmark = pytest.mark.gpu

# (n, h, w, c_in, c_out, c_base, kernel, stride, channels of the 1x1), and for the one-launch ones the layer's tile (pixel fragments, channel halves) and
# whether its K steps lie inside taps; test_kernels_of_calls_cpu.py holds these.  None: layers on other kernels and 1x1s that do not run in small
# pieces, i.e. two launches.
FORMS = [
    ((1, 7, 7, 512, 512, 128, 3, 1, 512), (1, 1, True)),         # several batches of K steps in the 1x1
    ((1, 13, 11, 64, 128, 16, 3, 2, 64), (1, 1, False)),         # ragged ends of pixels
    ((1, 12, 12, 48, 96, 16, 1, 1, 64), (1, 1, False)),          # two wavefronts a workgroup; a last K step of two chunks
    ((2, 28, 28, 128, 256, 32, 3, 2, 256), (1, 2, True)),
    ((1, 56, 56, 64, 128, 16, 3, 2, 128), (1, 2, False)),
    ((3, 28, 29, 128, 256, 32, 3, 2, 320), (1, 4, True)),
    ((2, 56, 56, 64, 128, 16, 3, 2, 128), (1, 4, False)),
    ((3, 56, 56, 64, 128, 64, 3, 2, 128), (2, 4, True)),         # a dense layer
    ((5, 56, 55, 64, 128, 16, 3, 2, 64), (2, 4, False)),
    ((40, 28, 28, 128, 128, 32, 3, 1, 128), None),
    ((2, 30, 30, 64, 64, 16, 3, 1, 512), None),
]

# the same of layers with channel groups, the last number: blocks of 64 channels inside a group (one launch), over several (two)
GROUPED = [(2, 14, 14, 128, 256, 32, 3, 2, 256, 4), (2, 14, 14, 128, 96, 32, 3, 2, 128, 4)]

# the layer's workgroups and the 1x1's pieces to one of the further ones
SHARES = [((1, 14, 14, 256, 512, 64, 3, 2, 512), 128, 1), ((5, 14, 14, 256, 512, 64, 3, 2, 512), 256, 1), ((10, 14, 14, 256, 512, 64, 3, 2, 512), 248, 2),
          ((1, 28, 28, 128, 256, 32, 3, 2, 256), 208, 4), ((12, 14, 14, 256, 512, 64, 3, 2, 512), 152, 8), ((3, 27, 29, 48, 96, 16, 3, 2, 64), 240, 5)]


@pytest.mark.parametrize("form", [f for f, _ in FORMS] + [f for f, _, _ in SHARES] + GROUPED, ids=lambda f: "x".join(map(str, f)))
@pytest.mark.parametrize("scaled", [True, False])
def test_beside_is_the_two_calls(form, scaled):
    n, h, w, c_in, c_out, c_base, k, stride, c1, *groups = form
    gen = torch.Generator(device="cuda").manual_seed(h * c_in + n)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")
    x = torch.relu(rand(n, h, w, c_in)).to(torch.bfloat16)
    wt = (rand(c_out, k, k, c_in) * (2.0 / (k * k * c_in)) ** 0.5).to(torch.bfloat16)
    w1 = (rand(c1, c_in) * (2.0 / c_in) ** 0.5).to(torch.bfloat16)
    sc, sh = torch.rand(c1, generator=gen, device="cuda") + 0.5, rand(c1) * 0.1
    gate = dict(gate_mean=np.zeros(c_out), gate_var=np.ones(c_out), delta=np.full(c_out, 0.3)) if c_base < c_in else {}
    layer = B.GatedConv(n_max=n, h=h, w=w, c_in=c_in, c_out=c_out, c_base=c_base, w_base=wt[..., :c_base].contiguous(),
                        w_cond=wt[..., c_base:].contiguous() if c_base < c_in else None, in_dtype=B.CG_BF16, out_dtype=B.CG_BF16, kh=k, kw=k, stride=stride,
                        pad=k // 2, groups=groups[0] if groups else 0, **gate)
    want, _, _ = layer.forward(x, bitmap=False, counts=False)
    want1 = torch.empty((n, layer.ho, layer.wo, c1), dtype=torch.bfloat16, device="cuda")
    B.cg_pointwise_conv(x.data_ptr(), w1.data_ptr(), sc.data_ptr() if scaled else 0, sh.data_ptr() if scaled else 0, want1.data_ptr(), n, h, w, c_in, c1,
                        stride, False, B.current_stream_ptr())
    for _ in range(2):
        y, y1 = layer.forward_beside(x, w1, sc if scaled else None, sh if scaled else None, c1)
        assert torch.equal(y, want) and torch.equal(y1, want1)
    layer.close()


@pytest.mark.parametrize("form", [(2, 28, 28, 128, 256, 32, 3, 2, 256), (3, 56, 56, 64, 128, 64, 3, 2, 128), (40, 28, 28, 128, 128, 32, 3, 1, 128)],
                         ids=lambda f: "x".join(map(str, f)))
def test_beside_of_layers_with_float_outputs(form):
    """One launch, of a gated and a dense layer, and two."""
    n, h, w, c_in, c_out, c_base, k, stride, c1 = form
    gen = torch.Generator(device="cuda").manual_seed(h * c_in + n)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")
    x = torch.relu(rand(n, h, w, c_in)).to(torch.bfloat16)
    wt, w1 = rand(c_out, k, k, c_in).to(torch.bfloat16), rand(c1, c_in).to(torch.bfloat16)
    gate = dict(gate_mean=np.zeros(c_out), gate_var=np.ones(c_out), delta=np.full(c_out, 0.3)) if c_base < c_in else {}
    layer = B.GatedConv(n_max=n, h=h, w=w, c_in=c_in, c_out=c_out, c_base=c_base, w_base=wt[..., :c_base].contiguous(),
                        w_cond=wt[..., c_base:].contiguous() if c_base < c_in else None, in_dtype=B.CG_BF16, out_dtype=B.CG_F32, kh=k, kw=k, stride=stride,
                        pad=k // 2, **gate)
    want, _, _ = layer.forward(x, bitmap=False, counts=False)
    want1 = torch.empty((n, layer.ho, layer.wo, c1), dtype=torch.bfloat16, device="cuda")
    B.cg_pointwise_conv(x.data_ptr(), w1.data_ptr(), 0, 0, want1.data_ptr(), n, h, w, c_in, c1, stride, False, B.current_stream_ptr())
    y, y1 = layer.forward_beside(x, w1, None, None, c1)
    assert y.dtype == torch.float32 and torch.equal(y, want) and torch.equal(y1, want1)
    layer.close()


def test_beside_refuses_what_it_does_not_cover():
    x = torch.zeros((1, 8, 8, 64), dtype=torch.bfloat16, device="cuda")
    wt, w1, one = torch.zeros((64, 3, 3, 64), dtype=torch.bfloat16, device="cuda"), torch.zeros((64, 64), dtype=torch.bfloat16, device="cuda"), torch.ones(64, device="cuda")
    make = lambda **kw: B.GatedConv(**{**dict(n_max=1, h=8, w=8, c_in=64, c_out=64, c_base=64, w_base=wt, w_cond=None, in_dtype=B.CG_BF16, out_dtype=B.CG_BF16), **kw})
    for kw in (dict(pad=0), dict(epilogue=B.CG_EPI_RESIDUAL), dict(c_in=64, x_pixel_stride=128)):
        with pytest.raises(B.CGError):
            make(**kw).forward_beside(x, w1, one, one, 64)
    with pytest.raises(B.CGError):
        make().forward_beside(x, w1, one, one, 96)
    with pytest.raises(B.CGError):
        make().forward_beside(torch.zeros((2, 8, 8, 64), dtype=torch.bfloat16, device="cuda"), w1, one, one, 64)
