"""A forward call through the native extension and the same call through ctypes (which takes what is no plain tensor): the same outputs, kinds of
result and errors."""
import numpy as np
import pytest
import torch

from paper_1805_12549_amd import binding as B

pytestmark = pytest.mark.gpu


class Marked(torch.Tensor):
    """A tensor subclass: not a plain tensor."""


def _layer(tau_c=0.0, gated=True):
    g = torch.Generator().manual_seed(5)
    w = torch.randn((48, 3, 3, 32), generator=g).cuda()
    x = torch.randn((5, 9, 7, 32), generator=g).relu().cuda()
    kw = dict(gate_mean=np.zeros(48), gate_var=np.ones(48), delta=np.full(48, 0.3)) if gated else {}
    cb = 8 if gated else 32
    layer = B.GatedConv(n_max=5, h=9, w=7, c_in=32, c_out=48, c_base=cb, w_base=w[..., :cb].contiguous(), w_cond=w[..., cb:].contiguous() if gated else None,
                        in_dtype=B.CG_F32, out_dtype=B.CG_F32, epilogue=B.CG_EPI_RELU | B.CG_EPI_RESIDUAL, tau_c=tau_c, **kw)
    return layer, x, torch.randn((5, 9, 7, 48), generator=g).cuda()


@pytest.mark.parametrize("tau_c,gated", [(0.0, True), (0.4, True), (0.0, False)], ids=["gate", "channel_gate", "dense"])
@pytest.mark.parametrize("bitmap", [True, False, None, "given"])
@pytest.mark.parametrize("counts", [True, False, "given"])
def test_native_and_ctypes_calls_agree(tau_c, gated, bitmap, counts):
    layer, x, res = _layer(tau_c, gated)

    def outputs():
        b = torch.full((5 * 63, 2), -1, dtype=torch.int32, device="cuda") if bitmap == "given" else bitmap
        c = torch.full((2 + 5 * 48,), -1, dtype=torch.int32, device="cuda") if counts == "given" else counts
        return b, c

    for n in (5, 2):
        b, c = outputs()
        native = layer.forward(x[:n], residual=res[:n], bitmap=b[:n * 63] if bitmap == "given" else b, counts=c)
        b2, c2 = outputs()
        other = layer.forward(x[:n].as_subclass(Marked), residual=res[:n], bitmap=b2[:n * 63] if bitmap == "given" else b2, counts=c2)
        for p, q in zip(native, other):
            assert (p is None) == (q is None)
            if p is not None:
                assert p.shape == q.shape and p.dtype == q.dtype and p.stride() == q.stride() and p.device == q.device
                k = 2 + n * 48 if p.dim() == 1 else None             # (a smaller batch leaves the rest of a larger buffer alone)
                assert torch.equal(torch.as_tensor(p)[:k], torch.as_tensor(q)[:k])
        assert (native[1] is not None) == (bitmap not in (False, None)) and (native[2] is not None) == (counts is not False)
    layer.close()


def test_errors_and_streams():
    layer, x, res = _layer()
    with pytest.raises(B.CGError) as err:
        layer.forward(torch.cat([x, x]), residual=torch.cat([res, res]))
    assert err.value.code == B.CG_EINVAL and "n_max" in str(err.value)
    with pytest.raises(B.CGError) as err:
        layer.forward(x)
    assert err.value.code == B.CG_EINVAL and "residual" in str(err.value)
    want = layer.forward(x, residual=res)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        here = layer.forward(x, residual=res)
    layer.stream = side                                              # the layer's own stream, whatever the current one is
    own = layer.forward(x, residual=res)
    side.synchronize()
    for got in (here, own):
        assert all(torch.equal(p, q) for p, q in zip(want, got))
    with pytest.raises(AttributeError):
        layer.forward(None, residual=res)                            # (as the other path says it)
    layer.close()
    with pytest.raises(B.CGError):
        layer.forward(x, residual=res)


def test_calls_without_the_extension():
    """The extension is what a built tree runs on; without it the same call goes through ctypes."""
    assert B._calls is not None
    layer, x, res = _layer()
    assert layer._native is not None
    want = layer.forward(x, residual=res)
    layer._native = None
    assert all(torch.equal(p, q) for p, q in zip(want, layer.forward(x, residual=res)))
    layer.close()
