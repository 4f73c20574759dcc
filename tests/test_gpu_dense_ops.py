"""GPU parity of the dense pieces of a ResNet around the gated layers (small-channel input
convolution, 3x3 stride-2 max pooling, average pooling + fully connected layer, 1x1 stride-2
shortcut convolution) against the CPU oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import cg_oracle as O
from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def _bf16(a):
    return W.bf16_round(np.asarray(a, np.float32))


def _dev(a, dtype=torch.bfloat16):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda().to(dtype).contiguous()


def _stream():
    return torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("n,h,w,c_in,c_out,k,stride,pad", [
    (2, 224, 224, 3, 64, 7, 2, 3),        # the ImageNet input layer
    (3, 37, 29, 3, 64, 7, 2, 3),          # ragged tiles
    (2, 32, 32, 3, 128, 3, 1, 1),         # a CIFAR-style input layer, two channel blocks
    (1, 9, 9, 4, 64, 5, 2, 2),
    (2, 8, 8, 1, 64, 1, 1, 0),
])
def test_small_cin_conv(n, h, w, c_in, c_out, k, stride, pad):
    rng = np.random.default_rng(n * 100 + h + k)
    x = _bf16(rng.standard_normal((n, h, w, c_in)))
    wt = _bf16(rng.standard_normal((c_out, k, k, c_in)) * np.sqrt(2.0 / (k * k * c_in)))
    sc = rng.uniform(0.5, 1.5, c_out).astype(np.float32)
    sh = (rng.standard_normal(c_out) * 0.1).astype(np.float32)
    ho, wo = O.out_hw(h, w, k, k, stride, pad)
    xd, wd_ = _dev(x), _dev(wt)
    scd, shd = _dev(sc, torch.float32), _dev(sh, torch.float32)
    for relu, with_affine in ((True, True), (False, False)):
        y = torch.empty((n, ho, wo, c_out), dtype=torch.bfloat16, device="cuda")
        B.cg_small_cin_conv(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr() if with_affine else 0,
                            shd.data_ptr() if with_affine else 0, y.data_ptr(), n, h, w, c_in, c_out, k, stride, pad,
                            relu, _stream())
        torch.cuda.synchronize()
        ref = O.dense_conv(x, wt, stride=stride, pad=pad, scale=sc if with_affine else None,
                           shift=sh if with_affine else None, relu=relu)
        got = y.float().cpu().numpy().astype(np.float64)
        tol = P.ATOL + P.RTOL * np.abs(ref) + P.bf16_ulp(ref)
        assert (np.abs(got - ref) <= tol).all(), float(np.abs(got - ref).max())


@pytest.mark.parametrize("n,h,w,c_out,pad", [(2, 224, 224, 64, 3), (3, 61, 45, 64, 3), (2, 33, 70, 128, 3), (1, 9, 9, 64, 2),
                                              (70, 64, 64, 64, 3)])
def test_conv7x7s2_maxpool_fused(n, h, w, c_out, pad):
    """The fused kernel against the two separate entry points (bit for bit) and against the oracle."""
    rng = np.random.default_rng(n + h + w)
    x = _bf16(rng.standard_normal((n, h, w, 3)))
    wt = _bf16(rng.standard_normal((c_out, 7, 7, 3)) * np.sqrt(2.0 / 147))
    sc = rng.uniform(0.5, 1.5, c_out).astype(np.float32)
    sh = (rng.standard_normal(c_out) * 0.3).astype(np.float32)
    ho, wo = O.out_hw(h, w, 7, 7, 2, pad)
    pho, pwo = (ho - 1) // 2 + 1, (wo - 1) // 2 + 1
    xd, wd_, scd, shd = _dev(x), _dev(wt), _dev(sc, torch.float32), _dev(sh, torch.float32)
    for relu in (True, False):
        y = torch.empty((n, ho, wo, c_out), dtype=torch.bfloat16, device="cuda")
        p2 = torch.empty((n, pho, pwo, c_out), dtype=torch.bfloat16, device="cuda")
        pf = torch.full((n, pho, pwo, c_out), 7.0, dtype=torch.bfloat16, device="cuda")
        B.cg_small_cin_conv(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr(), shd.data_ptr(), y.data_ptr(), n, h, w, 3, c_out,
                            7, 2, pad, relu, _stream())
        B.cg_maxpool3x3s2(y.data_ptr(), p2.data_ptr(), n, ho, wo, c_out, _stream())
        B.cg_conv7x7s2_maxpool(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr(), shd.data_ptr(), pf.data_ptr(), n, h, w, c_out,
                               pad, relu, _stream())
        torch.cuda.synchronize()
        assert torch.equal(pf, p2)
        if n <= 3:
            ref = O.maxpool3x3s2(O.dense_conv(x, wt, stride=2, pad=pad, scale=sc, shift=sh, relu=relu))
            got = pf.float().cpu().numpy().astype(np.float64)
            tol = P.ATOL + P.RTOL * np.abs(ref) + P.bf16_ulp(ref)
            assert (np.abs(got - ref) <= tol).all(), float(np.abs(got - ref).max())


@pytest.mark.parametrize("n,h,w,c_out,pad", [(24, 224, 224, 64, 3), (40, 131, 90, 128, 3), (300, 33, 40, 64, 2)])
def test_conv7x7s2_single_images_equal_the_batch(n, h, w, c_out, pad):
    """32 channels a workgroup (few images) and 64: every output is the same chain of products, so bit for bit the same."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    x = torch.randn((n, h, w, 3), generator=gen, device="cuda").to(torch.bfloat16)
    wt = (torch.randn((c_out, 7, 7, 3), generator=gen, device="cuda") * 0.12).to(torch.bfloat16)
    sc = torch.randn(c_out, generator=gen, device="cuda")              # negative ones among them
    sh = torch.randn(c_out, generator=gen, device="cuda")
    ho, wo = O.out_hw(h, w, 7, 7, 2, pad)
    ph, pw = (ho - 1) // 2 + 1, (wo - 1) // 2 + 1
    def run(k0, k1):
        y = torch.empty((k1 - k0, ho, wo, c_out), dtype=torch.bfloat16, device="cuda")
        p = torch.empty((k1 - k0, ph, pw, c_out), dtype=torch.bfloat16, device="cuda")
        B.cg_small_cin_conv(x[k0:k1].data_ptr(), wt.data_ptr(), sc.data_ptr(), sh.data_ptr(), y.data_ptr(), k1 - k0, h, w, 3, c_out,
                            7, 2, pad, True, _stream())
        B.cg_conv7x7s2_maxpool(x[k0:k1].data_ptr(), wt.data_ptr(), sc.data_ptr(), sh.data_ptr(), p.data_ptr(), k1 - k0, h, w, c_out,
                               pad, True, _stream())
        return y, p
    y, p = run(0, n)
    for k in (0, n // 2, n - 1):
        y1, p1 = run(k, k + 1)
        assert torch.equal(y[k:k + 1], y1) and torch.equal(p[k:k + 1], p1)


@pytest.mark.parametrize("w,pad", [(w, 3) for w in (1, 2, 3, 5, 8, 9, 12, 14, 23, 47, 86, 127)] + [(w, 2) for w in (3, 5, 8, 9, 12, 14, 23, 47, 86, 127)])
def test_conv7x7s2_rows_that_end_inside_a_piece(w, pad):
    """Widths whose rows end at every place of a 16-byte piece of the input, rows shorter than one among them; odd numbers of output rows."""
    n, h, c_out = 2, 25, 64
    rng = np.random.default_rng(w + pad)
    x = _bf16(rng.standard_normal((n, h, w, 3)))
    wt = _bf16(rng.standard_normal((c_out, 7, 7, 3)) * np.sqrt(2.0 / 147))
    sc = rng.uniform(-0.5, 1.5, c_out).astype(np.float32)
    sh = (rng.standard_normal(c_out) * 0.3).astype(np.float32)
    ho, wo = O.out_hw(h, w, 7, 7, 2, pad)
    xd, wd_, scd, shd = _dev(x), _dev(wt), _dev(sc, torch.float32), _dev(sh, torch.float32)
    y = torch.empty((n, ho, wo, c_out), dtype=torch.bfloat16, device="cuda")
    p = torch.empty((n, (ho - 1) // 2 + 1, (wo - 1) // 2 + 1, c_out), dtype=torch.bfloat16, device="cuda")
    B.cg_small_cin_conv(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr(), shd.data_ptr(), y.data_ptr(), n, h, w, 3, c_out, 7, 2, pad, True, _stream())
    B.cg_conv7x7s2_maxpool(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr(), shd.data_ptr(), p.data_ptr(), n, h, w, c_out, pad, True, _stream())
    torch.cuda.synchronize()
    dense = O.dense_conv(x, wt, stride=2, pad=pad, scale=sc, shift=sh, relu=True)
    for got, ref in ((y, dense), (p, O.maxpool3x3s2(dense))):
        tol = P.ATOL + P.RTOL * np.abs(ref) + P.bf16_ulp(ref)
        assert (np.abs(got.float().cpu().numpy().astype(np.float64) - ref) <= tol).all()


@pytest.mark.parametrize("n,h,w,c", [(2, 112, 112, 64), (3, 9, 7, 8), (1, 1, 1, 16), (2, 6, 5, 72)])
def test_maxpool_bit_exact(n, h, w, c):
    rng = np.random.default_rng(h * 10 + c)
    x = _bf16(rng.standard_normal((n, h, w, c)) - 2.0)
    xd = _dev(x)
    y = torch.empty((n, (h - 1) // 2 + 1, (w - 1) // 2 + 1, c), dtype=torch.bfloat16, device="cuda")
    B.cg_maxpool3x3s2(xd.data_ptr(), y.data_ptr(), n, h, w, c, _stream())
    torch.cuda.synchronize()
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), O.maxpool3x3s2(x))     # a maximum of bf16 values is exact


@pytest.mark.parametrize("n,hw,c,classes", [(4, 49, 512, 1000), (2, 16, 64, 10), (1, 1, 24, 7),
                                              (2, 9, 640, 33), (2, 5, 768, 12), (1, 4, 1200, 9)])
def test_avgpool_fc(n, hw, c, classes):
    rng = np.random.default_rng(hw + classes)
    x = _bf16(np.maximum(rng.standard_normal((n, hw, c)), 0))
    wfc = _bf16(rng.standard_normal((classes, c)) / np.sqrt(c))
    b = rng.standard_normal(classes).astype(np.float32)
    xd, wd_, bd = _dev(x), _dev(wfc), _dev(b, torch.float32)
    out = torch.empty((n, classes), dtype=torch.float32, device="cuda")
    B.cg_avgpool_fc(xd.data_ptr(), wd_.data_ptr(), bd.data_ptr(), out.data_ptr(), n, hw, c, classes, _stream())
    B.cg_avgpool_fc(xd.data_ptr(), wd_.data_ptr(), 0, out.data_ptr(), 0, hw, c, classes, _stream())   # n = 0: nothing
    torch.cuda.synchronize()
    ref = O.avgpool_fc(x, wfc, b)
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=P.RTOL, atol=P.ATOL)


@pytest.mark.parametrize("c_in,c_out,hw", [(64, 128, 56), (128, 256, 28), (256, 512, 14)])
def test_shortcut_conv_1x1_stride2_dense(c_in, c_out, hw):
    """The ResNet shortcut: a dense (c_base == c_in) 1x1 stride-2 layer of cg_conv_create, with scale/shift."""
    shape = W.LayerShape("sc_%d" % c_in, 2, hw, hw, c_in, c_out, stride=2, pad=0, groups=1, k=1)
    inp = W.make_inputs(shape, 600 + c_in, kind="iid", round_bf16=True)
    rng = np.random.default_rng(c_in)
    aff = dict(scale0=rng.uniform(0.5, 1.5, c_out), shift0=rng.normal(0, 0.1, c_out),
               scale1=rng.uniform(0.5, 1.5, c_out), shift1=rng.normal(0, 0.1, c_out))
    rep = P.run_float(inp, None, out_dtype=B.CG_BF16, epilogue=B.CG_EPI_AFFINE, affine=aff, name=shape.name)
    assert rep.variant == B.CG_VARIANT_TILE and rep.fired_frac == 0.0


@pytest.mark.parametrize("n,hw,c_in,c_out,stride", [(2, 56, 64, 128, 2), (3, 28, 128, 256, 2), (2, 14, 256, 512, 2),
                                                    (1, 9, 16, 64, 1), (2, 7, 512, 64, 3)])
def test_pointwise_conv(n, hw, c_in, c_out, stride):
    rng = np.random.default_rng(c_in + hw)
    x = _bf16(rng.standard_normal((n, hw, hw + 1, c_in)))
    wt = _bf16(rng.standard_normal((c_out, 1, 1, c_in)) * np.sqrt(2.0 / c_in))
    sc = rng.uniform(0.5, 1.5, c_out).astype(np.float32)
    sh = (rng.standard_normal(c_out) * 0.1).astype(np.float32)
    ho, wo = (hw - 1) // stride + 1, hw // stride + 1
    xd, wd_, scd, shd = _dev(x), _dev(wt.reshape(c_out, c_in)), _dev(sc, torch.float32), _dev(sh, torch.float32)
    for relu, aff in ((True, True), (False, False)):
        y = torch.empty((n, ho, wo, c_out), dtype=torch.bfloat16, device="cuda")
        B.cg_pointwise_conv(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr() if aff else 0, shd.data_ptr() if aff else 0,
                            y.data_ptr(), n, hw, hw + 1, c_in, c_out, stride, relu, _stream())
        torch.cuda.synchronize()
        ref = O.dense_conv(x, wt, stride=stride, pad=0, scale=sc if aff else None, shift=sh if aff else None, relu=relu)
        assert ref.shape == (n, ho, wo, c_out)
        got = y.float().cpu().numpy().astype(np.float64)
        tol = P.ATOL + P.RTOL * np.abs(ref) + P.bf16_ulp(ref)
        assert (np.abs(got - ref) <= tol).all(), float(np.abs(got - ref).max())


def test_dense_ops_reject_bad_arguments_before_any_launch():
    with pytest.raises(B.CGError) as e:
        B.cg_small_cin_conv(16, 16, 0, 0, 16, 1, 8, 8, 5, 64, 3, 1, 1, True)
    assert e.value.code == B.CG_EUNSUPPORTED
    with pytest.raises(B.CGError) as e:
        B.cg_maxpool3x3s2(16, 16, 1, 8, 8, 12)
    assert e.value.code == B.CG_EUNSUPPORTED
    with pytest.raises(B.CGError) as e:
        B.cg_avgpool_fc(0, 16, 0, 16, 1, 4, 8, 2)
    assert e.value.code == B.CG_EINVAL


def _check(got, ref):
    tol = P.ATOL + P.RTOL * np.abs(ref) + P.bf16_ulp(ref)
    err = np.abs(got - ref)
    assert (err <= tol).all(), "max err %.4g at %s" % (float(err.max()), np.unravel_index(int(err.argmax()), err.shape))


@pytest.mark.parametrize("seed", range(12))
def test_dense_ops_on_random_shapes(seed):
    """Seeded random shapes inside each entry point's documented limits: odd image sizes, every kernel
    size and stride the input layer takes, channel counts away from the powers of two."""
    rng = np.random.default_rng(4100 + seed)
    # input-layer convolution
    n, h, w = int(rng.integers(1, 4)), int(rng.integers(7, 50)), int(rng.integers(7, 50))
    c_in, c_out = int(rng.integers(1, 5)), 64 * int(rng.integers(1, 4))
    k = int(rng.choice([1, 3, 5, 7]))
    stride, pad = int(rng.integers(1, 3)), int(rng.integers(0, k))
    x = _bf16(rng.standard_normal((n, h, w, c_in)))
    wt = _bf16(rng.standard_normal((c_out, k, k, c_in)) * np.sqrt(2.0 / (k * k * c_in)))
    sc = rng.uniform(0.5, 1.5, c_out).astype(np.float32)
    sh = (rng.standard_normal(c_out) * 0.1).astype(np.float32)
    ho, wo = O.out_hw(h, w, k, k, stride, pad)
    y = torch.empty((n, ho, wo, c_out), dtype=torch.bfloat16, device="cuda")
    scd, shd = _dev(sc, torch.float32), _dev(sh, torch.float32)
    print("\n  small_cin_conv n=%d %dx%d c_in=%d c_out=%d k=%d s=%d p=%d" % (n, h, w, c_in, c_out, k, stride, pad), flush=True)
    xd, wd_ = _dev(x), _dev(wt)           # (held until the kernel has run)
    B.cg_small_cin_conv(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr(), shd.data_ptr(), y.data_ptr(), n, h, w,
                        c_in, c_out, k, stride, pad, True, _stream())
    torch.cuda.synchronize()
    _check(y.float().cpu().numpy().astype(np.float64), O.dense_conv(x, wt, stride=stride, pad=pad, scale=sc, shift=sh, relu=True))
    # max pooling
    n, h, w, c = int(rng.integers(1, 4)), int(rng.integers(1, 40)), int(rng.integers(1, 40)), 8 * int(rng.integers(1, 20))
    x = _bf16(rng.standard_normal((n, h, w, c)))
    y = torch.empty((n, (h - 1) // 2 + 1, (w - 1) // 2 + 1, c), dtype=torch.bfloat16, device="cuda")
    print("  maxpool n=%d %dx%d c=%d" % (n, h, w, c), flush=True)
    xd = _dev(x)
    B.cg_maxpool3x3s2(xd.data_ptr(), y.data_ptr(), n, h, w, c, _stream())
    torch.cuda.synchronize()
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), O.maxpool3x3s2(x))
    # 1x1 convolution with stride
    n, h, w = int(rng.integers(1, 4)), int(rng.integers(1, 30)), int(rng.integers(1, 30))
    c_in, c_out, stride = 16 * int(rng.integers(1, 33)), 64 * int(rng.integers(1, 6)), int(rng.integers(1, 4))
    x = _bf16(rng.standard_normal((n, h, w, c_in)))
    wt = _bf16(rng.standard_normal((c_out, 1, 1, c_in)) * np.sqrt(2.0 / c_in))
    sc = rng.uniform(0.5, 1.5, c_out).astype(np.float32)
    sh = (rng.standard_normal(c_out) * 0.1).astype(np.float32)
    y = torch.empty((n, (h - 1) // stride + 1, (w - 1) // stride + 1, c_out), dtype=torch.bfloat16, device="cuda")
    scd, shd = _dev(sc, torch.float32), _dev(sh, torch.float32)
    print("  pointwise n=%d %dx%d c_in=%d c_out=%d s=%d" % (n, h, w, c_in, c_out, stride), flush=True)
    xd, wd_ = _dev(x), _dev(wt.reshape(c_out, c_in))
    B.cg_pointwise_conv(xd.data_ptr(), wd_.data_ptr(), scd.data_ptr(), shd.data_ptr(),
                        y.data_ptr(), n, h, w, c_in, c_out, stride, False, _stream())
    torch.cuda.synchronize()
    _check(y.float().cpu().numpy().astype(np.float64), O.dense_conv(x, wt, stride=stride, pad=0, scale=sc, shift=sh, relu=False))
    # average pooling + classifier
    n, hw, c, classes = int(rng.integers(1, 6)), int(rng.integers(1, 60)), 8 * int(rng.integers(1, 200)), int(rng.integers(1, 1100))
    x = _bf16(np.maximum(rng.standard_normal((n, hw, c)), 0))
    wfc = _bf16(rng.standard_normal((classes, c)) / np.sqrt(c))
    b = rng.standard_normal(classes).astype(np.float32)
    out = torch.empty((n, classes), dtype=torch.float32, device="cuda")
    print("  avgpool_fc n=%d hw=%d c=%d classes=%d" % (n, hw, c, classes), flush=True)
    xd, wd_, bd = _dev(x), _dev(wfc), _dev(b, torch.float32)
    B.cg_avgpool_fc(xd.data_ptr(), wd_.data_ptr(), bd.data_ptr(), out.data_ptr(), n, hw, c, classes, _stream())
    torch.cuda.synchronize()
    np.testing.assert_allclose(out.cpu().numpy(), O.avgpool_fc(x, wfc, b), rtol=P.RTOL, atol=P.ATOL)


@pytest.mark.parametrize("n,h,w,c_in,c_out,stride", [
    (1, 4, 4, 16, 64, 1), (1, 1, 17, 48, 64, 1), (3, 9, 7, 272, 128, 2), (1, 31, 33, 512, 192, 2),      # few pixels: 16 x 32 tiles
    (70, 56, 57, 64, 128, 2), (19, 43, 41, 16, 64, 1), (64, 28, 28, 512, 64, 1), (130, 30, 29, 208, 256, 2)])    # many: 64 x 128 or 128 x 64
def test_pointwise_conv_forms(n, h, w, c_in, c_out, stride):
    gen = torch.Generator(device="cuda").manual_seed(c_in + h)
    x = torch.randn((n, h, w, c_in), generator=gen, device="cuda").to(torch.bfloat16)
    wt = (torch.randn((c_out, c_in), generator=gen, device="cuda") * (2.0 / c_in) ** 0.5).to(torch.bfloat16)
    sc, sh = torch.rand(c_out, generator=gen, device="cuda") + 0.5, torch.randn(c_out, generator=gen, device="cuda") * 0.1
    y = torch.empty((n, (h - 1) // stride + 1, (w - 1) // stride + 1, c_out), dtype=torch.bfloat16, device="cuda")
    B.cg_pointwise_conv(x.data_ptr(), wt.data_ptr(), sc.data_ptr(), sh.data_ptr(), y.data_ptr(), n, h, w, c_in, c_out, stride, True, _stream())
    xs = x[:, ::stride, ::stride].reshape(-1, c_in).double().cpu()
    ref = torch.relu(xs @ wt.double().cpu().t() * sc.double().cpu() + sh.double().cpu()).reshape(y.shape)
    _check(y.double().cpu().numpy(), ref.numpy())


# workgroups of 64 pixels x 128 channels, the last block of channels half empty, and of 128 x 64 (test_kernels_of_calls_cpu.py holds which)
HALF_EMPTY = [((1, 1, 9600, 192, 64, 1), True), ((3, 57, 61, 208, 192, 1), True), ((2, 73, 61, 48, 320, 1), True), ((9, 60, 61, 512, 64, 1), True), ((1, 150, 61, 112, 192, 1), True),
              ((5, 64, 61, 320, 64, 1), False), ((13, 71, 77, 128, 64, 1), False), ((11, 139, 131, 512, 64, 2), False), ((3, 61, 57, 64, 192, 1), False),
              ((5, 66, 70, 384, 320, 2), False)]


@pytest.mark.parametrize("scaled,relu", [(True, True), (False, False)])
@pytest.mark.parametrize("shape", [s for s, _ in HALF_EMPTY], ids=lambda s: "x".join(map(str, s)))
def test_pointwise_conv_half_empty_blocks(shape, scaled, relu):
    n, h, w, c_in, c_out, stride = shape
    gen = torch.Generator(device="cuda").manual_seed(c_in + h)
    x = torch.randn((n, h, w, c_in), generator=gen, device="cuda").to(torch.bfloat16)
    wt = (torch.randn((c_out, c_in), generator=gen, device="cuda") * (2.0 / c_in) ** 0.5).to(torch.bfloat16)
    sc, sh = torch.rand(c_out, generator=gen, device="cuda") + 0.5, torch.randn(c_out, generator=gen, device="cuda") * 0.1
    ho, wo = (h - 1) // stride + 1, (w - 1) // stride + 1
    y = torch.full((n * ho * wo + 1, c_out), 7.0, dtype=torch.bfloat16, device="cuda")          # (a pixel more, that stays as it is)
    B.cg_pointwise_conv(x.data_ptr(), wt.data_ptr(), sc.data_ptr() if scaled else 0, sh.data_ptr() if scaled else 0, y.data_ptr(), n, h, w, c_in, c_out, stride, relu,
                        _stream())
    ref = x[:, ::stride, ::stride].reshape(-1, c_in).double().cpu() @ wt.double().cpu().t()
    if scaled:
        ref = ref * sc.double().cpu() + sh.double().cpu()
    _check(y[:-1].double().cpu().numpy(), (torch.relu(ref) if relu else ref).numpy())
    assert torch.equal(y[-1], torch.full_like(y[-1], 7.0))


@pytest.mark.parametrize("n,hw,c,classes", [(1, 49, 512, 1000), (1, 3, 32, 33), (5, 49, 2048, 40), (17, 16, 96, 1000), (70, 9, 352, 257),
                                              (300, 4, 64, 700)])
def test_avgpool_fc_splits(n, hw, c, classes):
    """32 to 256 classes to a workgroup, whose K steps up to eight wavefronts share."""
    gen = torch.Generator(device="cuda").manual_seed(n + c)
    x = torch.relu(torch.randn((n, hw, c), generator=gen, device="cuda")).to(torch.bfloat16)
    wfc = (torch.randn((classes, c), generator=gen, device="cuda") / c ** 0.5).to(torch.bfloat16)
    b = torch.randn(classes, generator=gen, device="cuda")
    out = torch.empty((n, classes), dtype=torch.float32, device="cuda")
    B.cg_avgpool_fc(x.data_ptr(), wfc.data_ptr(), b.data_ptr(), out.data_ptr(), n, hw, c, classes, _stream())
    ref = x.double().cpu().mean(1) @ wfc.double().cpu().t() + b.double().cpu()
    np.testing.assert_allclose(out.cpu().numpy(), ref.numpy(), rtol=P.RTOL, atol=P.ATOL)
