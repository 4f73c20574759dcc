"""GPU parity of the small-tile matrix-core kernel (operands straight from global memory) against the CPU
oracle, through the C ABI: channel counts that are multiples of nothing large, base groups that end
inside a 16-byte chunk, single images, fp32, both forms (K split over wavefronts / one wavefront per tile)."""
import numpy as np
import pytest
import torch

from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def _say(rep):
    print("\n  " + str(rep), flush=True)
    return rep


def S(n, h, w, ci, co, **kw):
    return W.LayerShape("%dx%dx%d_%d>%d" % (n, h, w, ci, co) + "".join("_%s%d" % i for i in sorted(kw.items())), n, h, w, ci, co, **kw)


SHAPES = [
    S(1, 32, 32, 16, 16),                     # the smallest configuration
    S(5, 45, 33, 96, 80),                     # c_out ends inside a fragment
    S(1, 3, 3, 16, 8, pad=0),                 # one output pixel, eight channels
    S(2, 9, 11, 48, 33),                      # c_out odd: element stores
    S(3, 7, 7, 16, 48, groups=8),             # base groups of two channels: inside a chunk
    S(2, 13, 9, 80, 96, groups=5, stride=2),  # three fragments across the channels
    S(1, 14, 14, 256, 256),                   # one image, deep
    S(1, 7, 7, 512, 512),
    S(40, 33, 31, 16, 64),                    # enough tiles for one wavefront each
    S(9, 5, 6, 96, 112, k=1, pad=0),
    S(70, 1, 1, 160, 48, k=1, pad=0),
    S(2, 14, 14, 64, 128, k=1, pad=0, stride=2, groups=8),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[s.name for s in SHAPES])
def test_small_tiles(shape):
    rng = np.random.default_rng(shape.n * 7 + shape.c_out)
    c = shape.c_out
    aff = dict(scale0=rng.uniform(0.5, 1.5, c), shift0=rng.normal(0, 0.1, c),
               scale1=rng.uniform(0.5, 1.5, c), shift1=rng.normal(0, 0.1, c))
    res = rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32)
    full = B.CG_EPI_RELU | B.CG_EPI_AFFINE | B.CG_EPI_RESIDUAL
    kind = "coherent" if min(shape.h, shape.w) >= 8 else "iid"
    inp = W.make_inputs(shape, 7000 + c + shape.h, kind=kind, rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.3, sample_images=None)
    _say(P.run_float(inp, gate, in_dtype=B.CG_F32, out_dtype=B.CG_F32, affine=aff, residual=res, epilogue=full, name=shape.name + " fp32"))
    _say(P.run_float(inp, gate, in_dtype=B.CG_F32, out_dtype=B.CG_BF16, n_run=1, tau_c=0.3, name=shape.name + " fp32 channel-wise gate"))
    if shape.c_in % 8 == 0:
        _say(P.run_float(inp, gate, out_dtype=B.CG_BF16, affine=aff, residual=res, epilogue=full, name=shape.name + " bf16"))
        _say(P.run_float(inp, gate, out_dtype=B.CG_F32, delta_hi=gate.delta + 0.8, n_run=(shape.n + 1) // 2, name=shape.name + " bf16 two-sided"))
        _say(P.run_float(inp, None, out_dtype=B.CG_F32, name=shape.name + " bf16 dense")) if shape.groups == 1 else None
    if shape.c_in % 16 == 0:
        q = W.quantize_int8(W.make_inputs(shape, 7100 + c + shape.h, kind=kind, rho=0.35))
        thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
        res8 = rng.integers(-128, 128, (shape.n, shape.ho, shape.wo, c)).astype(np.int8)
        _say(P.run_int8(q, thr, name=shape.name + " int8"))
        _say(P.run_int8(q, thr, out_i8=True, rq=W.requant_params(q, rng), residual=res8, rq_res_mult=1 << 14,
                        epilogue=B.CG_EPI_RESIDUAL | B.CG_EPI_RELU, n_run=1, name=shape.name + " int8 requantised"))


@pytest.mark.parametrize("shape", [S(3, 9, 9, 64, 64, groups=4), S(2, 8, 10, 96, 48, groups=4), S(1, 10, 10, 48, 144, groups=3)],
                         ids=lambda s: s.name)
def test_small_tiles_grouped(shape):
    inp = W.make_inputs(shape, 7300 + shape.c_out, kind="coherent", rho=0.3, round_bf16=True, grouped=True)
    gate = W.calibrate_gate(inp, 0.3, sample_images=None)
    for dt in (B.CG_F32, B.CG_BF16):
        _say(P.run_float(inp, gate, in_dtype=dt, shuffle=True, name=shape.name + " grouped shuffled"))
        _say(P.run_float(inp, gate, in_dtype=dt, n_run=1, out_dtype=B.CG_BF16, name=shape.name + " grouped n=1"))


def test_base_group_inside_a_chunk_keeps_the_paths_apart():
    """A value that is not finite in a conditional channel of the base group's last chunk reaches no base sum."""
    import torch
    w_b, w_c = torch.ones((32, 3, 3, 4), dtype=torch.bfloat16, device="cuda"), torch.ones((32, 3, 3, 12), dtype=torch.bfloat16, device="cuda")
    x = torch.ones((1, 8, 8, 16), dtype=torch.bfloat16, device="cuda")
    x[..., 4:] = float("inf")
    layer = B.GatedConv(n_max=1, h=8, w=8, c_in=16, c_out=32, c_base=4, w_base=w_b, w_cond=w_c, in_dtype=B.CG_BF16,
                        out_dtype=B.CG_F32, gate_mean=np.zeros(32), gate_var=np.ones(32), delta=np.full(32, 1e6))
    y, bitmap, counts = layer.forward(x)
    torch.cuda.synchronize()
    assert int(bitmap.abs().sum()) == 0 and int(counts[0]) == 0
    assert float(y.max()) == 36.0 and float(y.min()) == 16.0
    layer.close()


@pytest.mark.parametrize("in_dtype", [B.CG_F32, B.CG_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("n,h,w,cin,cout,groups", [(1, 9, 7, 64, 64, 4), (2, 8, 10, 96, 48, 4), (1, 8, 8, 32, 48, 16), (40, 33, 31, 16, 64, 4)],
                         ids=["split", "one_group_a_fragment", "groups_inside_a_chunk", "one_wavefront_a_tile"])
def test_grouped_layers_keep_infinities_in_their_group(in_dtype, n, h, w, cin, cout, groups):
    """An infinite input reaches the base sums of its own group and the conditional sums of the others, and nothing else.
    Weights are ones and finite inputs small whole numbers, so every sum is exact and the reference is a plain sum."""
    import torch
    dt = torch.float32 if in_dtype == B.CG_F32 else torch.bfloat16
    cb, cpg = cin // groups, cout // groups
    x = torch.ones((n, h, w, cin), dtype=torch.float64)
    x[:, :, w // 2:, :] = 2.0
    for g in range(groups):
        x[g % n, (3 * g) % h, (5 * g) % w, g * cb + g % cb] = float("inf")
    thr = 9.0 * cb + 0.5                                               # the left half's base sums stay below
    layer = B.GatedConv(n_max=n, h=h, w=w, c_in=cin, c_out=cout, c_base=cb, groups=groups, in_dtype=in_dtype, out_dtype=B.CG_F32,
                        w_base=torch.ones((cout, 3, 3, cb), dtype=dt, device="cuda"),
                        w_cond=torch.ones((cout, 3, 3, cin - cb), dtype=dt, device="cuda"),
                        gate_mean=np.zeros(cout), gate_var=np.ones(cout), delta=np.full(cout, thr))
    y, bitmap, _ = layer.forward(x.to(dt).cuda())
    torch.cuda.synchronize()
    layer.close()
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    per_group = [sum(xp[:, r:r + h, c:c + w, g * cb:(g + 1) * cb].sum(-1) for r in range(3) for c in range(3)) for g in range(groups)]
    want = torch.empty((n, h, w, cout), dtype=torch.float64)
    for g in range(groups):
        rest = sum(per_group[k] for k in range(groups) if k != g)
        want[..., g * cpg:(g + 1) * cpg] = torch.where(per_group[g] >= thr, per_group[g] + rest, per_group[g])[..., None]
    assert torch.isfinite(want).any() and torch.isinf(want).any()
    assert torch.equal(y.cpu().double(), want)
    fired = torch.from_numpy(W.unpack_bitmap(bitmap.cpu().numpy().view(np.uint32), cout)).reshape(n, h, w, cout).bool()
    base = torch.stack(per_group, -1).repeat_interleave(cpg, -1)
    assert torch.equal(fired, base >= thr)


# Layers whose base group ends inside a chunk, (type, images, size, channels in and out, base channels) with the tile and the wavefronts that share
# its K; and grouped ones.  (tests/test_kernels_of_calls_cpu.py checks the forms.)
INSIDE = [
    (B.CG_F32, (1, 20, 40, 40, 10, 1), (1, 1, True)), (B.CG_F32, (4, 20, 40, 40, 10, 1), (1, 2, True)), (B.CG_F32, (8, 64, 16, 16, 3, 1), (2, 2, True)),
    (B.CG_F32, (16, 28, 48, 48, 10, 1), (2, 4, True)), (B.CG_F32, (90, 28, 16, 40, 3, 1), (2, 2, False)), (B.CG_F32, (200, 28, 16, 40, 3, 1), (2, 4, False)),
    (B.CG_BF16, (1, 20, 40, 40, 12, 1), (1, 1, True)), (B.CG_BF16, (4, 20, 40, 40, 12, 1), (1, 2, True)), (B.CG_BF16, (8, 64, 16, 16, 4, 1), (2, 2, True)),
    (B.CG_BF16, (16, 28, 48, 48, 12, 1), (2, 4, True)), (B.CG_BF16, (40, 32, 16, 64, 4, 1), (1, 4, False)), (B.CG_BF16, (200, 28, 16, 40, 4, 1), (2, 4, False)),
    (B.CG_F32, (1, 20, 48, 48, 6, 8), (1, 1, True)), (B.CG_BF16, (200, 28, 16, 80, 4, 4), (2, 4, False)),
]


@pytest.mark.parametrize("bad", [float("inf"), float("nan")], ids=["inf", "nan"])
@pytest.mark.parametrize("dtype,shape,form", INSIDE, ids=["%s_%s%s" % ({0: "fp32", 1: "bf16"}[d], "_".join(map(str, f)), "_grouped" if s[5] > 1 else "")
                                                          for d, s, f in INSIDE])
def test_a_value_that_is_not_finite_changes_no_other_sum(dtype, shape, form, bad):
    """Inputs of any size, so that a sum in another order is another sum.  A bad value in a channel of the conditional path next to the last base channel: no
    decision changes, and no output but those of fired gates that it reaches.  In the last base channel: nothing outside its window
    changes.  Both to the bit.  Grouped: outside the window."""
    n, h, c, co, cb, groups = shape
    tdt = torch.float32 if dtype == B.CG_F32 else torch.bfloat16
    g = torch.Generator().manual_seed(c + co)
    x = torch.randn((n, h, h, c), generator=g).relu().to(tdt).cuda()
    w = (torch.randn((co, 3, 3, c), generator=g) / (9 * c) ** 0.5).to(tdt).cuda()
    kw = dict(groups=groups) if groups > 1 else {}
    layer = B.GatedConv(n_max=n, h=h, w=h, c_in=c, c_out=co, c_base=cb, w_base=w[..., :cb].contiguous(), w_cond=w[..., cb:].contiguous(), in_dtype=dtype,
                        out_dtype=B.CG_F32, epilogue=0, gate_mean=np.zeros(co), gate_var=np.ones(co), delta=np.full(co, 0.2), **kw)
    y0, bits0 = [t.clone() for t in layer.forward(x, counts=False)[:2]]
    fired = torch.from_numpy(W.unpack_bitmap(bits0.cpu().numpy().view(np.uint32), co)).reshape(n, h, h, co).bool().cuda()
    assert 0.05 < fired.float().mean() < 0.7 and torch.isfinite(y0).all()
    for channel in (cb, cb - 1):
        bad_x, near = x.clone(), torch.zeros((n, h, h, 1), dtype=torch.bool, device="cuda")
        for img, r, s in ((0, 3, 4), (0, h - 1, 0), (n - 1, h // 2, h - 2)):
            bad_x[img, r, s, channel] = bad
            near[img, max(0, r - 1):r + 2, max(0, s - 1):s + 2] = True
        y, bits = layer.forward(bad_x, counts=False)[:2]
        own = groups == 1 and channel == cb                        # only fired gates may see it
        same_bits = torch.ones_like(near) if own else ~near
        assert torch.equal(bits.reshape(n, h, h, -1)[same_bits[..., 0]], bits0.reshape(n, h, h, -1)[same_bits[..., 0]])
        same = ~(near & fired) if own else (~near).expand_as(fired)
        assert torch.equal(y[same], y0[same])
        assert not torch.isfinite(y).all()
    layer.close()


# Images one pixel wide whose pixels are of more than 4 MiB: the difference of a row and three pixels is beyond 24 bits of bytes.
LONG_PIXELS = [(B.CG_F32, (1 << 20) + 4), (B.CG_BF16, (1 << 21) + 8), (B.CG_I8, (1 << 22) + 16)]


@pytest.mark.parametrize("dtype,c", LONG_PIXELS, ids=["fp32", "bf16", "int8"])
def test_long_pixels(dtype, c):
    """Whole numbers, whose sums stay below 2^24: exact."""
    g = torch.Generator(device="cuda").manual_seed(c)
    tdt = {B.CG_F32: torch.float32, B.CG_BF16: torch.bfloat16, B.CG_I8: torch.int8}[dtype]
    x = torch.randint(0, 2, (1, 3, 1, c), generator=g, device="cuda", dtype=torch.int8).to(tdt)
    w = torch.randint(-1, 2, (8, 3, 3, c), generator=g, device="cuda", dtype=torch.int8).to(tdt)
    layer = B.GatedConv(n_max=1, h=3, w=1, c_in=c, c_out=8, c_base=c, w_base=w, w_cond=None, in_dtype=dtype,
                        out_dtype=B.CG_I32 if dtype == B.CG_I8 else B.CG_F32, epilogue=0)
    y = layer.forward(x, bitmap=False, counts=False)[0].double().reshape(3, 8)
    layer.close()
    want = torch.zeros((3, 8), dtype=torch.float64, device="cuda")
    for r in range(3):
        column = w[:, r, 1].double()
        for row in range(max(0, 1 - r), min(3, 4 - r)):
            want[row] += column @ x[0, row + r - 1, 0].double()
    assert want.abs().max() > 100 and torch.equal(y, want)


@pytest.mark.parametrize("tau_c", [0.0, 0.3], ids=["plain_gate", "channel_gate"])
def test_batches_beyond_the_offsets_run_in_pieces(tau_c):
    """x of 1.02 GiB: one piece of 255 images and a rest of six, against calls of 29 images at a time; whole numbers, so equal."""
    import torch
    n, c = 261, 16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    x = torch.randint(0, 60, (n, 512, 512, c), generator=gen, device="cuda", dtype=torch.int8)
    w = torch.randint(-60, 60, (c, 3, 3, c), generator=gen, device="cuda", dtype=torch.int8)
    layer = B.GatedConv(n_max=n, h=512, w=512, c_in=c, c_out=c, c_base=4, w_base=w[..., :4].contiguous(), w_cond=w[..., 4:].contiguous(),
                        in_dtype=B.CG_I8, out_dtype=B.CG_I8, gate_thr_i32=np.linspace(-30000, 30000, c).astype(np.int32), tau_c=tau_c,
                        epilogue=B.CG_EPI_RELU | B.CG_EPI_RESIDUAL, rq_mult0=3, rq_mult1=2, rq_shift=10, rq_res_mult=900)
    res = torch.randint(-128, 128, (n, 512, 512, c), generator=gen, device="cuda", dtype=torch.int8)
    y, bitmap, counts = layer.forward(x, residual=res)
    total = 0
    for i in range(0, n, 29):
        y2, bitmap2, counts2 = layer.forward(x[i:i + 29], residual=res[i:i + 29])
        px = 512 * 512
        assert torch.equal(y[i:i + 29], y2) and torch.equal(bitmap[i * px:(i + 29) * px], bitmap2)
        assert torch.equal(counts[2 + i * c:2 + (i + 29) * c], counts2[2:])
        total += int(counts2[0]) & 0xffffffff
    assert (int(counts[0]) & 0xffffffff) + (int(counts[1]) << 32) == total and 0 < total < n * 512 * 512 * c
    layer.close()


# Edges of the tiles of 16 or 32 pixels by 16, 32 or 64 channels: pixels around multiples of 16, channels that end inside a
# sixteen (the bitmap's other half word is written as well), K of one step and of many, wavefronts without a K step of their own.
FORMS = [
    S(1, 1, 1, 16, 16, k=1, pad=0), S(3, 1, 5, 48, 17, k=1, pad=0), S(1, 4, 4, 32, 48), S(1, 1, 17, 64, 40),
    S(2, 3, 11, 128, 72, k=1, pad=0, stride=2), S(1, 7, 7, 128, 128), S(33, 2, 2, 96, 33), S(5, 9, 9, 64, 144, stride=2),
    S(1, 1, 1, 1344, 208, k=1, pad=0, groups=2), S(3, 13, 13, 192, 96, groups=8), S(60, 12, 12, 32, 80), S(16, 40, 40, 16, 32, k=1, pad=0),
]


@pytest.mark.parametrize("shape", FORMS, ids=[s.name for s in FORMS])
@pytest.mark.parametrize("grouped", [False, True], ids=["plain", "grouped"])
def test_tile_edges(shape, grouped):
    if grouped and (shape.c_out % shape.groups or shape.k != 3):
        pytest.skip("no such grouping")
    kind = "iid"
    inp = W.make_inputs(shape, 7300 + shape.c_out + shape.h, kind=kind, rho=0.3, round_bf16=True, grouped=grouped)
    gate = W.calibrate_gate(inp, 0.3, sample_images=None)
    kw = dict(shuffle=grouped)
    for dtype in (B.CG_F32, B.CG_BF16):
        if shape.c_in % (4 if dtype == B.CG_F32 else 8) == 0:
            _say(P.run_float(inp, gate, in_dtype=dtype, out_dtype=dtype, name=shape.name + " %d" % dtype, **kw))
    if shape.c_in % 16 == 0:
        q = W.quantize_int8(W.make_inputs(shape, 7400 + shape.c_out + shape.h, kind=kind, rho=0.35, grouped=grouped))
        thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
        _say(P.run_int8(q, thr, name=shape.name + " int8", **kw))


# The forms that the layers above do not run in, a layer for up to three types: tile (16 pixels, 16 channels), whether K is split.  Pixels and
# channels end inside a tile.  (tests/test_kernels_of_calls_cpu.py checks that they run in these forms.)
F, H, I = B.CG_F32, B.CG_BF16, B.CG_I8
TILES = [
    (S(1, 28, 39, 16, 35, k=1, pad=0, groups=2), False, {F: (1, 2, True), H: (1, 2, True), I: (1, 2, True)}),
    (S(173, 15, 1, 48, 33, k=1, pad=0, groups=2), False, {F: (1, 4, True), H: (1, 4, True), I: (1, 4, True)}),
    (S(904, 1, 19, 16, 39, k=1, pad=0, groups=2), False, {F: (1, 2, False), H: (2, 4, False), I: (2, 4, False)}),
    (S(1269, 1, 13, 16, 72, k=1, pad=0), False, {F: (2, 2, False), H: (2, 2, False), I: (2, 2, False)}),
    (S(62, 9, 39, 16, 83, k=1, pad=0, groups=2), False, {H: (1, 2, False), I: (1, 2, False)}),
    (S(19, 39, 27, 16, 133, k=1, pad=0, groups=2), False, {F: (2, 4, False)}),
    (S(11, 38, 36, 96, 35, k=1, pad=0, groups=2), False, {F: (2, 4, True)}),
    (S(40, 33, 31, 16, 64), False, {F: (1, 4, False), H: (1, 4, False), I: (1, 4, False)}),
    (S(60, 12, 12, 32, 80), False, {F: (2, 2, True), H: (2, 2, True), I: (2, 2, True)}),
    (S(5, 45, 33, 96, 80), False, {H: (2, 4, True), I: (2, 4, True)}),
    (S(19, 4, 27, 16, 18, groups=2), True, {F: (1, 2, True), H: (1, 2, True)}),
    (S(3, 12, 19, 16, 692, stride=2), True, {F: (1, 4, True), H: (1, 4, True)}),
    (S(158, 38, 3, 16, 74, groups=2), True, {F: (2, 2, False), H: (2, 2, False)}),
    (S(45, 40, 15, 16, 100), True, {F: (2, 4, False), H: (2, 4, False)}),
    (S(13, 40, 34, 16, 172, stride=2), True, {F: (2, 4, True)}),
    (S(527, 6, 4, 16, 100), True, {F: (1, 4, False)}),
    (S(49, 15, 6, 16, 344), True, {F: (1, 2, False)}),
    (S(1698, 1, 52, 8, 10, k=1, pad=0, stride=2, groups=2), True, {H: (1, 2, False)}),
    (S(578, 2, 12, 96, 33, k=1, pad=0), False, {F: (2, 4, True)}),
]

# The same where every K step lies inside one tap, which are kernels of their own.  (All but fp32, 32 x 64, not split, which no layer was found to run in.)
UNIFORM = [
    (S(4, 33, 32, 128, 33, k=1, pad=0, stride=2, groups=2), False, {F: (1, 2, True), H: (1, 2, True), I: (1, 2, True)}),
    (S(94, 7, 21, 128, 18, k=1, pad=0, stride=2, groups=2), False, {F: (2, 2, True), H: (2, 2, True), I: (2, 2, True)}),
    (S(69, 21, 6, 128, 34, k=1, pad=0, stride=2, groups=2), False, {H: (1, 4, True), I: (1, 4, True)}),
    (S(21, 11, 18, 128, 36, k=1, pad=0, groups=2), False, {H: (2, 4, True), I: (2, 4, True)}),
    (S(204, 21, 11, 128, 17, k=1, pad=0, groups=2), False, {F: (1, 2, False), H: (1, 2, False), I: (1, 2, False)}),
    (S(232, 23, 5, 128, 34, k=1, pad=0, groups=2), False, {F: (2, 2, False), H: (2, 4, False), I: (2, 4, False)}),
    (S(27, 9, 12, 128, 299, k=1, pad=0, stride=2, groups=2), False, {F: (1, 4, True)}),
    (S(43, 35, 35, 128, 20, k=1, pad=0, groups=2), False, {H: (2, 2, False), I: (2, 2, False)}),
    (S(81, 32, 14, 128, 33, k=1, pad=0, groups=2), False, {H: (1, 4, False), I: (1, 4, False)}),
    (S(29, 17, 11, 128, 358, k=1, pad=0), False, {F: (1, 4, False)}),
    (S(8, 54, 35, 96, 33, k=1, pad=0, groups=2), False, {F: (2, 4, True)}),
    (S(20, 13, 11, 128, 72, groups=2), False, {F: (1, 2, True), H: (2, 4, True), I: (2, 4, True)}),      # 3x3: K goes over taps and around the base group
    (S(4, 14, 14, 512, 512), False, {I: (2, 4, True)}),
]


@pytest.mark.parametrize("shape,grouped,forms", TILES + UNIFORM, ids=[t[0].name + ("_grouped" if t[1] else "") for t in TILES + UNIFORM])
def test_every_tile(shape, grouped, forms):
    inp = W.make_inputs(shape, 7500 + shape.c_out + shape.h, kind="iid", rho=0.3, round_bf16=True, grouped=grouped)
    gate = W.calibrate_gate(inp, 0.3, sample_images=None)
    for dtype in (F, H):
        if dtype in forms:
            _say(P.run_float(inp, gate, in_dtype=dtype, out_dtype=dtype, shuffle=grouped, name="%s %s" % (shape.name, forms[dtype])))
    if I in forms:
        q = W.quantize_int8(W.make_inputs(shape, 7600 + shape.c_out + shape.h, kind="iid", rho=0.35, grouped=grouped))
        thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
        _say(P.run_int8(q, thr, shuffle=grouped, name="%s int8 %s" % (shape.name, forms[I])))


# Dense layers, (images, height, width, channels in and out, kernel), with the tile and the wavefronts that share its K, and the roundings that a product
# passes through, in roundings of the last sum: a chain of m additions makes (m + 1) / 2.  Sums of eight wavefronts are added up in
# pairs, 3; of four, 2.
def _chain(m):
    return (m + 1) / 2


SUMS = [
    (H, (261, 20, 8, 752, 40, 1), (1, 4, 1), _chain(23.5 / 2) + 1),                          # whole: even and odd steps by themselves
    (H, (22, 25, 38, 1424, 80, 1), (2, 2, 1), _chain(44.5 / 2) + 1),
    (H, (30, 40, 24, 1376, 72, 1), (2, 4, 1), _chain(43 / 2) + 1),
    (H, (1, 57, 18, 2032, 64, 3), (1, 2, 8), _chain(2) + 1 + _chain(571.5 / 8 / 4) + 3),     # two blocks of two steps at a time
    (H, (1, 44, 41, 560, 280, 3), (1, 2, 4), _chain(2) + 1 + _chain(157.5 / 4 / 4) + 2),
    (H, (7, 41, 19, 768, 328, 1), (1, 4, 4), _chain(2) + _chain(24 / 4 / 2) + 2),            # blocks of two steps
    (H, (24, 25, 21, 352, 88, 3), (2, 2, 4), _chain(2) + _chain(99 / 4 / 2) + 2),
    (H, (2, 33, 8, 272, 1800, 1), (2, 4, 8), _chain(8.5 / 8 + 1) + 3),                       # a chain to a wavefront
    (F, (10, 10, 25, 80, 392, 3), (1, 2, 2), _chain(8) + 1 + _chain(45 / 2 / 4) + 1),        # (fp32: four products to a step)
    (F, (1, 22, 53, 768, 440, 3), (1, 4, 8), _chain(8) + _chain(432 / 8 / 2) + 3),
    (F, (5, 46, 18, 560, 184, 3), (2, 2, 4), _chain(8) + _chain(315 / 4 / 2) + 2),
    (F, (3, 47, 35, 496, 136, 3), (2, 4, 8), _chain(279 / 8 * 4) + 3),
    (F, (7, 55, 18, 128, 432, 3), (1, 4, 1), _chain(8) + _chain(72 / 2)),
    (F, (11, 49, 54, 144, 48, 3), (2, 2, 1), _chain(8) + _chain(81 / 2)),
]


@pytest.mark.parametrize("dtype,shape,form,roundings", SUMS, ids=["%s_%s" % ({F: "fp32", H: "bf16"}[d], "_".join(map(str, f))) for d, _, f, _ in SUMS])
def test_sums_of_every_form_against_64_bits(dtype, shape, form, roundings):
    """The error of a layer's sums, in the rms, is at most that of the roundings: 0.58 * 2^-24 of the sum each, a 15th more for what a product of 32
    bf16 pairs rounds inside, which adds at most a seventh to the variance of one chain over K (measured: 24 to 25 for 22 of 44.5 and 43 steps)."""
    n, h, w_, c, co, k = shape
    g = torch.Generator(device="cuda").manual_seed(c + co)
    tdt = torch.float32 if dtype == F else torch.bfloat16
    x = torch.relu(torch.randn(n, h, w_, c, generator=g, device="cuda")).to(tdt)
    w = (torch.randn(co, k, k, c, generator=g, device="cuda") * (2.0 / (k * k * c)) ** 0.5).to(tdt)
    layer = B.GatedConv(n_max=n, h=h, w=w_, c_in=c, c_out=co, c_base=c, w_base=w, w_cond=None, in_dtype=dtype, out_dtype=F, kh=k, kw=k, stride=1, pad=k // 2,
                        epilogue=0)
    y = layer.forward(x, bitmap=False, counts=False)[0].double().reshape(-1, co)
    layer.close()
    cols = x.double().permute(0, 3, 1, 2)
    cols = torch.nn.functional.unfold(cols, k, padding=k // 2).transpose(1, 2).reshape(-1, c * k * k)
    ref = cols @ w.double().permute(0, 3, 1, 2).reshape(co, -1).T
    rms = (y - ref).pow(2).mean().sqrt().item()
    bound = 0.58 * 2.0 ** -24 * (1.14 * roundings) ** 0.5 * ref.pow(2).mean().sqrt().item()
    print("%s: %.3g of %.3g" % (shape, rms, bound))
    assert rms <= bound


@pytest.mark.parametrize("dtype,shape", [("f32", (1, 20, 512, 256, 2)), ("f32", (1, 9, 128, 80, 1)), ("bf16", (1, 14, 512, 64, 1)),
                                         ("bf16", (4, 4, 512, 128, 1))])
def test_sums_of_a_split_against_64_bits(dtype, shape):
    """A deep dense layer of few pixels, tiles of 16 x 16: K is split over eight wavefronts, each adding up blocks of four K steps, of
    which the even and the odd ones have a sum of their own.

    A rounding is at most 2^-24 of the sum it makes and 0.58 of that in the rms.  On its way a product passes through those of
    its half block (two steps; fp32: four products each), of the wavefront's blocks and of the eight wavefronts' sums, none of which
    is larger than the result in the rms.  (As one chain to a wavefront the fp32 errors were 1.3 and 2.4 times the bound.)"""
    n, h, c, co, s = shape
    g = torch.Generator().manual_seed(c + co)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.randn(n, h, h, c, generator=g).to(tdt)
    w = (torch.randn(co, 3, 3, c, generator=g) / (9 * c) ** 0.5).to(tdt)
    layer = B.GatedConv(n_max=n, h=h, w=h, c_in=c, c_out=co, c_base=c, w_base=w.cuda(), w_cond=None,
                        in_dtype=B.CG_F32 if dtype == "f32" else B.CG_BF16, out_dtype=B.CG_F32, kh=3, kw=3, stride=s, pad=1, epilogue=0)
    y = layer.forward(x.cuda(), bitmap=False, counts=False)[0].cpu().double()
    ref = torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), w.double().permute(0, 3, 1, 2), stride=s, padding=1).permute(0, 2, 3, 1)
    steps = 9 * c // (16 if dtype == "f32" else 32)                  # K steps of the layer
    roundings = (8 if dtype == "f32" else 2) + -(-steps // 32) + 8
    rms = (y - ref).pow(2).mean().sqrt().item()
    bound = 0.58 * 2.0 ** -24 * roundings ** 0.5 * ref.pow(2).mean().sqrt().item()
    print("%s %s: %.3g of %.3g" % (dtype, shape, rms, bound))
    assert rms <= bound


@pytest.mark.parametrize("shape,chain,sums", [
    ((67, 42, 45, 192, 64, 1, 2, 4), 8, 5), ((27, 30, 31, 128, 64, 1, 1, 4), 8, 3), ((1011, 1, 1, 256, 1664, 1, 1, 8), 8, 7),
    ((23, 27, 27, 32, 80, 3, 1, 2), 8, 5), ((89, 11, 11, 128, 256, 3, 2, 2), 36, 4)],
    ids=["whole_192>64s2", "whole_128>64", "whole_fc", "whole_3x3", "split_of_eight_units"])
def test_sums_of_gated_fp32_layers_against_64_bits(shape, chain, sums):
    """The whole form adds up blocks of two K steps (eight 16x16x4 products); a split's tiles of eight units take a wavefront's share in
    one chain (nine steps here).

    A rounding is at most 2^-24 of the sum it makes and 0.58 of that in the rms.  In a chain of m additions of equal terms the sum grows with
    them, so that they come to (m + 1) / 2 roundings of the last sum: those of a block, of the `sums` blocks or wavefronts of the
    conditional path, and one for base and conditional sum.  (With one chain over K the whole form's errors were 1.45, 1.20, 1.71 and 1.52 times the bound.)"""
    n, h, w_, c, co, k, s, groups = shape
    cb = c // groups
    g = torch.Generator().manual_seed(c + co)
    x = torch.relu(torch.randn(n, h, w_, c, generator=g))
    w = torch.randn(co, k, k, c, generator=g) * (2.0 / (k * k * c)) ** 0.5
    layer = B.GatedConv(n_max=n, h=h, w=w_, c_in=c, c_out=co, c_base=cb, w_base=w[..., :cb].contiguous().cuda(), w_cond=w[..., cb:].contiguous().cuda(),
                        in_dtype=B.CG_F32, out_dtype=B.CG_F32, kh=k, kw=k, stride=s, pad=k // 2, epilogue=0, gate_mean=np.zeros(co),
                        gate_var=np.ones(co), delta=np.full(co, -np.inf))
    y = layer.forward(x.cuda(), bitmap=False, counts=False)[0].cpu().double()
    layer.close()
    ref = torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), w.double().permute(0, 3, 1, 2), stride=s, padding=k // 2).permute(0, 2, 3, 1)
    rms = (y - ref).pow(2).mean().sqrt().item()
    bound = 0.58 * 2.0 ** -24 * ((chain + 1) / 2 + (sums + 1) / 2 + 1) ** 0.5 * ref.pow(2).mean().sqrt().item()
    print("%s: %.3g of %.3g" % (shape, rms, bound))
    assert rms <= bound
