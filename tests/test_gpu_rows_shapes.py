"""GPU parity of the row-tiled matrix-core kernel at the edges of its tiles: every fragment shape, tiles that end inside an
image or an image row, weights that stay in LDS or stream, the shuffled store, one and two fragments per wavefront."""
import numpy as np
import pytest
import torch

from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import workloads as W
from tests import parity as P
from tests.test_gpu_requantise import fits_32_bits

pytestmark = pytest.mark.gpu


def S(n, h, w, ci, co, **kw):
    return W.LayerShape("%dx%dx%d_%d>%d" % (n, h, w, ci, co) + "".join("_%s%d" % i for i in sorted(kw.items())), n, h, w, ci, co, **kw)


SHAPES = [
    S(1, 3, 3, 64, 64),                        # one fragment, most of it past the image
    S(3, 5, 250, 64, 64),                      # the widest rows
    S(2, 20, 33, 64, 64),                      # last fragment of a row holds one column
    S(5, 14, 14, 256, 256),
    S(7, 27, 27, 192, 192),
    S(2, 31, 9, 128, 64, stride=2),
    S(4, 17, 40, 128, 128, groups=2),          # channel groups: a block inside one
    S(3, 13, 21, 128, 128, groups=8),          # a block of several
    S(130, 14, 14, 256, 256),                  # several tiles per workgroup that straddle images
    S(100, 14, 14, 256, 256),                  # two fragments per wavefront, in runs of 32 pixels
    S(30, 14, 14, 256, 1024),                  # the same, more channel blocks
    S(16, 28, 28, 384, 384),                   # the same in fragments of 4 x 8 pixels
]


@pytest.mark.parametrize("shape", SHAPES, ids=[s.name for s in SHAPES])
def test_rows_kernel_shapes(shape):
    rng = np.random.default_rng(shape.n * 11 + shape.c_out)
    c, big = shape.c_out, shape.n * shape.h * shape.w > 5000
    aff = dict(scale0=rng.uniform(0.5, 1.5, c), shift0=rng.normal(0, 0.1, c),
               scale1=rng.uniform(0.5, 1.5, c), shift1=rng.normal(0, 0.1, c))
    res = rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32)
    full = B.CG_EPI_RELU | B.CG_EPI_AFFINE | B.CG_EPI_RESIDUAL
    inp = W.make_inputs(shape, 9000 + c + shape.h, kind="coherent", rho=0.3, round_bf16=True, grouped=shape.groups != 4)
    gate = W.calibrate_gate(inp, 0.3, sample_images=2)
    kw = dict(variant=B.CG_VARIANT_MFMA_ROWS)
    runs = [dict(out_dtype=B.CG_BF16, affine=aff, residual=res, epilogue=full, n_run=max(1, shape.n - 1))]
    if not big:
        runs += [dict(out_dtype=B.CG_BF16, affine=aff, epilogue=full & ~B.CG_EPI_RESIDUAL, shuffle=inp.grouped),
                 dict(out_dtype=B.CG_F32, delta_hi=gate.delta + 0.8)]
    for r in runs:
        print("\n  " + str(P.run_float(inp, gate, name=shape.name, **kw, **r)), flush=True)
    if not big:
        q = W.quantize_int8(W.make_inputs(shape, 9100 + c + shape.h, kind="coherent", rho=0.35, grouped=inp.grouped))
        thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
        print("  " + str(P.run_int8(q, thr, name=shape.name + " int8", **kw)), flush=True)


POINT = [
    S(24, 14, 14, 256, 512, k=1, pad=0),
    S(23, 13, 11, 512, 1024, k=1, pad=0),               # last tile ends inside a fragment
    S(70, 16, 16, 256, 64, k=1, pad=0),                 # weights stay in LDS
    S(20, 15, 15, 256, 512, k=1, pad=0, groups=2),      # channel groups: a block inside one
    S(20, 15, 15, 512, 256, k=1, pad=0, groups=8),      # a block of several
]


@pytest.mark.parametrize("shape", POINT, ids=[s.name for s in POINT])
def test_point_wise_shapes(shape):
    rng = np.random.default_rng(shape.n * 13 + shape.c_out)
    c = shape.c_out
    aff = dict(scale0=rng.uniform(0.5, 1.5, c), shift0=rng.normal(0, 0.1, c),
               scale1=rng.uniform(0.5, 1.5, c), shift1=rng.normal(0, 0.1, c))
    res = rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32)
    full = B.CG_EPI_RELU | B.CG_EPI_AFFINE | B.CG_EPI_RESIDUAL
    inp = W.make_inputs(shape, 9400 + c + shape.h, kind="coherent", rho=0.3, round_bf16=True, grouped=shape.groups != 4)
    gate = W.calibrate_gate(inp, 0.3, sample_images=2)
    for r in (dict(out_dtype=B.CG_BF16, affine=aff, residual=res, epilogue=full, n_run=shape.n - 1),
              dict(out_dtype=B.CG_BF16, affine=aff, epilogue=full & ~B.CG_EPI_RESIDUAL, shuffle=inp.grouped),
              dict(out_dtype=B.CG_F32, tau_c=0.3)):
        print("\n  " + str(P.run_float(inp, gate, name=shape.name, **r)), flush=True)
    q = W.quantize_int8(W.make_inputs(shape, 9500 + c + shape.h, kind="coherent", rho=0.35, grouped=inp.grouped))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    print("  " + str(P.run_int8(q, thr, name=shape.name + " int8")), flush=True)


@pytest.mark.parametrize("n", [100, 130], ids=["two_fragments", "one_fragment"])
def test_residual_may_be_the_output(n):
    """y written over the residual (two fragments per wavefront write y twice, which that must not see)."""
    shape = S(n, 14, 14, 256, 256)
    inp = W.make_inputs(shape, 9300, kind="coherent", rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.3, sample_images=2)
    bf = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16)
    layer = B.GatedConv(n_max=shape.n, h=14, w=14, c_in=256, c_out=256, c_base=inp.w_base.shape[-1], w_base=bf(inp.w_base),
                        w_cond=bf(inp.w_cond), in_dtype=B.CG_BF16, out_dtype=B.CG_BF16,
                        epilogue=B.CG_EPI_RELU | B.CG_EPI_RESIDUAL, gate_mean=gate.mean, gate_var=gate.var, delta=gate.delta)
    x = bf(inp.x)
    res = torch.randn(shape.n, 14, 14, 256, device="cuda").to(torch.bfloat16)
    y, bits, counts = [t.clone() for t in layer.forward(x, residual=res)]
    over = res.clone()
    _, bits2, counts2 = layer.forward(x, residual=over, y=over)
    torch.cuda.synchronize()
    layer.close()
    assert torch.equal(y, over) and torch.equal(bits, bits2) and torch.equal(counts, counts2)


@pytest.mark.parametrize("n", [2048, 1900, 5], ids=["large_tile", "row_tiled", "small_tile"])
def test_dense_deep_point_wise_layers(n):
    """A dense bf16 layer of 2048 channels runs on three kernels, by the batch: whole rounds of large tiles, others, few pixels."""
    shape = S(2048, 1, 1, 2048, 1024, k=1, pad=0, groups=1)
    inp = W.make_inputs(shape, 9800, kind="iid", round_bf16=True)
    rng = np.random.default_rng(98)
    aff = dict(scale0=rng.uniform(0.5, 1.5, 1024), shift0=rng.normal(0, 0.1, 1024), scale1=rng.uniform(0.5, 1.5, 1024),
               shift1=rng.normal(0, 0.1, 1024))
    print("\n  " + str(P.run_float(inp, None, out_dtype=B.CG_BF16, affine=aff, epilogue=B.CG_EPI_RELU | B.CG_EPI_AFFINE, n_run=n,
                                    name=shape.name)), flush=True)


@pytest.mark.parametrize("pairs", ["equal", "differ_in_one_shift", "none"])
def test_one_scale_shift_pair(pairs):
    """Fragments that take one pair throughout: nothing fired, a dense layer, equal pairs, no scale/shift at all."""
    rng = np.random.default_rng(5)
    c = 128
    scale, shift = rng.uniform(0.5, 1.5, c), rng.normal(0, 0.1, c)
    other = shift.copy()
    other[c - 1] += 0.0 if pairs == "equal" else 0.5
    aff = None if pairs == "none" else dict(scale0=scale, shift0=shift, scale1=scale, shift1=other)
    epi = B.CG_EPI_RELU | (0 if aff is None else B.CG_EPI_AFFINE)
    for groups in (4, 1):
        inp = W.make_inputs(S(3, 13, 18, c, c, groups=groups), 8800, kind="coherent", rho=0.3, round_bf16=True)
        gate = W.calibrate_gate(inp, 0.3, sample_images=None) if groups > 1 else None
        rep = P.run_float(inp, gate, out_dtype=B.CG_BF16, affine=aff, epilogue=epi, variant=B.CG_VARIANT_MFMA_ROWS, name=pairs)
        assert rep.variant == B.CG_VARIANT_MFMA_ROWS


PAIRED = [
    S(128, 8, 8, 256, 256),                    # full fragments of four rows
    S(40, 7, 7, 512, 512),                     # runs of 32 pixels over five rows and images, stages of four chunks
    S(2, 3, 4, 64, 128),                       # part of one fragment
    S(9, 13, 13, 64, 192),
    S(3, 17, 31, 128, 128),                    # the widest rows whose number goes into the chunk permutation
    S(3, 12, 33, 64, 64),                      # fragments of eight columns or runs, the fixed permutation
    S(11, 17, 15, 64, 128, stride=2),
    S(6, 12, 18, 64, 128, groups=1),           # dense
]


@pytest.mark.parametrize("shape", PAIRED, ids=[s.name for s in PAIRED])
def test_two_wavefronts_to_a_fragment(shape):
    """Tiles of at most four fragments: each wavefront has 32 of the block's 64 channels.  Every gate and output option."""
    c, full = shape.c_out, B.CG_EPI_RELU | B.CG_EPI_AFFINE | B.CG_EPI_RESIDUAL
    rng = np.random.default_rng(c + shape.w)
    aff = dict(scale0=rng.uniform(0.5, 1.5, c), shift0=rng.normal(0, 0.1, c), scale1=rng.uniform(0.5, 1.5, c), shift1=rng.normal(0, 0.1, c))
    res = rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32)
    inp = W.make_inputs(shape, 9600 + shape.h, kind="coherent", rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.3, sample_images=2) if shape.groups > 1 else None
    runs = [dict(epilogue=B.CG_EPI_RELU), dict(affine=aff, residual=res, epilogue=full, n_run=max(1, shape.n - 1))]
    if gate:
        runs += [dict(affine=aff, epilogue=full & ~B.CG_EPI_RESIDUAL, delta_hi=gate.delta + 0.8), dict(epilogue=0, tau_c=0.3)]
    for r in runs:
        rep = P.run_float(inp, gate, out_dtype=B.CG_BF16, variant=B.CG_VARIANT_MFMA_ROWS, name=shape.name, **r)
        assert rep.variant == B.CG_VARIANT_MFMA_ROWS
    if not gate or c * shape.n > 12000:
        return
    q = W.quantize_int8(W.make_inputs(shape, 9700 + shape.h, kind="coherent", rho=0.35))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    r8 = rng.integers(-128, 128, (shape.n, shape.ho, shape.wo, c)).astype(np.int8)
    for lo, hi, shift, fits in ((-200, 200, 14, False), (-(1 << 20), 1 << 20, 24, False), (20, 200, 14, True)):      # in 64 bits and in 32
        rq = dict(rq_mult0=rng.integers(lo, hi, c).astype(np.int32), rq_mult1=rng.integers(lo, hi, c).astype(np.int32),
                  rq_bias=rng.integers(-hi, hi, c).astype(np.int32), rq_shift=shift)
        assert fits_32_bits(rq, hi // 2, True) == fits_32_bits(rq, 0, False) == fits
        P.run_int8(q, thr, out_i8=True, rq=rq, epilogue=B.CG_EPI_RELU, variant=B.CG_VARIANT_MFMA_ROWS, name=shape.name)
        P.run_int8(q, thr, out_i8=True, rq=rq, residual=r8, rq_res_mult=hi // 2, epilogue=B.CG_EPI_RESIDUAL, variant=B.CG_VARIANT_MFMA_ROWS,
                   name=shape.name)


# (the first four: two wavefronts to a fragment; the next three: one, stages of two chunks and of four)
ENDS = [S(6, 9, 13, 64, 64), S(40, 14, 14, 256, 256), S(16, 20, 20, 128, 128), S(3, 30, 70, 64, 192, stride=2),
        S(2, 6, 141, 128, 64), S(31, 18, 45, 64, 64, groups=2), S(17, 33, 44, 128, 64, groups=2), S(23, 13, 11, 512, 1024, k=1, pad=0)]


@pytest.mark.parametrize("one_pair", [False, True])
@pytest.mark.parametrize("shape", ENDS, ids=[s.name for s in ENDS])
def test_outputs_with_and_without_scale_shift_and_residual(shape, one_pair):
    """Each way through the end of a tile: no scale/shift, one pair, a pair by each decision; with and without a residual; one and two wavefronts to
    a fragment (tests/test_kernels_of_calls_cpu.py checks the forms); tiles whose last fragment has lanes without a pixel, whose places must neither be
    read nor written."""
    c, rng = shape.c_out, np.random.default_rng(shape.h)
    pair = [rng.uniform(0.5, 1.5, c), rng.normal(0, 0.1, c)]
    other = pair if one_pair else [rng.uniform(0.5, 1.5, c), rng.normal(0, 0.1, c)]
    aff = dict(scale0=pair[0], shift0=pair[1], scale1=other[0], shift1=other[1])
    res = rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32)
    inp = W.make_inputs(shape, 9800 + shape.h, kind="coherent", rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.3, sample_images=2)
    relu, scaled, added = B.CG_EPI_RELU, B.CG_EPI_AFFINE, B.CG_EPI_RESIDUAL
    for epi in (scaled, scaled | added | relu) if one_pair else (0, added, scaled | relu, scaled | added):
        more = dict(residual=res) if epi & added else {}
        if epi & scaled:
            more["affine"] = aff
        if shape.k == 3:                       # (1x1 layers choose it by themselves)
            more["variant"] = B.CG_VARIANT_MFMA_ROWS
        P.run_float(inp, gate, out_dtype=B.CG_BF16, epilogue=epi, n_run=max(1, shape.n - 1), name=shape.name, **more)


@pytest.mark.parametrize("shape", ENDS, ids=[s.name for s in ENDS])
def test_outputs_of_four_bytes(shape):
    """Float and 32-bit outputs, 16 channels of a pixel by four lanes: the same ways through the end, and sums that a residual
    takes past 32 bits either way (the sums of 64 to 512 channels times nine taps stay below 2^27, residuals go to 2^32), with ReLU too."""
    c, rng = shape.c_out, np.random.default_rng(shape.w)
    aff = dict(scale0=rng.uniform(0.5, 1.5, c), shift0=rng.normal(0, 0.1, c), scale1=rng.uniform(0.5, 1.5, c), shift1=rng.normal(0, 0.1, c))
    one = dict(aff, scale1=aff["scale0"], shift1=aff["shift0"])
    res = rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32)
    inp = W.make_inputs(shape, 9900 + shape.h, kind="coherent", rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.3, sample_images=2)
    relu, scaled, added, n = B.CG_EPI_RELU, B.CG_EPI_AFFINE, B.CG_EPI_RESIDUAL, max(1, shape.n - 1)
    rows = dict(variant=B.CG_VARIANT_MFMA_ROWS) if shape.k == 3 else {}
    for epi, more in ((0, {}), (added, dict(residual=res)), (scaled | relu, dict(affine=aff)), (scaled | added, dict(affine=aff, residual=res)),
                      (scaled | added | relu, dict(affine=one, residual=res))):
        P.run_float(inp, gate, epilogue=epi, n_run=n, name=shape.name, **more, **rows)
    q = W.quantize_int8(W.make_inputs(shape, 9950 + shape.h, kind="coherent", rho=0.35))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    r8 = rng.integers(-128, 128, (shape.n, shape.ho, shape.wo, c)).astype(np.int8)
    for epi, more in ((relu, {}), (added, dict(residual=r8, rq_res_mult=-(1 << 25))), (added | relu, dict(residual=r8, rq_res_mult=1 << 25))):
        P.run_int8(q, thr, epilogue=epi, n_run=n, name=shape.name, **more, **rows)


@pytest.mark.parametrize("shape", ENDS, ids=[s.name for s in ENDS])
def test_int8_outputs_with_and_without_residual(shape):
    c, rng = shape.c_out, np.random.default_rng(shape.n)
    q = W.quantize_int8(W.make_inputs(shape, 9960 + shape.h, kind="coherent", rho=0.35))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    r8 = rng.integers(-128, 128, (shape.n, shape.ho, shape.wo, c)).astype(np.int8)
    rows = dict(variant=B.CG_VARIANT_MFMA_ROWS) if shape.k == 3 else {}
    for lo, hi, shift, fits in ((-200, 200, 14, False), (20, 200, 14, True)):      # in 64 bits and in 32
        rq = dict(rq_mult0=rng.integers(lo, hi, c).astype(np.int32), rq_mult1=rng.integers(lo, hi, c).astype(np.int32),
                  rq_bias=rng.integers(-hi, hi, c).astype(np.int32), rq_shift=shift)
        assert fits_32_bits(rq, hi // 2, True) == fits_32_bits(rq, 0, False) == fits
        P.run_int8(q, thr, out_i8=True, rq=rq, epilogue=B.CG_EPI_RELU, n_run=max(1, shape.n - 1), name=shape.name, **rows)
        P.run_int8(q, thr, out_i8=True, rq=rq, residual=r8, rq_res_mult=hi // 2, epilogue=B.CG_EPI_RESIDUAL, n_run=max(1, shape.n - 1), name=shape.name, **rows)


# 1x1 layers of several tiles to a workgroup, whose stages the loading wavefronts take in turn: stages of eight chunks (four buffers) and of four,
# weights that stay in LDS and stages of two (eight buffers), the last tile shorter than the others, gates that hardly ever fire (stages passed by before they land).
IN_TURN = [
    (S(43, 14, 14, 1024, 1024, k=1, pad=0), 0.3, False), (S(43, 14, 14, 1024, 1024, k=1, pad=0), 0.01, False), (S(43, 14, 14, 1024, 1024, k=1, pad=0), 0.3, True),
    (S(61, 25, 25, 192, 128, k=1, pad=0), 0.3, False), (S(117, 25, 25, 192, 128, k=1, pad=0), 0.01, False), (S(29, 13, 13, 384, 1024, k=1, pad=0), 0.3, False),
    (S(19, 16, 16, 384, 1024, k=1, pad=0), 0.02, True)]


@pytest.mark.parametrize("shape,rho,grouped", IN_TURN, ids=["%s_%g_%d" % (s.name, r, g) for s, r, g in IN_TURN])
def test_point_wise_stages_in_turn(shape, rho, grouped):
    inp = W.make_inputs(shape, 9600 + shape.c_in, kind="coherent", rho=rho, round_bf16=True, grouped=grouped)
    gate = W.calibrate_gate(inp, rho, sample_images=2)
    print("\n  " + str(P.run_float(inp, gate, name=shape.name, out_dtype=B.CG_BF16, epilogue=B.CG_EPI_RELU)), flush=True)


def test_point_wise_stages_in_turn_int8():
    shape = S(29, 13, 13, 768, 1024, k=1, pad=0)
    q = W.quantize_int8(W.make_inputs(shape, 9650, kind="coherent", rho=0.3))
    thr = W.calibrate_gate_int8(q, 0.3, sample_images=None)
    print("\n  " + str(P.run_int8(q, thr, name=shape.name + " int8")), flush=True)


# The same with other outputs, whose kernels are others: two-byte outputs beside a residual (stages of two, four and eight chunks), in shuffled order, of four
# bytes, int8 ones of a shift below two; (shape, what is asked for, the form in test_kernels_of_calls_cpu.py).
IN_TURN_OUTPUTS = [
    (S(61, 25, 25, 192, 128, k=1, pad=0), "residual", 2, 14), (S(29, 13, 13, 384, 1024, k=1, pad=0), "residual", 4, 14), (S(43, 14, 14, 1024, 1024, k=1, pad=0), "residual", 8, 14),
    (S(83, 25, 25, 192, 128, k=1, pad=0), "shuffled", 4, 11), (S(61, 25, 25, 192, 128, k=1, pad=0), "float", 2, 13), (S(61, 25, 25, 192, 128, k=1, pad=0), "tau", 2, 8),
    (S(106, 14, 14, 512, 1024, k=1, pad=0), "residual", 8, 6), (S(106, 14, 14, 512, 1024, k=1, pad=0), "natural", 8, 0)]     # (eight stages, four buffers: not in turn)
IN_TURN_INT8 = [("bytes", 8), ("residual", 14), ("shift of one", 12), ("32 bits, residual", 13)]


@pytest.mark.parametrize("shape,what", [(s, w) for s, w, _, _ in IN_TURN_OUTPUTS], ids=["%s_%s" % (s.name, w) for s, w, _, _ in IN_TURN_OUTPUTS])
def test_point_wise_stages_in_turn_outputs(shape, what):
    c, rng = shape.c_out, np.random.default_rng(shape.n)
    inp = W.make_inputs(shape, 9660 + shape.c_in, kind="coherent", rho=0.3, round_bf16=True, grouped=what == "shuffled")
    gate = W.calibrate_gate(inp, 0.3, sample_images=2)
    aff = dict(scale0=rng.uniform(0.5, 1.5, c), shift0=rng.normal(0, 0.1, c), scale1=rng.uniform(0.5, 1.5, c), shift1=rng.normal(0, 0.1, c))
    more = dict(out_dtype=B.CG_F32 if what == "float" else B.CG_BF16, epilogue=B.CG_EPI_RELU | B.CG_EPI_AFFINE, affine=aff, shuffle=what == "shuffled")
    if what == "residual":
        more.update(epilogue=more["epilogue"] | B.CG_EPI_RESIDUAL, residual=rng.standard_normal((shape.n, shape.ho, shape.wo, c)).astype(np.float32))
    if what == "tau":
        more.update(tau_c=0.3)
    print("\n  " + str(P.run_float(inp, gate, name=shape.name, **more)), flush=True)


@pytest.mark.parametrize("what", [w for w, _ in IN_TURN_INT8])
def test_point_wise_stages_in_turn_int8_outputs(what):
    shape = S(29, 13, 13, 768, 1024, k=1, pad=0)
    c, rng = shape.c_out, np.random.default_rng(77)
    q = W.quantize_int8(W.make_inputs(shape, 9651, kind="coherent", rho=0.3))
    thr = W.calibrate_gate_int8(q, 0.3, sample_images=None)
    r8 = rng.integers(-128, 128, (shape.n, shape.ho, shape.wo, c)).astype(np.int8)
    shift = 1 if what == "shift of one" else 14
    rq = dict(rq_mult0=rng.integers(20, 200, c).astype(np.int32), rq_mult1=rng.integers(20, 200, c).astype(np.int32), rq_bias=rng.integers(-200, 200, c).astype(np.int32),
              rq_shift=shift)
    more = dict(out_i8=True, rq=rq) if what != "32 bits, residual" else {}
    if "residual" in what:
        more.update(residual=r8, rq_res_mult=100, epilogue=B.CG_EPI_RESIDUAL)
    print("\n  " + str(P.run_int8(q, thr, name=shape.name + " int8", **more)), flush=True)
