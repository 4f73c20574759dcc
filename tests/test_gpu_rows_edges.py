"""Edge cases of the row-tiled matrix-core kernel through the C ABI: partial batches, a large batch,
wide images, an input whose pixels are further apart than c_in, repeated calls."""
import numpy as np
import pytest
import torch

from oracle import cg_oracle as O
from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def _say(rep):
    print("\n  " + str(rep), flush=True)
    return rep


@pytest.mark.parametrize("shape,n_run", [
    (W.LayerShape("pb_256@14", 5, 14, 14, 256, 256), 3),       # tiles straddle images, last tile ragged
    (W.LayerShape("pb_512@7", 9, 7, 7, 512, 512), 1),          # one image of nine
    (W.LayerShape("pb_128@28", 4, 28, 28, 128, 128), 3),
])
def test_partial_batch(shape, n_run):
    inp = W.make_inputs(shape, 8000 + shape.c_out, kind="coherent", rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.30, sample_images=None)
    rep = _say(P.run_float(inp, gate, n_run=n_run, name="%s n=%d of %d" % (shape.name, n_run, shape.n)))
    assert rep.variant == B.CG_VARIANT_MFMA_ROWS
    q = W.quantize_int8(W.make_inputs(shape, 8100 + shape.c_out, kind="coherent", rho=0.35))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    _say(P.run_int8(q, thr, n_run=n_run, name="%s int8 n=%d" % (shape.name, n_run)))


def test_large_batch_and_wide_image():
    for shape in (W.LayerShape("big_128@28", 256, 28, 28, 128, 128), W.LayerShape("wide_64@112", 4, 112, 112, 64, 64),
                  W.LayerShape("tall_64", 2, 150, 20, 64, 128)):
        inp = W.make_inputs(shape, 8200 + shape.h, kind="coherent", rho=0.3, round_bf16=True)
        gate = W.calibrate_gate(inp, 0.30, sample_images=4)
        rep = _say(P.run_float(inp, gate, out_dtype=B.CG_BF16, name=shape.name))
        assert rep.variant == B.CG_VARIANT_MFMA_ROWS


def test_strided_input_pixels_and_repeatability():
    """x lives in a buffer with 160 elements per pixel of which the first 128 are the layer's channels."""
    shape = W.LayerShape("strided_128@14", 3, 14, 14, 128, 128)
    inp = W.make_inputs(shape, 8300, kind="coherent", rho=0.3, round_bf16=True)
    gate = W.calibrate_gate(inp, 0.30, sample_images=None)
    wide = torch.full((3, 14, 14, 160), 7.0, dtype=torch.bfloat16, device="cuda")
    wide[..., :128] = torch.from_numpy(inp.x).cuda().to(torch.bfloat16)
    layer = B.GatedConv(n_max=3, h=14, w=14, c_in=128, c_out=128, c_base=32, x_pixel_stride=160,
                        w_base=torch.from_numpy(inp.w_base).cuda().to(torch.bfloat16),
                        w_cond=torch.from_numpy(inp.w_cond).cuda().to(torch.bfloat16), in_dtype=B.CG_BF16,
                        out_dtype=B.CG_F32, gate_mean=gate.mean, gate_var=gate.var, delta=gate.delta)
    assert layer.variant == B.CG_VARIANT_MFMA_ROWS
    a = [t.clone() for t in layer.forward(wide)]
    b = layer.forward(wide)
    torch.cuda.synchronize()
    for u, v in zip(a, b):
        assert torch.equal(u, v)
    f32 = lambda v: np.asarray(v, np.float32).astype(np.float64)
    ref = O.forward_float(inp.x, inp.w_base, inp.w_cond, gate_mean=f32(gate.mean), gate_var=f32(gate.var),
                          delta=f32(gate.delta), want_partials=False)
    _say(P.compare_float("strided input", a[0].cpu().numpy().astype(np.float64), a[1].cpu().numpy().view(np.uint32),
                         a[2].cpu().numpy().view(np.uint32), ref, 128, B.CG_F32, layer.variant))
    layer.close()


# More output channels than a tile's outputs have 32-bit offsets for, and as many as they just do: (type, output type, channels, shuffled, the kernel's
# form, which tests/test_kernels_of_calls_cpu.py checks).
F, H, I = B.CG_F32, B.CG_BF16, B.CG_I8
MANY_CHANNELS = [(H, H, (1 << 20) + 128, False, "1"), (H, H, (1 << 20) + 128, True, "3"), (H, F, (1 << 20) + 128, False, "5"), (H, F, (1 << 21) + 128, False, "4"),
                 (H, H, (1 << 22) + 512, False, "4"), (H, H, (1 << 22) + 512, True, "4"), (I, I, (1 << 20) + 128, False, "1")]


@pytest.mark.parametrize("dtype,out,c,shuffle,form", MANY_CHANNELS, ids=["%d_%d_%d_%s" % (d, o, c, f) for d, o, c, _, f in MANY_CHANNELS])
def test_many_output_channels(dtype, out, c, shuffle, form):
    """Small whole numbers against the plain kernel: equal."""
    g = torch.Generator(device="cuda").manual_seed(c)
    tdt = torch.int8 if dtype == I else torch.bfloat16
    odt = {F: torch.float32, H: torch.bfloat16, I: torch.int8}[out]
    x = torch.randint(0, 4, (1, 2, 2, 32), generator=g, device="cuda", dtype=torch.int8).to(tdt)
    w_b, w_c = (torch.randint(-2, 3, (c, 3, 3, 16), generator=g, device="cuda", dtype=torch.int8).to(tdt) for _ in range(2))
    res = torch.randint(-9, 10, (1, 2, 2, c), generator=g, device="cuda", dtype=torch.int8).to(odt)
    kw = dict(gate_thr_i32=np.full(c, 5, np.int32), rq_mult0=3, rq_mult1=2, rq_shift=8, rq_res_mult=100) if dtype == I else dict(
        gate_mean=np.zeros(c), gate_var=np.ones(c), delta=np.full(c, 5.0))
    got = []
    for variant in (B.CG_VARIANT_MFMA_ROWS, B.CG_VARIANT_NAIVE):
        layer = B.GatedConv(n_max=1, h=2, w=2, c_in=32, c_out=c, c_base=16, w_base=w_b, w_cond=w_c, in_dtype=dtype, out_dtype=out, variant=variant,
                            epilogue=B.CG_EPI_RELU | (0 if shuffle else B.CG_EPI_RESIDUAL), **kw, **(dict(groups=2, shuffle=True) if shuffle else {}))
        assert layer.variant == variant
        got.append(layer.forward(x, residual=None if shuffle else res))
        torch.cuda.synchronize()
        layer.close()
    assert all(torch.equal(a, b) for a, b in zip(*got)) and int(got[0][2][0]) > c
