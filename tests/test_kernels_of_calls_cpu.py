"""That the layers of the GPU tests run on the kernels, and in the forms, which those tests are there for: the choice of kernel and plan is the
library's own, asked for through forward calls without a GPU."""
import itertools

import pytest

from paper_1805_12549_amd import binding as B
from tests import kernels_of_calls as K
from tests import test_gpu_beside as beside
from tests import test_gpu_dense_ops as dense_ops
from tests import test_gpu_nan_outputs as nan_outputs
from tests import test_gpu_rows_edges as rows_edges
from tests import test_gpu_rows_shapes as rows_shapes
from tests import test_gpu_small_tiles as small_tiles


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    path = K.build(tmp_path_factory.mktemp("driver"))
    if path is None:
        pytest.skip("needs hipcc and the built library")
    return path


def _layer(dtype, s, grouped=False):
    return K.layer(dtype, s.n, s.h, s.w, s.c_in, s.c_out, c_base=s.c_base, k=s.k, stride=s.stride, pad=s.pad, groups=s.groups if grouped else 0,
                   shuffle=grouped, out_dtype=dtype if dtype != B.CG_I8 else None)


TYPE = {B.CG_F32: "F32Direct", B.CG_BF16: "Bf16Direct", B.CG_I8: "I8Direct"}


def test_small_tile_forms(exe):
    seen = set()
    for at, (shape, grouped, forms) in enumerate(small_tiles.TILES + small_tiles.UNIFORM):
        for dtype, (pf, nh, split) in forms.items():
            kernel, args, _, types = K.ask(exe, [_layer(dtype, shape, grouped)])[0]
            assert (kernel, args) == ("gated_conv_direct_kernel", (TYPE[dtype], str(pf), str(nh), str(split).lower(), str(grouped).lower())), shape
            assert at < len(small_tiles.TILES) or types == ("UniformArgs",), shape
            seen.add(args + types)
    for shape in small_tiles.FORMS + small_tiles.SHAPES:
        for dtype, ch in ((B.CG_F32, 4), (B.CG_BF16, 8), (B.CG_I8, 16)):
            for grouped in (False, True):
                if shape.c_in % ch == 0 and not (grouped and (shape.c_out % shape.groups or shape.k != 3)):
                    _, args, _, types = K.ask(exe, [_layer(dtype, shape, grouped)])[0]
                    seen.add(args + types)
    tiles = [("1", "1", "true")] + [(pf, nh, split) for pf, nh in (("1", "2"), ("1", "4"), ("2", "2"), ("2", "4")) for split in ("true", "false")]
    forms = [(TYPE[d],) + t + ("false", args) for d in TYPE for t in tiles for args in ("DirectArgs", "UniformArgs")]
    forms += [(TYPE[d],) + t + ("true", "DirectArgs") for d in TYPE if d != B.CG_I8 for t in tiles]
    missing = [f for f in forms if f not in seen]
    assert missing == [("F32Direct", "2", "4", "false", "false", "UniformArgs")]


def test_layers_with_a_base_group_that_ends_inside_a_chunk(exe):
    for dtype, (n, h, c, co, cb, groups), (pf, nh, split) in small_tiles.INSIDE:
        kernel, args, *_ = K.ask(exe, [K.layer(dtype, n, h, h, c, co, c_base=cb, groups=groups if groups > 1 else 0)])[0]
        assert (kernel, args) == ("gated_conv_direct_kernel", (TYPE[dtype], str(pf), str(nh), str(split).lower(), str(groups > 1).lower())), (dtype, n, h, c, co)


def test_layers_of_long_pixels(exe):
    for dtype, c in small_tiles.LONG_PIXELS:
        assert K.ask(exe, [K.layer(dtype, 1, 3, 1, c, 8)])[0][0] == "gated_conv_direct_kernel"


@pytest.mark.parametrize("dtype,c", [(B.CG_F32, 1900004), (B.CG_BF16, 3800008), (B.CG_I8, 7600016)], ids=["fp32", "bf16", "int8"])
def test_weights_of_a_tile_are_within_32_bits(exe, dtype, c):
    """K of 2^20 steps and more: 2 GiB of weights to 32 channels, so no tiles of 64."""
    for c_out in (512, 2048, 4096):
        kernel, args, *_ = K.ask(exe, [K.layer(dtype, 1, 100, 1, c, c_out)])[0]
        assert kernel == "gated_conv_direct_kernel" and args[2] in ("1", "2"), args


def test_row_tiled_outputs_of_many_channels(exe):
    """The row-tiled kernel takes as many channels as before its outputs were at 32-bit offsets, beyond them in the form for any output."""
    for dtype, out, c_out, shuffle, form in rows_edges.MANY_CHANNELS:
        kernel, args, *_ = K.ask(exe, [K.layer(dtype, 1, 2, 2, 32, c_out, c_base=16, groups=2 if shuffle else 0, shuffle=shuffle, out_dtype=out, rq_shift=8,
                                              variant=B.CG_VARIANT_MFMA_ROWS)])[0]
        assert (kernel, args[4]) == ("gated_conv_rows_kernel", form), (dtype, out, c_out)


def test_row_tiled_forms_of_the_ends(exe):
    """One and two wavefronts to a fragment, with and without a residual, stages of two chunks and of four, and 1x1: both types."""
    seen = set()
    for s in rows_shapes.ENDS:
        for dtype in (B.CG_BF16, B.CG_I8):
            for epilogue in (0, B.CG_EPI_RESIDUAL):
                kernel, args, *_ = K.ask(exe, [K.layer(dtype, s.n, s.h, s.w, s.c_in, s.c_out, c_base=s.c_base, k=s.k, stride=s.stride, pad=s.pad, out_dtype=dtype,
                                                       epilogue=epilogue, rq_shift=14, variant=B.CG_VARIANT_MFMA_ROWS if s.k == 3 else B.CG_VARIANT_AUTO)])[0]
                assert kernel == "gated_conv_rows_kernel", s
                seen.add(args)
    for kind in ("Bf16Rows", "I8Rows"):
        assert {(kind, cps, "1", "9", out) for cps in "24" for out in "0167"} <= seen and {(kind, "8", "1", "1", out) for out in "06"} <= seen


def test_forms_of_the_sums(exe):
    for dtype, (n, h, w, c, co, k), (pf, nh, waves), _ in small_tiles.SUMS:
        kernel, args, threads, _ = K.ask(exe, [K.layer(dtype, n, h, w, c, co, k=k)])[0]
        assert (kernel, args[:4]) == ("gated_conv_direct_kernel", (TYPE[dtype], str(pf), str(nh), str(waves > 1).lower())), (dtype, n, h, w, c, co, k)
        assert threads == (64 * waves if waves > 1 else 256), (dtype, n, h, w, c, co, k)


def test_layers_of_the_nan_test(exe):
    want = [("gated_conv_rows_kernel", ("1", "9", "0")), ("gated_conv_rows_kernel", ("1", "9", "1")), ("gated_conv_rows_kernel", ("2", "9", "0")),
            ("gated_conv_rows_kernel", ("1", "1", "0")), ("gated_conv_tile_kernel", None), ("gated_conv_tile_kernel", None),
            ("gated_conv_direct_kernel", ("true",)), ("gated_conv_direct_kernel", ("false",)), ("naive_kernel", None)]
    for (variant, n, hw, c, k), (kernel, args) in zip(nan_outputs.LAYERS, want):
        got = K.ask(exe, [K.layer(B.CG_BF16, n, hw, hw, c, c, c_base=c // 4, k=k, out_dtype=B.CG_BF16, variant=variant)])[0]
        assert got[0] == kernel, (variant, n, hw, c, k)
        if kernel == "gated_conv_rows_kernel":
            assert got[1][2:] == args, (variant, n, hw, c, k)
        elif kernel == "gated_conv_direct_kernel":
            assert got[1][3] == args[0], (variant, n, hw, c, k)


def test_layers_with_a_1x1_beside(exe):
    """The tiles that the layers of test_gpu_beside.py name, and that the 1x1 of the last ones or their own kernel is not for one launch."""
    for (n, h, w, c_in, c_out, c_base, k, stride, c1), tile in beside.FORMS:
        kernel, args, _, types = K.ask(exe, [K.layer(B.CG_BF16, n, h, w, c_in, c_out, c_base=c_base, k=k, stride=stride, out_dtype=B.CG_BF16)])[0]
        pieces = (n * -(-h // stride) * -(-w // stride) + 127) // 128 * (c1 // 64) * 4 < 256
        one = kernel == "gated_conv_direct_kernel" and args[3] == "true" and pieces
        assert one == (tile is not None), (n, h, w, c_in)
        if one:
            assert (int(args[1]), int(args[2]), types == ("UniformArgs",)) == tile, (n, h, w, c_in)


def test_launches_of_layers_with_a_1x1_beside(exe):
    """One launch, of the kernel and tile that test_gpu_beside.py names, or two."""
    got = K.beside(exe, [form + (0,) for form, _ in beside.FORMS])
    for (form, tile), launches in zip(beside.FORMS, got):
        if tile is None:
            assert [l[0] for l in launches][1:] in (["pointwise_small_kernel"], ["pointwise_tile_kernel"]) and launches[0][0] != "gated_conv_beside_kernel", form
        else:
            assert [l[0] for l in launches] == ["gated_conv_beside_kernel"], form
            args = launches[0][1]
            assert (args[0], int(args[1]), int(args[2]), args[3] == "UniformArgs") == ("Bf16Direct",) + tile, form
    # grouped layers: 64-channel blocks inside one group are a kernel's that may have a 1x1 beside it, blocks over several not
    for form, names in ((beside.GROUPED[0], ["gated_conv_beside_kernel"]), (beside.GROUPED[1], ["gated_conv_direct_kernel", "pointwise_small_kernel"])):
        assert [l[0] for l in K.beside(exe, [form])[0]] == names, form


def test_pieces_of_a_1x1_beside_are_spread_over_compute_units(exe):
    """(eight of 24 KB to a workgroup took longer than the layer and a launch of their own)"""
    for (form, layer, share), launches in zip(beside.SHARES, K.beside(exe, [form + (0,) for form, _, _ in beside.SHARES])):
        n, h, w, *_, stride, c1 = form
        pieces = -(-n * -(-h // stride) * -(-w // stride) // 16) * (c1 // 32)
        assert [l[0] for l in launches] == ["gated_conv_beside_kernel"] and launches[0][4] == layer + -(-pieces // share), (form, launches)


def test_layers_whose_stages_are_taken_in_turn(exe):
    for (s, _, grouped), cps in zip(rows_shapes.IN_TURN, "8882244"):
        kernel, args, *_ = K.ask(exe, [K.layer(B.CG_BF16, s.n, s.h, s.w, s.c_in, s.c_out, c_base=s.c_base, k=1, pad=0, groups=s.groups if grouped else 0,
                                              out_dtype=B.CG_BF16)])[0]
        assert (kernel, args[1], args[4]) == ("gated_conv_rows_kernel", cps, "8"), (s.name, args)
    for s, what, cps, form in rows_shapes.IN_TURN_OUTPUTS:
        grouped = what == "shuffled"
        kernel, args, *_ = K.ask(exe, [K.layer(B.CG_BF16, s.n, s.h, s.w, s.c_in, s.c_out, c_base=s.c_base, k=1, pad=0, groups=s.groups if grouped else 0, shuffle=grouped,
                                              out_dtype=B.CG_F32 if what == "float" else B.CG_BF16, epilogue=B.CG_EPI_RESIDUAL if what == "residual" else 0)])[0]
        assert (kernel, args[1], args[4]) == ("gated_conv_rows_kernel", str(cps), str(form)), (s.name, what, args)
    for what, form in rows_shapes.IN_TURN_INT8:
        wide, residual = what.startswith("32"), "residual" in what
        kernel, args, *_ = K.ask(exe, [K.layer(B.CG_I8, 29, 13, 13, 768, 1024, c_base=192, k=1, pad=0, out_dtype=B.CG_I32 if wide else B.CG_I8,
                                              rq_shift=1 if what == "shift of one" else 14, epilogue=B.CG_EPI_RESIDUAL if residual else 0)])[0]
        assert (kernel, args[1], args[4]) == ("gated_conv_rows_kernel", "4", str(form)), (what, args)
    kernel, args, *_ = K.ask(exe, [K.layer(B.CG_I8, 29, 13, 13, 768, 1024, c_base=192, k=1, pad=0)])[0]
    assert (kernel, args[4]) == ("gated_conv_rows_kernel", "13"), args
    kernel, args, *_ = K.ask(exe, [K.layer(B.CG_BF16, 8, 28, 28, 512, 512, c_base=128, k=1, pad=0, out_dtype=B.CG_BF16)])[0]      # one tile to a workgroup
    assert (kernel, args[4]) == ("gated_conv_rows_kernel", "0"), args


def test_1x1_convolutions_of_many_pixels_end(exe):
    """More output pixels than one launch holds: in one row, in rows of one image, in images; every one once."""
    for n, h, w, c_out, stride in [(1, 1, 1 << 30, 64, 1), (1, 1, (1 << 30) + 64, 64, 1), (1, 1, 1 << 29, 192, 1), (2, 2, 1 << 30, 64, 2), (3, 40000, 40000, 64, 1),
                                   (2000, 1000, 999, 128, 1)]:
        got = K.pieces(exe, "pointwise", [(n, h, w, 16, c_out, stride)])[0]
        at = 0
        for x, y, m, ho, wo in got:
            assert 0 < m <= 1 << 30 and m % (ho * wo) == 0 and y == at * c_out * 2
            at += m
        assert len(got) > 1 and at == n * -(-h // stride) * -(-w // stride), (n, h, w)


def test_pieces_of_1x1_convolutions_cover_every_pixel_once(exe):
    calls = [(n, h, w, 16, 64, s, cap) for n, h, w, s in itertools.product((1, 2, 5), (1, 2, 7), (1, 3, 9), (1, 2, 3)) for cap in (1, 2, 3, 4, 8, 20, 63, 1000)]
    for (n, h, w, c_in, c_out, s, cap), pieces in zip(calls, K.pieces(exe, "cut", calls)):
        ho, wo = -(-h // s), -(-w // s)
        want = [((((i * h + r * s) * w) + c * s) * c_in * 2, ((i * ho + r) * wo + c) * c_out * 2) for i in range(n) for r in range(ho) for c in range(wo)]
        got = []
        for x, y, m_total, pho, pwo in pieces:
            assert 0 < m_total <= cap
            for m in range(m_total):                          # (the pixel of the kernel's point_pixel)
                q, img = m // pwo, m // pwo // pho
                got.append((x + ((img * h + (q - img * pho) * s) * w + (m - q * pwo) * s) * c_in * 2, y + m * c_out * 2))
        assert sorted(got) == want, (n, h, w, s, cap)


def test_1x1_convolutions_whose_last_block_is_half_empty(exe):
    """(64 x 128 everywhere was up to 17 % slower than 128 x 64, where that comes to fewer workgroups to a compute unit)"""
    for (shape, tiles), line in zip(dense_ops.HALF_EMPTY, K.lines(exe, "pointwise", [s for s, _ in dense_ops.HALF_EMPTY])):
        (n, h, w, _, _, stride), wide = shape, "pointwise_conv_kernel" in line
        assert wide == (not tiles) and (wide or int(line.split()[2]) == n * -(-h // stride) * -(-w // stride)), (shape, line)
