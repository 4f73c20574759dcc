"""Requantisation to int8 in 32 bits (where every channel's factors allow it) and in 64: whole numbers, so equal to the oracle bit
for bit, on the row-tiled and the small-tile kernel, with sums on both sides of the range that the output covers."""
import numpy as np
import pytest

from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu

#           name               mult0       mult1            bias        shift  residual factor   fits 32 bits (without and with a residual)
SETTINGS = [("usual",          (40, 900),  (40, 900),       (-8, 9),    16,    30000,            (True, True)),
            ("wide",           (1, 2),     (1, 2),          (-128, 128), 2,    5,                (True, True)),       # bounds of hundreds
            ("pairs_apart",    (1, 2),     (4000, 8000),    (-8, 9),    16,    0,                (False, False)),     # bound times the larger mult
            ("large",          (2 ** 20, 2 ** 22), (2 ** 20, 2 ** 22), (-3, 4), 22, -(2 ** 20),  (True, False)),      # bounds of hundreds
            ("large_narrow",   (2 ** 20, 2 ** 21), (2 ** 20, 2 ** 21), (-3, 4), 22, -(2 ** 20),  (True, True)),       # sums near 2^31
            ("beyond_24_bits", (2 ** 23, 2 ** 24), (2 ** 23, 2 ** 24), (-3, 4), 22, 0,           (False, False)),
            ("bias_too_large", (40, 900),  (40, 900),       (-40000, 40000), 16, 0,              (False, False)),
            ("negative",       (-900, 900), (40, 900),      (-8, 9),    16,    -30000,           (False, False)),
            ("shift_of_none",  (1, 3),     (1, 3),          (-8, 9),    0,     1,                (True, True))]       # plain outputs


def fits_32_bits(rq, res_mult, residual):
    """Whether every channel's requantisation fits 32 bits: factors below 2^23, sums below 2^31 once the sum of products is clamped to where the
    output's byte still changes."""
    limit, shift = 1 << 23, rq["rq_shift"]
    res = 128 * abs(res_mult) if residual else 0
    for m0, m1, bias in zip(rq["rq_mult0"].tolist(), rq["rq_mult1"].tolist(), rq["rq_bias"].tolist()):
        least, most = min(m0, m1), max(m0, m1)
        add = abs(bias * (1 << shift) + (1 << (shift - 1) if shift > 0 else 0))
        span = (128 << shift) + add + res
        if least <= 0 or most >= limit or res >= 128 * limit or span >= 1 << 31:
            return False
        bound = span // least + 1
        if bound >= limit or bound * most + add + res >= 1 << 31:
            return False
    return True


@pytest.mark.parametrize("setting", SETTINGS, ids=[s[0] for s in SETTINGS])
@pytest.mark.parametrize("n", [1, 40], ids=["small_tiles", "rows"])
def test_requantise_bit_exact(setting, n):
    name, m0, m1, bias, shift, res_mult, fits = setting
    shape = W.LayerShape("rq_" + name, n, 14, 15, 64, 64)
    rng = np.random.default_rng(n + shift)
    q = W.quantize_int8(W.make_inputs(shape, 9100 + n, kind="coherent", rho=0.35))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    res = rng.integers(-128, 128, (n, shape.ho, shape.wo, 64)).astype(np.int8)
    rq = dict(rq_mult0=rng.integers(*m0, 64).astype(np.int32), rq_mult1=rng.integers(*m1, 64).astype(np.int32),
              rq_bias=rng.integers(*bias, 64).astype(np.int32), rq_shift=shift)
    variant = B.CG_VARIANT_AUTO if n == 1 else B.CG_VARIANT_MFMA_ROWS
    assert fits == (fits_32_bits(rq, 0, False), fits_32_bits(rq, res_mult, True))
    for epilogue, r in ((B.CG_EPI_RELU, None), (0, None), (B.CG_EPI_RESIDUAL, res)):
        P.run_int8(q, thr, out_i8=True, rq=rq, residual=r, rq_res_mult=res_mult if r is not None else 0, epilogue=epilogue,
                   variant=variant, name=shape.name)
