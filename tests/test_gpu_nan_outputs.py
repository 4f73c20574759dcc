"""bf16 outputs without ReLU: a NaN in the input or the residual comes out as a NaN on every kernel, and nowhere else.  Weights are ones
and finite inputs one or two, so that every finite value is exact."""
import numpy as np
import pytest
import torch

from paper_1805_12549_amd import binding as B

pytestmark = pytest.mark.gpu

LAYERS = [  # variant, images, size, channels, kernel
    (B.CG_VARIANT_MFMA_ROWS, 32, 56, 64, 3), (B.CG_VARIANT_MFMA_ROWS, 2, 14, 64, 3), (B.CG_VARIANT_MFMA_ROWS, 12, 28, 512, 3),
    (B.CG_VARIANT_AUTO, 64, 28, 128, 1), (B.CG_VARIANT_TILE, 4, 14, 64, 3), (B.CG_VARIANT_TILE, 4, 14, 128, 1), (B.CG_VARIANT_AUTO, 1, 14, 64, 3),
    (B.CG_VARIANT_AUTO, 60, 14, 144, 1), (B.CG_VARIANT_NAIVE, 2, 9, 64, 3)]


@pytest.mark.parametrize("variant,n,hw,c,k", LAYERS,
                         ids=["rows", "rows_paired", "rows_two_fragments", "rows_1x1", "tile", "tile_1x1", "small_split", "small_whole", "plain"])
@pytest.mark.parametrize("epilogue", [0, B.CG_EPI_AFFINE, B.CG_EPI_RESIDUAL, B.CG_EPI_AFFINE | B.CG_EPI_RESIDUAL],
                         ids=["plain", "affine", "residual", "affine_residual"])
def test_nan_without_relu(variant, n, hw, c, k, epilogue):
    cb, p = c // 4, k // 2
    x = torch.ones((n, hw, hw, c))
    x[:, :, hw // 2:] = 2.0
    x[0, 2, 3, 1] = x[n - 1, hw - 1, hw - 2, cb - 1] = float("nan")                  # in the base group
    x[0, 7, 1, cb] = x[n - 1, 5, hw - 3, c - 1] = float("nan")                       # a conditional channel, of unfired and of fired pixels
    thr = float(k * k * cb) + 0.5                                                    # the left half stays below
    affine, residual = epilogue & B.CG_EPI_AFFINE, epilogue & B.CG_EPI_RESIDUAL
    kw = dict(scale0=np.full(c, 0.5), shift0=np.zeros(c), scale1=np.full(c, 2.0), shift1=np.zeros(c)) if affine else {}
    res = None
    if residual:
        res = torch.zeros((n, hw, hw, c))
        res[0, 4, 4, :] = float("nan")
        res[n - 1, 1, hw - 1, c - 1] = float("nan")
    ones = torch.ones((c, k, k, c), dtype=torch.bfloat16, device="cuda")
    layer = B.GatedConv(n_max=n, h=hw, w=hw, c_in=c, c_out=c, c_base=cb, kh=k, kw=k, pad=p, w_base=ones[..., :cb].contiguous(),
                        w_cond=ones[..., cb:].contiguous(), in_dtype=B.CG_BF16, out_dtype=B.CG_BF16, epilogue=epilogue, variant=variant,
                        gate_mean=np.zeros(c), gate_var=np.ones(c), delta=np.full(c, thr), **kw)
    y = layer.forward(x.bfloat16().cuda(), residual=None if res is None else res.bfloat16().cuda(), bitmap=False, counts=False)[0].cpu().float()
    layer.close()
    xp = torch.nn.functional.pad(torch.stack([x[..., :cb].sum(-1), x[..., cb:].sum(-1)], -1), (0, 0, p, p, p, p))
    base, cond = sum(xp[:, r:r + hw, s:s + hw] for r in range(k) for s in range(k)).unbind(-1)
    fired = base >= thr
    want = torch.where(fired, (base + cond) * (2.0 if affine else 1.0), base * (0.5 if affine else 1.0))[..., None].expand(y.shape)
    if residual:
        want = want + res
    want = want.bfloat16().float()
    assert want.isnan().any() and not want.isnan().all()
    assert torch.equal(y.isnan(), want.isnan())
    assert torch.equal(torch.nan_to_num(y), torch.nan_to_num(want))
