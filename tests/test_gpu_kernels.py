"""GPU tests of single kernels at the sizes where their splits and dispatch
rules can go wrong: remainders of tiles, the smallest and largest of a range,
misaligned buffers; each against the same operation in float64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _offset_copy(t, by):
    """A contiguous copy of t whose first element lies `by` elements into its buffer."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    v = buf[by:].view(t.shape)
    v.copy_(t)
    return v


# channel counts: one per lane (odd, or not a multiple of 16 bytes), whole 16-byte groups, more
# groups than a block has threads; rows: fewer than one chunk, chunk remainders, several chunks a block
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,c,shift", [(1, 1, 0), (63, 7, 0), (65, 16, 0), (1000, 48, 0), (1000, 48, 1), (777, 264, 0),
                                       (130, 2080, 0), (70001, 64, 0)])
def test_affine_act_bwd_shapes(dtype, n, c, shift):
    from paper_1904_08755_amd import gsc
    g = torch.Generator(DEV).manual_seed(n * 31 + c)
    scale = 0.5 + torch.rand(c, generator=g, device=DEV)
    if c > 4:
        scale[1] = 0.0
    sh = 0.3 * torch.randn(c, generator=g, device=DEV)
    S = torch.randn((n, c), generator=g, device=DEV)
    Y = _offset_copy(torch.clamp(S * scale + sh, min=0).to(dtype), shift)
    dY = _offset_copy(torch.randn((n, c), generator=g, device=DEV).to(dtype), shift)
    dZ, ds, dt = gsc.gsc_affine_act_bwd(Y, dY, scale, sh, relu=True)
    y, gr, sc, s0 = Y.double(), dY.double(), scale.double(), sh.double()
    G = torch.where(y > 0, gr, 0.0)
    # the product in float32 (half an ulp), rounded to the dtype (half an ulp)
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    assert ((dZ.double() - G * sc).abs() <= (G * sc).abs() * eps + 1e-40).all()
    # sums: at most rows-per-lane + lanes float32 additions, each within 2^-24 of the sum of magnitudes
    bound = (n + 512) * 2.0 ** -24
    assert ((dt.double() - G.sum(0)).abs() <= G.abs().sum(0) * bound + 1e-30).all()
    ok = scale != 0
    z = (y - s0)[:, ok] / sc[ok]
    zmag = (G[:, ok].abs() * (y.abs() + s0.abs())[:, ok] / sc[ok]).sum(0)
    assert ((ds.double()[ok] - (G[:, ok] * z).sum(0)).abs() <= zmag * (bound + 2.0 ** -22) + 1e-30).all()
    if c > 4:   # a channel with scale 0: not finite when a row counts, 0 when none does
        counts = bool((G[:, 1] != 0).any())
        assert torch.isfinite(ds[1]).item() != counts
    again = gsc.gsc_affine_act_bwd(Y, dY, scale, sh, relu=True)
    assert torch.equal(again[1].nan_to_num(7.0), ds.nan_to_num(7.0)) and torch.equal(again[2], dt)
