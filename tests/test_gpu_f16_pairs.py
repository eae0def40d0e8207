"""fg_linear at 33 to 48 rows on tiled 4-bit weights with FP16 {min, scale} pairs (gemm_decode16h_kernel in csrc/fg_gemm_stream.hip)
against the same matrix with its pairs in FP32: another kernel and another dequantization, but the same weights and the same order
of additions, so the same bits.  Sizes beyond those of the few-rows kernel: one K step, even and odd numbers of them, ranges that
end inside a tile, whole tiles and ranges in one call, a ragged last column block, all rows of the tiles and few; scales from FP16's subnormals up, below and from the 0.25 at which the dequantization changes, of one column or of all."""
import pytest
import torch

from paper_2303_06865_amd import binding as B
from tests import routes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scales", ["small", "one column", "all", "subnormal"])
@pytest.mark.parametrize("m,n,k", [(33, 32800, 64), (48, 33056, 128), (37, 36896, 192), (40, 14368, 4160), (41, 70016, 320),
                                   (35, 28672, 2112), (48, 7200, 8192)])
def test_f16_pairs_same_bits_as_f32_pairs(m, n, k, scales):
    # neither matrix is the few-rows kernel's: both run on tiles of three 16-row tiles, which 33 to 48 rows take
    assert not any(routes.few_rows(t, n, k, m) for t in (B.FG_Q4G64_H16_TILED, B.FG_Q4G64_TILED))
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    codes = torch.randint(0, 256, (n, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    pairs = half(n, k // 64, 2) * 0.05   # {min, scale}, scales of either sign
    if scales == "one column":
        pairs.view(-1, 2)[7::97, 1] = 0.25   # (the layout keeps a 32-column tile's pairs together)
    elif scales == "all":
        pairs[..., 1] *= 40.0
    elif scales == "subnormal":
        pairs *= 2.0 ** -12
    x, bias, res = half(m, k), half(n), half(m, n)
    h16 = B.Mat(n, k, B.FG_Q4G64_H16_TILED, codes, pairs)
    f32 = B.Mat(n, k, B.FG_Q4G64_TILED, codes, pairs.float())
    got = B.fg_linear(h16, bias, x, residual=res, relu=True)
    ref = B.fg_linear(f32, bias, x, residual=res, relu=True)
    assert torch.isfinite(ref).all() and ref.abs().max() > 0
    assert torch.equal(got, ref)
