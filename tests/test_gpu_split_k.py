"""fg_linear where the contraction is shared by workgroups and a second pass adds the partial sums: less work than
workgroups (down to one range), ranges that end inside a tile, begin at one or hold several, rows and columns that end
inside a tile, one and two items per thread of the second pass, and the same bits on every call."""
import pytest
import torch

from paper_2303_06865_amd import binding as B
from tests.test_gpu_kernels import _linear_case
from tests.util import assert_close

pytestmark = pytest.mark.gpu

FORMATS = {"f16": (False, False, False), "q4t": (True, True, False), "q4h": (True, True, True)}

CASES = [
    # m, n, k
    (33, 32, 64),        # one unit in all
    (40, 768, 192),      # 9 units: 3 ranges, one per tile
    (48, 1056, 128),     # 10 units, 3 ranges over 5 tiles
    (70, 544, 1984),
    (128, 4096, 1024),
    (144, 12288, 192),
    (144, 12832, 448),   # 51 tiles
    (129, 2080, 832),
    (257, 1056, 256),    # two row blocks
    (321, 288, 640),     # 256-row tiles, one row in the second block's 9th eight
    (333, 2304, 768),
    (700, 3104, 320),
    (161, 25600, 64),    # one K step per tile
]


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", CASES)
def test_linear_shared_contraction(m, n, k, fmt):
    quant, tiled, h16 = FORMATS[fmt]
    got, ref = _linear_case(m, n, k, quant, True, m % 2 == 0, True, seed=m + n + k, tiled=tiled, meta_f16=h16)
    assert_close(got, ref, "shared contraction m=%d n=%d k=%d %s" % (m, n, k, fmt))


@pytest.mark.parametrize("m,n,k", [(144, 36864, 512), (400, 30720, 256)])   # two items per thread
def test_linear_shared_contraction_of_many_tiles(m, n, k):
    g = torch.Generator(device="cuda").manual_seed(m)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    w, x = half(n, k) * 0.05, half(m, k)
    mat = B.Mat.from_f16(w, True, tiled=True)
    wd = B.fg_dequantize_groupwise(*B.fg_quantize_groupwise(w)).view(n, k).half().float()   # the products take FP16 weights
    ref = x.float() @ wd.t()
    got = B.fg_linear(mat, None, x)
    assert_close(got.cpu().numpy(), ref.cpu().numpy(), "m=%d n=%d" % (m, n))
    assert torch.equal(B.fg_linear(mat, None, x), got)
