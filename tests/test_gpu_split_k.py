"""fg_linear where the contraction is shared by workgroups and a second pass adds the partial sums: less work than
workgroups (down to one range), ranges that end inside a tile, begin at one or hold several, rows and columns that end
inside a tile, one and two items per thread of the second pass, and the same bits on every call.  The sizes are beyond
those that csrc/fg_gemm_fewrows.hip takes, but for two (FP16 and tiled 4-bit, 500 rows); FP16 weights of most of them run on
csrc/fg_gemm_f16_tiles.hip, so those kernels on 256 columns have FP16 sizes of their own below."""
import pytest
import torch

from paper_2303_06865_amd import binding as B
from tests import routes
from tests.util import assert_close

pytestmark = pytest.mark.gpu

FORMATS = {"f16": (False, False, False), "q4t": (True, True, False), "q4h": (True, True, True)}

CASES = [
    # m, n, k
    (1025, 32, 64),        # tiles of one K step, a range each
    (1300, 8224, 64),
    (1025, 4128, 128),     # of two
    (700, 16416, 128),
    (1100, 2080, 256),     # of four
    (500, 2080, 256),      # ... halved where there are few tiles
    (1100, 2080, 320),     # of five
    (500, 2080, 320),      # ... in ranges of three or more, across tiles
    (1040, 768, 192),      # 45 units, 15 ranges over 15 tiles
    (1100, 1056, 448),     # a last column block of one 32-column tile, a last row block of 76 rows
    (1281, 288, 640),      # one row in the last block
    (1500, 3104, 320),
    (161, 12832, 1536),    # 16-row tiles, two row blocks
    (257, 9248, 1984),
    (321, 7200, 2624),     # 256-row tiles
    (333, 2304, 4800),
    (33, 12832, 4416),     # 3, 4, 5, ... 10 tiles of 16 rows
    (64, 4128, 14016),
    (70, 12832, 3072),
    (81, 12832, 3072),
    (112, 8224, 3520),
    (128, 4128, 6720),
    (144, 12832, 1856),
    (160, 4128, 5440),
    (144, 36864, 640),     # two items per thread
    (400, 30720, 384),
]


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", CASES)
def test_linear_shared_contraction(m, n, k, fmt):
    _check(m, n, k, *FORMATS[fmt])


def _check(m, n, k, quant, tiled, h16):
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    w, x, bias, res = half(n, k) * 0.05, half(m, k), half(n), half(m, n)
    mat = B.Mat.from_f16(w, quant, tiled=tiled, meta_f16=h16)
    if quant:   # the products take FP16 weights
        w = B.fg_dequantize_groupwise(*B.fg_quantize_groupwise(w, meta_f16=h16)).view(n, k).half()
    ref = torch.relu(x.float() @ w.float().t() + bias.float()) + res.float()
    got = B.fg_linear(mat, bias, x, residual=res, relu=True)
    assert_close(got.cpu().numpy(), ref.cpu().numpy(), "shared contraction m=%d n=%d k=%d %s" % (m, n, k, (quant, tiled, h16)))
    assert torch.equal(B.fg_linear(mat, bias, x, residual=res, relu=True), got)


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", [
    (321, 32800, 64),      # two blocks of 192 rows: whole rounds of one K step, a last column block of 32
    (384, 33024, 128),     # both blocks full, two K steps
    (385, 16416, 192),     # one row more: blocks of 256 again
    (513, 22112, 256),     # three blocks, one row in the last
    (576, 22112, 448),     # whole rounds and a shared rest
    (577, 8224, 512),
    (1152, 11040, 320),
    (1344, 9248, 192),
    (1281, 4096, 7168),
    (1281, 4064, 7168),
    (1281, 4096, 7104),
    (1344, 12320, 7168),
    (1152, 4096, 7168),
])
def test_linear_blocks_of_192_rows(m, n, k, fmt):
    test_linear_shared_contraction(m, n, k, fmt)


# FP16 weights that neither the few-rows kernel nor the FP16 tiles take: the kernels on 256 columns, at every number of 32-row tiles,
# one and two row blocks of them, blocks of 192 and of 256 rows, whole tiles and ranges, ragged rows and columns, one K step and many.
@pytest.mark.parametrize("m,n,k,residual", [
    (24, 33056, 1088, True), (60, 57376, 1088, True), (81, 65536, 320, True), (72, 8352, 13312, True), (80, 8352, 21824, False),
    (82, 4256, 17536, True), (112, 12832, 18048, True), (128, 18464, 12864, True), (129, 33056, 6400, True),
    (200, 38912, 2560, False), (231, 41120, 2816, False), (257, 36896, 3072, False), (320, 33056, 6400, True),
    (321, 32800, 64, False), (384, 33024, 128, False), (343, 36896, 192, False), (385, 33024, 192, False), (513, 33056, 256, True),
    (576, 33056, 448, True), (577, 33056, 320, True), (1100, 33056, 64, True), (1152, 32800, 320, True),
    (1281, 12288, 17152, True),   # blocks of 256 rows
    (1281, 12320, 17152, True),   # ... and of 192
    (2049, 8224, 64, True), (2100, 8224, 320, True), (2100, 96, 4160, True), (2304, 2080, 4160, True), (3000, 8224, 448, False),
])
def test_linear_f16_past_the_tiles(m, n, k, residual):
    assert not routes.few_rows(B.FG_F16, n, k, m) and not routes.f16_tiles(n, k, m, residual)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    w, x, bias, res = half(n, k) * 0.05, half(m, k), half(n), half(m, n) if residual else None
    y = x.float() @ w.float().t() + bias.float()
    want = torch.relu(y) + (res.float() if residual else 0.0)
    mat = B.Mat.from_f16(w, False)
    got = B.fg_linear(mat, bias, x, residual=res, relu=True)
    # results are rounded to FP16: half a unit of the largest, 2^-11 of it
    assert_close(got.cpu().numpy(), want.cpu().numpy(), "f16 past the tiles m=%d n=%d k=%d" % (m, n, k),
                 mabs=max(1e-2, float(want.abs().max()) * 2.0 ** -11))
    assert torch.equal(B.fg_linear(mat, bias, x, residual=res, relu=True), got)


# Canonical 4-bit weights past the lines of the few-rows kernel, and FP16 weights whose columns 32 does not divide, which
# neither streaming kernel takes: every row tile count, ragged columns, contractions that end inside a step of 128.
@pytest.mark.parametrize("fmt,m,n,k", [
    ("q4", 33, 36864, 12288), ("q4", 64, 33800, 8896), ("q4", 96, 20488, 9792), ("q4", 128, 16392, 9280),
    ("q4", 144, 12872, 9664), ("q4", 160, 12296, 9792), ("q4", 300, 8200, 7360), ("q4", 512, 6152, 6208),
    ("q4", 600, 4104, 3904), ("q4", 1000, 3080, 3072),
    ("f16", 20, 32776, 128), ("f16", 32, 32792, 192), ("f16", 50, 5000, 3456), ("f16", 64, 5000, 3456), ("f16", 100, 3016, 2880),
    ("f16", 128, 3016, 2880), ("f16", 144, 4104, 3520), ("f16", 300, 2056, 3456), ("f16", 512, 1544, 2880), ("f16", 600, 1032, 3648),
])
def test_linear_small_and_large_m_past_the_few_rows_lines(fmt, m, n, k):
    _check(m, n, k, fmt == "q4", False, False)


# Both sides of the lines between blocks of 32 rows over whole contractions and the kernels that take the rest.
@pytest.mark.parametrize("fmt,m,n,k", [
    ("f16", 1, 1024, 10304), ("f16", 1, 1056, 10304), ("f16", 8, 1280, 10304), ("f16", 8, 1312, 10304), ("f16", 16, 1696, 10304),
    ("f16", 16, 1728, 10304), ("f16", 24, 2560, 10304), ("f16", 24, 2592, 10304), ("f16", 40, 320, 8256), ("f16", 7, 200, 9280),
    ("q4t", 17, 32768, 192), ("q4h", 32, 32800, 192), ("q4t", 33, 32768, 192), ("q4t", 64, 32800, 192), ("q4h", 512, 8192, 256),
    ("q4t", 513, 8192, 256), ("q4t", 33, 49152, 256), ("q4t", 40, 49184, 256),
    ("f16", 33, 4096, 192), ("f16", 50, 4096, 128), ("f16", 65, 4096, 256), ("f16", 128, 6144, 128), ("f16", 100, 6176, 128),
    ("f16", 129, 13088, 192), ("f16", 130, 13120, 192), ("f16", 512, 8192, 256), ("f16", 513, 8192, 256),
    ("q4", 161, 13648, 128), ("q4", 161, 13664, 128), ("q4", 330, 18608, 256), ("q4", 330, 18632, 256), ("q4", 320, 18632, 256),
    ("q4", 161, 16384, 3456), ("q4", 161, 16384, 3520), ("q4", 321, 12288, 3712), ("q4", 321, 12288, 3840),
])
def test_linear_around_the_few_rows_lines(fmt, m, n, k):
    _check(m, n, k, *dict(FORMATS, q4=(True, False, False))[fmt])
