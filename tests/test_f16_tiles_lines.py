"""Which FP16 projections run on csrc/fg_gemm_f16_tiles.hip: those at which it was measured to be the faster kernel, and none of
those at which it was measured to be slower than the one that it took them from."""
import pytest

from tests import routes

SLOWER = [
    # m, n, k, residual
    (92, 8352, 13312, False), (80, 8352, 21824, False), (84, 8672, 13376, True), (82, 4256, 17536, True), (65, 4160, 14464, True),
    (78, 5408, 15488, False), (72, 5504, 28928, False), (97, 4256, 24320, True), (108, 8576, 10176, False),
    (1089, 27488, 64, False), (982, 26240, 64, False), (343, 36896, 192, False), (352, 42688, 128, False), (1662, 18624, 128, False),
    (347, 29856, 256, False), (530, 38912, 64, False), (800, 15328, 128, False),
    (1000, 16384, 320, False), (1000, 16384, 4096, False), (2000, 8192, 768, False), (1800, 8192, 2048, False), (500, 32768, 1024, False),
    (384, 32768, 512, False), (320, 32768, 1024, False), (160, 65536, 2048, False), (80, 12288, 16384, True), (383, 33408, 2496, False), (322, 38752, 4928, False), (330, 49568, 4096, False), (231, 41120, 2816, False),
    (1595, 19584, 10496, False), (1314, 28928, 5184, False), (1491, 12416, 13248, False), (1732, 9920, 17856, True),
    (1260, 27200, 4864, False), (1703, 21504, 7168, False),
]
FASTER = [
    (333, 12288, 4096, False), (333, 4096, 4096, True), (333, 16384, 4096, False), (333, 4096, 16384, True), (512, 7168, 7168, True),
    (128, 12288, 4096, False), (128, 4096, 16384, True), (80, 4096, 10560, True), (85, 7168, 16768, False), (66, 7168, 7168, True),
    (800, 15328, 128, True), (618, 3648, 64, False), (1018, 4352, 128, False), (9000, 768, 3072, True), (1024, 6144, 2048, False),
    (1485, 7168, 11584, False), (1680, 4160, 23424, False), (1138, 9504, 15552, False), (300, 40000, 1024, False), (1000, 16384, 4096, True), (2000, 8192, 768, True), (2048, 7936, 4096, False), (1024, 15872, 512, False),
    (256, 32768, 1024, False), (320, 32768, 1024, True), (69, 4864, 28480, False), (89, 6016, 9408, False), (89, 5760, 20928, False), (201, 17568, 7104, True),
    (259, 35744, 3840, True),
]


@pytest.mark.parametrize("m,n,k,residual", SLOWER)
def test_left_to_the_other_kernels(m, n, k, residual):
    assert not routes.f16_tiles(n, k, m, residual)


@pytest.mark.parametrize("m,n,k,residual", FASTER)
def test_taken(m, n, k, residual):
    assert routes.f16_tiles(n, k, m, residual)
