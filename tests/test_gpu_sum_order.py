"""The order of additions that results downstream depend on: LayerNorm's sums, bit for bit, at every width that its launch
rules tell apart.

A projection behind a LayerNorm whose sums run in another order differs by last bits, and where its output is quantized
into the cache a last bit can be a whole code step; so the order is held fixed here, not only the value."""
import numpy as np
import pytest

from paper_2303_06865_amd import binding as B
from tests.util import dev, host

pytestmark = pytest.mark.gpu

F = np.float32


def _fma(a, b, c):
    """binary32 a * b + c with one rounding (the product of two binary32 numbers is exact in binary64)."""
    return (a.astype(np.float64) * b + c).astype(F)


def _row_sum(t):
    """t [rows, 256]: the workgroup's sum of what its 256 threads hold.  64 lanes fold in halves (lane i and i ^ 32
    first, neighbours last), then the four waves' sums are added in order."""
    t = t.reshape(t.shape[0], 4, 64)
    for o in (32, 16, 8, 4, 2, 1):
        t = t + t[:, :, np.arange(64) ^ o]
    w = t[:, :, 0]
    return ((w[:, 0] + w[:, 1]) + w[:, 2]) + w[:, 3]


def layernorm_in_order(x16, g16, b16, eps):
    """LayerNorm in binary32 with every addition in its place: thread t takes pieces t, t + 256, ... of eight elements
    and adds them one after the other."""
    rows, cols = x16.shape
    pieces = -(-cols // (8 * 256)) * 256
    v = np.zeros((rows, pieces * 8), F)
    v[:, :cols] = x16.astype(F)
    live = (np.arange(pieces * 8) < cols).reshape(-1, 256, 8)
    v = v.reshape(rows, -1, 256, 8)
    s = np.zeros((rows, 256), F)
    for j in range(v.shape[1]):
        for i in range(8):
            s = s + v[:, j, :, i]
    mean = (_row_sum(s) / F(cols))[:, None]
    q = np.zeros((rows, 256), F)
    for j in range(v.shape[1]):
        d = np.where(live[j][None], v[:, j] - mean[:, None], F(0))
        start = 0
        if j == 0 and cols <= 16384:   # the row is held in registers: of the first two squares the second one is rounded
            q, start = _fma(d[..., 0], d[..., 0], d[..., 1] * d[..., 1]), 2
        for i in range(start, 8):
            q = _fma(d[..., i], d[..., i], q)
    rstd = (F(1) / np.sqrt(_row_sum(q) / F(cols) + F(eps)))[:, None]
    return _fma((x16.astype(F) - mean) * rstd, g16.astype(F), b16.astype(F)).astype(np.float16)


@pytest.mark.parametrize("rows,cols", [(513, 64), (513, 768), (600, 2056), (513, 4096), (600, 4104), (513, 7168), (513, 12288),
                                       (600, 16384), (513, 16392), (1, 49152),
                                       (1, 8), (256, 768), (200, 2048), (512, 4096), (100, 4104), (256, 8192), (37, 8200),
                                       (144, 12288), (512, 16384)])
def test_layernorm_sums_in_order(rows, cols):
    rng = np.random.default_rng(rows + cols)
    x = (rng.standard_normal((rows, cols)) * 3 + 0.7).astype(np.float16)
    g, b = (1 + 0.1 * rng.standard_normal(cols)).astype(np.float16), (0.1 * rng.standard_normal(cols)).astype(np.float16)
    out = host(B.fg_layernorm(dev(x), dev(g), dev(b), 1e-5))
    assert np.array_equal(out.view(np.uint16), layernorm_in_order(x, g, b, 1e-5).view(np.uint16))

