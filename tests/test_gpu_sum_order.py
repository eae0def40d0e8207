"""The order of additions that results downstream depend on: LayerNorm's sums, bit for bit, at every width that its launch
rules tell apart; and a 12288-wide decode layer on an FP16 cache, where no 4-bit code can move.

A projection behind a LayerNorm whose sums run in another order differs by last bits, and where its output is quantized
into the cache a last bit can be a whole code step; so the order is held fixed here, not only the value."""
import numpy as np
import pytest
import torch

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


def test_decode_layer_175b_wide_f16_cache():
    """144 sequences, tiled 4-bit weights, against binary32 with an FP16 rounding wherever the layer stores FP16.  Seven
    stored tensors lie in a row.  If a last bit of a sum turned every one of their roundings over, they would add up to
    sqrt(7) 2^-11 = 1.3e-3 in the 2-norm; half of that, and single values within 1e-2 of the root mean square, are far
    from what a moved code of a 4-bit cache does (up to 0.06)."""
    b, nh, dh, t = 144, 96, 128, 130
    h1, h2 = nh * dh, 4 * nh * dh
    cfg = B.Cfg(h1, nh, h2, 1000, 4096)
    g = torch.Generator(device="cuda").manual_seed(12)
    half = lambda shape, std=1.0: torch.empty(shape, dtype=torch.float16, device="cuda").normal_(0.0, std, generator=g)
    mats, dense = [], []
    for n, k in ((3 * h1, h1), (h1, h1), (h2, h1), (h1, h2)):
        w = half((n, k), 0.02)
        mats.append(B.Mat.from_f16(w, True, tiled=True))
        dense.append(B.fg_dequantize_groupwise(*B.fg_quantize_groupwise(w)).view(n, k).half())
    ones, zeros = torch.ones(h1, dtype=torch.float16, device="cuda"), torch.zeros(h1, dtype=torch.float16, device="cuda")
    kv = B.KVCache(cfg, b, t + 2, False, zero=False)
    for c in (kv.k_codes, kv.v_codes):
        c.normal_(0.0, 1.0, generator=g)
    x = half((b, h1))
    r16 = lambda a: a.half().float()
    lin = lambda a, w: a @ w.float().t()
    norm = lambda a: r16(torch.nn.functional.layer_norm(a.double(), (h1,), eps=1e-5))
    q, k, v = r16(lin(norm(x.float()), dense[0])).view(b, 3, nh, dh).unbind(1)
    rows = lambda c, new: torch.cat([c.view(b, nh, t + 2, dh)[:, :, :t].float(), new[:, :, None]], 2)
    kk, vv = rows(kv.k_codes, k), rows(kv.v_codes, v)
    p = torch.softmax((kk * q[:, :, None]).sum(-1) / dh ** 0.5, -1)
    o = r16((p[..., None] * vv).sum(2).reshape(b, h1))
    x1 = r16(lin(o, dense[1]) + x.float())
    want = r16(lin(r16(torch.relu(lin(norm(x1), dense[2]))), dense[3]) + x1)
    got = B.fg_decode_layer(cfg, B.LayerWeights(*mats, ones, zeros, ones, zeros), x, t, kv).float()
    d, rms = (got - want).abs(), want.square().mean().sqrt()
    assert float(d.norm() / want.norm()) <= 6.3e-4
    assert float(d.max() / rms) <= 1e-2
