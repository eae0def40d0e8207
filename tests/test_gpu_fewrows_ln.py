"""The decode layer of a few rows, whose projections take the LayerNorm before them in (csrc/fg_gemm_fewrows_ln.hip), against
the same layer put together from fg_layernorm, fg_linear and fg_decode_attention, bit for bit: both sum in the same order."""
import pytest
import torch

from paper_2303_06865_amd import binding as B

pytestmark = pytest.mark.gpu

FORMATS = {"f16": (False, False, False), "q4": (True, False, False), "q4t": (True, True, False), "q4h": (True, True, True)}


# widths of one group (half a step), an odd number of groups, a step for every wave and one more, one and two pieces of a row
# per lane, and beyond the kernel; rows at which groups of waves have one row more than the other, and beyond the kernel
@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("b,nh,dh,h2", [(1, 1, 64, 64), (2, 3, 64, 192), (4, 12, 64, 3072), (6, 8, 128, 1088), (3, 17, 64, 4160),
                                        (8, 9, 128, 64), (7, 32, 64, 2048), (5, 33, 64, 8256), (1, 32, 128, 4160), (9, 6, 64, 832),
                                        (2, 65, 64, 320), (1, 31, 64, 16448)])
def test_decode_layer_is_its_parts(b, nh, dh, h2, fmt):
    quant, tiled, h16 = FORMATS[fmt]
    h1, t = nh * dh, 5
    g = torch.Generator(device="cuda").manual_seed(b * 1000 + h1)
    half = lambda *s, std=1.0, mean=0.0: torch.empty(s, dtype=torch.float16, device="cuda").normal_(mean, std, generator=g)
    cfg = B.Cfg(h1, nh, h2, 1000, 64)
    mats = [B.Mat.from_f16(half(n, k, std=0.1), quant, tiled=tiled, meta_f16=h16)
            for n, k in ((3 * h1, h1), (h1, h1), (h2, h1), (h1, h2))]
    ln = [half(h1, std=0.1, mean=m) for m in (1.0, 0.0, 1.0, 0.0)]
    bias = [half(n, std=0.1) if b != 3 else None for n in (3 * h1, h1, h2, h1)]
    kv, parts = B.KVCache(cfg, b, t + 1, False), B.KVCache(cfg, b, t + 1, False)
    for p in ("k_codes", "v_codes"):
        getattr(kv, p).normal_(0.0, 1.0, generator=g)
        getattr(parts, p).copy_(getattr(kv, p))
    x = half(b, h1, std=2.0, mean=0.5)
    out = B.fg_decode_layer(cfg, B.LayerWeights(*mats, *ln, *bias), x, t, kv)

    qkv = B.fg_linear(mats[0], bias[0], B.fg_layernorm(x, ln[0], ln[1], 1e-5))
    B.fg_kv_append(cfg, qkv[:, h1:], qkv[:, 2 * h1:], 3 * h1, b, 1, parts, 0, t)
    o = B.fg_decode_attention(cfg, qkv, 3 * h1, b, t + 1, parts, 0)
    x1 = B.fg_linear(mats[1], bias[1], o, residual=x)
    act = B.fg_linear(mats[2], bias[2], B.fg_layernorm(x1, ln[2], ln[3], 1e-5), relu=True)
    assert torch.equal(kv.k_codes, parts.k_codes) and torch.equal(kv.v_codes, parts.v_codes)
    assert torch.equal(out, B.fg_linear(mats[3], bias[3], act, residual=x1))
