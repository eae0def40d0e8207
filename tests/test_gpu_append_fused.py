"""The decode layer of few heads, whose attention stores the token's own cache row (csrc/fg_attn_decode.hip), against the same
layer put together from fg_kv_append and fg_decode_attention, bit for bit: the row first, last and alone in a chunk, with one,
two, four and eight waves per head, at both sides of the line between the two ways; what the cache held in the row's place is
not a number."""
import pytest
import torch

from paper_2303_06865_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kvf", ["q4", "q4h", "f16"])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("b,nh,t", [(1, 1, 0), (3, 1, 63), (2, 3, 64), (4, 12, 40), (5, 5, 127), (33, 8, 128), (130, 8, 129),
                                    (1, 9, 1400), (9, 7, 319), (1030, 1, 9), (64, 32, 70), (65, 32, 200), (16, 32, 90), (57, 9, 90), (20, 15, 639)])
def test_decode_layer_appends(b, nh, t, dh, kvf):
    h1, off = nh * dh, 2
    g = torch.Generator(device="cuda").manual_seed(b * 1000 + t)
    half = lambda *s, std=1.0: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, std, generator=g)
    cfg = B.Cfg(h1, nh, 64, 1000, 4096)
    mats = [B.Mat.from_f16(half(n, k, std=0.1), False) for n, k in ((3 * h1, h1), (h1, h1), (64, h1), (h1, 64))]
    ones, zeros = torch.ones(h1, dtype=torch.float16, device="cuda"), torch.zeros(h1, dtype=torch.float16, device="cuda")
    caches = [B.KVCache(cfg, b + off, t + 2, kvf != "f16", meta_f16=kvf == "q4h") for _ in range(2)]
    for p in ("k_codes", "v_codes", "k_meta", "v_meta"):
        c, d = getattr(caches[0], p), getattr(caches[1], p)
        if c is None:
            continue
        if c.dtype == torch.uint8:
            c.random_(0, 256, generator=g)
        else:
            c.normal_(0.0, 0.3, generator=g)
            c[:, :, t:] = float("nan")
        d.copy_(c)
    x = half(b, h1)
    out = B.fg_decode_layer(cfg, B.LayerWeights(*mats, ones, zeros, ones, zeros), x, t, caches[0], batch_offset=off)

    qkv = B.fg_linear(mats[0], None, B.fg_layernorm(x, ones, zeros, 1e-5))
    B.fg_kv_append(cfg, qkv[:, h1:], qkv[:, 2 * h1:], 3 * h1, b, 1, caches[1], off, t)
    o = B.fg_decode_attention(cfg, qkv, 3 * h1, b, t + 1, caches[1], off)
    x1 = B.fg_linear(mats[1], None, o, residual=x)
    act = B.fg_linear(mats[2], None, B.fg_layernorm(x1, ones, zeros, 1e-5), relu=True)
    assert torch.equal(out, B.fg_linear(mats[3], None, act, residual=x1))
    assert bool(torch.isfinite(out).all())
    for p in ("k_codes", "v_codes", "k_meta", "v_meta"):
        c, d = getattr(caches[0], p), getattr(caches[1], p)
        if c is not None:
            bits = {1: torch.uint8, 2: torch.int16, 4: torch.int32}[c.element_size()]
            assert torch.equal(c.view(bits), d.view(bits)), p
