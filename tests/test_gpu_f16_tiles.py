"""fg_linear on FP16 weights from 33 rows up (csrc/fg_gemm_f16_tiles.hip) against binary32: every tile shape, with the contraction
whole and in two, four and eight ranges, fewer steps than the stages that are copied ahead, rows and columns that end inside a
tile.  That a size runs there, and on which tiles, is asked of the library's own rule; tests/test_f16_tiles_lines.py has sizes
on both sides of it, tests/test_gpu_split_k.py what the former kernels keep."""
import pytest
import torch

from paper_2303_06865_amd import binding as B
from tests import routes
from tests.util import assert_close

pytestmark = pytest.mark.gpu

CASES = [
    # m, n, k, (tile rows / 32, tile columns / 32, ranges of the contraction)
    (1500, 32, 320, (1, 2, 1)),       # one column tile of which half is there
    (1500, 32, 2048, (1, 2, 4)),
    (1500, 32, 64, (2, 2, 1)),        # a single step
    (2049, 32, 3072, (2, 2, 4)),      # one row in the last block
    (1500, 32, 4096, (2, 2, 8)),
    (2049, 512, 64, (2, 3, 1)),
    (33, 8224, 8192, (2, 3, 2)),      # 33 rows, the fewest
    (33, 6144, 4096, (2, 3, 4)),
    (33, 2080, 8192, (2, 3, 8)),
    (129, 8224, 2048, (2, 4, 1)),
    (3000, 512, 64, (3, 2, 1)),
    (65, 6144, 4096, (3, 2, 2)),
    (2049, 96, 4096, (3, 2, 4)),
    (2049, 32, 4096, (3, 2, 8)),
    (2049, 768, 128, (4, 2, 1)),      # two steps
    (1500, 288, 8192, (4, 2, 4)),
    (97, 21504, 1088, (4, 4, 1)),     # 96 rows and one
    (128, 20512, 1024, (4, 4, 1)),    # 128 rows, a last column tile of 32
    (66, 17408, 7168, (4, 3, 1)),
    (2049, 1056, 192, (4, 4, 1)),     # three steps
    (100, 4128, 8192, (4, 4, 4)),
    (333, 1056, 8192, (4, 4, 8)),
    (2049, 2080, 64, (6, 3, 1)),
    (129, 8224, 4096, (6, 3, 2)),
    (129, 4128, 8192, (6, 3, 4)),
    (192, 2080, 8256, (6, 3, 8)),     # ranges of 16 and 17 steps
    (193, 2080, 8256, (3, 2, 2)),     # ... and one row more
    (2048, 2304, 256, (6, 4, 1)),     # four steps
    (385, 12288, 1984, (8, 4, 1)),
    (1500, 4128, 320, (8, 4, 1)),
    (257, 20512, 704, (4, 4, 1)),
]


def _inputs(m, n, k):
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    return half(n, k) * 0.05, half(m, k), half(n), half(m, n)


@pytest.mark.parametrize("m,n,k,tile", CASES)
def test_linear_f16_tiles(m, n, k, tile):
    assert all(routes.f16_tiles(n, k, m, residual) for residual in (True, False)) and not routes.few_rows(B.FG_F16, n, k, m)
    assert routes.f16_tile(n, k, m) == tile
    w, x, bias, res = _inputs(m, n, k)
    mat = B.Mat.from_f16(w, False)
    # the sums, then the results rounded to FP16: 2^-11 of up to about 5 sqrt(k) 0.05 in single values, 1e-2 at sums up to 20
    y = x.float() @ w.float().t() + bias.float()
    got = B.fg_linear(mat, bias, x, residual=res, relu=True)
    top = float(y.abs().max()) + 5.0
    want = torch.relu(y) + res.float()
    assert_close(got.cpu().numpy(), want.cpu().numpy(), "m=%d n=%d k=%d" % (m, n, k), mabs=max(1e-2, top * 2.0 ** -11))
    plain = B.fg_linear(mat, None, x)
    assert_close(plain.cpu().numpy(), (x.float() @ w.float().t()).cpu().numpy(), "m=%d n=%d k=%d plain" % (m, n, k),
                 mabs=max(1e-2, top * 2.0 ** -11))
    assert torch.equal(B.fg_linear(mat, None, x), plain)   # the same bits on every call


@pytest.mark.parametrize("m,n,k,few", [(333, 4096, 4096, False), (512, 7168, 7168, False), (100, 4128, 8192, False),
                                       (129, 8224, 2048, False), (333, 1056, 8192, False), (200, 2304, 768, True)])
def test_bias_and_residual_at_any_address(m, n, k, few):
    """Both are FP16 arrays without an alignment of their own: one element past a 16-byte boundary the results are the same bits,
    from whole contractions and from ranges of them, and from the few-rows kernel."""
    assert routes.f16_tiles(n, k, m) and routes.few_rows(B.FG_F16, n, k, m) == few
    w, x, bias, res = _inputs(m, n, k)
    off = lambda t: torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape)
    b1, r1 = off(bias), off(res)
    assert b1.data_ptr() % 16 and r1.data_ptr() % 16
    mat = B.Mat.from_f16(w, False)
    want = B.fg_linear(mat, bias, x, residual=res)
    for b, r in ((b1, r1), (bias, r1), (b1, res)):
        assert torch.equal(B.fg_linear(mat, b, x, residual=r), want)


def test_logits_at_any_address():
    rows, vocab, h1 = 100, 34016, 768
    assert routes.f16_tiles(vocab, h1, rows) and not routes.few_rows(B.FG_F16, vocab, h1, rows)
    g = torch.Generator(device="cuda").manual_seed(3)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    cfg = B.Cfg(h1, h1 // 64, 4 * h1, vocab, 64)
    emb, x = half(vocab, h1), half(rows, h1)
    ones, zeros = torch.ones(h1, dtype=torch.float16, device="cuda"), torch.zeros(h1, dtype=torch.float16, device="cuda")
    ids, logits = B.fg_lm_head_greedy(cfg, x, ones, zeros, emb)
    ids1, buf = torch.empty_like(ids), torch.zeros(rows * vocab + 2, dtype=torch.float32, device="cuda")
    n = B.lib().fg_lm_head_workspace_bytes(B.C.byref(cfg.c), rows)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    rc = B.lib().fg_lm_head_greedy(B.C.byref(cfg.c), x.data_ptr(), h1, rows, ones.data_ptr(), zeros.data_ptr(), emb.data_ptr(),
                                   ids1.data_ptr(), 1, buf.data_ptr() + 4, ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert torch.equal(buf[1:-1], logits.view(-1)) and torch.equal(ids1, ids)
    assert buf[0] == 0 and buf[-1] == 0


@pytest.mark.parametrize("rows,vocab,h1", [(100, 34016, 768), (129, 20000, 768), (300, 8032, 1024), (512, 33024, 320)])
def test_lm_head_rows(rows, vocab, h1):
    assert routes.f16_tiles(vocab, h1, rows, False) and not routes.few_rows(B.FG_F16, vocab, h1, rows)
    g = torch.Generator(device="cuda").manual_seed(rows + vocab)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    cfg = B.Cfg(h1, h1 // 64, 4 * h1, vocab, 64)
    emb, x = half(vocab, h1), half(rows, h1)
    ones, zeros = torch.ones(h1, dtype=torch.float16, device="cuda"), torch.zeros(h1, dtype=torch.float16, device="cuda")
    ids, logits = B.fg_lm_head_greedy(cfg, x, ones, zeros, emb)
    want = B.fg_layernorm(x, ones, zeros, 1e-5).float() @ emb.float().t()
    # binary32 sums in another order: about sqrt(h1) 2^-24 of sums of h1 products of about 1
    assert float((logits.view(rows, vocab) - want).abs().max()) <= 1e-3
    best = logits.view(rows, vocab).max(1).values
    assert torch.equal(logits.view(rows, vocab).gather(1, ids.long().view(-1, 1))[:, 0], best)
