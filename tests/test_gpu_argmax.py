"""Greedy token over rows of logits (csrc/fg_norm.hip: argmax_kernel): widths around what its threads
take in one pass, widths and addresses that it has to read element by element, ties between far columns."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2303_06865_amd import binding as B
from tests.util import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("vocab", [8, 256, 264, 1000, 1024, 1032, 2048, 2056, 4096, 4104, 8192, 8200, 16384, 16392, 50272, 65536,
                                   65544, 131080])
def test_argmax_is_the_lowest_index_of_the_maximum(vocab, offset):
    """Every embedding row that attains the largest logit occurs at three columns, one near the end; with
    offset 1 the logits start 4 bytes off a 16-byte boundary."""
    rows, h1 = 5 if vocab >= 1000 else 1, 64   # (few columns hold the three of one row)
    cfg = B.Cfg(h1, 1, 64, vocab, 8)
    g = torch.Generator(device="cuda").manual_seed(vocab)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    x, gamma, beta, emb = half(rows, h1), half(h1), half(h1), half(vocab, h1)
    for r in range(rows):                     # the row's strongest embedding, at three columns
        at = [7 * r + 3, vocab // 2 + r, vocab - 1 - r]
        y = torch.nn.functional.layer_norm(x[r].float(), (h1,), gamma.float(), beta.float())
        emb[at] = (3.0 * y.sign()).half()
    buf = torch.empty(rows * vocab + 1, dtype=torch.float32, device="cuda")
    logits = buf[offset:offset + rows * vocab].view(rows, vocab)
    ids = torch.empty(rows, dtype=torch.int32, device="cuda")
    n = B.lib().fg_lm_head_workspace_bytes(C.byref(cfg.c), rows)
    ws = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
    p = lambda t: C.c_void_p(t.data_ptr())
    rc = B.lib().fg_lm_head_greedy(C.byref(cfg.c), p(x), h1, rows, p(gamma), p(beta), p(emb), p(ids), 1, p(logits), p(ws),
                                   n, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    lg = host(logits)
    assert (lg == lg.max(axis=1, keepdims=True)).sum(axis=1).min() == 3   # the ties are there
    assert np.array_equal(host(ids), np.argmax(lg, axis=1).astype(np.int32))
