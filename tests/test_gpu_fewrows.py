"""fg_linear with up to 32 rows (csrc/fg_gemm_fewrows.hip) on every weight format, against the oracle: every number of
four-row pieces, every count of column tiles per workgroup and of waves, ragged columns, contractions of one group, of
an odd number of groups (the last step is half empty), shorter and longer than the steps the waves keep in flight."""
import pytest
import torch

from paper_2303_06865_amd import binding as B
from tests.test_gpu_kernels import _linear_case
from tests.util import assert_close

pytestmark = pytest.mark.gpu

# format: (quantized, tiled, FP16 pairs)
FORMATS = {"f16": (False, False, False), "q4": (True, False, False), "q4t": (True, True, False), "q4h": (True, True, True)}

CASES = [
    # m, n, k, bias, relu, residual
    (1, 32, 64, True, False, True),          # one group: one half-empty step, seven waves without work
    (4, 96, 192, False, True, False),
    (5, 544, 1984, True, False, True),       # 31 groups: 16 steps, two per wave, the last half empty
    (8, 160, 3072, True, True, False),       # three steps per wave
    (9, 256, 4160, False, False, True),      # 33 steps: four and five per wave
    (16, 2304, 768, True, False, True),
    (17, 768, 832, True, False, True),
    (32, 1056, 1024, True, True, True),
    (3, 7168, 128, True, False, False),      # two column tiles per workgroup
    (12, 12288, 64, False, False, True),     # three
    (16, 16384, 192, True, False, True),     # four
    (29, 12256, 128, False, False, True),    # three, ragged
    (2, 128, 8256, True, False, True),       # 65 steps: sixteen waves (tiled), eight (canonical); FP16: not this kernel
    (2, 832, 8256, True, False, True),       # ... this one again, with eight
    (13, 64, 16448, True, False, True),      # 129 steps
    (3, 1664, 16448, True, False, True),     # ... sixteen waves on FP16 weights too
    (7, 6144, 8256, True, False, False),     # sixteen waves, two column tiles (tiled)
]


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k,bias,relu,residual", CASES)
def test_linear_few_rows(m, n, k, bias, relu, residual, fmt):
    quant, tiled, h16 = FORMATS[fmt]
    got, ref = _linear_case(m, n, k, quant, bias, relu, residual, seed=m + n + k, tiled=tiled, meta_f16=h16)
    assert_close(got, ref, "few rows m=%d n=%d k=%d %s" % (m, n, k, fmt))


@pytest.mark.parametrize("quant", [True, False])
@pytest.mark.parametrize("m,n", [(1, 8), (6, 1000), (31, 264)])
def test_linear_few_rows_columns_not_a_multiple_of_16(m, n, quant):
    got, ref = _linear_case(m, n, 320, quant, True, False, True, seed=m + n)
    assert_close(got, ref, "few rows m=%d n=%d q=%s" % (m, n, quant))


# more rows of a small matrix: blocks of 32 rows, the last one with one row or all but one, up to the rows and sizes at
# which the other kernels take over (tests/test_gpu_split_k.py has those)
@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", [(33, 96, 192), (63, 2304, 768), (64, 1056, 1984), (129, 800, 448), (1023, 64, 256),
                                   (1024, 544, 64)])
def test_linear_blocks_of_rows(m, n, k, fmt):
    quant, tiled, h16 = FORMATS[fmt]
    got, ref = _linear_case(m, n, k, quant, True, True, True, seed=m + n + k, tiled=tiled, meta_f16=h16)
    assert_close(got, ref, "blocks of rows m=%d n=%d k=%d %s" % (m, n, k, fmt))


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", [(1, 64, 64), (6, 96, 192), (16, 2304, 832), (31, 288, 1984)])
def test_infinite_weight_in_the_half_empty_last_step(m, n, k, fmt):
    """An infinite weight in the last group of an odd number of groups: infinity in its column (the activations are
    positive), the other columns as they are.  The lanes that have no elements in that step must not bring it in."""
    quant, tiled, h16 = FORMATS[fmt]
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    w, x = half(n, k) * 0.05, half(m, k).abs() + 0.01
    mat = B.Mat.from_f16(w, quant, meta_f16=h16)
    if quant:
        ref = B.fg_dequantize_groupwise(*B.fg_quantize_groupwise(w, meta_f16=h16)).view(n, k).half().float()
        mat.meta.view(n, k // 64, 2)[5, -1] = torch.tensor([float("inf"), 0.0])   # {min, scale}: the whole group
        mat = mat.tiled() if tiled else mat
    else:
        ref = w.float().clone()
        mat.data[5, k - 7] = float("inf")
    out = B.fg_linear(mat, None, x).float()
    want = x.float() @ ref.t()
    assert bool((out[:, 5] == float("inf")).all())
    keep = torch.arange(n) != 5
    assert_close(out[:, keep].cpu().numpy(), want[:, keep].cpu().numpy(), "beside an infinite column, %s" % fmt)
