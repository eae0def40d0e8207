"""What csrc/fg_gemm_stream.hip relies on its generated gfx950 code for, looked at in that code."""
import os
import re
import subprocess

import pytest

from paper_2303_06865_amd import build as FB


@pytest.fixture(scope="module")
def stream_code(tmp_path_factory):
    asm = str(tmp_path_factory.mktemp("asm") / "stream.s")
    subprocess.run([FB._hipcc(), *FB.COMMON, "--cuda-device-only", "-S", os.path.join(FB.CSRC, "fg_gemm_stream.hip"), "-o", asm],
                   check=True, capture_output=True)
    with open(asm) as f:
        return f.read()


def test_whole_tiles_without_a_residual_store_without_waits(stream_code):
    """A lane stores one piece of each of its 16 RG rows of a finished tile, in FP16 or in FP32.  Where no residual is added
    none of these stores may wait for the memory (that would be for the store before it)."""
    kernels = re.findall(r"^\S*gemm_prefill16(?:_f16)?_kernelILi(\d+)E\S*:.*?\n(.*?)s_endpgm", stream_code, re.S | re.M)
    assert len(kernels) == 6   # 192 and 256 rows; FP16 weights, FP32 and FP16 pairs
    for rg, body in kernels:
        seq = "".join("S" if m.group(0).startswith("global") else "W"
                      for m in re.finditer(r"global_store_dword(?:x2)?\b|s_waitcnt[^\n]*vmcnt", body))
        assert max(len(run) for run in seq.split("W")) >= 2 * 16 * int(rg) - 2, seq   # (the first of either follows the bias)
