"""LayerNorm's results are the same bits whichever kernel normalizes a row (csrc/fg_norm.hip, or a projection that takes the
LayerNorm in, csrc/fg_gemm_fewrows_ln.hip).  So which products are rounded before they are added is written in the source, and
not left to what the compiler makes of a * b + c: with and without leave to fuse, the generated code is the same.  And a result
is rounded to binary32 before it is rounded to FP16 (where an instruction that rounds once is used, it dequantizes weights)."""
import os
import re
import subprocess

import pytest

from paper_2303_06865_amd import build as FB


@pytest.mark.parametrize("source", ["fg_norm.hip", "fg_gemm_fewrows_ln.hip"])
def test_nothing_is_left_to_contraction(source, tmp_path):
    codes = []
    for contract in ("fast", "off"):
        asm = str(tmp_path / contract)
        subprocess.run([FB._hipcc(), *FB.COMMON, "-ffp-contract=" + contract, "--cuda-device-only", "-S",
                        os.path.join(FB.CSRC, source), "-o", asm], check=True, capture_output=True)
        with open(asm) as f:
            codes.append(f.read())
    instructions = [re.findall(r"^\t[a-z]+_.*", code, re.M) for code in codes]
    assert len(instructions[0]) > 1000 and instructions[0] == instructions[1]
    normalize = [body for name, body in re.findall(r"^(_ZN\S*):[^\n]*\n(.*?)^\.Lfunc_end", codes[0], re.S | re.M)
                 if re.search("layernorm_(reg_)?kernel|gemm_fewrows_ln_kernelILi0E", name)]   # (0: FP16 weights)
    assert len(normalize) >= 5
    assert not any("v_fma_mixlo" in body or "v_fma_mixhi" in body for body in normalize)
