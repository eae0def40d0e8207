"""csrc/fg_gemm_fewrows.hip takes the arrival of a step's first weight register for the arrival of the activation copies
issued before it (loads complete in order).  That holds as long as no weight load is moved ahead of the copies, which the
kernel's fence between them forbids: the generated gfx950 code is looked at, every instantiation, every step."""
import os
import re
import subprocess

from paper_2303_06865_amd import build as FB


def test_activation_copies_are_issued_before_the_weights(tmp_path):
    src, asm = os.path.join(FB.CSRC, "fg_gemm_fewrows.hip"), str(tmp_path / "fewrows.s")
    subprocess.run([FB._hipcc(), *FB.COMMON, "--cuda-device-only", "-S", src, "-o", asm], check=True, capture_output=True)
    with open(asm) as f:
        text = f.read()
    kernels = re.findall(r"^\S*gemm_fewrows_kernelILi\d+ELi(\d+)E\S*:.*?\n(.*?)s_endpgm", text, re.S | re.M)
    assert len(kernels) >= 4 * 4 * 4   # formats, four-row pieces, column tiles
    for pieces, body in kernels:
        # C: an activation copy, F: the fence, W: a 16-byte weight load, in the order of the code
        seq = "".join("C" if m.group(0).startswith("global_load_lds") else "F" if m.group(0).startswith(";") else "W"
                      for m in re.finditer(r"global_load_lds_dwordx4|; activation copies issued|global_load_dwordx4\b", body))
        steps = re.findall(r"(C+)F(W+)", seq)
        assert steps and "".join("%sF%s" % s for s in steps) == seq, seq
        assert all(len(c) == int(pieces) for c, _ in steps), seq
