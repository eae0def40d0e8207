"""What the projection kernels rely on their generated gfx950 code for, looked at in that code."""
import os
import re
import subprocess

import pytest

from paper_2303_06865_amd import build as FB


def _code(source, folder):
    asm = str(folder / (source + ".s"))
    subprocess.run([FB._hipcc(), *FB.COMMON, "--cuda-device-only", "-S", os.path.join(FB.CSRC, source), "-o", asm],
                   check=True, capture_output=True)
    with open(asm) as f:
        return f.read()


@pytest.fixture(scope="module")
def stream_code(tmp_path_factory):
    return _code("fg_gemm_stream.hip", tmp_path_factory.mktemp("asm"))


@pytest.fixture(scope="module")
def tiles_code(tmp_path_factory):
    return _code("fg_gemm_f16_tiles.hip", tmp_path_factory.mktemp("asm"))


def test_whole_tiles_without_a_residual_store_without_waits(stream_code):
    """A lane stores one piece of each of its 16 RG rows of a finished tile, in FP16 or in FP32.  Where no residual is added
    none of these stores may wait for the memory (that would be for the store before it)."""
    kernels = re.findall(r"^\S*gemm_prefill16(?:_f16)?_kernelILi(\d+)E\S*:.*?\n(.*?)s_endpgm", stream_code, re.S | re.M)
    assert len(kernels) == 6   # 192 and 256 rows; FP16 weights, FP32 and FP16 pairs
    for rg, body in kernels:
        seq = "".join("S" if m.group(0).startswith("global") else "W"
                      for m in re.finditer(r"global_store_dword(?:x2)?\b|s_waitcnt[^\n]*vmcnt", body))
        assert max(len(run) for run in seq.split("W")) >= 2 * 16 * int(rg) - 2, seq   # (the first of either follows the bias)


def _registers(text):
    out = set()
    for m in re.finditer(r"\bv(?:(\d+)|\[(\d+):(\d+)\])", text):
        out.update([int(m[1])] if m[1] else range(int(m[2]), int(m[3]) + 1))
    return out


def _blocks(body):
    """[label, [(instruction, hand-placed)]], cut at labels and behind branches"""
    blocks, by_hand = [["", []]], False
    for line in body.splitlines():
        line = line.strip()
        if line.startswith(";;#ASM"):
            by_hand = line.startswith(";;#ASMSTART")
            continue
        label = re.match(r"(\.L\w+):", line)
        if label:
            blocks.append([label[1], []])
            continue
        code = line.split(";")[0].strip()
        if code and not code.startswith("."):
            blocks[-1][1].append((code, by_hand))
            if re.match(r"s_c?branch|s_endpgm", code):
                blocks.append(["", []])
    return blocks


def _reads_in_flight(body):
    """Follows every path of a kernel.  Hand-placed LDS reads, and instructions that touch a register of one before a wait
    for all of them, and branches before it."""
    blocks = _blocks(body)
    at = {b[0]: i for i, b in enumerate(blocks) if b[0]}
    state, touched, branches = {0: frozenset()}, [], []

    def follow(i, record):
        flight, next_blocks, falls = set(state[i]), [], True
        for code, by_hand in blocks[i][1]:
            op = code.split()[0]
            if op == "s_waitcnt" and "lgkmcnt(0)" in code:
                flight.clear()
            elif op.startswith("s_cbranch") or op == "s_branch":
                if record and flight:
                    branches.append(code)
                next_blocks.append(at[code.split()[1]])
                falls = op != "s_branch"
            elif op == "s_endpgm":
                falls = False
            else:
                if record and flight & _registers(code):
                    touched.append(code)
                if by_hand and op.startswith("ds_read"):
                    flight |= _registers(code.split(",")[0])
        return flight, next_blocks + ([i + 1] if falls and i + 1 < len(blocks) else [])

    todo = [0]
    while todo:
        flight, next_blocks = follow(todo.pop(), False)
        for b in next_blocks:
            if b not in state or not flight <= state[b]:
                state[b] = frozenset(flight | state.get(b, frozenset()))
                todo.append(b)
    for i in list(state):
        follow(i, True)
    reads = sum(by_hand and code.startswith("ds_read") for b in blocks for code, by_hand in b[1])
    return reads, touched, branches


def _kernels(text):
    return re.findall(r"^(_ZN\S*_kernel\S*):[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M)


def test_reads_in_flight_are_seen():
    """The search itself: a register used before the wait on one of two paths, and on none."""
    code = """\ts_cbranch_scc0 .LBB0_1
\t;;#ASMSTART
\tds_read_b128 v[4:7], v1 offset:16
\t;;#ASMEND
.LBB0_1:
\t%s
\ts_waitcnt lgkmcnt(0)
\tv_add_f32_e32 v0, v5, v2
\ts_cbranch_scc1 .LBB0_1
\ts_endpgm
"""
    assert _reads_in_flight(code % "v_mov_b32_e32 v3, v6") == (1, ["v_mov_b32_e32 v3, v6"], [])
    assert _reads_in_flight(code % "s_cbranch_scc0 .LBB0_1") == (1, [], ["s_cbranch_scc0 .LBB0_1"])
    assert _reads_in_flight(code % "v_mov_b32_e32 v3, v8") == (1, [], [])


def test_no_register_of_an_lds_read_in_flight_is_touched(stream_code, tiles_code, tmp_path):
    """The compiler takes the registers of hand-placed LDS reads as written at once."""
    found = 0
    for text in (stream_code, tiles_code, _code("fg_gemm_f16w.hip", tmp_path)):
        for name, body in _kernels(text):
            reads, touched, branches = _reads_in_flight(body)
            found += reads > 0
            assert not touched, (name, touched[:4])
            # gemm_decode16h_kernel chooses between two dequantizations in every step
            if "gemm_decode16h_kernel" in name or "gemm_f16_tiles_kernel" in name:
                assert reads and not branches, (name, branches)
    assert found >= 60


def test_lanes_that_exchange_through_lds_are_fenced(tiles_code, tmp_path):
    """Where a wave's lanes read from LDS what its other lanes wrote, with no barrier of the workgroup between, a barrier of the
    wave stands there, which is no instruction but holds the compiler: the finished sums of the FP16 tiles, and the new cache
    row of the decode attention that stores it."""
    for name, body in _kernels(tiles_code):
        if "gemm_f16_tiles_kernel" in name:
            tail = body[body.rindex("; wave barrier"):] if "; wave barrier" in body else body
            first = body.index("ds_write")
            assert first < len(body) - len(tail) and "ds_read" in tail and "ds_write" not in tail, name
            assert "ds_read" not in body[first:len(body) - len(tail)], name
    stores = [(name, body) for name, body in _kernels(_code("fg_attn_decode.hip", tmp_path))
              if re.search(r"attn_decode_q4_kernelILi\d+ELi\d+ELb[01]ELb0ELb1E", name)]
    assert len(stores) == 16   # two head sizes, one to eight waves per head, FP32 and FP16 pairs
    assert all("; wave barrier" in body for _, body in stores)


def test_residual_is_on_its_way_with_the_partial_sums(stream_code, tiles_code):
    """The reduction passes ask for the residual's four rows, and wait for none of them before they ask for partial sums."""
    finish = [(name, body) for text in (stream_code, tiles_code) for name, body in _kernels(text) if "_finish_kernel" in name]
    assert len(finish) == 5   # one and two items per thread on two layouts, and the FP16 tiles'
    for name, body in finish:
        kinds = {"global_load_ushort": "R", "global_load_dwordx4": "P"}
        seq = "".join(kinds.get(m.group(0), "W") for m in re.finditer(r"global_load_ushort|global_load_dwordx4|s_waitcnt[^\n]*vmcnt", body))
        assert "RRRR" in seq and "P" in seq, name
        assert not re.search("RRRRR*W", seq), (name, seq)
