"""Required distances between instructions in the built library.  The compiler keeps them for what it selects itself; the result of
inline assembly it does not count as a vector operation's, so nothing but the schedule separates it from an instruction that needs
wait states behind such a result.  No GPU is needed: the library's own gfx950 code is disassembled."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_05176_amd", "libpatternkv.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(OBJDUMP), reason="no built library or no disassembler")


def _registers(text):
    out = set()
    for one, lo, hi in re.findall(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]", text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def _too_close(asm, needed=2):
    """(reads of the three kinds, those with fewer than `needed` wait states behind the vector operation that wrote them)"""
    kernel, seen, bad, recent = None, {"lane swap": 0, "lane permutation": 0, "matrix": 0}, [], []
    for line in asm.splitlines():
        line = line.split("//")[0].strip()
        start = re.match(r"^[0-9a-f]* ?<(.*)>:", line)
        if start:
            kernel, recent = start.group(1), []
            continue
        op, _, rest = line.partition(" ")
        if not op or not re.match(r"[a-z]+_", op):
            continue
        operands = [o.strip() for o in rest.split(",")]
        swap, matrix = op.startswith("v_permlane"), op.startswith("v_mfma")
        kind, reads = None, set()
        if swap:
            kind, reads = "lane swap", _registers(rest)
        elif matrix:
            kind, reads = "matrix", _registers(",".join(operands[1:]))
        elif re.search(r"\b(quad_perm|row_\w+|wave_\w+):|\brow_(half_)?mirror\b", rest):
            kind, reads = "lane permutation", _registers(operands[1].split(" ")[0])
        if kind:
            seen[kind] += 1
            for written, distance, by in recent:
                if written & reads and distance < needed:
                    bad.append((kernel, kind, distance, by, line))
                    break
        step = 1 + int(rest) if op == "s_nop" else 1
        recent = [(w, d + step, by) for w, d, by in recent if d + step < needed]
        if op.startswith("v_") and not matrix and not op.startswith(("v_cmp", "v_readlane", "v_readfirstlane", "v_dot")):
            recent.insert(0, (_registers(operands[0]) | (_registers(operands[1]) if "swap" in op else set()), 0, line))
    return seen, bad


def test_the_check_sees_a_missing_wait():
    head = "0 <kernel>:\n v_max_f32_e32 v5, v5, v6\n"
    assert len(_too_close(head + " v_permlane32_swap_b32_e32 v4, v5\n")[1]) == 1
    assert len(_too_close(head + " s_nop 0\n v_permlane32_swap_b32_e32 v4, v5\n")[1]) == 1
    assert len(_too_close(head + " s_nop 1\n v_permlane32_swap_b32_e32 v4, v5\n")[1]) == 0
    assert len(_too_close(head + " v_mov_b32_e32 v1, v2\n v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], v[0:3]\n")[1]) == 1
    assert len(_too_close(head + " v_mov_b32_dpp v1, v5 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n")[1]) == 1


def test_vector_results_are_not_read_too_early(tmp_path):
    """Two wait states from a vector operation to a lane swap, a permuted operand or a matrix operation that reads its result."""
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    images = [f for f in sorted(os.listdir(tmp_path)) if f.endswith("gfx950") and os.path.getsize(tmp_path / f)]
    assert images
    total, bad = {}, []
    for f in images:
        r = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", "--no-leading-addr", f], cwd=tmp_path, check=True,
                           capture_output=True, text=True)
        seen, found = _too_close(r.stdout)
        bad += found
        total = {k: total.get(k, 0) + n for k, n in seen.items()}
    assert all(total.values()), total
    assert not bad, (len(bad), bad[:4])
