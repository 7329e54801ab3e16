"""The matrix instructions of the tiled kernel and of the matrix loop that it is measured against stand in inline assembly,
where the compiler adds none of the wait states that they need: read from the assembly of the kernels' own build that every
one of them has its wait states all the same."""
import os
import re
import subprocess

import pytest

from paper_2503_06823_amd import build as B

# source, kernel, its instances: three epilogues, K with and without a tail; with and without fragment reads
KERNELS = [("ffn_bf16_tiled.hip", "grouped_gemm_bf16", 6), ("peaks.hip", "mfma_loop_kernel", 2)]
VALU_TO_MFMA = 2   # wait states from a VALU write of a vector register to a matrix instruction that reads it
MFMA_TO_READ = 18  # from a matrix instruction to a read of its result, the longest of all shapes


@pytest.fixture(scope="module", params=KERNELS, ids=lambda p: p[1])
def kernels(tmp_path_factory, request):
    """name -> instructions of every instance of a kernel, as text, inline assembly and labels as they come"""
    source, kernel, instances = request.param
    out = tmp_path_factory.mktemp("asm") / "kernel.s"
    subprocess.run([B._hipcc(), *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, source), "-o", str(out)], check=True,
                   capture_output=True)
    found, lines, name = {}, None, None
    for line in open(out):
        m = re.match(r"(_ZN4emoe\S*" + kernel + r"\S*):", line)
        if m:
            name, lines = m.group(1), []
        elif line.startswith(".Lfunc_end") and lines is not None:
            found[name] = lines
            lines = None
        elif lines is not None:
            text = line.split(";")[0].strip() if "#ASM" not in line else line.strip().lstrip(";")
            if text and not text.startswith("."):
                lines.append(text)
    assert len(found) == instances, sorted(found)
    return found


def registers(operand, bank):
    """the registers of `bank` ("v" or "a") that an operand names"""
    m = re.fullmatch(bank + r"\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(bank + r"(\d+)", operand)
    return {int(m.group(1))} if m else set()


def operands(text):
    return [o.strip() for o in text.split(None, 1)[1].split(",")] if " " in text or "\t" in text else []


def wait_states(text):
    if text.startswith("#"):
        return 0
    m = re.match(r"s_nop (\d+)", text)
    return int(m.group(1)) + 1 if m else 1


def test_operands_are_written_long_enough_before(kernels):
    for name, code in kernels.items():
        n = 0
        for i, text in enumerate(code):
            if not text.startswith("v_mfma"):
                continue
            n += 1
            ops = operands(text)
            read = registers(ops[1], "v") | registers(ops[2], "v")
            assert read, text
            states, j = 0, i - 1
            while states < VALU_TO_MFMA and j >= 0:
                before = code[j]
                if before.startswith("v_") and not before.startswith(("v_mfma", "v_cmp")):
                    written = registers(operands(before)[0], "v")
                    if before.startswith("v_permlane") or before.startswith("v_swap"):
                        written |= registers(operands(before)[1], "v")
                    assert not written & read, f"{name}: '{before}' {states} wait states before '{text}'"
                states += wait_states(before)
                j -= 1
        assert n >= 3 * 64, name


def test_clearing_instructions_bring_their_own_wait_states(kernels):
    """Their operand is a constant, which the compiler may write again at any place between them."""
    for name, code in kernels.items():
        n = 0
        for i, text in enumerate(code):
            if text.startswith("v_mfma") and operands(text)[3] == "0":
                n += 1
                assert code[i - 1].startswith("s_nop") and wait_states(code[i - 1]) >= VALU_TO_MFMA, f"{name}: {text}"
                assert code[i - 2].startswith("#ASMSTART"), f"{name}: {text}"
        assert n >= 64, name


def test_accumulators_are_matrix_results_read_long_enough_after(kernels):
    for name, code in kernels.items():
        reads = 0
        for i, text in enumerate(code):
            if text.startswith("#") or not re.search(r"\ba(\d+|\[)", text):
                continue
            if text.startswith("v_accvgpr_read"):
                reads += 1
                states, j = 0, i - 1
                while states < MFMA_TO_READ and j >= 0:
                    assert not code[j].startswith("v_mfma"), f"{name}: '{text}' {states} wait states after '{code[j]}'"
                    states += wait_states(code[j])
                    j -= 1
            else:  # nothing else touches an accumulator: no copies, no loads, no spills
                assert text.startswith("v_mfma"), f"{name}: {text}"
        assert reads >= 64 * 4, name
