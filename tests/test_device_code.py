"""Properties of the gfx950 code in the built library that no result shows for certain."""
import os
import re
import shutil
import subprocess

from paper_2109_04312_amd import mate

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
MATRIX = re.compile(r"\s(v_mfma_\w+) (\S+), (\S+), (\S+), ([^\s/]+)")


def registers(operand):
    """(file, first, last) of a register operand; None for a constant."""
    m = re.fullmatch(r"([av])(?:\[(\d+):(\d+)\]|(\d+))", operand)
    return m and (m[1], int(m[2] or m[4]), int(m[3] or m[4]))


def partly_overlapping(line):
    """Does the line's matrix instruction write a part of the registers that its accumulator starts from, and others?"""
    m = MATRIX.search(line)
    result, start = m and registers(m[2]), m and registers(m[5])
    return bool(result and start and result != start and result[0] == start[0] and result[1] <= start[2] and start[1] <= result[2])


def device_code(tmp_path):
    library = shutil.copy(mate.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", library], check=True, capture_output=True, cwd=tmp_path)
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" in f:
            yield from subprocess.run([OBJDUMP, "-d", os.path.join(tmp_path, f)], check=True, capture_output=True,
                                      text=True).stdout.splitlines()


def test_what_counts_as_partly_overlapping():
    for line, overlaps in [(" v_mfma_f32_16x16x32_bf16 v[92:95], v[152:155], v[38:41], v[94:97]// 00000001D21C: D3B5005C 057A4D98", True),
                           (" v_mfma_f32_16x16x32_bf16 v[94:97], v[152:155], v[38:41], v[92:95]", True),
                           (" v_mfma_f32_16x16x32_bf16 v[92:95], v[152:155], v[38:41], v[92:95]", False),
                           (" v_mfma_f32_16x16x32_bf16 v[92:95], v[92:95], v[38:41], v[96:99]", False),
                           (" v_mfma_f32_16x16x32_bf16 v[92:95], v[152:155], v[38:41], a[94:97]", False),
                           (" v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], 0", False),
                           (" v_add_f32_e32 v1, v2, v3", False)]:
        assert partly_overlapping(line) == overlaps, line


def test_no_matrix_instruction_partly_overwrites_its_accumulator(tmp_path):
    matrix = [line for line in device_code(tmp_path) if MATRIX.search(line)]
    assert len(matrix) > 1000
    assert not [line.split("//")[0].strip() for line in matrix if partly_overlapping(line)]
