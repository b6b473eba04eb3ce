"""The 6-bit GEMM's accumulators in the compiled code (CPU only).

Its matrix instructions are inline assembly, for which the compiler adds no
waits: the source keeps the distances.  The kernels' assembly is scanned in
layout order for the shortest one between a matrix instruction and a read of
an accumulation register by anything else (at most 19 wait states are needed,
for the longest instructions) and between a write of one and the next matrix
instruction (the 8 of the source's s_nop)."""
import os
import re
import subprocess

import pytest

from paper_2609_34867_amd import build

SRC = os.path.join(build.CSRC, "w4a4_f6.hip")


def distances(asm):
    """{kernel: (accumulator reads, least wait states MFMA -> read, write -> MFMA)}"""
    out, kern = {}, None
    for line in asm.splitlines():
        t = line.split(";")[0].strip()
        if m := re.match(r"(_Z\S*k_w4a4_gemm_f6\S*):$", t):
            kern, reads, to_read, to_mfma = m.group(1), 0, 10 ** 9, 10 ** 9
            since_mfma = since_write = 10 ** 9
        elif kern and t.startswith(".Lfunc_end"):
            out[kern], kern = (reads, to_read, to_mfma), None
        elif kern and t and not t.startswith(".") and not t.endswith(":"):
            op = t.split()[0]
            if op.startswith("v_mfma"):
                to_mfma, since_mfma, since_write = min(to_mfma, since_write), 0, 10 ** 9
                continue
            if op.startswith("v_accvgpr_write"):
                since_write = -1
            elif re.search(r"\ba(\d+|\[\d+:\d+\])", t):
                reads, to_read = reads + 1, min(to_read, since_mfma)
            n = int(t.split()[1], 0) + 1 if op == "s_nop" else 1
            since_mfma, since_write = since_mfma + n, since_write + n
    return out


def test_distances_to_the_matrix_instructions(tmp_path):
    if not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("no hipcc")
    asm = tmp_path / "f6.s"
    subprocess.run(["/opt/rocm/bin/hipcc", *build.HIPCC_FLAGS, "--cuda-device-only", "-S", SRC, "-o",
                    str(asm)], check=True, capture_output=True)
    found = distances(asm.read_text())
    assert len(found) == 4
    for kern, (reads, to_read, to_mfma) in found.items():
        assert reads >= 256, kern
        assert to_read >= 19, (kern, to_read)
        assert 8 <= to_mfma < 10 ** 9, (kern, to_mfma)
