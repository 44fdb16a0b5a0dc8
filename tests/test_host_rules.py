"""Host-side sizing rules of the HIP library, compiled for the CPU from its header.

Rows of the cells' expansions start on 16 bytes at every maximum degree that a
context accepts."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1712_10116_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")


def _run(tmp_path, body):
    src = tmp_path / "rules.hip"
    src.write_text('#include "common.h"\n#include <stdio.h>\nint main() {\n%s\n}\n' % body)
    exe = str(tmp_path / "rules")
    subprocess.run([HIPCC, "-std=c++17", "-O0", "--cuda-host-only", "-Wno-unused-value",
                    "-Wno-unused-result", "-I", CSRC, str(src), "-o", exe], check=True,
                   capture_output=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()


def test_rows_start_on_16_bytes(tmp_path):
    out = _run(tmp_path, 'for (int p = 1; p <= 8; ++p) printf("%d %d ", coeff_row(p), folded_row(p));')
    for p in range(1, 9):
        coeffs, folded = int(out[2 * p - 2]), int(out[2 * p - 1])
        for row, values in ((coeffs, (p + 1) * (p + 2) * (p + 3) // 6), (folded, (p + 1) ** 2)):
            assert row % 2 == 0 and values <= row <= values + 1
