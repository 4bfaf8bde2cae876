"""Vocabulary rows that the LM head's products over the kept probabilities take at a time (layout.hpp, host arithmetic): the loops over
them advance at every shape that a call accepts, and each product's operands stay within 31-bit byte offsets."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_27085_amd", "csrc")
MAIN = """
#include <stdio.h>
#include "layout.hpp"
size_t k_attn_ds_bytes(int, int) { return 0; }
int main() {
  long T; int h;
  while (scanf("%ld %d", &T, &h) == 2) printf("%d\\n", rp::head_rows_per_product((size_t)T, h));
}
"""


def test_rows_per_product_are_positive_and_addressable(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(tmp_path / "main.cpp"), "-o",
                    str(tmp_path / "main")], check=True)
    # around the sizes where 256 rows stop fitting, and the largest call (2^24 tokens)
    Ts = [8, 4096, 8192, 2 ** 21, 2 ** 22 - 8, 2 ** 22, 2 ** 22 + 8, 2 ** 23, 2 ** 24 - 8, 2 ** 24]
    args = [(T, h) for T in Ts for h in (8, 64, 248, 2048, 8192)]
    out = subprocess.run([str(tmp_path / "main")], input="".join("%d %d\n" % a for a in args), capture_output=True, text=True, check=True)
    rows = [int(x) for x in out.stdout.split()]
    assert len(rows) == len(args)
    for (T, h), n in zip(args, rows):
        assert n >= 8 and n % 8 == 0, (T, h, n)
        assert n * max(T, h) * 2 < 2 ** 31, (T, h, n)
        assert n % 256 == 0 or 256 * max(T, h) * 2 >= 2 ** 31, (T, h, n)
