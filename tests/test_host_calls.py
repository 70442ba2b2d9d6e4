"""The library's host code with a stand-in HIP runtime: what it allocates and
launches (no GPU)."""

import os
import re
import shutil
import subprocess

import pytest

from fakehip import ROOT, fake_hip, run  # noqa: F401


CSRC = os.path.join(ROOT, "paper_2607_21985_amd", "csrc")


def test_word_records_end_with_the_width(fake_hip):
    # tiles wider than a chunk (64 columns) pad the width by whole chunks,
    # whose activations would be loaded from past the end of X: the records
    # (2560 bytes a chunk, three spare) cover the chunks that hold a column
    out = run(fake_hip, """
    for tk in (16, 64, 128, 256):
        for cols in (8, 64, 72, 1032, 1152, 2056, 4160):
            hip.fake_clear()
            m = ones(300, cols, (256, tk))
            sizes = [int(l[1]) for l in log() if l[0] == "malloc"]
            out[f"{tk} {cols}"] = (2 * -(-cols // 64) + 3) * 2560 in sizes
            m.close()
    """)
    assert out and all(out.values()), out


def test_activation_loads_stay_inside_the_row(tmp_path):
    # every 16-byte piece that the all-columns decode form loads, over every
    # width (multiples of 8) up to 1088 and every chunk of it
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "t.cpp"
    src.write_text("""
#include "chunks.h"
#include <cstdio>
using namespace spdp_dev;
int main() {
  long n = 0;
  for (int cols = 8; cols <= 1088; cols += 8) {
    int seen = 0;
    for (int c = 0; c < chunk_count(cols); ++c)
      for (int p = 0; p < 8; ++p, ++n) {
        const int k = c * kChunkCols + 8 * p, from = k - 8 * pieces_back(c, p, cols);
        if (from < 0 || from + 8 > cols || (k < cols && from != k)) return std::printf("%d %d %d\\n", cols, c, p), 1;
        seen += k < cols;
      }
    if (seen != cols / 8) return std::printf("%d: %d pieces\\n", cols, seen), 1;
  }
  return std::printf("%ld\\n", n) < 0;
}
""")
    exe = str(tmp_path / "t")
    subprocess.run([gxx, "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
