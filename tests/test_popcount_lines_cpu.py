"""The popcount tile's look-ahead over the next block of library rows, checked
on the host for every row length (D = 512 to 32,768) and block size: each word
it touches lies inside the rows, and no 128-byte piece of them is left out."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2211_16422_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "popcount_lines.h"
using namespace homs::popc;
int main()
{
    for (uint32_t words = 16; words <= 1024; words += 16)
        for (uint32_t rows = 1; rows <= 32; ++rows)
            for (uint32_t row : {0u, 1u, 97u, 2147483000u}) {
                const size_t first = (size_t)row * words, end = first + (size_t)rows * words;
                const uint32_t n = ahead_lines(rows, words);
                size_t covered = first;  // touched so far, in whole pieces
                for (uint32_t i = 0; i < n; ++i) {
                    const size_t w = ahead_word(row, words, i);
                    if (w < first || w >= end || w != covered) {
                        std::printf("words %u rows %u row %u piece %u: word %zu of [%zu, %zu)\n",
                                    words, rows, row, i, w, first, end);
                        return 1;
                    }
                    covered = w + kLineWords;
                }
                if (covered < end) {
                    std::printf("words %u rows %u: %zu words not touched\n", words, rows,
                                end - covered);
                    return 1;
                }
            }
    std::puts("all lines inside the rows");
    return 0;
}
"""


def test_every_line_lies_inside_the_rows(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    src, exe = tmp_path / "lines.cpp", str(tmp_path / "lines")
    src.write_text(PROGRAM)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined",
                        "-fno-sanitize-recover=all", f"-I{CSRC}", str(src), "-o", exe],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_the_tile_code_takes_its_addresses_from_there():
    text = open(os.path.join(CSRC, "popcount_tile.h")).read()
    assert "lib_hv[ahead_word(next, words, i)]" in text
    assert "words / 32" not in text  # 0 for rows of 16 words
