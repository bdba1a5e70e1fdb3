"""The element-aligned backward kernel reads a kept t four entries at a time: no read may lie outside an array that ends
with the last row's token T - 1, and every token below T must come out of the words read (no GPU: the index function is compiled for the host)."""
import os
import subprocess

from paper_2605_24058_amd import binding

PROGRAM = r"""
#include <cstdio>
#include "lordba_rows.h"
int main() {
    for (int row = 0; row < 3; ++row)
        for (int T = 1; T <= 700; ++T) {
            const int stride = (T + 127) / 128 * 128, end = 2 * stride + T;   // an array that ends with token T - 1 of the last row
            for (int tok = 0; tok < stride; tok += 4) {
                const int at = row * stride + row_piece(tok, T, row);
                if (at < 0 || at + 4 > end) { std::printf("T %d, row %d, token %d: reads from %d\n", T, row, tok, at); return 1; }
                for (int e = 0; e < 4 && tok + e < T; ++e) {
                    const int n = row * stride + tok - at, word = n + e;   // the kernel moves the words down by n, which must not exceed 3
                    if (word < 0 || word > 3 || n > 3) { std::printf("T %d, row %d, token %d: word %d\n", T, row, tok + e, word); return 1; }
                }
            }
        }
    return 0;
}
"""


def test_pieces_stay_inside_the_row(tmp_path):
    src = tmp_path / "rows.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "rows"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", binding._CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


def test_the_kernel_reads_through_it():
    """Every read of du and t by the element-aligned variants takes its place from row_piece."""
    with open(os.path.join(binding._CSRC, "lordba_backward.hip")) as f:
        text = f.read()
    reads = [line for line in text.splitlines() if "load16_word(" in line]
    assert len(reads) == 3 and all("row_piece(" in line for line in reads), reads
