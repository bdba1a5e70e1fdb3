"""A share's value carries the parity of its sweep beside its 53 bits: storing it, taking the mark off and adding it up gives the bits of the
plain sum (no GPU: the functions are compiled for the host)."""
import os
import re
import subprocess

from paper_2605_24058_amd import binding

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include "lordba_share_mark.h"
static uint64_t bits(double v) { uint64_t u; std::memcpy(&u, &v, 8); return u; }
static double from(uint64_t u) { double v; std::memcpy(&v, &u, 8); return v; }
static int bad(const char* what, double v) { std::printf("%s: %a\n", what, v); return 1; }
int main() {
    std::mt19937_64 rng(7);
    double sum = 0.0, marked = 0.0;
    for (long n = 0; n < 4000000; ++n) {
        const uint64_t significand = n % 3 == 0 ? rng() & 0xfffffffffffffull : n % 3 == 1 ? 0xfffffffffffffull : rng() & 1;
        const int exponent = n % 2 ? static_cast<int>(rng() % 1014) - 510 : static_cast<int>(rng() % 60) - 40;
        double v = from(significand | static_cast<uint64_t>(exponent + 1023) << 52 | (rng() & 1) << 63);
        if (n % 101 == 0) v = n % 2 ? 0.0 : -0.0;
        const uint32_t mark = rng() & 1;
        const double stored = with_mark(v, mark);
        if (other_mark(mark_word(stored, mark)) || !other_mark(mark_word(stored, 1 - mark))) return bad("mark", v);
        const double back = without_mark(stored);
        if (bits(back * kShareUnit) != bits(v)) return bad("value", v);
        if (n % kMaxShares == 0) sum = marked = 0.0;
        sum += v;
        marked = std::fma(back, kShareUnit, marked);
        if (bits(sum) != bits(share_sum(marked))) return bad("sum", v);
    }
    const double none[] = {INFINITY, -INFINITY, NAN, -NAN, from(0x7ff0000000000001ull), from(0x7fffffffffffffffull), 0x1p504, -0x1p504, 0x1p513, 1.7976931348623157e308};
    for (double v : none)
        for (uint32_t mark = 0; mark < 2; ++mark) {
            const double stored = with_mark(v, mark);
            if (other_mark(mark_word(stored, mark)) || !other_mark(mark_word(stored, 1 - mark))) return bad("mark", v);
            const double largest = 0x1.fffffffffffffp503;   // of either sign, before it and behind it
            for (int at = 0; at < kMaxShares; ++at)
                for (double other : {0.0, largest, -largest}) {
                    double sum = 0.0;
                    for (int k = 0; k < kMaxShares; ++k) sum = std::fma(without_mark(k == at ? stored : with_mark(other, mark)), kShareUnit, sum);
                    if (share_sum(sum) == share_sum(sum)) return bad("a number all the same", v);
                }
        }
    double most = 0.0, least = 0.0;
    for (int k = 0; k < kMaxShares; ++k) {
        most = std::fma(without_mark(with_mark(0x1.fffffffffffffp503, k & 1)), kShareUnit, most);
        least = std::fma(without_mark(with_mark(-0x1.fffffffffffffp503, k & 1)), kShareUnit, least);
    }
    if (bits(share_sum(most)) != bits(0x1.fffffffffffffp509) || bits(share_sum(least)) != bits(-0x1.fffffffffffffp509)) return bad("the largest sum", most);
    for (double v : {0x1p-511, 0x1.fffffffffffffp-511, 0x1p-562, -0x1.8p-540, 0x1p-600, 5e-324}) {   // the smallest lose what lies below 2^-562
        const double stored = with_mark(v, 1);
        if (other_mark(mark_word(stored, 1)) || !(std::fabs(without_mark(stored) * kShareUnit - v) <= 0x1p-563)) return bad("small", v);
    }
    return 0;
}
"""


def test_a_mark_costs_no_bit(tmp_path):
    src = tmp_path / "mark.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "mark"
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-I", binding._CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


def test_the_kernel_adds_shares_up_through_it():
    with open(os.path.join(binding._CSRC, "lordba_ptq_run.h")) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    assert len(re.findall(r"\bwith_mark\(", text)) == 1 and len(re.findall(r"\bwithout_mark\(", text)) == 1
    assert len(re.findall(r"without_mark\([^;]*, kShareUnit, acc\);", text)) == 1 and len(re.findall(r"share_sum\(acc\)", text)) == 1
