// How a value of a share (the quantiser's partial Gram sums) carries one bit, the parity of its sweep, beside all of its 53 bits of significand.
// Plain C++ (no HIP), so that a host program can go through every case.
#pragma once
#include <stdint.h>

// A share's value is stored divided by 2^512, which leaves the upper one of a double's exponent bits free below 2: bit 62 is the mark.
// Exact from 2^-510 up to 2^504 (smaller values lose what lies below 2^-562).  What is larger, infinite or not a number is stored as almost 2, and
// makes the sum more than a sum of the others can be: see share_sum.  (The sums are of products of fp16 factors, numbers near +-1 and
// the scales that fit them.)
constexpr double kShareUnit = 0x1p512, kShareLimit = 0x1p-8, kNoNumber = 0x1.fffffp0;
constexpr int kMaxShares = 64;

constexpr uint64_t share_bits(double v) { return __builtin_bit_cast(uint64_t, v); }
// Whether a stored value (or one of several whose words are or-ed) carries the other mark: other_mark(mark_word(stored, mark)).
constexpr uint32_t mark_word(double stored, uint32_t mark) { return static_cast<uint32_t>(share_bits(stored) >> 32) ^ mark << 30; }
constexpr bool other_mark(uint32_t word) { return (word & 0x40000000u) != 0u; }
constexpr double with_mark(double v, uint32_t mark) {
    const double scaled = v * (1.0 / kShareUnit);
    return __builtin_bit_cast(double, share_bits(scaled < kShareLimit && scaled > -kShareLimit ? scaled : kNoNumber) | static_cast<uint64_t>(mark) << 62);
}
// In units of 2^512, so that adding it up takes one multiply-add and no rounding but the sum's: sum = fma(without_mark(stored), kShareUnit, sum).
constexpr double without_mark(double stored) { return __builtin_bit_cast(double, share_bits(stored) & ~(1ull << 62)); }
// The sum of up to kMaxShares values: not a number where one of them was not.
constexpr double share_sum(double sum) { return sum < kMaxShares * kShareLimit * kShareUnit ? sum : __builtin_nan(""); }
