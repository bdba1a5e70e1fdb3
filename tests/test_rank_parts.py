"""d_s_rank, a sum over all tokens per rank, is dealt to several workgroups on long batches: every token to one of them, sums and arrivals inside the
workspace, and no workgroup left with more than its share (no GPU: the functions are compiled for the host)."""
import subprocess

from paper_2605_24058_amd import binding

PROGRAM = r"""
#include <cstdio>
#include "lordba_rows.h"
static int look(long long T, int splits) {
    const int room = splits - 1, parts = rank_parts(T, room);
    const long long span = rank_span(T, parts);
    const bool fits = parts >= 1 && parts <= kMaxRankParts && (parts == 1 || 1 + parts <= splits);   // one plane of arrivals, one per part
    const bool covered = span % 4 == 0 && (parts - 1) * span < T && parts * span >= T;              // whole pieces, no part empty
    const long long needed = (T + kRankTokens - 1) / kRankTokens;
    const bool share = T <= 2 * kRankTokens || needed > room || needed > kMaxRankParts || span <= kRankTokens;
    if (fits && covered && share) return 0;
    std::printf("T %lld, splits %d: parts %d of %lld\n", T, splits, parts, span);
    return 1;
}
int main() {
    const int splits[] = {1, 2, 3, 4, 5, 9, 16, 33, 64, 255, 256, 257, 258, 512};
    for (int s : splits) {
        for (long long T = 1; T <= 70000; ++T)
            if (look(T, s)) return 1;
        for (long long T = 70000; T <= 2147483519ll; T += T / 97 + 1)   // (up to the most rows that are taken)
            for (long long at = T; at < T + 4 && at <= 2147483519ll; ++at)
                if (look(at, s)) return 1;
        if (look(2147483519ll, s)) return 1;
    }
    return 0;
}
"""


def test_every_token_has_one_part(tmp_path):
    src = tmp_path / "parts.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "parts"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", binding._CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout
