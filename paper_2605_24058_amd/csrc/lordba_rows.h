// Rows of T entries: reading them four at a time without reading past the end of the last one, and dealing one to several workgroups.  Plain C++ (no HIP), so that a host
// program can go through every case.
#pragma once

// Where to read four entries for tokens tok .. tok + 3 of row `row`, relative to the row's start: at tok, or the last four up to
// token T - 1.  Rows of fewer than four entries lie at least four apart and there are two or more of them: the four of the first
// row start with it, those of the others before it.  The entry of token tok + e is the (tok + e - row_piece(tok, T, row))-th of the four, for every
// token below T.
constexpr int row_piece(int tok, int T, int row) {
    const int last = T < 4 && row == 0 ? 0 : T - 4;
    return tok < last ? tok : last;
}

// d_s_rank of a rank is a sum over T tokens.  A workgroup of 256 threads requests 4096 of them at a time; longer batches are dealt to several, one per
// kRankTokens (`room`: at most as many as there is workspace for), which costs two more trips to memory: the parts' sums and arrivals, then all
// sums.  Four rounds of one workgroup take no longer than that (T = 16384, 2048 -> 2048, r = 4 80.7 us for the backward call, in two parts 81.7); with
// 16384 each T = 65536 takes 280 (278), and one workgroup for everything took 148 us of a call of 1023 at T = 1048576, 64 -> 64, r = 1 (now 7 of 880).
constexpr int kRankTokens = 8192, kMaxRankParts = 256;   // (a thread for every part in the smallest workgroup)
constexpr int rank_parts(long long T, long long room) {
    const long long wanted = T <= 2 * kRankTokens ? 1 : (T + kRankTokens - 1) / kRankTokens, most = room < kMaxRankParts ? room : kMaxRankParts;
    return wanted <= 1 || most <= 1 ? 1 : static_cast<int>(wanted < most ? wanted : most);
}
// Tokens of each part but the last (whole pieces of four).
constexpr long long rank_span(long long T, int parts) { return ((T + parts - 1) / parts + 3) / 4 * 4; }
