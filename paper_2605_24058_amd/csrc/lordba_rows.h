// Reading rows of T entries four at a time without reading past the end of the last one.  Plain C++ (no HIP), so that a host
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
