// Reading a row of T entries four at a time without reading past its end.  Plain C++ (no HIP), so that a host program can go
// through every case.
#pragma once

// Where to read four entries for tokens tok .. tok + 3 of a row: at tok, or at the row's last four (T < 4: at its start; such a
// row is followed by memory of its own).  The entry of token tok + e is then the (tok + e - row_piece(tok, T))-th of the four, for
// every token below T.
constexpr int row_piece(int tok, int T) {
    const int last = T > 4 ? T - 4 : 0;
    return tok < last ? tok : last;
}
