// Where the packed terms of an operand B[rows][K] lie (K a multiple of 8, any number of rows): chunks of
// eight k of a row, 16 bytes, ordered [row / 8][k / 8][term][row % 8], so that the 16 rows x 32 k that a
// wave loads at once are whole 128-byte lines, its terms side by side.  The last group of eight rows has
// its full size whatever rows is (input gradients: the rows are the input features, a multiple of 4).
// Behind two fp16 terms the rows' exponents, one int each.
#pragma once
#include <stddef.h>

namespace mg {

constexpr int PACK_TERM = 128;                            // bytes from term to term
constexpr size_t pack_row(long long row, int K, int terms) {
  return (size_t)(row >> 3) * (K >> 3) * (PACK_TERM * terms) + (row & 7) * 16;
}
constexpr long long pack_rows(long long rows) { return (rows + 7) / 8 * 8; }
// offset of the exponents behind two terms; bytes of both
constexpr size_t pack_exponents_at(long long rows, int K) { return pack_row(pack_rows(rows), K, 2); }
constexpr size_t pack2_bytes(long long rows, int K) {
  return pack_exponents_at(rows, K) + (size_t)pack_rows(rows) * sizeof(int);
}

}  // namespace mg
