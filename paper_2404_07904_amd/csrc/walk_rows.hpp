// Where the rows of a chunk lie for the reverse walk: 32-bit byte offsets inside a buffer descriptor that covers exactly
// the chunk's tokens.  Plain arithmetic, in a header of its own so that it can be compiled and checked without a GPU.
#pragma once
#include <limits.h>
#include <stdint.h>

namespace hgrn2 {

constexpr int kWalkRows = 64;      // rows of a chunk

// Whether a descriptor reaches all rows of a chunk, from token to token ld_k (q, f) or ld_v (v, grad_o) elements apart: all
// offsets and their products fit an int, and rows before the chunk's first, whose offsets are negative, stay out of range as
// unsigned ones.  The first stride that does not is 8.4 million elements (fp32 gates), the heads of a token side by side: 65536 heads
// of 128.  Such a batch has more sequences than there are compute units: no run, span or light walk cuts one.
constexpr bool walk_rows_near(long long ld_k, long long ld_v, int gate_bytes)
{
    const long long k = ld_k * gate_bytes, v = ld_v * 2;
    return kWalkRows * (k > v ? k : v) <= INT_MAX;
}

// Bytes from the first token's row to the end of the last one's, `rows` in all; a row is `width` elements of es bytes.
constexpr uint32_t walk_chunk_bytes(int rows, int ld, int width, int es)
{
    return rows > 0 ? ((uint32_t)(rows - 1) * (uint32_t)ld + (uint32_t)width) * (uint32_t)es : 0u;
}

// Row `row` of the chunk, column `col`, from the first row that stands for a token, `lo`.  Rows before it wrap round to offsets
// that are out of range, like those behind the last one.
constexpr uint32_t walk_row_offset(int row, int lo, int ld, int col, int es)
{
    return (uint32_t)(((row - lo) * ld + col) * es);
}

}   // namespace hgrn2
