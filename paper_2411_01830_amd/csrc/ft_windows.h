// How a wavefront cuts a piece of a transfer into windows: which bytes window j of a contiguous run or of
// a set of pitched rows covers. Plain arithmetic, the same on host and device, so that the ranges
// the copy kernel touches can be checked without a GPU.
#pragma once
#include <stdint.h>

#include "ft_tables.h"

namespace ft {

FT_HD uint32_t mul_hi32(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }

// A contiguous run of n >= 16 bytes (n < 2^30): windows of 16 bytes on the destination's 16-byte boundaries, the
// first moved forward and the last moved back to begin and end with the run. They overlap their
// neighbours with the same bytes, so no edge bytes are left over.
struct RunWindows {
  uint32_t count;
  int32_t adj, last;  // window j begins at byte clamp(16 * j + adj, 0, last)
};

FT_HD RunWindows run_windows(uint64_t dst, uint32_t n) {
  const uint32_t head = (16 - ((uint32_t)dst & 15)) & 15;  // bytes before the first boundary
  const uint32_t h = head != 0 ? 1u : 0u;
  RunWindows w;
  w.count = h + (n - head + 15) / 16;
  w.adj = (int32_t)head - (int32_t)(h << 4);
  w.last = (int32_t)n - 16;
  return w;
}

FT_HD uint32_t run_window_at(const RunWindows &w, uint32_t j) {
  int32_t off = (int32_t)(j << 4) + w.adj;
  off = off < 0 ? 0 : off;
  return (uint32_t)(off > w.last ? w.last : off);
}

// Bytes [c0, ...) of row r0 up to but not including column last_end of row r0 + more of a pitched descriptor,
// in windows of W bytes: a row of n bytes has ceil(n / W) windows at columns 0, W, 2 W, ..., each moved as
// far as it must to lie inside the row and inside the piece (it then overlaps a neighbour with the same bytes).
// Windows are numbered through, row by row. The part of the first or the last row that the piece holds may be
// shorter than a window: it has none, its short_first bytes from column c0 of row r0 and its short_last bytes from
// column 0 of row r0 + more go one by one.
struct RowWindows {
  uint32_t c0, more, row_bytes, last_end;
  uint32_t per_row;  // windows of a whole row
  uint32_t magic;    // g / per_row = mulhi(g, magic) or one less than that; 0: per_row is 1
  uint32_t first;    // number of the piece's first window if row r0's windows count from 0
  uint32_t count;
  uint32_t short_first, short_last;
};

// row_bytes >= W and < 2^30, take < 2^30 bytes from column c0 on.
template <uint32_t W>
FT_HD RowWindows row_windows(uint32_t row_bytes, uint32_t c0, uint32_t take) {
  RowWindows w;
  const uint32_t room = row_bytes - c0;
  w.c0 = c0;
  w.row_bytes = row_bytes;
  w.per_row = (row_bytes + W - 1) / W;
  w.magic = 0xffffffffu / w.per_row + 1;  // 2^32 / per_row rounded up
  w.more = 0;
  w.last_end = c0 + take;
  uint32_t first_len = take, last_len = take;
  if (take > room) {
    const uint32_t rest = take - room;
    w.more = (rest + row_bytes - 1) / row_bytes;
    w.last_end = last_len = rest - (w.more - 1) * row_bytes;
    first_len = room;
  }
  w.short_first = first_len < W ? first_len : 0u;
  w.short_last = w.more != 0 && last_len < W ? last_len : 0u;
  w.first = w.short_first != 0 ? w.per_row : c0 / W;
  const uint32_t last = last_len < W ? w.more * w.per_row : w.more * w.per_row + (w.last_end + W - 1) / W;  // one past it
  w.count = last > w.first ? last - w.first : 0u;
  return w;
}

// Where a lane is: window `col / W` of row r0 + row.
struct RowCursor {
  uint32_t row, col;
};

template <uint32_t W>
FT_HD RowCursor row_window(const RowWindows &w, uint32_t q) {
  const uint32_t g = w.first + q;
  RowCursor c;
  c.row = w.magic == 0 ? g : mul_hi32(g, w.magic);
  c.row -= (c.row * w.per_row > g) ? 1u : 0u;
  c.col = (g - c.row * w.per_row) * W;
  return c;
}

// `rows` whole rows and `cols` columns further (cols a multiple of W, less than a row's windows).
template <uint32_t W>
FT_HD void row_window_next(const RowWindows &w, uint32_t rows, uint32_t cols, RowCursor *c) {
  c->row += rows;
  c->col += cols;
  const uint32_t end = w.per_row * W;
  const bool over = c->col >= end;
  c->row += over ? 1u : 0u;
  c->col -= over ? end : 0u;
}

// The window's first byte: its column moved into the row and the piece.
template <uint32_t W>
FT_HD uint32_t row_window_col(const RowWindows &w, const RowCursor &c) {
  const uint32_t lo = c.row == 0 ? w.c0 : 0u;
  const uint32_t hi = (c.row == w.more ? w.last_end : w.row_bytes) - W;
  const uint32_t col = c.col < lo ? lo : c.col;
  return col > hi ? hi : col;
}

}  // namespace ft
