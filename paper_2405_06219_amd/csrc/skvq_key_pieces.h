// Where a lane of the decode kernels finds its pieces of a tile's key rows, for the key formats whose rows are fetched a
// quarter per lane.  Plain constexpr arithmetic without device types: the host can check it at cache lengths that no test fills.
#pragma once

namespace skvq {

// Rows that the tile has after its first one, at most 63.  (The distance to the last packed token itself, up to 2^31, times
// a row's bytes does not fit 32 bits from 2^26 tokens of 4-bit keys on.)
constexpr unsigned rows_after_first(int last_token, int tile) {
  const int rows = last_token - tile * 64;  // >= 0
  return (unsigned)(rows < 63 ? rows : 63);
}

// Byte offset, from the tile's first row, of piece x (0..3) of a lane: quarter lane / 16 of the row of token 16 x + lane % 16;
// tokens past the tile's last one: the last quarter of its row.
template <unsigned ROW_BYTES>
constexpr unsigned key_piece_offset(unsigned lane, unsigned x, unsigned rows_after) {
  const unsigned at = ROW_BYTES * (16 * x + lane % 16) + ROW_BYTES / 4 * (lane / 16);
  const unsigned last = ROW_BYTES * rows_after + ROW_BYTES / 4 * 3;
  return at < last ? at : last;
}

}  // namespace skvq
