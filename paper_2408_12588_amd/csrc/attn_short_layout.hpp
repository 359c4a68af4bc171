// Where a wavefront of attn_short.hpp keeps its K and V tile in LDS.  Plain arithmetic without any device code, so that a host
// program can go through the addresses of all lanes.
#pragma once

namespace pab {

// elements of a K or V row: D of data, then a chunk of eight.  40 (20) banks, which no 16-byte operand read conflicts on
template <int D> constexpr int SHORT_PITCH = D + 8;

// Column at which a lane reads the V rows of sub-tile dt: four elements of which the lanes of piece 0 .. 3 make the rows 16 dt +
// 4 piece of V^T.  Heads of 32 have 40 columns and the third sub-tile asks for 48: what it would find behind a row only feeds rows
// of O^T that are never stored, but behind the last row it lies in another wavefront's tile or past the end of LDS.  Those
// lanes take the last four columns of their own row.
template <int D> constexpr int short_v_column(int dt, int piece) {
  const int column = 16 * dt + 4 * piece;
  return column + 4 <= SHORT_PITCH<D> ? column : SHORT_PITCH<D> - 4;
}

}  // namespace pab
