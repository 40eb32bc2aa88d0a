// Index arithmetic of walks over rows, in plain C++ (constexpr functions are
// host and device functions both), so that it can be checked on the host at
// sizes of which no graph is built for a test.
#pragma once

#include <cstdint>

namespace hg {

// Positions and row numbers are int32 below 2^31; a walk in strides steps past
// its end, by up to a stride, where an int32 would wrap and never end.
typedef uint32_t row_pos;

// for p = beg, beg + step, ... below end
#define HG_ROW_WALK(p, beg, end, step) \
  for (::hg::row_pos p = (::hg::row_pos)(beg); p < (::hg::row_pos)(end); p += (::hg::row_pos)(step))

// Stretches of rows without entries, in pieces of kRpPiece rows that blocks
// fill on their own; hi is at most 2^31 - 1.
constexpr int32_t kRpPiece = 16384;
struct RowRange {
  int32_t beg, end;
};
constexpr int32_t gap_pieces(int32_t lo, int32_t hi) { return (hi - lo - 1) / kRpPiece + 1; }
constexpr RowRange gap_piece(int32_t lo, int32_t hi, int32_t i) {
  const int32_t beg = lo + i * kRpPiece;
  return {beg, hi - beg < kRpPiece ? hi : beg + kRpPiece};
}

}  // namespace hg
