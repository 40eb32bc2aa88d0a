// Index arithmetic of walks over rows, in plain C++ (constexpr functions are
// host and device functions both), so that it can be checked on the host at
// sizes of which no graph is built for a test.
#pragma once

#include <algorithm>
#include <cstdint>

namespace hg {

// Positions and row numbers are int32 below 2^31; a walk in strides steps past
// its end, by up to a stride, where an int32 would wrap and never end.
typedef uint32_t row_pos;

// for p = beg, beg + step, ... below end
#define HG_ROW_WALK(p, beg, end, step) \
  for (::hg::row_pos p = (::hg::row_pos)(beg); p < (::hg::row_pos)(end); p += (::hg::row_pos)(step))

// Entries that a wave takes at base: 64, or those left.
constexpr int wave_entries(row_pos base, row_pos end) { return end - base < 64 ? (int)(end - base) : 64; }

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

// Most CSC entries that one backward work item (one wave) handles.  A wave walks
// its entries serially, 16 or more rows in flight, so a hub's items are the
// pass's tail: 1024 entries take about 45 us, which is all of the pass on a
// graph whose edges would give each of the chip's 8192 waves a few dozen
// (100k edges: 50 us at 1024, 14 at 64), and nothing beside it at 200M, where
// short items would only cost partial rows.  E: the input graph's edges (the
// plan's capacity follows from them).
constexpr int32_t kMaxChunk = 1024;
constexpr int32_t plan_chunk(int64_t E) {
  return E < ((int64_t)1 << 20) ? 64 : (E < ((int64_t)1 << 23) ? 256 : kMaxChunk);
}

// How the long rows of the CSC are cut into work items.  A row of up to
// `whole` entries is one item; one of more is m * blocks pieces of equal
// length, m = ceil(len / (row_chunk * blocks)), laid out block by block: the b-th
// m pieces of every split row stand together.
//
// A row's entries ascend by destination and the rows draw on the same
// destinations, so the pieces of one block gather from one part of the
// destinations' rows: of kBlockNodes nodes, 128 MB at 512 bytes a row, half of
// the Infinity Cache.  Gathers of 512-byte rows run at 9.3 TB/s from 64 MB,
// 7.2 from 256 MB and 4.5 from 2.5 GB and more; blocks of 128k and 512k nodes
// measured 0-3 % slower.  A piece costs a float64 partial row written and read
// (2 KB at d = 128, 0.4 ns of the whole chip), so a row is split only into pieces
// of kMinPiece entries and more (16 and 32 measured 0-3 % slower).  Destinations
// that fit one block are gathered from the cache as they are: rows are cut by
// length alone.
struct PlanCut {
  int32_t chunk, blocks, whole;
};
constexpr int64_t kBlockNodes = (int64_t)1 << 18;
constexpr int32_t kMaxBlocks = 128;
constexpr int32_t kMinPiece = 24;

constexpr PlanCut plan_cut(int64_t E, int64_t ns) {
  const int32_t chunk = plan_chunk(E);
  const int32_t blocks = (int32_t)std::max<int64_t>(1, std::min<int64_t>((ns - 1) / kBlockNodes + 1, kMaxBlocks));
  return {chunk, blocks, blocks == 1 ? chunk : kMinPiece * blocks - 1};
}

// The cut by length alone.
constexpr PlanCut by_length(PlanCut k) { return {k.chunk, 1, k.chunk}; }

// Whether the cut by blocks pays in a subgraph of e edges, of which it splits
// rows of `split` entries into `pieces`.  Blocks gain where hubs' long pieces run
// beside many short rows: Zipf sources of 20 edges a node have 150 to 480 edges to
// a piece and 0.2 to 0.9 of them in split rows, and their backward takes up to 17 %
// less at 2.5M nodes and more and 0 to 3 % at a million.  Where all rows are alike
// and long the waves walk the destinations in step, and blocks only cost the
// partial rows: 0.3M to 2M nodes of 50 to 200 edges in one relation take 2 to 17 %
// more in blocks (25 to 100 edges to a piece, all split), 4M and 10M nodes whose
// edges leave a few rows of 400 to 1000 up to 16 %, a million nodes of 60 edges
// (log-normal, 120 to a piece) 2 to 5 %.  The bound also keeps the partial rows
// below a hundredth of the edges.
constexpr int32_t kFewBlocks = 8;
constexpr int64_t kEdgesPerPiece = 100, kEdgesPerPieceFew = 200;
constexpr bool blocks_pay(PlanCut k, int64_t e, int64_t pieces, int64_t split) {
  return pieces * (k.blocks <= kFewBlocks ? kEdgesPerPieceFew : kEdgesPerPiece) <= e && 16 * split <= 15 * e;
}

// Most entries of a piece of a row of len: a row of more than kMostPieces chunks
// takes longer ones, up to kMaxChunk entries.  One wave adds a row's partial rows
// in order, at 25 to 70 ns each, so a row's pieces beyond some hundreds cost more
// there than they save in the pass: a row of 500k of a million edges in pieces
// of 64 had 340 us (d = 128; 1083 at d = 256) added up behind a pass of 37 us,
// where 512 take 12 to 30.  256 and 128 pieces measured up to 10 % slower.
constexpr int32_t kMostPieces = 512;
constexpr int32_t row_chunk(int32_t len, PlanCut k) {
  const int32_t c = len / kMostPieces;
  return c <= k.chunk ? k.chunk : (c < kMaxChunk ? c : kMaxChunk);
}

// Pieces of a row per block of destinations: 0 for a row that is one item or none.
constexpr int32_t cuts_of(int32_t len, PlanCut k) {
  return len > k.whole ? (len - 1) / (row_chunk(len, k) * k.blocks) + 1 : 0;
}

// Entries of piece c of the n of row [beg, end).
constexpr RowRange row_piece(int32_t beg, int32_t end, int32_t c, int32_t n) {
  const int64_t len = end - beg;
  return {beg + (int32_t)(len * c / n), beg + (int32_t)(len * (c + 1) / n)};
}

// Destination rows (all relations of one node j in the CSR) longer than
// this are not walked by one wave: the plan cuts them into chunks of this
// many entries whose partial results are merged in chunk order.
constexpr int32_t kFwdChunk = 2048;
constexpr int32_t fwd_chunks_of(int32_t len) { return len > kFwdChunk ? (len - 1) / kFwdChunk + 1 : 0; }

}  // namespace hg
