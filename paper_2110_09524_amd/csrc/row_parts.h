// Rows cut into parts, for the persistent kernels that walk the column blocks of a plan with the rows' sums in LDS.  A workgroup's
// rows are in the order of their degrees; a row of 2^l parts takes 2^l slots, which the groups draw like rows.
#pragma once

#include <algorithm>

#include "common.h"

namespace gnn {

constexpr int kPartLevels = 7;
// the first rows[i] rows of a workgroup are cut into at least 2^(i + 1) parts
struct RowParts {
  int rows[kPartLevels];
};

// parts of the workgroup's j-th row, as a power of two
__device__ __forceinline__ int log_parts(const RowParts& cut, int j) {
  int l = 0;
#pragma unroll
  for (int i = 0; i < kPartLevels; ++i) l += j < cut.rows[i] ? 1 : 0;
  return l;
}
// slots of the rows before it
__device__ __forceinline__ int slots_before(const RowParts& cut, int j) {
  int s = j;
#pragma unroll
  for (int i = 0; i < kPartLevels; ++i) s += min(j, cut.rows[i]) << i;  // level i doubles: 2^i more slots
  return s;
}
// the end of the rows from j0 on whose slots are at most `room` (at least 2^log_parts(j0)), at most `rows`
__device__ __forceinline__ int rows_that_fit(const RowParts& cut, int j0, int rows, int room) {
  const int s0 = slots_before(cut, j0);
  int j1 = min(rows, j0 + room);
  if (slots_before(cut, j1) - s0 > room) {
    int over = j1;
    j1 = j0 + 1;
    while (over - j1 > 1) {
      const int mid = (j1 + over) >> 1;
      if (slots_before(cut, mid) - s0 <= room) j1 = mid; else over = mid;
    }
  }
  return j1;
}
// the row in [j0, j1) that slot q, counted from j0, belongs to
__device__ __forceinline__ int row_of_slot(const RowParts& cut, int j0, int j1, int q) {
  const int s0 = slots_before(cut, j0);
  int lo = j0, hi = j1;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (slots_before(cut, mid) - s0 <= q) lo = mid; else hi = mid;
  }
  return lo;
}
// part i of 2^l of a segment, cut at whole chunks
__device__ __forceinline__ int2 part_of_segment(int2 seg, int i, int l, int chunk) {
  const int64_t len = seg.y - seg.x;
  const int beg = seg.x + (int)((len * i >> l) & ~(int64_t)(chunk - 1));
  const int end = i + 1 == 1 << l ? seg.y : seg.x + (int)((len * (i + 1) >> l) & ~(int64_t)(chunk - 1));
  return make_int2(beg, end);
}

// Which graphs have their long rows cut, and into what, where `groups` groups share the edges of a slice.  A row as long as its share (what a
// group has of the edges on average) is what its workgroup waits for in every block, unless all rows are about as long: GAT layer,
// 15 523 rows of 132 even edges, 1 x 64, uncut 122 us a training pass, cut 138.  So: rows longer than four times the mean and 0.7 shares
// (232 965 power-law rows, 8 x 8, longest 1.08 shares: 6042 -> 5187; longest row 0.27 shares, 4 x 64: 15.41 ms cut, 15.35 uncut).
// Pieces of a quarter to half a share, and of at least half a chunk in a block: 22 308 rows, 10^7 edges, 1 x 64 325 us (twice as long
// 344, half 330), 100 000 rows, 4 10^7 edges, 8 x 8 1807 (2086, 1775).
constexpr int64_t kPieceEdges = 32;  // to a block: rows shorter than two such pieces stay whole
inline bool has_long_rows(const gnn_graph_t* g, int side, int64_t groups) {
  const int64_t longest = g->max_degree[side];
  return 10 * longest > 7 * (g->nnz / groups) && longest > 2 * kPieceEdges * g->nblk && longest * g->n > 4 * g->nnz;
}
// into parts of more than half of `piece` edges, and at most twice that
inline RowParts cut_rows(const gnn_graph_t* g, int side, int64_t piece, int64_t workgroups, int slots) {
  RowParts cut{};
  for (int i = 0; i < kPartLevels && (2 << i) <= slots; ++i) {
    int k = 0;  // rows of at least 2^k edges are cut into 2^(i + 1): the first power of two above piece 2^i
    while (k < 31 && ((int64_t)1 << k) <= piece << i) ++k;
    cut.rows[i] = k >= 31 ? 0 : (int)cdiv(g->h_bucket_offsets[side][32 - k], workgroups);
  }
  return cut;
}
inline RowParts cut_long_rows(const gnn_graph_t* g, int side, int64_t groups, int64_t workgroups, int slots) {
  return cut_rows(g, side, std::max<int64_t>(kPieceEdges * g->nblk, g->nnz / groups / 2), workgroups, slots);
}

}  // namespace gnn
