// Launch shape of the edge gradients (bwd_split.hip): a block takes kEdgeRows rows of
// kEdgeCols voxels along the last axis and strides over the rows that the grid does
// not cover; a last axis of more than kEdgeLaunchCols takes several launches.  The
// runtime takes at most 2^32 - 1 threads along an axis of the grid, and 65535
// blocks along its second.  (A loop over columns in the kernel instead costs 5 % of
// a reverse: 256^3 x 2 at lambda 0.5 5.42 -> 5.80 ms.)
#pragma once

namespace ggdt {

constexpr unsigned kEdgeCols = 64, kEdgeRows = 4, kEdgeThreads = kEdgeCols * kEdgeRows;
constexpr unsigned kEdgeLaunchCols = 1u << 26;  // 2^28 threads

// The launch for the columns from col0, of `cols` in all.
inline void edge_grid(unsigned cols, unsigned col0, long long rows, unsigned* gx, unsigned* gy) {
  constexpr long long kMaxY = 32768;
  const unsigned n = cols - col0 < kEdgeLaunchCols ? cols - col0 : kEdgeLaunchCols;
  const long long by = (rows + kEdgeRows - 1) / kEdgeRows;
  *gx = n / kEdgeCols + (n % kEdgeCols != 0);
  *gy = (unsigned)(by < kMaxY ? by : kMaxY);
}

}  // namespace ggdt
