// Host check of the edge gradients' launches (the library's edge_grid.h, included
// verbatim): within the runtime's limits for every shape of fewer than 2^31
// voxels, and together over each column once.
#include <stdio.h>

#include <initializer_list>

#include "edge_grid.h"

using namespace ggdt;

int main() {
  const unsigned long long widths[] = {1, 2, 63, 64, 65, 4097, 1u << 20, (1u << 26) - 1, 1u << 26, (1u << 26) + 1,
                                       1u << 30, (1u << 30) + 1, (1u << 30) + 4097, 0x7ffffffeu, 0x7fffffffu};
  int bad = 0;
  for (unsigned long long w : widths) {
    for (unsigned long long rows : {1ull, 2ull, 5ull, 131072ull, 131073ull, 0x7fffffffull / w}) {
      if (rows < 1 || rows * w > 0x7fffffffull) continue;
      unsigned long long next = 0;  // columns covered so far
      bool ok = true;
      for (unsigned col0 = 0; col0 < w; col0 += kEdgeLaunchCols) {
        unsigned gx = 0, gy = 0;
        edge_grid((unsigned)w, col0, (long long)rows, &gx, &gy);
        ok &= gx >= 1 && gy >= 1 && (unsigned long long)gx * kEdgeThreads < (1ull << 32) && gy <= 65535;
        ok &= col0 == next && (unsigned long long)col0 + (unsigned long long)gx * kEdgeCols < (1ull << 32);
        next = col0 + (unsigned long long)gx * kEdgeCols;
      }
      ok &= next >= w && next < w + kEdgeCols;
      if (!ok) {
        printf("width %llu rows %llu\n", w, rows);
        ++bad;
      }
    }
  }
  printf("failures %d\n", bad);
  return bad ? 1 : 0;
}
