// Rows in 32-lane segments over every block and thread: each row lane owned once, its
// x2 neighbours held by the lanes next to it, every loaded lane inside the row.
#include <cstdio>
#include <initializer_list>
#include <vector>

#include "index_math.h"

using namespace lddmm;
void __syncthreads() {}

static int check(int n0, int n1, int RW) {
  const RowSegments r = row_segments(RW);
  const FieldTiling t = segment_tiling(n0, n1, r);
  const bool halo = r.chunks > 1;
  if (t.BX != 32 || t.BX * t.BY > 256) return 1;
  std::vector<int> seen(size_t(n0) * n1 * RW, 0);
  for (unsigned b = 0; b < t.blocks; ++b)
    for (int ty = 0; ty < t.BY; ++ty) {
      int lane_j[32], lane_ok[32], i0, i1, q;
      bool any = false;
      for (int tx = 0; tx < 32; ++tx) {
        lane_ok[tx] = -1;
        if (!tile_voxel_at(t, int(b), tx, ty, n1, halo ? t.TX * 32 : RW, i0, i1, q)) continue;
        if (i0 < 0 || i0 >= n0 || i1 < 0 || i1 >= n1) return 2;
        any = true;
        int j = q;
        lane_ok[tx] = halo ? segment_lane(r, q >> 5, q & 31, j) : 1;
        if (j < 0 || j >= RW) return 3;
        lane_j[tx] = j;
      }
      if (!any) continue;
      for (int tx = 0; tx < 32; ++tx) {
        if (lane_ok[tx] != 1) continue;
        int l = (tx - 1) & 31, h = (tx + 1) & 31;
        if (!halo) row_lanes(tx, RW, l, h);
        if (lane_ok[l] < 0 || lane_ok[h] < 0) return 4;
        if (lane_j[l] != (lane_j[tx] + RW - 1) % RW || lane_j[h] != (lane_j[tx] + 1) % RW) return 5;
        ++seen[(size_t(i0) * n1 + i1) * RW + lane_j[tx]];
      }
    }
  for (int s : seen)
    if (s != 1) return 6;
  return 0;
}

int main() {
  for (int n1 : {4, 7, 12, 30, 64, 105, 128, 210, 216})
    for (int RW : {4, 5, 9, 16, 25, 31, 32, 33, 45, 60, 61, 64, 90, 91, 105, 128, 180, 245})
      if (const int rc = check(3, n1, RW)) {
        std::printf("%d rows of %d lanes: %d\n", n1, RW, rc);
        return 1;
      }
  return 0;
}
