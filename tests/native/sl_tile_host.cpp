// Tiles and windows of the semi-Lagrangian kernels over every block and lane: each
// voxel owned once, every window element a grid element, and every corner that the
// gather may read the voxel's own periodic neighbour.
#include <cstdio>
#include <initializer_list>
#include <vector>

#include "index_math.h"

using namespace lddmm;
void __syncthreads() {}

static int check(int n0, int n1, int n2, int T0) {
  const SlTile t = sl_tile(n0, n1, n2, T0);
  if (t.T1 * t.T2 > kSlLanes || t.T2 > kSlRow || t.count > sl_window_loads(T0) * kSlLanes) return 1;
  std::vector<int> seen(size_t(n0) * n1 * n2, 0), win(t.count);
  for (unsigned b = 0; b < t.blocks; ++b) {
    int b0, b1, b2;
    if (!sl_tile_block(t, int(b), b0, b1, b2)) continue;
    if (b0 < 0 || b0 >= n0 || b1 < 0 || b1 >= n1 || b2 < 0 || b2 >= n2) return 2;
    for (int e = 0; e < t.count; ++e) {
      const int w0 = index_quot(e, t.inv_plane), r = e - w0 * t.plane, w1 = index_quot(r, t.inv_row), w2 = r - w1 * t.row;
      const int g0 = sl_tile_wrap(b0, w0, n0), g1 = sl_tile_wrap(b1, w1, n1), g2 = sl_tile_wrap(b2, w2, n2);
      if (g0 < 0 || g0 >= n0 || g1 < 0 || g1 >= n1 || g2 < 0 || g2 >= n2) return 3;
      win[e] = (g0 * n1 + g1) * n2 + g2;
    }
    for (int lane = 0; lane < kSlLanes; ++lane) {
      const int l1 = index_quot(lane, t.inv_T2), l2 = lane - l1 * t.T2, i1 = b1 + l1, i2 = b2 + l2;
      if (!(l1 < t.T1 && i1 < n1 && i2 < n2)) continue;
      for (int k = 0; k < T0; ++k) {
        if (b0 + k < n0) ++seen[(size_t(b0 + k) * n1 + i1) * n2 + i2];
        const int centre = t.plane + (l1 + 1) * t.row + l2 + 1 + k * t.plane;
        for (int c = 0; c < 27; ++c) {
          const int d0 = c / 9 - 1, d1 = c / 3 % 3 - 1, d2 = c % 3 - 1;
          const int o = centre + d0 * t.plane + d1 * t.row + d2;
          if (o < 0 || o >= t.count) return 4;
          const int j0 = (b0 + k + d0 + n0) % n0, j1 = (i1 + d1 + n1) % n1, j2 = (i2 + d2 + n2) % n2;
          if (b0 + k < n0 && win[o] != (j0 * n1 + j1) * n2 + j2) return 5;
        }
      }
    }
  }
  for (int s : seen)
    if (s != 1) return 6;
  return 0;
}

int main() {
  for (int T0 : {1, 2, 4})
    for (int n0 : {4, 5, 9, 20})
      for (int n1 : {4, 7, 30, 64, 105})
        for (int n2 : {4, 6, 16, 32, 50, 64, 70, 128, 180, 250})
          if (const int rc = check(n0, n1, n2, T0)) {
            std::printf("%d x %d x %d, %d planes: %d\n", n0, n1, n2, T0, rc);
            return 1;
          }
  return 0;
}
