// Cuts of the transforms' planes over all grids that a context takes, at 160 KB of LDS:
// where whole planes (or the split path) can run with a tile width, so can the cut that
// is chosen, and what it chooses fits.
#include <cstdio>
#include <vector>

#include "fft_rt.h"

using namespace lddmm;
void __syncthreads() {}

static bool uncut_runs(const SpectralSizes& z, int tb) {
  if (pencil_lds(z, z.n0, tb) > z.max_lds) return false;
  return units_fit(z, 1, tb) || (pencil_lds(z, z.n1, tb) <= z.max_lds && rows_lds(z, 1) <= z.max_lds);
}

static int check(const SpectralSizes& z, int want = 0) {
  const int xs = plane_units(z);
  if (want && (units_fit(z, xs, default_pencil_tb(z)) ? xs : 1) != want) return 1;
  if (xs > 1 && !units_fit(z, xs, default_pencil_tb(z))) return 4;  // planned as cut, runs whole or split
  for (int tb : {default_pencil_tb(z), 1, 2, 4, 6, 8, 16, 32}) {
    if (xs == 1 || !units_fit(z, xs, tb)) continue;  // runs uncut
    if (z.n1 % xs || unit_lds(z, z.n1 / xs) > z.max_lds) return 2;
    if (uncut_runs(z, tb) && pencil_lds(z, z.n0, pencil_groups(tb, xs) * xs) > z.max_lds) return 3;
  }
  return 0;
}

// Launches of the split path's x1 pencils have n0 rows of workgroups per component, and
// a launch at most 65536 of them.
static int check_pass(const SpectralSizes& z) {
  const size_t one = 3 * size_t(z.n0) * z.n1 * (z.H + 1) * z.cb;
  for (int count : {2, 11, 181, 100000}) {
    const int k = fields_per_pass(one, count, z.n0);
    if (k < 1 || k > count || (k > 1 && (3LL * k * z.n0 > 65536 || k * one > size_t(96) << 20))) return 5;
  }
  return 0;
}

int main() {
  const size_t lds = 160 * 1024;
  std::vector<int> len;
  for (int n = 4; n <= 20480; ++n) {
    int m = n;
    for (int p : {2, 3, 5, 7})
      while (m % p == 0) m /= p;
    if (m == 1) len.push_back(n);
  }
  // halves, quarters and thirds; long x0 axes whose pencils leave no room for a group
  const struct { int n0, n1, n2; size_t cb; int want; } known[] = {
      {180, 210, 180, 16, 2},   {128, 128, 128, 8, 2},  {8, 320, 288, 8, 4},    {6, 256, 256, 16, 4},
      {5, 225, 240, 8, 3},      {10, 45, 30, 8, 1},     {2100, 256, 256, 16, 1}, {2400, 300, 210, 16, 1},
      {4000, 320, 320, 8, 1},   {1875, 32, 1152, 16, 1}, {2304, 945, 18, 16, 1}, {2304, 2625, 4, 16, 1}};
  for (const auto& k : known)
    if (const int rc = check({k.n0, k.n1, k.n2 / 2, k.cb, lds}, k.want)) {
      std::printf("%d x %d x %d, %zu bytes: %d\n", k.n0, k.n1, k.n2, k.cb, rc);
      return 1;
    }
  for (size_t cb : {size_t(8), size_t(16)})
    for (int n0 : len)
      for (int n1 : len)
        for (int n2 : len) {
          if (n2 % 2) continue;
          if (3LL * n0 * n1 * n2 >= 1LL << 31) break;
          const SpectralSizes z{n0, n1, n2 / 2, cb, lds};
          int rc = check(z);
          if (!rc) rc = check_pass(z);
          if (rc) {
            std::printf("%d x %d x %d, %zu bytes: %d\n", n0, n1, n2, cb, rc);
            return 1;
          }
        }
  return 0;
}
