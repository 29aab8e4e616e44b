// index_math.h - index arithmetic of the field kernels, shared by the GPU code
// and host checks.
//
//   field_tiling / tile_voxel_at   voxel tiling of the stencil and SL kernels
//                                  (XCD-aware order of the x1 tiles)
//   periodic_next / periodic_prev  neighbours on the periodic grid
//   xcd_grouped, xcd_run_if_split  unit of a block so that each XCD takes runs
//                                  of consecutive units that share cache lines
//   index_quot                     integer quotient by a float reciprocal
//   row_lanes                      x2 neighbours inside a row of lanes of the
//                                  row-vectorised stencils
//   sl_tile, sl_tile_block         tiles of the semi-Lagrangian kernels and their LDS
//                                  windows (sl_tile_wrap: periodic index of a window)
//   sl_axis                        cell and weight of a displaced point along one
//                                  axis for the semi-Lagrangian gathers
//
// Every function is __host__ __device__ (or host-only where marked) so that a host
// program can run the exact code the kernels run over every block and thread of a
// launch, with bounds checks, address and undefined-behaviour sanitizers.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>

namespace lddmm {

#define LDI_HD __host__ __device__ __forceinline__

// Voxel tiling of the field kernels: a block covers BX x BY voxels of one x0
// plane (BX spans a whole x2 row when N2 <= 256, so x2 halos stay inside the
// tile).  With XCD-aware mapping the 8 XCDs (which take blocks round-robin)
// each own a contiguous slab of x1 rows for every x0, so x1 halos and the
// neighbouring x0 planes a block needs were loaded into the same L2.  XCD x
// owns tile rows [x TY / 8, (x + 1) TY / 8) (rounded down), so where 8 does not
// divide TY the slabs differ by one row; the grid then holds 8 slab blocks per
// (x2 tile, x0 plane) and the blocks past an XCD's own rows do nothing.
struct FieldTiling {
  int BX, BY;      // block shape (threads)
  int TX, TY;      // tiles along x2 and x1
  int slab;        // most tile rows of x1 one XCD owns (0: plain linear order)
  unsigned blocks; // TX * N0 * (8 slab, or TY in linear order)
};

// Host: tile rows of the largest slab when 8 XCDs share TY of them, 0 where that is
// more than 15 % above the mean or there are fewer than 8.
inline int slab_rows(int TY) {
  const int s = (TY + 7) / 8;
  return TY >= 8 && 800 * s <= 115 * TY ? s : 0;
}

// Host: x1 rows per block, `most` of them or the largest half, quarter, ... (at least
// `least`) whose tile rows share evenly over the XCDs; linear order where none does.
// 90 x 108 x 100 FP64, 50-lane rows: 27 tile rows of 4 in linear order 72 us a tangent
// corrector, 54 of 2 in slabs 50 us.
inline void tile_rows(FieldTiling& t, int n1, int most, int least) {
  t.BY = most;
  for (int by = most; by >= least; by /= 2)
    if (slab_rows((n1 + by - 1) / by)) {
      t.BY = by;
      break;
    } else if (by % 2 != 0) {
      break;
    }
  t.TY = (n1 + t.BY - 1) / t.BY;
  t.slab = slab_rows(t.TY);
}

// Host: the tiling of an n0 x n1 x n2 grid (n2 = row length in lanes for the
// row-vectorised kernels).
inline FieldTiling field_tiling(int n0, int n1, int n2) {
  FieldTiling t;
  int bx = (n2 + 31) / 32 * 32;
  if (bx > 256) bx = 256;
  t.BX = bx;
  t.TX = (n2 + t.BX - 1) / t.BX;
  tile_rows(t, n1, 256 / bx > 0 ? 256 / bx : 1, bx % 64 == 0 ? 1 : 2);  // whole waves
  t.blocks = unsigned(t.TX) * unsigned(t.slab ? 8 * t.slab : t.TY) * unsigned(n0);
  return t;
}

// Voxel (i0, i1, i2) of thread (tx, ty) of block b under tiling t; false for the
// threads of an edge tile that fall outside the grid and for every thread of a
// block past its XCD's own slab.
LDI_HD bool tile_voxel_at(const FieldTiling& t, int b, int tx, int ty, int n1, int n2, int& i0, int& i1, int& i2) {
  int bx, by;
  bool own = true;
  if (t.slab) {
    const int x = b & 7, k = b >> 3;
    const int r = k / t.TX;
    bx = k - r * t.TX;
    const int rz = r / t.slab;
    const int ry = r - rz * t.slab;
    const int lo = (x * t.TY) >> 3, rows = (((x + 1) * t.TY) >> 3) - lo;
    own = ry < rows;
    by = lo + ry;
    i0 = rz;
  } else {
    const int r = b / t.TX;
    bx = b - r * t.TX;
    i0 = r / t.TY;
    by = r - i0 * t.TY;
  }
  i2 = bx * t.BX + tx;
  i1 = by * t.BY + ty;
  return own && i2 < n2 && i1 < n1;
}

// Unit of block b (of B) such that each XCD takes runs of g consecutive units:
// blocks go to the 8 XCDs round-robin (block b to XCD b mod 8), so within each
// span of 8 g blocks XCD x gets units [x g, x g + g) of the span, in order; a
// last span of fewer than 8 g blocks keeps unit = block.  Units next to each
// other in memory then share an L2 (a cache line split between two of them is
// fetched once), while the units in flight stay as close together as in
// round-robin order.
LDI_HD int xcd_grouped(int b, int B, int g) {
  const int span = 8 * g, s = b / span;
  if ((s + 1) * span > B) return b;
  const int r = b - s * span;
  return s * span + (r & 7) * g + (r >> 3);
}

// Host: run length for xcd_grouped.  Units share a 128-byte cache line with
// their neighbours unless every byte offset and stride that places them (a row,
// a tile, a plane of the spectrum) is a whole number of lines: then `run`, else
// 1 (round-robin order).
inline int xcd_run_if_split(long long a, long long b, long long c, long long d, int run) {
  return (a % 128 == 0 && b % 128 == 0 && c % 128 == 0 && d % 128 == 0) ? 1 : run;
}

// b / d for 0 <= b < 2^20 and 1 <= d < 2^20 from inv = 1.0f / d: the product of
// b + 1/2 with the rounded reciprocal stays within b 2^-22 / d of (b + 1/2) / d,
// which is at least 1 / 2d away from every integer.
LDI_HD int index_quot(int b, float inv) { return int((float(b) + 0.5f) * inv); }
// a * b of indices below 2^23: the 24-bit multiply issues at four times the rate of
// the 32-bit one.
LDI_HD int mul24(int a, int b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __mul24(a, b);
#else
  return a * b;
#endif
}

LDI_HD int periodic_next(int i, int n) { return i + 1 == n ? 0 : i + 1; }
LDI_HD int periodic_prev(int i, int n) { return i == 0 ? n - 1 : i - 1; }

// Row-vectorised stencils: a row of RW lanes (32 <= RW <= 64) starts a 32-lane
// half of a wave (RW = 32: two rows per wave) or a whole wave (RW > 32; lanes
// RW..63 hold no voxel).  The lanes holding the x2 neighbours of `lane`,
// periodic inside its row.
LDI_HD void row_lanes(int lane, int RW, int& left, int& right) {
  const int seg = RW <= 32 ? 32 : 64;
  const int base = lane & ~(seg - 1);
  const int pos = lane - base;
  left = base + (pos == 0 ? RW - 1 : (pos - 1) % RW);
  right = base + (pos + 1) % RW;
}

// Host: a row-vectorised width vw (voxels per lane: 1, 2, 3 or 4) is valid when
// a row of n2 voxels is 32 to 64 lanes.
inline bool row_vector_valid(int n2, int vw) {
  if (vw < 1 || vw > 4) return false;
  return n2 % vw == 0 && n2 / vw >= 32 && n2 / vw <= 64;
}

// Rows in segments of 32 lanes (half a wave): a row of RW lanes is cut into `chunks`
// of `out` lanes, each with a halo lane on either side that only holds the x2
// neighbour of the first and last (RW <= 32: one chunk, the whole periodic row, no
// halo).
struct RowSegments {
  int RW, chunks, out;
};
inline RowSegments row_segments(int RW) {
  RowSegments r{RW, 1, RW};
  if (RW > 32) {
    r.chunks = (RW + 29) / 30;
    r.out = (RW + r.chunks - 1) / r.chunks;
  }
  return r;
}
// Host: segments of vw voxels per lane for rows of n2 voxels: 2 or 4 where the row is
// one segment, 2 where it is cut.
inline bool row_segments_valid(int n2, int vw) {
  return (vw == 2 || vw == 4) && n2 % vw == 0 && n2 / vw >= 4 && (vw == 2 || n2 / vw <= 32);
}

// Host: voxels per lane of the segments a grid takes by default (0: the rows of 32 to
// 64 lanes of `rowvec`, or one voxel per thread).  A segment holds two x1 rows per
// wave, so one x1 row in two comes by a lane swap, and a wide aligned access per lane;
// it pays with its halo and spare lanes.  Sum over the six tangent, adjoint and EPDiff
// stages in us, rows of 32 to 64 lanes / segments:
//   FP32, one segment of width 4 against a row that is not 32 lanes: N2 = 72 119 / 81,
//     84 153 / 111, 100 168 / 129, 112 226 / 167, 120 184 / 143 (96, 32 lanes of width
//     3: 115 / 119; cut rows lose: 180 923 / 1099)
//   FP64, one segment of width 2: 64^3 76 / 60, N2 = 50 68 / 54
//   FP64, cut rows of width 2 against widths 3 (24 unaligned bytes) and 4: N2 = 140
//     730 / 637, 160 765 / 657, 180 1970 / 1820 (head grid), 240 1022 / 932; against
//     one voxel per thread: 210 1298 / 890.  Rows of 64 lanes stay (192 788 / 827,
//     256 4640 / 4630), as do widths 2 up to N2 = 128 (112 264 / 284)
//   FP32, cut rows against one voxel per thread, N1 even: 210 507 / 483
inline int default_segments(int n1, int n2, bool fp64, int rowvec) {
  const int lanes = rowvec ? n2 / rowvec : 0;
  if (fp64) {
    if (n2 % 2 != 0 || lanes == 64 && rowvec > 1) return 0;
    return (n2 / 2 > 16 && n2 / 2 <= 32) || n2 > 128 ? 2 : 0;
  }
  if (lanes != 32 && n2 > 64 && n2 % 4 == 0 && n2 / 4 <= 32) return 4;
  return !rowvec && n1 % 2 == 0 && n2 % 2 == 0 && n2 > 128 ? 2 : 0;
}

// Host: tiling in segments, up to 8 x1 rows per block.
inline FieldTiling segment_tiling(int n0, int n1, const RowSegments& r) {
  FieldTiling t;
  t.BX = 32;
  t.TX = r.chunks;
  tile_rows(t, n1, 8, 2);
  t.blocks = unsigned(t.TX) * unsigned(t.slab ? 8 * t.slab : t.TY) * unsigned(n0);
  return t;
}

// Lane pos (0 .. 31) of chunk k of a cut row: the row lane it loads (periodic) and
// whether it owns voxels.
LDI_HD bool segment_lane(const RowSegments& r, int k, int pos, int& j) {
  const int q = k * r.out + pos - 1;
  j = q < 0 ? q + r.RW : q >= r.RW ? q - r.RW : q;
  return pos >= 1 && pos <= r.out && q < r.RW;
}

// Semi-Lagrangian gather along one axis: grid index i displaced by d voxels.
// Offsets beyond a million voxels (or NaN) are clamped first, so the integer
// conversion cannot overflow and the periodic wrap keeps every index in
// [0, n).  a = lower cell index, b = the next one (periodic), t in [0, 1] the
// weight of b.
constexpr double kSlMaxVoxels = 1.0e6;
template <typename T>
LDI_HD void sl_axis(int i, T d, int n, int& a, int& b, T& t) {
  constexpr T lim = T(kSlMaxVoxels);
  d = fmin(fmax(d, -lim), lim);
  const T f = floor(d);
  t = d - f;
  int j = (i + int(f)) % n;
  a = j < 0 ? j + n : j;
  b = a + 1 == n ? 0 : a + 1;
}

// Tiles of the semi-Lagrangian kernels: a workgroup of 256 lanes covers T0 x0 planes
// of T1 x1 rows of T2 voxels (T1 T2 <= 256, T2 <= 64: an x2 row is cut into equal
// chunks), lane l the column (l / T2, l % T2) of every plane.  Its LDS window is the
// tile with one voxel more on every side, (T0 + 2) planes of (T1 + 2) rows of T2 + 2.
// Blocks are ordered so that each XCD owns a slab of x1 tiles, as in FieldTiling.
constexpr int kSlLanes = 256, kSlRow = 64;
// most window elements per lane: (T1 + 2) (T2 + 2) <= 396
constexpr int sl_window_loads(int T0) { return ((T0 + 2) * 396 + kSlLanes - 1) / kSlLanes; }

struct SlTile {
  int T0, T1, T2;
  int TX, TY, slab;  // tiles along x2 and x1; slab as in FieldTiling
  unsigned blocks;
  int row, plane, count;  // elements of a window's row, plane and all of it
  float inv_T2, inv_row, inv_plane;
};

inline SlTile sl_tile(int n0, int n1, int n2, int T0) {
  SlTile t;
  t.T0 = T0;
  const int chunks = (n2 + kSlRow - 1) / kSlRow;
  t.T2 = (n2 + chunks - 1) / chunks;
  t.T1 = kSlLanes / t.T2 < n1 ? kSlLanes / t.T2 : n1;
  t.TX = (n2 + t.T2 - 1) / t.T2;
  t.TY = (n1 + t.T1 - 1) / t.T1;
  t.slab = slab_rows(t.TY);
  t.blocks = unsigned(t.TX) * unsigned(t.slab ? 8 * t.slab : t.TY) * unsigned((n0 + T0 - 1) / T0);
  t.row = t.T2 + 2;
  t.plane = (t.T1 + 2) * t.row;
  t.count = (T0 + 2) * t.plane;
  t.inv_T2 = 1.0f / float(t.T2);
  t.inv_row = 1.0f / float(t.row);
  t.inv_plane = 1.0f / float(t.plane);
  return t;
}

// First voxel of block b's tile; false for a block past its XCD's own slab.
LDI_HD bool sl_tile_block(const SlTile& t, int b, int& i0, int& i1, int& i2) {
  bool own = true;
  int by, bz;
  const int k = t.slab ? b >> 3 : b, r = k / t.TX, bx = k - r * t.TX;
  if (t.slab) {
    const int x = b & 7, lo = (x * t.TY) >> 3, rows = (((x + 1) * t.TY) >> 3) - lo;
    bz = r / t.slab;
    const int ry = r - bz * t.slab;
    own = ry < rows;
    by = lo + ry;
  } else {
    bz = r / t.TY;
    by = r - bz * t.TY;
  }
  i0 = bz * t.T0;
  i1 = by * t.T1;
  i2 = bx * t.T2;
  return own;
}

// Grid index of window index w (0 .. tile length + 1) of a tile that starts at i:
// i + w - 1, periodic (an edge tile's window reaches at most one tile past n, and no
// tile is longer than n).
LDI_HD int sl_tile_wrap(int i, int w, int n) {
  const int j = i + w - 1;
  return j < 0 ? j + n : j >= n ? j - n : j;
}

// ---------------------------------------------------------------------------
// Host: trajectory storage policy (vector fields held per policy, c = interval)
//   store-all   4 nt + 2             (mu_n, v_n for n <= nt; mu*_n, v*_n for n < nt)
//   checkpoint  ceil(nt/c) + 4 c + 1 (mu every c steps; one segment: mu, v, mu*, v*)
//   recompute   7                    (mu_0; rolling mu, v pairs; mu*, v*)
// ---------------------------------------------------------------------------
enum { TRAJ_STORE_ALL = 0, TRAJ_CHECKPOINT = 1, TRAJ_RECOMPUTE = 2 };

inline size_t traj_fields(int policy, int nt, int c) {
  if (policy == TRAJ_STORE_ALL) return size_t(4) * nt + 2;
  if (policy == TRAJ_CHECKPOINT) return size_t((nt + c - 1) / c) + size_t(4) * c + 1;
  return 7;
}

struct TrajChoice {
  int policy;
  int every;  // checkpoint interval (0 unless TRAJ_CHECKPOINT)
};

// checkpoint_every > 0: checkpoint every min(c, nt) steps; < 0: recompute; 0:
// store-all, unless budget > 0 and fixed + store-all would exceed it: then the
// largest interval whose total fits, else recompute.  fixed = bytes held besides
// the trajectory, vbytes = bytes of one vector field.
inline TrajChoice choose_trajectory(int nt, int checkpoint_every, long long budget, size_t fixed, size_t vbytes) {
  if (checkpoint_every > 0) return {TRAJ_CHECKPOINT, checkpoint_every < nt ? checkpoint_every : nt};
  if (checkpoint_every < 0) return {TRAJ_RECOMPUTE, 0};
  if (budget <= 0 || fixed + traj_fields(TRAJ_STORE_ALL, nt, 0) * vbytes <= size_t(budget))
    return {TRAJ_STORE_ALL, 0};
  for (int c = nt; c >= 1; --c)
    if (fixed + traj_fields(TRAJ_CHECKPOINT, nt, c) * vbytes <= size_t(budget)) return {TRAJ_CHECKPOINT, c};
  return {TRAJ_RECOMPUTE, 0};
}

}  // namespace lddmm
