// fft_rt.h - transform passes for lengths known at run time (any product of 2,
// 3, 5, 7): what the kernels of fft_rt.hip take and how their launch is planned.
//
// The (x1, x2) planes of the fused path are cut into XS units, unit h holding the
// x1 rows XS m + h: n1 / XS rows, transformed along x1 at length n1 / XS.  The x0
// pencil pass takes the XS partial spectra at one (k1, k2) slot together, forms
// the pencils of k1, k1 + n1 / XS, ... (the first radix-XS step of the x1 transform
// by decimation in x1) as it loads and undoes that as it stores.  XS = 1: whole
// planes.
#pragma once

#include <cstddef>
#include <initializer_list>

#include "fft_core.h"
#include "index_math.h"

namespace lddmm {

// Host: what decides the launch shapes of a grid's transforms.
struct SpectralSizes {
  int n0, n1, H;   // H = n2 / 2
  size_t cb;       // bytes of a complex value
  size_t max_lds;  // of a workgroup
};

// LDS of the split path's row kernels for rb rows, with the x2 tables.
inline size_t rows_lds(const SpectralSizes& z, int rb) {
  return size_t(rb) * (z.H + 1) * z.cb + size_t(z.H + z.H / 2 + 1) * z.cb + size_t(z.H + 1) * sizeof(int);
}
// LDS of a plane kernel for `rows` x1 rows at a row stride of H + 1 + `pad` values.
inline size_t unit_lds(const SpectralSizes& z, int rows, int pad = 0) {
  return rows_lds(z, rows) + size_t(rows) * (pad + 1) * z.cb;
}
// LDS of a pencil kernel for `seqs` sequences of n values, with a symbol term for each.
inline size_t pencil_lds(const SpectralSizes& z, int n, int seqs) {
  return (size_t(n) * seqs + n) * z.cb + size_t(n + seqs) * (z.cb / 2);
}
// Groups of xs sequences per x0 pencil workgroup at a tile of tb pencils.
inline int pencil_groups(int tb, int xs) { return tb / xs > 0 ? tb / xs : 1; }

// Pencils per workgroup by default: 256-byte rows, fewer on axes that do not fit the LDS.
inline int default_pencil_tb(const SpectralSizes& z) {
  int tb = int(256 / z.cb);
  while (tb > 1 && ((size_t(z.n0) * tb + z.n0) * z.cb + z.n0 * (z.cb / 2) > z.max_lds ||
                    (size_t(z.n1) * tb + z.n1) * z.cb > z.max_lds))
    tb /= 2;
  return tb;
}

// True if planes in xs units (1: whole) can run with pencil tiles of tb: a unit fits the
// LDS, and so do the pencils of a group of xs, which may be more than tb.
inline bool units_fit(const SpectralSizes& z, int xs, int tb) {
  if (unit_lds(z, z.n1 / xs) > z.max_lds) return false;
  if (xs == 1) return true;
  return z.n1 % xs == 0 && z.n1 / xs >= 4 && tb % 2 == 0 &&
         pencil_lds(z, z.n0, pencil_groups(tb, xs) * xs) <= z.max_lds;
}

// Units that a plane is cut into (their tables are part of the plan): halves, or
// quarters or thirds where halves do not fit; odd n1 gets thirds where the whole plane
// does not fit.  1: whole planes, or the split path where those do not fit.
inline int plane_units(const SpectralSizes& z) {
  const int tb = default_pencil_tb(z);
  if (z.n1 % 2 != 0 && units_fit(z, 1, tb)) return 1;
  for (int xs : {2, 4, 3})
    if (units_fit(z, xs, tb)) return xs;
  return 1;
}

// Vector fields of a stack of `count` that one spectral pass takes: spectra (`one` bytes a
// field) within 96 MB, at most 256, and no more than the split path's x1 pencils can
// launch (three rows of n0 workgroups a field; a grid's second dimension ends at 65536).
inline int fields_per_pass(size_t one, int count, int n0) {
  const size_t most = size_t(96) << 20;
  size_t k = one > 0 ? most / one : 1;
  if (k > size_t(count)) k = size_t(count);
  if (k > 256) k = 256;
  if (k > size_t(65536 / (3 * n0))) k = size_t(65536 / (3 * n0));
  return k < 1 ? 1 : int(k);
}

// One stage of a run-time plan with what its kernels would otherwise divide for.
struct RtStage {
  int R;      // radix
  int S;      // element stride inside a sub-block: L / R
  int L;      // sub-block length
  int tws;    // twiddle step n / L
  float invS; // 1 / S (index_quot)
};

constexpr int kRtStages = 8;  // lengths whose pencil fits the LDS (20480 values) have at most 7

struct RtPlan {
  int n, nf;
  RtStage st[kRtStages];
};

// Run-time form of a plan; false if it has more stages than the kernels take.
inline bool make_rt_plan(const FftPlan& pl, RtPlan& r) {
  r = RtPlan{};
  r.n = pl.n;
  r.nf = pl.nf;
  if (pl.nf < 1 || pl.nf > kRtStages) return false;
  int L = pl.n;
  for (int i = 0; i < pl.nf; ++i) {
    RtStage& s = r.st[i];
    s.R = pl.radix[i];
    s.L = L;
    s.S = L / s.R;
    s.tws = pl.n / L;
    s.invS = 1.0f / float(s.S);
    L = s.S;
  }
  return true;
}

// True if a plan holds a radix above 10: those take the kernels' BIG form (the others
// keep the registers of a radix-10 butterfly).
inline bool has_big_radix(const FftPlan& pl) {
  for (int i = 0; i < pl.nf; ++i)
    if (pl.radix[i] > 10) return true;
  return false;
}

template <typename T>
struct RtPlaneArgs {
  int threads;          // of a workgroup
  int n0, n1u, H, M;    // n1u = n1 / XS rows per unit
  int LM;               // row stride in the LDS (odd: rows one below the other miss each other's banks)
  int xs;
  long long N;          // n0 * n1 * n2
  RtPlan r1, r2;        // lengths n1u and H
  float inv_n1u, inv_H; // index_quot
  const cplx<T>* tw1;
  const cplx<T>* tw2;
  const cplx<T>* twr;
  const int* slot2;
  const T* add;         // inverse pass: out = add + add_scale * (transform) where not null
  T add_scale;
  int xcd_run;          // units per XCD run (xcd_grouped); 1: round-robin order
};

template <typename T>
struct RtPencilArgs {
  int threads;             // of a workgroup
  RtPlan r0;
  int es;                  // element stride (complex units)
  int nin;                 // groups of XS sequences per component
  long long outer_stride;  // complex units between components
  int tb;                  // groups per workgroup
  float inv_tb, inv_ts, inv_M;
  int hs;                  // offset of the next unit's spectrum: n1u * M
  int n1u, M;
  const cplx<T>* tw;
  const cplx<T>* twx;      // W_{n1}^{k1} per slot of the unit transform (XS > 1)
  T alpha;
  int s, op;
  T scale;
  const T* ksq0;
  const T* ksq1;           // |k1 + p n1u|^2 at p * n1u + slot
  const T* ksq2;
  int xcd_run;
};

template <typename T>
using RtPlaneFwdFn = void (*)(const T*, cplx<T>*, RtPlaneArgs<T>);
template <typename T>
using RtPlaneInvFn = void (*)(const cplx<T>*, T*, RtPlaneArgs<T>);
template <typename T>
using RtPencilFn = void (*)(cplx<T>*, RtPencilArgs<T>);

// Kernel entry points (fft_rt.hip).  Plane kernels take any workgroup of up to
// 1024 threads, pencils up to 512.
template <typename T>
RtPlaneFwdFn<T> rt_plane_fwd(bool big);
template <typename T>
RtPlaneInvFn<T> rt_plane_inv(bool big);
template <typename T>
RtPencilFn<T> rt_pencil(int xs, bool big);  // xs 1 to 4

}  // namespace lddmm
