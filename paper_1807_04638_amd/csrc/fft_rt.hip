// fft_rt.hip - the three passes of the spectral operator for lengths known at run
// time (see fft_rt.h; fft.hip has the compile-time forms of the common lengths).
//
// Same algorithm as the compile-time kernels: every pass meets global memory
// inside a butterfly stage, stages run in place in the LDS, the symbol is applied
// in registers between the last forward and the first inverse stage.  What would
// be constants there are kernel arguments here: stage strides and twiddle steps
// per stage, and the reciprocals that index_quot divides with (an integer division
// costs about 40 instructions, as much as a radix-5 butterfly; the quotient by a
// float reciprocal 4).  Each radix has its own copy of each stage's code behind a
// uniform branch.  Stages of radix 2 to 5 take several butterflies per turn of the
// loops that read global memory, so that about eight loads per lane are in flight.
#include "fft_rt.h"

#include "lddmm.h"

namespace lddmm {

namespace {

// Run f<R>() for a uniform run-time radix R.
#define LDDMM_RT_RADIX(r, CALL) \
  switch (r) {                  \
    case 2: CALL(2); break;     \
    case 3: CALL(3); break;     \
    case 4: CALL(4); break;     \
    case 5: CALL(5); break;     \
    case 6: CALL(6); break;     \
    case 7: CALL(7); break;     \
    case 8: CALL(8); break;     \
    case 9: CALL(9); break;     \
    case 10: CALL(10); break;   \
    default:                    \
      if constexpr (BIG) {      \
        if (r == 12) CALL(12);  \
        if (r == 14) CALL(14);  \
        if (r == 15) CALL(15);  \
        if (r == 16) CALL(16);  \
      }                         \
      break;                    \
  }

// Element o of a uniform pointer by a 32-bit byte offset: one address register per
// lane beside the scalar base, where a 64-bit index takes a 64-bit addition per
// access (o sizeof(cplx) < 2^32: checked on the host).
template <typename T>
__device__ __forceinline__ const cplx<T>& at(const cplx<T>* p, unsigned o) {
  return *reinterpret_cast<const cplx<T>*>(reinterpret_cast<const char*>(p) + o * unsigned(sizeof(cplx<T>)));
}
template <typename T>
__device__ __forceinline__ cplx<T>& at(cplx<T>* p, unsigned o) {
  return *reinterpret_cast<cplx<T>*>(reinterpret_cast<char*>(p) + o * unsigned(sizeof(cplx<T>)));
}

// Butterflies per turn of a loop over global memory.
constexpr int rt_unroll(int R) { return R <= 2 ? 4 : R <= 3 ? 3 : R <= 5 ? 2 : 1; }

// All butterflies of stage s over `count` sequences held in LDS (element e of
// sequence q at buf[q * ss + e * es]), consecutive lanes on consecutive sequences.
template <typename T, int R, bool INV, bool TW>
__device__ __forceinline__ void rt_stage_r(cplx<T>* buf, const RtStage& s, int total, int count, float inv_count,
                                           int es, int ss, const cplx<T>* tw, int nthr) {
  for (int b = threadIdx.x; b < total; b += nthr) {
    const int u = index_quot(b, inv_count), q = b - mul24(u, count);
    const int blk = TW ? index_quot(u, s.invS) : u;
    const int j = TW ? u - mul24(blk, s.S) : 0;
    const int base = mul24(q, ss) + mul24(mul24(blk, s.L) + j, es);
    if (INV)
      dit_butterfly<T, R, TW, true>(buf, base, s.S * es, j, s.tws, tw);
    else
      dif_butterfly<T, R, TW, true>(buf, base, s.S * es, j, s.tws, tw);
  }
}

// Stages [from, to) of the plan in DIF order forward, in reverse order inverse,
// a barrier after each.
template <typename T, bool INV, bool BIG>
__device__ __forceinline__ void rt_stages(cplx<T>* buf, const RtPlan& pl, int from, int to, int count,
                                          float inv_count, int es, int ss, const cplx<T>* tw, int nthr) {
  for (int i = from; i < to; ++i) {
    const RtStage& s = pl.st[INV ? to - 1 - (i - from) : i];
    const int total = count * (pl.n / s.R);
    if (s.S > 1) {
#define LDDMM_RT_CALL(r) rt_stage_r<T, r, INV, true>(buf, s, total, count, inv_count, es, ss, tw, nthr)
      LDDMM_RT_RADIX(s.R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
    } else {
#define LDDMM_RT_CALL(r) rt_stage_r<T, r, INV, false>(buf, s, total, count, inv_count, es, ss, tw, nthr)
      LDDMM_RT_RADIX(s.R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
    }
    __syncthreads();
  }
}

template <typename T>
struct RtPlaneLds {
  cplx<T>* A;
  cplx<T>* tw1;
  cplx<T>* tw2;
  cplx<T>* twr;
  int* slot2;
};

template <typename T>
__device__ __forceinline__ RtPlaneLds<T> rt_carve(unsigned char* smem, const RtPlaneArgs<T>& a) {
  RtPlaneLds<T> l;
  l.A = reinterpret_cast<cplx<T>*>(smem);
  l.tw1 = l.A + a.n1u * a.LM;
  l.tw2 = l.tw1 + a.n1u;
  l.twr = l.tw2 + a.H;
  l.slot2 = reinterpret_cast<int*>(l.twr + a.H / 2 + 1);
  for (int i = threadIdx.x; i < a.n1u; i += a.threads) l.tw1[i] = a.tw1[i];
  for (int i = threadIdx.x; i < a.H; i += a.threads) l.tw2[i] = a.tw2[i];
  for (int i = threadIdx.x; i <= a.H / 2; i += a.threads) l.twr[i] = a.twr[i];
  for (int i = threadIdx.x; i <= a.H; i += a.threads) l.slot2[i] = a.slot2[i];
  return l;
}

// Unit of the workgroup (component, x0, h): offset of its first row in the field
// and index of its spectrum.
template <typename T>
__device__ __forceinline__ int rt_unit(const RtPlaneArgs<T>& a, long long& row0) {
  const int lin = int(blockIdx.y) * int(gridDim.x) + int(blockIdx.x);
  const int p = a.xcd_run > 1 ? xcd_grouped(lin, int(gridDim.x * gridDim.y), a.xcd_run) : lin;
  const int per_comp = a.n0 * a.xs;
  const int comp = p / per_comp, r = p - comp * per_comp, x0 = r / a.xs, h = r - x0 * a.xs;
  row0 = comp * a.N + ((long long)x0 * a.n1u * a.xs + h) * (2 * a.H);
  return p;
}

// Slot (DIF output position) of frequency k (the inverse of digit_reverse).
__device__ __forceinline__ int rt_slot_of(const RtPlan& pl, int k) {
  int p = 0;
  for (int i = 0; i < pl.nf; ++i) {
    const int q = k / pl.st[i].R;
    p += (k - q * pl.st[i].R) * pl.st[i].S;
    k = q;
  }
  return p;
}

// First DIF stage of the rows straight from global memory, consecutive lanes on
// consecutive elements of a row.
template <typename T, int R>
__device__ __forceinline__ void rt_rows_first(cplx<T>* A, const cplx<T>* __restrict__ src, const RtPlaneArgs<T>& a) {
  constexpr int U = rt_unroll(R);
  const RtStage& s = a.r2.st[0];
  const int total = a.n1u * s.S, rs = a.xs * a.H;
  for (int b0 = threadIdx.x; b0 < total; b0 += U * a.threads) {
    cplx<T> v[U][R];
    int r[U], j[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int b = b0 + k * a.threads;
      r[k] = index_quot(b, s.invS);
      j[k] = b - mul24(r[k], s.S);
      if (b < total) {
#pragma unroll
        for (int q = 0; q < R; ++q) v[k][q] = at(src + q * s.S, mul24(r[k], rs) + j[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (b0 + k * a.threads >= total) break;
      Dft<T, R, -1>::run(v[k]);
      const int base = mul24(r[k], a.LM) + j[k];
      A[base] = v[k][0];
      cplx<T> w[R];
      // the table in global memory: the LDS copy is complete only after the barrier
      twiddle_reads<T, R>(w, j[k], 1, a.tw2);
#pragma unroll
      for (int q = 1; q < R; ++q) A[base + q * s.S] = s.S > 1 ? c_mul(v[k][q], w[q]) : v[k][q];
    }
  }
}

// Last DIT stage of the rows straight to global memory (with the addend).
template <typename T, int R>
__device__ __forceinline__ void rt_rows_last(const cplx<T>* A, cplx<T>* __restrict__ dst,
                                             const cplx<T>* __restrict__ add, const RtPlaneArgs<T>& a,
                                             const cplx<T>* tw2) {
  const RtStage& s = a.r2.st[0];
  const int total = a.n1u * s.S, rs = a.xs * a.H;
  for (int b = threadIdx.x; b < total; b += a.threads) {
    const int r = index_quot(b, s.invS), j = b - mul24(r, s.S);
    const int base = mul24(r, a.LM) + j, o = mul24(r, rs) + j;
    cplx<T> v[R], w[R];
    twiddle_reads<T, R>(w, j, 1, tw2);
    v[0] = A[base];
#pragma unroll
    for (int q = 1; q < R; ++q) v[q] = s.S > 1 ? c_mulc(A[base + q * s.S], w[q]) : A[base + q * s.S];
    cplx<T> ad[R];
    if (add) {
#pragma unroll
      for (int q = 0; q < R; ++q) ad[q] = at(add + q * s.S, o);
    }
    Dft<T, R, +1>::run(v);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (add) v[q] = {ad[q].x + a.add_scale * v[q].x, ad[q].y + a.add_scale * v[q].y};
      at(dst + q * s.S, o) = v[q];
    }
  }
}

// Last DIF stage of the columns (stride 1) straight to the spectrum; the packed
// column 0 goes back to LDS for the split.
template <typename T, int R>
__device__ __forceinline__ void rt_cols_last(cplx<T>* A, cplx<T>* __restrict__ dst, const RtPlaneArgs<T>& a) {
  const int total = a.H * (a.n1u / R);
  for (int b = threadIdx.x; b < total; b += a.threads) {
    const int u = index_quot(b, a.inv_H), col = b - mul24(u, a.H);
    const int row = mul24(u, R);
    cplx<T> v[R];
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = A[mul24(row, a.LM) + col + q * a.LM];
    Dft<T, R, -1>::run(v);
    if (col == 0) {
#pragma unroll
      for (int q = 0; q < R; ++q) A[mul24(row, a.LM) + q * a.LM] = v[q];
    } else {
#pragma unroll
      for (int q = 0; q < R; ++q) at(dst + q * a.M, mul24(row, a.M) + col) = v[q];
    }
  }
}

// First DIT stage of the columns (stride 1) straight from the spectrum, column H
// packed into column 0 as X[0] + i X[N2/2].
template <typename T, int R>
__device__ __forceinline__ void rt_cols_first(cplx<T>* A, const cplx<T>* __restrict__ src, const RtPlaneArgs<T>& a) {
  constexpr int U = rt_unroll(R);
  const int total = a.H * (a.n1u / R);
  for (int b0 = threadIdx.x; b0 < total; b0 += U * a.threads) {
    cplx<T> v[U][R];
    int u[U], col[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int b = b0 + k * a.threads;
      u[k] = index_quot(b, a.inv_H);
      col[k] = b - mul24(u[k], a.H);
      if (b < total) {
#pragma unroll
        for (int q = 0; q < R; ++q) v[k][q] = at(src + q * a.M, mul24(u[k], R * a.M) + col[k]);
        if (col[k] == 0) {
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const cplx<T> hi = at(src + q * a.M + a.H, mul24(u[k], R * a.M));
            v[k][q] = {v[k][q].x - hi.y, v[k][q].y + hi.x};
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (b0 + k * a.threads >= total) break;
      Dft<T, R, +1>::run(v[k]);
#pragma unroll
      for (int q = 0; q < R; ++q) A[mul24(u[k], R * a.LM) + col[k] + q * a.LM] = v[k][q];
    }
  }
}

// Waves per SIMD that the registers leave room for: two 1024-lane workgroups per
// compute unit in FP32.
constexpr int rt_plane_waves(size_t element, bool big) { return element == 4 && !big ? 8 : 4; }

// One unit of a plane: real rows -> x2 spectrum -> x1 columns.  The real columns
// k2 = 0 and k2 = N2/2 travel packed in column 0 through the x1 transform.
template <typename T, bool BIG>
__global__ void __launch_bounds__(1024, (rt_plane_waves(sizeof(T), BIG))) k_plane_fwd_rt(const T* __restrict__ in, cplx<T>* __restrict__ spec,
                                                       RtPlaneArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RtPlaneLds<T> l = rt_carve(smem, a);
  cplx<T>* A = l.A;
  long long row0;
  const int p = rt_unit(a, row0);
  const cplx<T>* src = reinterpret_cast<const cplx<T>*>(in + row0);
#define LDDMM_RT_CALL(r) rt_rows_first<T, r>(A, src, a)
  LDDMM_RT_RADIX(a.r2.st[0].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
  __syncthreads();
  rt_stages<T, false, BIG>(A, a.r2, 1, a.r2.nf, a.n1u, a.inv_n1u, 1, a.LM, l.tw2, a.threads);
  // split the half-length spectrum into the frequencies of the real row: item k
  // does the pair (k, H - k), the last k also k = 0 (X[0] + i X[H], packed)
  const int ki = a.H / 2;
  for (int idx = threadIdx.x; idx < a.n1u * ki; idx += a.threads) {
    const int k0 = index_quot(idx, a.inv_n1u), k = k0 + 1;
    cplx<T>* row = A + mul24(idx - mul24(k0, a.n1u), a.LM);
    const int sk = l.slot2[k], sm = l.slot2[a.H - k];
    const cplx<T> x = row[sk], y = row[sm];
    const cplx<T> e = {T(0.5) * (x.x + y.x), T(0.5) * (x.y - y.y)};
    const cplx<T> o = {T(0.5) * (x.x - y.x), T(0.5) * (x.y + y.y)};
    const cplx<T> wo = c_mul(l.twr[k], o);
    row[sk] = {e.x + wo.y, e.y - wo.x};
    if (sm != sk) row[sm] = {e.x - wo.y, -e.y - wo.x};
    if (k == ki) {
      const cplx<T> z = row[0];
      row[0] = {z.x + z.y, z.x - z.y};
    }
  }
  __syncthreads();
  rt_stages<T, false, BIG>(A, a.r1, 0, a.r1.nf - 1, a.H, a.inv_H, a.LM, 1, l.tw1, a.threads);
  cplx<T>* dst = spec + (long long)p * (a.n1u * a.M);
#define LDDMM_RT_CALL(r) rt_cols_last<T, r>(A, dst, a)
  LDDMM_RT_RADIX(a.r1.st[a.r1.nf - 1].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
  __syncthreads();
  for (int k = threadIdx.x; k <= a.n1u / 2; k += a.threads) {
    const int sk = rt_slot_of(a.r1, k), sm = rt_slot_of(a.r1, k == 0 ? 0 : a.n1u - k);
    const cplx<T> zk = A[sk * a.LM], zm = A[sm * a.LM];
    const cplx<T> lo = {T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y - zm.y)};
    const cplx<T> hi = {T(0.5) * (zk.y + zm.y), T(0.5) * (zm.x - zk.x)};
    dst[sk * a.M] = lo;
    dst[sk * a.M + a.H] = hi;
    dst[sm * a.M] = c_conj(lo);
    dst[sm * a.M + a.H] = c_conj(hi);
  }
}

// The inverse of k_plane_fwd_rt, times n1u * N2 (and the addend).
template <typename T, bool BIG>
__global__ void __launch_bounds__(1024, (rt_plane_waves(sizeof(T), BIG))) k_plane_inv_rt(const cplx<T>* __restrict__ spec, T* __restrict__ out,
                                                       RtPlaneArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RtPlaneLds<T> l = rt_carve(smem, a);
  cplx<T>* A = l.A;
  long long row0;
  const int p = rt_unit(a, row0);
  const cplx<T>* src = spec + (long long)p * (a.n1u * a.M);
#define LDDMM_RT_CALL(r) rt_cols_first<T, r>(A, src, a)
  LDDMM_RT_RADIX(a.r1.st[a.r1.nf - 1].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
  __syncthreads();
  rt_stages<T, true, BIG>(A, a.r1, 0, a.r1.nf - 1, a.H, a.inv_H, a.LM, 1, l.tw1, a.threads);
  const int ki = a.H / 2;
  for (int idx = threadIdx.x; idx < a.n1u * ki; idx += a.threads) {
    const int k0 = index_quot(idx, a.inv_n1u), k = k0 + 1;
    cplx<T>* row = A + mul24(idx - mul24(k0, a.n1u), a.LM);
    const int sk = l.slot2[k], sm = l.slot2[a.H - k];
    const cplx<T> x = row[sk], y = row[sm];
    const cplx<T> f = {x.x + y.x, x.y - y.y};  // X[k] + conj X[H-k]
    const cplx<T> d = {x.x - y.x, x.y + y.y};  // X[k] - conj X[H-k]
    const cplx<T> t = c_mulc(d, l.twr[k]);     // conj(w) d
    row[sk] = {f.x - t.y, f.y + t.x};          // f + i t
    if (sm != sk) row[sm] = {f.x + t.y, -f.y + t.x};  // conj(f) + i conj(t)
    if (k == ki) {
      const cplx<T> z = row[0];
      row[0] = {z.x + z.y, z.x - z.y};
    }
  }
  __syncthreads();
  rt_stages<T, true, BIG>(A, a.r2, 1, a.r2.nf, a.n1u, a.inv_n1u, 1, a.LM, l.tw2, a.threads);
  cplx<T>* dst = reinterpret_cast<cplx<T>*>(out + row0);
  const cplx<T>* add = a.add ? reinterpret_cast<const cplx<T>*>(a.add + row0) : nullptr;
#define LDDMM_RT_CALL(r) rt_rows_last<T, r>(A, dst, add, a, l.tw2)
  LDDMM_RT_RADIX(a.r2.st[0].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
}

// a / x: the hardware's FP32 reciprocal (1 ulp) and one correction of the quotient,
// which rounds as the division it replaces does (to half an ulp but for rare ties) at
// a third of its instructions; x >= 1 here.  A power that overflowed (x infinite) gives
// the division's 0: there the remainder x q would be infinity times 0.
__device__ __forceinline__ float rt_div(float a, float x) {
  const float r = __builtin_amdgcn_rcpf(x), q = a * r;
  return __builtin_isinf(x) ? q : fmaf(fmaf(-x, q, a), r, q);
}
__device__ __forceinline__ double rt_div(double a, double x) { return a / x; }

// The last DIF stage (stride 1), the symbol and the first DIT stage in registers.
template <typename T, int R>
__device__ __forceinline__ void rt_symbol(cplx<T>* A, const T* ksq0, const T* ksq12, const RtPencilArgs<T>& a, int ts) {
  const int total = ts * (a.r0.n / R);
  for (int b = threadIdx.x; b < total; b += a.threads) {
    const int u = index_quot(b, a.inv_ts), q = b - mul24(u, ts);
    cplx<T>* x = A + mul24(u, R * ts) + q;
    cplx<T> v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = x[i * ts];
    Dft<T, R, -1>::run(v);
    const T c12 = T(1) + a.alpha * ksq12[q];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const T bq = a.alpha * ksq0[u * R + i] + c12;
      T pw = bq * (a.s >= 2 ? bq : T(1));
      for (int k = 2; k < a.s; ++k) pw *= bq;
      v[i] = c_scale(v[i], a.op == LDDMM_OP_K ? rt_div(a.scale, pw) : a.scale * pw);
    }
    Dft<T, R, +1>::run(v);
#pragma unroll
    for (int i = 0; i < R; ++i) x[i * ts] = v[i];
  }
}

// The XS values of a group at one element become those of its XS pencils (the
// first radix-XS step of the x1 transform), and back.
template <typename T, int XS>
__device__ __forceinline__ void rt_merge(cplx<T>* y, const cplx<T>& wx) {
  if constexpr (XS > 1) {
    cplx<T> w = wx;
#pragma unroll
    for (int h = 1; h < XS; ++h) {
      y[h] = c_mul(y[h], w);
      if (h + 1 < XS) w = c_mul(w, wx);
    }
    Dft<T, XS, -1>::run(y);
  }
}
template <typename T, int XS>
__device__ __forceinline__ void rt_unmerge(cplx<T>* y, const cplx<T>& wx) {
  if constexpr (XS > 1) {
    Dft<T, XS, +1>::run(y);
    cplx<T> w = wx;
#pragma unroll
    for (int h = 1; h < XS; ++h) {
      y[h] = c_mulc(y[h], w);
      if (h + 1 < XS) w = c_mul(w, wx);
    }
  }
}

// Merge and first DIF stage of a tile's groups straight from the spectrum, and the
// last DIT stage with its unmerge straight to it (XS <= 2 and at least two stages:
// XS R values per lane).
template <typename T, int XS, int R>
__device__ __forceinline__ void rt_pencil_first(cplx<T>* A, const cplx<T>* __restrict__ base,
                                                const RtPencilArgs<T>& a, int q0, int cnt) {
  const RtStage& s = a.r0.st[0];
  const int tb = a.tb, ts = XS * tb, total = tb * s.S;
  for (int b = threadIdx.x; b < total; b += a.threads) {
    const int j = index_quot(b, a.inv_tb), t = b - mul24(j, tb);
    const bool live = t < cnt;
    const unsigned o = unsigned(j) * unsigned(a.es) + t;
    cplx<T> v[XS][R];
    const cplx<T> wx = XS > 1 && live ? a.twx[index_quot(q0 + t, a.inv_M)] : cplx<T>{T(1), T(0)};
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const cplx<T>* bq = base + (long long)(q * s.S) * a.es;
      cplx<T> y[XS];
#pragma unroll
      for (int h = 0; h < XS; ++h) y[h] = live ? at(bq + h * a.hs, o) : cplx<T>{T(0), T(0)};
      rt_merge<T, XS>(y, wx);
#pragma unroll
      for (int h = 0; h < XS; ++h) v[h][q] = y[h];
    }
    cplx<T> w[R];
    twiddle_reads<T, R>(w, j, 1, a.tw);
#pragma unroll
    for (int h = 0; h < XS; ++h) {
      Dft<T, R, -1>::run(v[h]);
      cplx<T>* x = A + mul24(j, ts) + h * tb + t;
      x[0] = v[h][0];
#pragma unroll
      for (int q = 1; q < R; ++q) x[q * s.S * ts] = c_mul(v[h][q], w[q]);
    }
  }
}
template <typename T, int XS, int R>
__device__ __forceinline__ void rt_pencil_last(const cplx<T>* A, cplx<T>* __restrict__ base, const cplx<T>* tw,
                                               const RtPencilArgs<T>& a, int q0, int cnt) {
  const RtStage& s = a.r0.st[0];
  const int tb = a.tb, ts = XS * tb, total = tb * s.S;
  for (int b = threadIdx.x; b < total; b += a.threads) {
    const int j = index_quot(b, a.inv_tb), t = b - mul24(j, tb);
    if (t >= cnt) continue;
    const unsigned o = unsigned(j) * unsigned(a.es) + t;
    cplx<T> v[XS][R], w[R];
    const cplx<T> wx = XS > 1 ? a.twx[index_quot(q0 + t, a.inv_M)] : cplx<T>{T(1), T(0)};
    twiddle_reads<T, R>(w, j, 1, tw);
#pragma unroll
    for (int h = 0; h < XS; ++h) {
      const cplx<T>* x = A + mul24(j, ts) + h * tb + t;
      v[h][0] = x[0];
#pragma unroll
      for (int q = 1; q < R; ++q) v[h][q] = c_mulc(x[q * s.S * ts], w[q]);
      Dft<T, R, +1>::run(v[h]);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      cplx<T>* bq = base + (long long)(q * s.S) * a.es;
      cplx<T> y[XS];
#pragma unroll
      for (int h = 0; h < XS; ++h) y[h] = v[h][q];
      rt_unmerge<T, XS>(y, wx);
#pragma unroll
      for (int h = 0; h < XS; ++h) at(bq + h * a.hs, o) = y[h];
    }
  }
}

// x0 pencils with the symbol: tb groups of XS sequences per workgroup.
template <typename T, int XS, bool BIG>
__global__ void __launch_bounds__(512) k_pencil_rt(cplx<T>* __restrict__ spec, RtPencilArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = a.r0.n, tb = a.tb, ts = XS * tb;
  cplx<T>* A = reinterpret_cast<cplx<T>*>(smem);
  cplx<T>* tw = A + n * ts;
  T* ksq0 = reinterpret_cast<T*>(tw + n);
  T* ksq12 = ksq0 + n;
  const int lin0 = int(blockIdx.y * gridDim.x + blockIdx.x);
  const int lin = a.xcd_run > 1 ? xcd_grouped(lin0, int(gridDim.x * gridDim.y), a.xcd_run) : lin0;
  const int comp = lin / int(gridDim.x), q0 = (lin - comp * int(gridDim.x)) * tb;
  const int cnt = (a.nin - q0) < tb ? (a.nin - q0) : tb;
  cplx<T>* base = spec + comp * a.outer_stride + q0;
  for (int i = threadIdx.x; i < n; i += a.threads) {
    tw[i] = a.tw[i];
    ksq0[i] = a.ksq0[i];
  }
  for (int i = threadIdx.x; i < ts; i += a.threads) {
    const int h = i / tb, q = q0 + i - h * tb;
    const int s1 = q / a.M, s2 = q - s1 * a.M;
    ksq12[i] = q < a.nin ? a.ksq1[h * a.n1u + s1] + a.ksq2[s2] : T(0);
  }
  const bool fuse = XS <= 2 && a.r0.nf >= 2;
  if (fuse) {
    if constexpr (XS <= 2) {
#define LDDMM_RT_CALL(r) rt_pencil_first<T, XS, r>(A, base, a, q0, cnt)
      LDDMM_RT_RADIX(a.r0.st[0].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
    }
    __syncthreads();
  } else {
    for (int b = threadIdx.x; b < n * tb; b += a.threads) {
      const int j = index_quot(b, a.inv_tb), t = b - mul24(j, tb);
      const bool live = t < cnt;
      cplx<T> y[XS];
#pragma unroll
      for (int h = 0; h < XS; ++h) y[h] = live ? at(base + h * a.hs, unsigned(j) * unsigned(a.es) + t) : cplx<T>{T(0), T(0)};
      const cplx<T> wx = XS > 1 && live ? a.twx[index_quot(q0 + t, a.inv_M)] : cplx<T>{T(1), T(0)};
      rt_merge<T, XS>(y, wx);
#pragma unroll
      for (int h = 0; h < XS; ++h) A[mul24(j, ts) + h * tb + t] = y[h];
    }
    __syncthreads();
  }
  const int from = fuse ? 1 : 0;
  rt_stages<T, false, BIG>(A, a.r0, from, a.r0.nf - 1, ts, a.inv_ts, ts, 1, tw, a.threads);
#define LDDMM_RT_CALL(r) rt_symbol<T, r>(A, ksq0, ksq12, a, ts)
  LDDMM_RT_RADIX(a.r0.st[a.r0.nf - 1].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
  __syncthreads();
  rt_stages<T, true, BIG>(A, a.r0, from, a.r0.nf - 1, ts, a.inv_ts, ts, 1, tw, a.threads);
  if (fuse) {
    if constexpr (XS <= 2) {
#define LDDMM_RT_CALL(r) rt_pencil_last<T, XS, r>(A, base, tw, a, q0, cnt)
      LDDMM_RT_RADIX(a.r0.st[0].R, LDDMM_RT_CALL)
#undef LDDMM_RT_CALL
    }
  } else {
    for (int b = threadIdx.x; b < n * tb; b += a.threads) {
      const int j = index_quot(b, a.inv_tb), t = b - mul24(j, tb);
      if (t >= cnt) continue;
      cplx<T> y[XS];
#pragma unroll
      for (int h = 0; h < XS; ++h) y[h] = A[mul24(j, ts) + h * tb + t];
      const cplx<T> wx = XS > 1 ? a.twx[index_quot(q0 + t, a.inv_M)] : cplx<T>{T(1), T(0)};
      rt_unmerge<T, XS>(y, wx);
#pragma unroll
      for (int h = 0; h < XS; ++h) at(base + h * a.hs, unsigned(j) * unsigned(a.es) + t) = y[h];
    }
  }
}

}  // namespace

template <typename T>
RtPlaneFwdFn<T> rt_plane_fwd(bool big) {
  return big ? k_plane_fwd_rt<T, true> : k_plane_fwd_rt<T, false>;
}
template <typename T>
RtPlaneInvFn<T> rt_plane_inv(bool big) {
  return big ? k_plane_inv_rt<T, true> : k_plane_inv_rt<T, false>;
}
template <typename T>
RtPencilFn<T> rt_pencil(int xs, bool big) {
  switch (xs) {
    case 1: return big ? k_pencil_rt<T, 1, true> : k_pencil_rt<T, 1, false>;
    case 2: return big ? k_pencil_rt<T, 2, true> : k_pencil_rt<T, 2, false>;
    case 3: return big ? k_pencil_rt<T, 3, true> : k_pencil_rt<T, 3, false>;
    case 4: return big ? k_pencil_rt<T, 4, true> : k_pencil_rt<T, 4, false>;
    default: return nullptr;
  }
}

#define LDDMM_RTINST(T)                       \
  template RtPlaneFwdFn<T> rt_plane_fwd(bool); \
  template RtPlaneInvFn<T> rt_plane_inv(bool); \
  template RtPencilFn<T> rt_pencil<T>(int, bool);
LDDMM_RTINST(float)
LDDMM_RTINST(double)

}  // namespace lddmm
