// sl.hip - semi-Lagrangian transport of the state equation (Section 2.3:
// d_t J + grad J . v = 0, J(0) = I_0) through the inverse-map displacement
// u = phi^-1 - id, and the final composition J_1 = I_0 o (id + u_1).
//
// One step, with grid-time velocities v_old = v_n and v_new = v_{n+1}:
//   foot point  X = x - dt/2 (v_new(x) + v_old(x - dt v_new(x)))   (Heun backtrace)
//   u_new(x)    = u_old(X) + (X - x)
// Interpolation is periodic trilinear.  Each voxel's query point is handled as
// its integer index plus a small offset in voxels, so the fractional weights
// keep full precision in FP32 at any grid index.
#include "lddmm.h"
#include "lddmm_internal.h"

namespace lddmm {

namespace {

template <typename T>
struct SlGeo {
  int n0, n1, n2;
  int N;
  T invh[3];
  FieldTiling ft;
};

template <typename T>
SlGeo<T> make_sl_geo(const Grid& g) {
  SlGeo<T> o;
  o.n0 = g.n0;
  o.n1 = g.n1;
  o.n2 = g.n2;
  o.N = g.N;
  o.invh[0] = T(1.0 / g.h0);
  o.invh[1] = T(1.0 / g.h1);
  o.invh[2] = T(1.0 / g.h2);
  o.ft = make_field_tiling(g);
  return o;
}

// Corners and weights of the trilinear stencil at voxel (i0, i1, i2) displaced by
// (d0, d1, d2) voxels.  The two x2 corners of each (x0, x1) pair are adjacent in
// memory unless the lower one is the last of its row (periodic wrap), so a pair
// is one two-element load: o[k] is the lower corner of pair k = 2 c0 + c1, wrap
// says the upper corner is the first of the row (o[k] - (N2 - 1)).
template <typename T>
struct Tri {
  int o[4];
  int n2m1;
  bool wrap;
  T w01[4];   // (x0, x1) weight of pair k
  T t2;       // x2 fraction: weights 1 - t2, t2 of the lower and upper corner
};

template <typename T>
__device__ __forceinline__ Tri<T> tri_setup(const SlGeo<T>& g, int i0, int i1, int i2, T d0, T d1, T d2) {
  // cells and weights per axis (offsets clamped, indices wrapped: sl_axis)
  int a0, b0, a1, b1, a2, b2;
  T t0, t1, t2;
  sl_axis(i0, d0, g.n0, a0, b0, t0);
  sl_axis(i1, d1, g.n1, a1, b1, t1);
  sl_axis(i2, d2, g.n2, a2, b2, t2);
  (void)b2;
  const int s0 = g.n1 * g.n2;
  const int r0[2] = {a0 * s0, b0 * s0};
  const int r1[2] = {a1 * g.n2, b1 * g.n2};
  const T w0[2] = {T(1) - t0, t0}, w1[2] = {T(1) - t1, t1};
  Tri<T> tr;
  // offsets fit in int: 3 N < 2^31
#pragma unroll
  for (int c0 = 0; c0 < 2; ++c0)
#pragma unroll
    for (int c1 = 0; c1 < 2; ++c1) {
      const int k = c0 * 2 + c1;
      tr.o[k] = r0[c0] + r1[c1] + a2;
      tr.w01[k] = w0[c0] * w1[c1];
    }
  tr.n2m1 = g.n2 - 1;
  tr.wrap = a2 == g.n2 - 1;
  tr.t2 = t2;
  return tr;
}

// Two consecutive elements f[o], f[o + 1] as one 8-byte load (4-byte aligned:
// the hardware takes element-aligned vector loads from global memory).
__device__ __forceinline__ void load_pair(const float* __restrict__ f, int o, float& lo, float& hi) {
  typedef float vec2 __attribute__((ext_vector_type(2)));
  vec2 v;
  __builtin_memcpy(&v, f + o, sizeof(vec2));
  lo = v.x;
  hi = v.y;
}

// Values of NC fields at the point.  FP32 reads each x2 pair with one load (half the
// gathers); at the end of a row the pair before it holds the lower corner, and only the
// upper one takes a load of its own.  All pairs' loads come first, so that they are in
// flight together and the row ends cost one branch (a step at 128^3 38 us, with a branch
// per pair 46).  FP64 reads the corners one by one, field by field (16-byte pairs
// measured slower than two loads, and all fields' loads first no faster).
template <typename T, int NC>
__device__ __forceinline__ void tri_eval(T (&out)[NC], const Tri<T>& tr, const T* const* f) {
  if constexpr (sizeof(T) == 4) {
    T lo[NC][4], hi[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) load_pair(f[c], tr.wrap ? tr.o[k] - 1 : tr.o[k], lo[c][k], hi[c][k]);
    if (tr.wrap) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          lo[c][k] = hi[c][k];
          hi[c][k] = f[c][tr.o[k] - tr.n2m1];
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      out[c] = T(0);
#pragma unroll
      for (int k = 0; k < 4; ++k) out[c] += tr.w01[k] * (lo[c][k] + tr.t2 * (hi[c][k] - lo[c][k]));
    }
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      out[c] = T(0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const T lo = f[c][tr.o[k]], hi = f[c][tr.wrap ? tr.o[k] - tr.n2m1 : tr.o[k] + 1];
        out[c] += tr.w01[k] * (lo + tr.t2 * (hi - lo));
      }
    }
  }
}
template <typename T>
__device__ __forceinline__ T tri_one(const Tri<T>& tr, const T* f) {
  T v[1];
  tri_eval<T, 1>(v, tr, &f);
  return v[0];
}

// ---------------------------------------------------------------------------
// One step along the characteristics: from the velocity vc at the voxel and vg
// gathered at the predicted point, the foot (or head) of the characteristic, and
// there the fields f[0 .. NF):
//   P = +-dt vc,  disp = +-dt/2 (vc + vg(x + P)),  val_c = f_c(x + disp)
// SL_START  u_new = disp                      (the shooting's first step, u = 0)
// SL_STEP   u_new = u_old(X) + disp           (f = u_old)
// SL_STATE  m_new = m_old(X)                  (PDE-LDDMM: the image itself)
// SL_INCR   dm_new = dm_old(X) + dt/2 (s_old(X) + s_new(x))
// SL_ADJOINT  lam_old = lam_new(Y) exp(dt/2 (D_old(x) + D_new(Y))), forward, D = div v
//
// Bound by the L1's return path when gathered from global memory (24 8-byte gathers
// per voxel: 38 us at 128^3 FP32 for 100 MB).  A step moves a point by less than a
// voxel as a rule, so the workgroup puts its tile of each field with one voxel around
// it into the LDS (2 planes of 4 x 64 voxels: 3.1 times the tile's values, of 8 x 32:
// 2.7; coalesced) and gathers there, without wrapping.  The second fields' window is in
// flight in registers while the first is gathered.  Lanes whose point leaves the window
// gather from global memory, and so does the whole tile, before it loads a window, where
// points leave it in many of its waves.  us per sl_step with steps of at most 0.5, 1.5,
// 3 and 6 voxels, in brackets all gathering (k_sl_points): 128^3 FP32 28, 27, 43, 52
// (38, 38, 41, 49), FP64 44, 44, 58, 74 (55, 55, 56, 74).
// ---------------------------------------------------------------------------
enum { SL_START, SL_STEP, SL_STATE, SL_INCR, SL_ADJOINT };
constexpr int sl_fields(int kind) { return kind == SL_START ? 0 : kind == SL_STEP ? 3 : kind == SL_STATE ? 1 : 2; }

// Waves with a point outside the window, per plane of a tile's four, above which the
// tile gathers from global memory.  FP32 one (128^3, 2 voxels a step: 33.8 us, none 36.5,
// two 33.2; 96^3, 1.5 voxels: 17.3, 17.4, 18.9); FP64 none (60 x 84 x 70, 1.5 voxels:
// 13.4 us, one 16.3): its lone lanes' loads are serial.
template <typename T>
constexpr int kSlSpread = sizeof(T) == 4 ? 1 : 0;

template <typename T>
struct SlIo {
  const T* vc;
  const T* vg;
  const T* f[3];
  const T* at_x;  // s_new (SL_INCR), D_old (SL_ADJOINT)
  T* out;
};

// Window elements of a lane, NF fields: registers <- global, LDS <- registers.  Lanes past
// the window's end load its last element again: a load behind a branch each would wait
// for the one before it.
template <typename T, int NF, int NL>
__device__ __forceinline__ void window_load(T (&r)[NF][NL], const T* const (&f)[3], const int (&go)[NL]) {
#pragma unroll
  for (int c = 0; c < NF; ++c)
#pragma unroll
    for (int l = 0; l < NL; ++l) r[c][l] = f[c][go[l]];
}
template <typename T, int NF, int NL>
__device__ __forceinline__ void window_store(T* w, const T (&r)[NF][NL], int count) {
#pragma unroll
  for (int c = 0; c < NF; ++c)
#pragma unroll
    for (int l = 0; l < NL; ++l)
      if (int(threadIdx.x) + l * kSlLanes < count) w[c * count + int(threadIdx.x) + l * kSlLanes] = r[c][l];
}

// Cell and weights of a displacement of less than a voxel in a window: lower corner
// relative to the voxel's own cell.
template <typename T>
struct WinTri {
  int o;  // lower corner in the window
  T t[3];
};

template <typename T>
__device__ __forceinline__ bool win_setup(WinTri<T>& w, const T d[3], int centre, const SlTile& t) {
  bool ok = true;
  int f[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const T fl = floor(d[e]);
    ok = ok && (fl == T(-1) || fl == T(0));
    w.t[e] = d[e] - fl;
    f[e] = fl < T(0) ? -1 : 0;
  }
  w.o = centre + f[0] * t.plane + f[1] * t.row + f[2];
  return ok;
}

template <typename T>
__device__ __forceinline__ T win_eval(const WinTri<T>& w, const T* win, const SlTile& t) {
  T acc = T(0);
#pragma unroll
  for (int c0 = 0; c0 < 2; ++c0)
#pragma unroll
    for (int c1 = 0; c1 < 2; ++c1) {
      const T* p = win + w.o + c0 * t.plane + c1 * t.row;
      const T lo = p[0], hi = p[1];
      const T w01 = (c0 ? w.t[0] : T(1) - w.t[0]) * (c1 ? w.t[1] : T(1) - w.t[1]);
      acc += w01 * (lo + w.t[2] * (hi - lo));
    }
  return acc;
}

// Result of a step at voxel o: disp and the fields' values there.
template <typename T, int KIND, int NR>
__device__ __forceinline__ void sl_write(const SlGeo<T>& g, const SlIo<T>& io, int o, const T (&d)[3], const T (&v)[NR],
                                         T dt) {
  if constexpr (KIND == SL_START || KIND == SL_STEP) {
#pragma unroll
    for (int c = 0; c < 3; ++c) io.out[c * g.N + o] = KIND == SL_STEP ? v[KIND == SL_STEP ? c : 0] + d[c] : d[c];
  } else if constexpr (KIND == SL_STATE) {
    io.out[o] = v[0];
  } else if constexpr (KIND == SL_INCR) {
    io.out[o] = v[0] + T(0.5) * dt * (v[NR - 1] + io.at_x[o]);
  } else {
    io.out[o] = v[0] * exp(T(0.5) * dt * (io.at_x[o] + v[NR - 1]));
  }
}

// A voxel's step by gathers from global memory, vc its velocity (not written where !own).
template <typename T, int KIND>
__device__ __forceinline__ void sl_point(const SlGeo<T>& g, const SlIo<T>& io, int i0, int i1, int i2, const T (&vc)[3],
                                         T dt, bool own) {
  constexpr int NF = sl_fields(KIND), NR = NF > 0 ? NF : 1;
  constexpr T sgn = KIND == SL_ADJOINT ? T(1) : T(-1);
  const T* const vg[3] = {io.vg, io.vg + g.N, io.vg + 2 * g.N};
  T d[3], v[NR] = {};
  tri_eval<T, 3>(d, tri_setup(g, i0, i1, i2, sgn * dt * vc[0] * g.invh[0], sgn * dt * vc[1] * g.invh[1],
                              sgn * dt * vc[2] * g.invh[2]),
                 vg);
#pragma unroll
  for (int c = 0; c < 3; ++c) d[c] = sgn * T(0.5) * dt * (vc[c] + d[c]);
  if constexpr (NF > 0)
    tri_eval<T, NF>(v, tri_setup(g, i0, i1, i2, d[0] * g.invh[0], d[1] * g.invh[1], d[2] * g.invh[2]), io.f);
  if (own) sl_write<T, KIND, NR>(g, io, (i0 * g.n1 + i1) * g.n2 + i2, d, v, dt);
}

template <typename T, int KIND>
__global__ void __launch_bounds__(256) k_sl_points(SlGeo<T> g, SlIo<T> io, T dt) {
  int i0, i1, i2;
  if (!tile_voxel(g.ft, g.n1, g.n2, i0, i1, i2)) return;
  const int o = (i0 * g.n1 + i1) * g.n2 + i2;
  const T vc[3] = {io.vc[o], io.vc[g.N + o], io.vc[2 * g.N + o]};
  sl_point<T, KIND>(g, io, i0, i1, i2, vc, dt, true);
}

// FP32 held to 128 registers (128^3 PDE steps 24 us, unbounded 26); FP64 needs no more
// than that by itself, and under a bound waits for the gathers one by one (6 voxels a
// step: 74 us, bounded 82).
template <typename T, int KIND, int T0>
__global__ void __launch_bounds__(kSlLanes, sizeof(T) == 4 ? 4 : 1) k_sl(SlGeo<T> g, SlTile t, SlIo<T> io, T dt) {
  constexpr int NF = sl_fields(KIND), NR = NF > 0 ? NF : 1;
  constexpr int NL = sl_window_loads(T0);
  constexpr T sgn = KIND == SL_ADJOINT ? T(1) : T(-1);
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int votes[kSlLanes / 64];
  T* win = reinterpret_cast<T*>(smem);
  int b0, b1, b2;
  if (!sl_tile_block(t, int(blockIdx.x), b0, b1, b2)) return;
  const int lane = int(threadIdx.x);
  const T* const vg[3] = {io.vg, io.vg + g.N, io.vg + 2 * g.N};
  const int l1 = index_quot(lane, t.inv_T2), l2 = lane - mul24(l1, t.T2);
  const int i1 = b1 + l1, i2 = b2 + l2;
  const bool column = l1 < t.T1 && i1 < g.n1 && i2 < g.n2;
  const int s0 = g.n1 * g.n2, o0 = (b0 * g.n1 + i1) * g.n2 + i2;
  const int centre = t.plane + (l1 + 1) * t.row + l2 + 1;
  T d[T0][3];  // vc, then the displacement
  WinTri<T> w[T0];
  unsigned far = 0;  // planes whose point leaves the window
#pragma unroll
  for (int k = 0; k < T0; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c) d[k][c] = column && b0 + k < g.n0 ? io.vc[c * g.N + o0 + k * s0] : T(0);
  int spread = 0;
#pragma unroll
  for (int k = 0; k < T0; ++k) {
    T p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = sgn * dt * d[k][c] * g.invh[c];
    const bool out = !win_setup(w[k], p, centre + k * t.plane, t);
    far |= out ? 1u << k : 0u;
    spread += __any(out) ? 1 : 0;
  }
  if ((lane & 63) == 0) votes[lane >> 6] = spread;
  __syncthreads();
  spread = 0;
#pragma unroll
  for (int i = 0; i < kSlLanes / 64; ++i) spread += votes[i];
  if (__builtin_amdgcn_readfirstlane(spread) > kSlSpread<T> * T0) {
    const int j1 = i1 < g.n1 ? i1 : 0, j2 = i2 < g.n2 ? i2 : 0;  // lanes without a voxel gather at another
#pragma unroll 1
    for (int k = 0; k < T0 && b0 + k < g.n0; ++k) {
      T vc[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if constexpr (T0 > 2) {  // from memory again: the choice among four planes' registers spills
          vc[c] = io.vc[c * g.N + ((b0 + k) * g.n1 + j1) * g.n2 + j2];
        } else {
          vc[c] = d[0][c];
#pragma unroll
          for (int m = 1; m < T0; ++m) vc[c] = k == m ? d[m][c] : vc[c];
        }
      }
      sl_point<T, KIND>(g, io, b0 + k, j1, j2, vc, dt, column);
    }
    return;
  }
  int go[NL];  // grid offsets of the lane's window elements
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int e = min(lane + l * kSlLanes, t.count - 1);
    const int w0 = index_quot(e, t.inv_plane), r = e - mul24(w0, t.plane);
    const int w1 = index_quot(r, t.inv_row), w2 = r - mul24(w1, t.row);
    go[l] = (sl_tile_wrap(b0, w0, g.n0) * g.n1 + sl_tile_wrap(b1, w1, g.n1)) * g.n2 + sl_tile_wrap(b2, w2, g.n2);
  }
  T rv[3][NL];
  window_load<T, 3, NL>(rv, vg, go);
  window_store<T, 3, NL>(win, rv, t.count);
  __syncthreads();
  T rf[NR][NL];
  if constexpr (NF > 0) window_load<T, NF, NL>(rf, io.f, go);
#pragma unroll
  for (int k = 0; k < T0; ++k) {
    const bool on = column && b0 + k < g.n0;
    T v[3] = {T(0), T(0), T(0)};
    if (far >> k & 1) {  // only where the lane is on
      const Tri<T> tp = tri_setup(g, b0 + k, i1, i2, sgn * dt * d[k][0] * g.invh[0], sgn * dt * d[k][1] * g.invh[1],
                                  sgn * dt * d[k][2] * g.invh[2]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        v[c] = tri_one(tp, vg[c]);
        // the fields' corners one after another (FP64 with one or two fields: all at once
        // pass 128 registers; with three they do not)
        if constexpr (NF < 3) __builtin_amdgcn_sched_barrier(0);
      }
    } else if (column) {
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] = win_eval(w[k], win + c * t.count, t);
    }
    T p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      d[k][c] = on ? sgn * T(0.5) * dt * (d[k][c] + v[c]) : T(0);
      p[c] = d[k][c] * g.invh[c];
    }
    if constexpr (NF > 0) {
      const unsigned bit = 1u << k;
      far = win_setup(w[k], p, centre + k * t.plane, t) ? far & ~bit : far | bit;
    }
  }
  if constexpr (NF > 0) {
    __syncthreads();  // the first window has been read
    window_store<T, NF, NL>(win, rf, t.count);
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < T0; ++k) {
    if (!(column && b0 + k < g.n0)) continue;
    T v[NR] = {};
    if constexpr (NF > 0) {
      if (far >> k & 1) {
        const Tri<T> tx =
            tri_setup(g, b0 + k, i1, i2, d[k][0] * g.invh[0], d[k][1] * g.invh[1], d[k][2] * g.invh[2]);
#pragma unroll
        for (int c = 0; c < NF; ++c) v[c] = tri_one(tx, io.f[c]);
      } else {
#pragma unroll
        for (int c = 0; c < NF; ++c) v[c] = win_eval(w[k], win + c * t.count, t);
      }
    }
    sl_write<T, KIND, NR>(g, io, o0 + k * s0, d[k], v, dt);
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_compose(SlGeo<T> g, const T* __restrict__ I, const T* __restrict__ u, T* __restrict__ J) {
  int i0, i1, i2;
  if (!tile_voxel(g.ft, g.n1, g.n2, i0, i1, i2)) return;
  const int o = (i0 * g.n1 + i1) * g.n2 + i2;
  const Tri<T> t = tri_setup(g, i0, i1, i2, u[o] * g.invh[0], u[g.N + o] * g.invh[1], u[2 * g.N + o] * g.invh[2]);
  J[o] = tri_one(t, I);
}

// D = div_h v (central differences)
template <typename T>
__global__ void __launch_bounds__(256) k_div(SlGeo<T> g, const T* __restrict__ v, T* __restrict__ D) {
  int i0, i1, i2;
  if (!tile_voxel(g.ft, g.n1, g.n2, i0, i1, i2)) return;
  const int s0 = g.n1 * g.n2;
  const int o = i0 * s0 + i1 * g.n2 + i2;
  const int p0 = periodic_next(i0, g.n0) * s0 + i1 * g.n2 + i2, m0 = periodic_prev(i0, g.n0) * s0 + i1 * g.n2 + i2;
  const int p1 = i0 * s0 + periodic_next(i1, g.n1) * g.n2 + i2, m1 = i0 * s0 + periodic_prev(i1, g.n1) * g.n2 + i2;
  const int p2 = i0 * s0 + i1 * g.n2 + periodic_next(i2, g.n2), m2 = i0 * s0 + i1 * g.n2 + periodic_prev(i2, g.n2);
  D[o] = T(0.5) * (g.invh[0] * (v[p0] - v[m0]) + g.invh[1] * (v[g.N + p1] - v[g.N + m1]) +
                   g.invh[2] * (v[2 * g.N + p2] - v[2 * g.N + m2]));
}

// With ssrc: s = -grad_h m . dv (the incremental state's source) into ssrc.
// Else out = bs base + w lam grad_h m (a time point's term of the gradient or Hessian;
// base may be out).
template <typename T>
__global__ void __launch_bounds__(256)
    k_pde_grad_m(SlGeo<T> g, const T* __restrict__ m, const T* __restrict__ lam, const T* __restrict__ dv, T w,
                 T bs, const T* base, T* out, T* __restrict__ ssrc) {
  int i0, i1, i2;
  if (!tile_voxel(g.ft, g.n1, g.n2, i0, i1, i2)) return;
  const int s0 = g.n1 * g.n2;
  const int o = i0 * s0 + i1 * g.n2 + i2;
  T gm[3];
  gm[0] = T(0.5) * g.invh[0] * (m[periodic_next(i0, g.n0) * s0 + i1 * g.n2 + i2] - m[periodic_prev(i0, g.n0) * s0 + i1 * g.n2 + i2]);
  gm[1] = T(0.5) * g.invh[1] * (m[i0 * s0 + periodic_next(i1, g.n1) * g.n2 + i2] - m[i0 * s0 + periodic_prev(i1, g.n1) * g.n2 + i2]);
  gm[2] = T(0.5) * g.invh[2] * (m[i0 * s0 + i1 * g.n2 + periodic_next(i2, g.n2)] - m[i0 * s0 + i1 * g.n2 + periodic_prev(i2, g.n2)]);
  if (ssrc) {
    ssrc[o] = -(gm[0] * dv[o] + gm[1] * dv[g.N + o] + gm[2] * dv[2 * g.N + o]);
    return;
  }
  const T a = w * lam[o];
#pragma unroll
  for (int c = 0; c < 3; ++c) out[c * g.N + o] = bs * base[c * g.N + o] + a * gm[c];
}

}  // namespace

namespace {

// Windows where the tiles give each compute unit one and a half workgroups or more, plain
// gathers below.  us per sl_step by gathers / by windows: FP32 32^3 (128 tiles) 4.2 / 6.0,
// 48^3 (240) 6.0 / 6.3, 64^3 (512) 7.9 / 6.9, 60 x 84 x 70 (720) 11.0 / 10.7; FP64, twice
// the bytes and registers, 48^3 7.3 / 8.7, 64^3 9.6 / 10.2, 60 x 84 x 70 17.2 / 13.5.
// Tiles of two planes.  Of four in FP32 from 16384 tiles on (216^3 has 24192): 2.3 window
// values per voxel instead of 3.1, where the fields no longer stay in the caches (256^3:
// sl_step 196 us, two planes 212; 200^3, 16000 tiles, 97 either way), though gathers then
// run in fewer waves (3 voxels a step: 350, 336); not the steps of two fields (197, 183).
template <typename T, int KIND>
void launch_sl(const char* name, const Grid& g, const SlIo<T>& io, double dt, hipStream_t st, Profiler* prof) {
  KernelTimer timer(prof, name);
  const SlGeo<T> geo = make_sl_geo<T>(g);
  SlTile t = sl_tile(g.n0, g.n1, g.n2, 2);
  if (t.blocks < (sizeof(T) == 4 ? 400u : 600u)) {
    LDDMM_LAUNCH(timer.start, timer.stop, (k_sl_points<T, KIND>), geo.ft.blocks, dim3(geo.ft.BX, geo.ft.BY), 0, st, geo, io, T(dt));
    return;
  }
  if constexpr (sizeof(T) == 4 && sl_fields(KIND) != 2)
    if (t.blocks >= 16384) {
      t = sl_tile(g.n0, g.n1, g.n2, 4);
      LDDMM_LAUNCH(timer.start, timer.stop, (k_sl<T, KIND, 4>), t.blocks, kSlLanes, size_t(3) * t.count * sizeof(T), st, geo, t, io, T(dt));
      return;
    }
  LDDMM_LAUNCH(timer.start, timer.stop, (k_sl<T, KIND, 2>), t.blocks, kSlLanes, size_t(3) * t.count * sizeof(T), st, geo, t, io, T(dt));
}

}  // namespace

template <typename T>
void launch_pde_state(const Grid& g, const T* m_old, const T* v_old, const T* v_new, T* m_new, double dt,
                      hipStream_t st, Profiler* prof) {
  launch_sl<T, SL_STATE>("pde_state", g, {v_new, v_old, {m_old, nullptr, nullptr}, nullptr, m_new}, dt, st, prof);
}

template <typename T>
void launch_pde_incr(const Grid& g, const T* dm_old, const T* s_old, const T* s_new, const T* v_old, const T* v_new,
                     T* dm_new, double dt, hipStream_t st, Profiler* prof) {
  launch_sl<T, SL_INCR>("pde_incremental_state", g, {v_new, v_old, {dm_old, s_old, nullptr}, s_new, dm_new}, dt, st,
                        prof);
}

template <typename T>
void launch_pde_adjoint(const Grid& g, const T* lam_new, const T* D_old, const T* D_new, const T* v_old,
                        const T* v_new, T* lam_old, double dt, hipStream_t st, Profiler* prof) {
  launch_sl<T, SL_ADJOINT>("pde_adjoint", g, {v_old, v_new, {lam_new, D_new, nullptr}, D_old, lam_old}, dt, st, prof);
}

template <typename T>
void launch_div(const Grid& g, const T* v, T* D, hipStream_t st, Profiler* prof) {
  KernelTimer t(prof, "divergence");
  const FieldTiling ft = make_field_tiling(g);
  LDDMM_LAUNCH(t.start, t.stop, k_div<T>, ft.blocks, dim3(ft.BX, ft.BY), 0, st, make_sl_geo<T>(g), v, D);
}

template <typename T>
void launch_pde_lambda_grad(const Grid& g, const T* m, const T* lam, double w, double bs, const T* base, T* out,
                            hipStream_t st, Profiler* prof) {
  KernelTimer t(prof, "pde_lambda_grad_m");
  const FieldTiling ft = make_field_tiling(g);
  LDDMM_LAUNCH(t.start, t.stop, k_pde_grad_m<T>, ft.blocks, dim3(ft.BX, ft.BY), 0, st, make_sl_geo<T>(g), m, lam, static_cast<const T*>(nullptr), T(w), T(bs), base, out, static_cast<T*>(nullptr));
}

template <typename T>
void launch_pde_source(const Grid& g, const T* m, const T* dv, T* s, hipStream_t st, Profiler* prof) {
  KernelTimer t(prof, "pde_source");
  const FieldTiling ft = make_field_tiling(g);
  LDDMM_LAUNCH(t.start, t.stop, k_pde_grad_m<T>, ft.blocks, dim3(ft.BX, ft.BY), 0, st, make_sl_geo<T>(g), m, static_cast<const T*>(nullptr), dv, T(0), T(0), static_cast<const T*>(nullptr), static_cast<T*>(nullptr), s);
}

template <typename T>
void launch_sl_step(const Grid& g, const T* u_old, const T* v_old, const T* v_new, T* u_new, double dt,
                    hipStream_t st, Profiler* prof) {
  if (!u_old) {
    launch_sl<T, SL_START>("sl_step", g, {v_new, v_old, {nullptr, nullptr, nullptr}, nullptr, u_new}, dt, st, prof);
    return;
  }
  launch_sl<T, SL_STEP>("sl_step", g, {v_new, v_old, {u_old, u_old + g.N, u_old + 2 * g.N}, nullptr, u_new}, dt, st,
                        prof);
}

template <typename T>
void launch_compose(const Grid& g, const T* I, const T* u, T* J, hipStream_t st, Profiler* prof) {
  KernelTimer t(prof, "compose");
  const FieldTiling ft = make_field_tiling(g);
  LDDMM_LAUNCH(t.start, t.stop, k_compose<T>, ft.blocks, dim3(ft.BX, ft.BY), 0, st, make_sl_geo<T>(g), I, u, J);
}

template void launch_sl_step<float>(const Grid&, const float*, const float*, const float*, float*, double,
                                    hipStream_t, Profiler*);
template void launch_sl_step<double>(const Grid&, const double*, const double*, const double*, double*, double,
                                     hipStream_t, Profiler*);
template void launch_compose<float>(const Grid&, const float*, const float*, float*, hipStream_t, Profiler*);
template void launch_compose<double>(const Grid&, const double*, const double*, double*, hipStream_t, Profiler*);

#define LDDMM_PDE_INST(T)                                                                                       \
  template void launch_pde_state<T>(const Grid&, const T*, const T*, const T*, T*, double, hipStream_t, Profiler*); \
  template void launch_pde_incr<T>(const Grid&, const T*, const T*, const T*, const T*, const T*, T*, double,      \
                                   hipStream_t, Profiler*);                                                     \
  template void launch_pde_adjoint<T>(const Grid&, const T*, const T*, const T*, const T*, const T*, T*, double,   \
                                      hipStream_t, Profiler*);                                                  \
  template void launch_div<T>(const Grid&, const T*, T*, hipStream_t, Profiler*);                               \
  template void launch_pde_lambda_grad<T>(const Grid&, const T*, const T*, double, double, const T*, T*,         \
                                          hipStream_t, Profiler*);                                              \
  template void launch_pde_source<T>(const Grid&, const T*, const T*, T*, hipStream_t, Profiler*);
LDDMM_PDE_INST(float)
LDDMM_PDE_INST(double)

}  // namespace lddmm
