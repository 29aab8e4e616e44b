// The run-time transform kernels of fft_rt.hip on the host: every lane of a
// workgroup is a host thread and the LDS an array of exactly the launch's size
// (its end poisoned), so a read or write out of range, a missing barrier's stale
// value or a wrong index shows against a plain transform.
#include <pthread.h>
#include <sanitizer/asan_interface.h>

#include <functional>
#include <thread>
#include <vector>

#include "fft_rt.hip"

using namespace lddmm;

namespace lddmm {
namespace {
alignas(16) unsigned char smem[1 << 18];
}
}  // namespace lddmm

static pthread_barrier_t g_barrier;
void __syncthreads() { pthread_barrier_wait(&g_barrier); }

namespace {

void launch(unsigned gx, unsigned gy, int threads, size_t lds, const std::function<void()>& kernel) {
  gridDim = {gx, gy, 1};
  blockDim = {unsigned(threads), 1, 1};
  for (unsigned y = 0; y < gy; ++y)
    for (unsigned x = 0; x < gx; ++x) {
      for (size_t i = 0; i < lds; ++i) smem[i] = 0xff;  // NaN until written
      __asan_poison_memory_region(smem + lds, sizeof(smem) - lds);
      pthread_barrier_init(&g_barrier, nullptr, threads);
      std::vector<std::thread> th;
      for (int t = 0; t < threads; ++t)
        th.emplace_back([&, t] {
          threadIdx = {unsigned(t), 0, 0};
          blockIdx = {x, y, 0};
          kernel();
        });
      for (auto& t : th) t.join();
      pthread_barrier_destroy(&g_barrier);
      __asan_unpoison_memory_region(smem, sizeof(smem));
    }
}

template <typename T>
std::vector<cplx<T>> roots(int n, int count) {
  std::vector<cplx<T>> t(count);
  for (int m = 0; m < count; ++m) t[m] = {T(std::cos(2 * M_PI * m / n)), T(-std::sin(2 * M_PI * m / n))};
  return t;
}

int fold(int k, int n) { return k <= n - k ? k * k : (n - k) * (n - k); }

// out = [add + add_scale *] K or L of `in` (ncomp components) with the three
// passes, xs units per plane, tb groups per pencil workgroup.
template <typename T>
int apply(const int n[3], int ncomp, int xs, int tb, int threads, int xcd_run, double alpha, int s, int op, int wide,
          const T* in, const T* add, double add_scale, T* out) {
  const int n0 = n[0], n1 = n[1], H = n[2] / 2, M = H + 1, u1 = n1 / xs, P = n1 * M;
  FftPlan p0, p1, p2;
  RtPlaneArgs<T> a{};
  RtPencilArgs<T> k{};
  // wide 0: the compile-time kernels' plans, 1: radices 2 to 10, 2: up to 16
  auto plan = [&](int m, FftPlan& p) { return wide ? make_wide_plan(m, wide > 1, p) : make_plan(m, p); };
  if (n1 % xs || !plan(n0, p0) || !plan(u1, p1) || !plan(H, p2)) return 1;
  if (!make_rt_plan(p0, k.r0) || !make_rt_plan(p1, a.r1) || !make_rt_plan(p2, a.r2)) return 2;
  const auto tw0 = roots<T>(n0, n0), tw1 = roots<T>(u1, u1), tw2 = roots<T>(H, H), twr = roots<T>(n[2], H / 2 + 1);
  std::vector<int> slot2(H + 1, H);
  std::vector<cplx<T>> twx(u1);
  std::vector<T> k0(n0), k1(n1), k2(M, T(H) * H);
  for (int p = 0; p < H; ++p) slot2[digit_reverse(p2, p)] = p;
  for (int p = 0; p < H; ++p) k2[p] = T(digit_reverse(p2, p)) * digit_reverse(p2, p);
  for (int p = 0; p < n0; ++p) k0[p] = T(fold(digit_reverse(p0, p), n0));
  for (int p = 0; p < u1; ++p) {
    const int f = digit_reverse(p1, p);
    twx[p] = roots<T>(n1, n1)[f];
    for (int h = 0; h < xs; ++h) k1[h * u1 + p] = T(fold(f + h * u1, n1));
  }
  a.threads = k.threads = threads;
  a.n0 = n0, a.n1u = u1, a.H = H, a.M = M, a.LM = M | 1, a.xs = xs;
  a.N = (long long)n0 * n1 * n[2];
  a.inv_n1u = 1.0f / u1, a.inv_H = 1.0f / H;
  a.tw1 = tw1.data(), a.tw2 = tw2.data(), a.twr = twr.data(), a.slot2 = slot2.data();
  a.add = add, a.add_scale = T(add_scale), a.xcd_run = xcd_run;
  const int groups = tb;
  k.es = P, k.nin = P / xs, k.outer_stride = (long long)n0 * P, k.tb = groups;
  k.inv_tb = 1.0f / groups, k.inv_ts = 1.0f / (groups * xs), k.inv_M = 1.0f / M;
  k.hs = xs > 1 ? P / xs : 0, k.n1u = u1, k.M = M;
  k.tw = tw0.data(), k.twx = twx.data(), k.alpha = T(alpha), k.s = s, k.op = op;
  k.scale = T(1.0 / (double(n0) * n1 * n[2]));
  k.ksq0 = k0.data(), k.ksq1 = k1.data(), k.ksq2 = k2.data(), k.xcd_run = xcd_run;
  std::vector<cplx<T>> spec(size_t(ncomp) * n0 * P);
  const size_t c = sizeof(cplx<T>);
  const size_t plane_lds = size_t(u1) * a.LM * c + (u1 + H + H / 2 + 1) * c + (H + 1) * sizeof(int);
  const size_t pencil_lds = (size_t(n0) * groups * xs + n0) * c + size_t(n0 + groups * xs) * sizeof(T);
  if (plane_lds > sizeof(smem) || pencil_lds > sizeof(smem)) return 3;
  const auto fwd = rt_plane_fwd<T>(has_big_radix(p1) || has_big_radix(p2));
  const auto inv = rt_plane_inv<T>(has_big_radix(p1) || has_big_radix(p2));
  const auto pen = rt_pencil<T>(xs, has_big_radix(p0));
  launch(n0 * xs, ncomp, threads, plane_lds, [&] { fwd(in, spec.data(), a); });
  launch((k.nin + groups - 1) / groups, ncomp, threads, pencil_lds, [&] { pen(spec.data(), k); });
  launch(n0 * xs, ncomp, threads, plane_lds, [&] { inv(spec.data(), out, a); });
  return 0;
}

}  // namespace

#include <cstdio>
#include <cstdlib>

// argv: n0 n1 n2 ncomp xs tb threads xcd_run s op f64 add wide; doubles in (and the
// addend) from stdin, doubles out on stdout.
template <typename T>
int run(char** v, const int n[3]) {
  const size_t N = size_t(n[0]) * n[1] * n[2] * std::atoi(v[4]);
  const bool with_add = std::atoi(v[12]) != 0;
  std::vector<double> raw(N * (with_add ? 2 : 1));
  if (std::fread(raw.data(), sizeof(double), raw.size(), stdin) != raw.size()) return 10;
  std::vector<T> in(raw.begin(), raw.begin() + N), add(raw.begin() + (raw.size() - N), raw.end()), out(N);
  const int rc = apply<T>(n, std::atoi(v[4]), std::atoi(v[5]), std::atoi(v[6]), std::atoi(v[7]), std::atoi(v[8]),
                          0.0025, std::atoi(v[9]), std::atoi(v[10]), std::atoi(v[13]), in.data(), with_add ? add.data() : nullptr, 0.3,
                          out.data());
  if (rc) return rc;
  const std::vector<double> o(out.begin(), out.end());
  std::fwrite(o.data(), sizeof(double), N, stdout);
  return 0;
}

int main(int argc, char** v) {
  if (argc != 14) return 11;
  const int n[3] = {std::atoi(v[1]), std::atoi(v[2]), std::atoi(v[3])};
  return std::atoi(v[11]) ? run<double>(v, n) : run<float>(v, n);
}
