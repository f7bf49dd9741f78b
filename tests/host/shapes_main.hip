// Host build: the launch shapes that the run-time-length passes choose for every line length
// the library takes, against the limits of the kernels they are meant for.  Prints the
// violations (at most 20) and a count.
#include <stdio.h>

#include "gp_generic_launch.hpp"
#include "gp_rfft_launch.hpp"
#include "gp_sweep_launch.hpp"

using namespace gpdbec;

static long long checked = 0, bad = 0;

static void check(bool ok, const char* what, const char* prec, int n, int n1, int n2, long long v) {
  ++checked;
  if (ok) return;
  if (++bad <= 20) printf("%s %s: line %d, others %d x %d: %lld\n", prec, what, n, n1, n2, v);
}

// what a sweep's gain tables and its block accept
static void check_sweep(const SweepCfg& c, const char* what, const char* prec, int n, int n1,
                        int n2, int most) {
  if (c.S == 0) return;
  check(c.chunks() >= 1 && c.chunks() <= kSweepMaxChunks, what, prec, n, n1, n2, c.chunks());
  check((long long)c.chunks() * c.S >= n, what, prec, n, n1, n2, (long long)c.chunks() * c.S);
  check(c.threads % 64 == 0 && c.threads <= most, what, prec, n, n1, n2, c.threads);
}

template <typename T>
static void lengths(const char* prec) {
  const int others[][2] = {{4, 1},  {21, 1},  {64, 1},   {101, 1},  {256, 1},   {500, 1}, {1000, 1},
                           {2000, 1}, {2049, 1}, {4000, 1}, {12, 10}, {63, 75}, {300, 300}};
  for (int n = 4; n <= gen_max_line<T>(); ++n) {
    if (!gen_size_ok<T>(n)) continue;
    for (const auto& o : others) {
      const int n1 = o[0], n2 = o[1];
      const RAxis a = r_axis<T>(n, (long long)n * n1 * n2);
      // prime factors to 31 have stages of their own; Bluestein's algorithm is for the others
      int rest = n;
      for (int q = 2; q <= 31; ++q)
        while (rest % q == 0) rest /= q;
      check(a.k == 0 || a.blue() == (rest > 1), "direct", prec, n, n1, n2, a.m);
      const RXCfg r = RLaunch<T>::x_r2c(a, n1, n2), c = RLaunch<T>::x_c2r(a, n1, n2);
      for (const RXCfg* x : {&r, &c}) {
        if (x->blocks == 0) continue;
        check(x->threads % 64 == 0 && x->threads <= r_max_threads<T>(), "x threads", prec, n, n1, n2,
              x->threads);
        check(x->lds <= kRLds, "x LDS", prec, n, n1, n2, (long long)x->lds);
        check(r_threads<T>(a, x->xt.np, false) <= x->threads, "x FFT", prec, n, n1, n2, x->threads);
      }
      // the x sweep leaves room for a second block on a CU wherever both lines of a pair and a
      // line's twiddles do (a few hundred bytes of carries and sums aside)
      if (c.blocks && !a.blue() && a.n <= (sizeof(T) == 8 ? 1500 : 3000))
        check(c.lds <= 81920, "x LDS of two blocks", prec, n, n1, n2, (long long)c.lds);
      if (c.blocks) {
        check_sweep(c.sweep(), "x sweep", prec, n, n1, n2, r_max_threads<T>());
        check(c.sweep().threads <= c.threads, "x sweep waves", prec, n, n1, n2, c.sweep().threads);
      }
      check_sweep(SweepLaunch<T>::cfg(n, n1, n2, n1), "strided sweep", prec, n, n1, n2, 1024);
    }
  }
}

// Strided lines past 2048 rows have no register sweep; many of them run one thread per line.
template <typename T>
static void columns(const char* prec) {
  for (int n : {2052, 2100}) {
    check(SweepLaunch<T>::cfg(2048, 182, 181, 182).S != 0, "2048 rows", prec, 2048, 182, 181, 0);
    check(SweepLaunch<T>::cfg(n, 182, 181, 182).S == 0, "past 2048 rows", prec, n, 182, 181, 0);
    check(gen_size_ok<T>(n), "accepted", prec, n, 182, 181, 0);
    check(GLaunch<T>::cn_by_columns(n, true, 182 * 181), "by columns", prec, n, 182, 181, 0);
    check(!GLaunch<T>::cn_by_columns(n, true, 18 * 22), "by tiles", prec, n, 18, 22, 0);
  }
}

int main() {
  columns<float>("fp32");
  columns<double>("fp64");
  lengths<float>("fp32");
  lengths<double>("fp64");
  printf("%s %lld checks, %lld violations\n", bad ? "bad" : "ok", checked, bad);
  return bad != 0;
}
