// FFTs of lines whose length is a kernel argument, with the data in registers between the
// stages: a thread runs whole butterflies of radix up to 16, and LDS only carries values from
// one stage to the next.
//
// A length whose prime factors are at most 13 runs Stockham stages of radices 2..16, as few
// as possible (200 = 5 x 5 x 8, 400 = 4 x 10 x 10, 240 = 15 x 16); the prime factors 17 to 31
// are stages of their own, before the others (290 = 29 x 10).  The first stage reads its
// operands from global memory and the last one leaves its results there, so an FFT of k
// stages crosses LDS k - 1 times.  A convolution (transform, product, inverse transform)
// runs the inverse with the radices in reverse order: the operands of its first stage are
// then the results of the forward transform's last one, which stay in the same registers
// through the product.  Other lengths run Bluestein's algorithm (Bluestein, "A linear
// filtering approach to the computation of discrete Fourier transform", 1970) as such a
// convolution of a length M >= 2 N - 1: with the chirp c_j = exp(-i pi j^2 / N),
// X_k = c_k sum_j (x_j c_j) conj(c_(k-j)).
#pragma once
#include "gp_device.hpp"
#include "gp_fdiv.hpp"
#include "gp_kernels.hpp"  // xcd_tile
#include "gp_sweep.hpp"    // buffer accesses

namespace gpdbec {

constexpr int kRMaxStages = 6;
constexpr int kRPrime = 31;  // largest prime factor with a stage of its own
// Largest block: FP32 kernels take at most 128 VGPRs.
template <typename T>
constexpr int r_max_threads() { return sizeof(T) == 4 ? 1024 : 512; }

// What a step reads, does to its butterflies' results, and writes.  Every transform runs
// forward: an inverse one is the conjugate of the forward transform of the conjugate, taken
// where the values are in registers anyway.
enum : int {
  // operands: LDS, or the caller's element e (of n; past the line zero for Bluestein)
  RI_LDS = 0, RI_PLAIN, RI_CONJ, RI_BLUE, RI_BLUE_CONJ,
  // results: none of these (one butterfly), or an operation and the first butterfly of the
  // transform back (the radices reversed): the caller's product, Bluestein's filter, the end
  // of one Bluestein transform with the product and the start of the next.  A radix past 16
  // ends with the product, and the transform back begins with a step of its own.
  RO_NONE = 0, RO_PRODUCT, RO_FILTER, RO_BLUE_PRODUCT,
  // destination: LDS, or the caller's element
  RD_LDS = 0, RD_PLAIN, RD_CONJ, RD_BLUE, RD_BLUE_CONJ
};
enum : int { RL_FWD = 0, RL_INV = 1, RL_CONV = 2 };

// One radix stage: butterflies of a line (nb = m / rad), product L of the earlier radices, the
// multipliers and shifts of the divisions by them (gp_fdiv.hpp), the twiddle stride m / (L rad).
// One 32-byte scalar read.
struct alignas(32) RStep {
  uint8_t rad, in, op, out;
  int32_t nb, L, ts;
  uint32_t mnb, ml;
  uint16_t snb, sl;
  uint32_t pad;
  __device__ __forceinline__ FDiv fnb() const { return FDiv{0u, mnb, snb}; }
  __device__ __forceinline__ FDiv fl() const { return FDiv{0u, ml, sl}; }
};

// The steps of a line of n points: m = n, or Bluestein's length.  One program per kind of
// pass; it lives in device memory (uniform reads: the fewer lines it takes, the fewer misses
// stand in the way of a small grid's few blocks).
constexpr int kRMaxSteps = 4 * (kRMaxStages - 1) + 1;
struct alignas(64) RProgram {
  int n, m, steps, pad;
  const void* chirp;  // Bluestein: c_j, j < n
  const void* filt;   // FFT_m of conj(c) wrapped to m, over m
  RStep st[kRMaxSteps];
  const void* tw;     // exp(-2 pi i k / m), k < m
};

// The radices (2..maxr, at most kRMaxStages) of n with the fewest stages, and among those the
// smallest largest radix (fewest registers); in increasing order.  0: none.
inline int r_radices(int n, int maxr, int* out) {
  struct Search {
    int maxr, best = 0, bestmax = 0;
    int cur[kRMaxStages], *out;
    void go(int n, int from, int depth) {
      if (n == 1) {
        if (depth == 0) return;
        const int mx = cur[depth - 1];
        if (best == 0 || depth < best || mx < bestmax) {
          best = depth;
          bestmax = mx;
          for (int i = 0; i < depth; ++i) out[i] = cur[i];
        }
        return;
      }
      if (depth >= kRMaxStages || (best && depth + 1 > best)) return;
      for (int r = from; r <= maxr; ++r) {
        if (n % r) continue;
        cur[depth] = r;
        go(n / r, r, depth + 1);
      }
    }
  } f;
  f.maxr = maxr;
  f.out = out;
  f.go(n, 2, 0);
  return f.best;
}

// Stages of an n-point line: k radices for m points (n, or Bluestein's length), by kernels
// that hold radices up to maxr.  k = 0: none, or a single radix up to 16 (such short lines
// take the other kernels).
struct RAxis {
  int n = 0, m = 0, k = 0, maxr = 0;
  int rad[kRMaxStages] = {};
  bool blue() const { return m != n; }
};

// Largest radices of the sets of kernels (besides the one with primes to 31): FP32 holds every
// radix up to 16 in 75-112 VGPRs; FP64 takes 87-128 with radices up to 10 (4 waves per SIMD)
// and 117-152 with 11 and 13 (3), so only lengths with such a factor run those.
template <typename T>
constexpr int r_max_radix(bool big) { return sizeof(T) == 4 ? 16 : big ? 13 : 10; }

// The contiguous passes (a few lines a block) of grids of few points are bound by the chain of
// instructions in one wave: radices up to 8 on more threads (r_spread) shorten it, a stage
// more or not.  A step of 60x50x40 FP64 47.1 -> 40.5 us, 720x700 57.4 -> 53.4, FP32 75^3
// 56.4 -> 51.9, 210x160 35.0 -> 31.6; of 46 grids in that range two lose 2 %.  Below it the
// stages count (90x70: 28.8, 29.5 so), above it the memory does (200^3 FP32 with radices up
// to 7: 201 -> 230).  Tiles of strided lines have the butterflies of all their columns and
// keep the fewest stages (with both: 90x80x70 FP32 51.0 -> 52.2).
constexpr int kRShortRadix = 8;
constexpr long long kRShortMin = 1 << 15, kRShortMax = 1 << 19;

// An axis of n points of a grid of `points` (0: strided lines).
template <typename T>
inline RAxis r_axis(int n, long long points) {
  RAxis a;
  a.n = n;
  if (points >= kRShortMin && points <= kRShortMax) {
    a.maxr = r_max_radix<T>(false);
    a.k = r_radices(n, kRShortRadix, a.rad);
  }
  for (int big = 0; big < 2 && a.k == 0; ++big) {
    a.maxr = r_max_radix<T>(big);
    a.k = r_radices(n, a.maxr, a.rad);
  }
  a.m = n;
  if (a.k == 0) {
    // Prime factors 17 to 31, then the rest.  (Bluestein's algorithm, two transforms and three
    // rounded products for the one, has 1.1 to 2.9 times their error: Phi of 340 points along x
    // FP64 8.6e-16 against 3.3e-16, of 380 along z 2.0e-15 against 6.8e-16.)
    int rest = n, k = 0;
    for (int q : {31, 29, 23, 19, 17})
      for (; rest % q == 0 && k < kRMaxStages; rest /= q) a.rad[k++] = q;
    int rad[kRMaxStages];
    const int kr = rest > 1 ? r_radices(rest, r_max_radix<T>(true), rad) : 0;
    if (k > 0 && k + kr <= kRMaxStages && (kr > 0 || rest == 1)) {
      for (int i = 0; i < kr; ++i) a.rad[k + i] = rad[i];
      a.k = k + kr;
      a.maxr = kRPrime;
    }
  }
  if (a.k == 0) {
    // Bluestein: among the lengths from 2n - 1 to a quarter more, the least values times
    // stages
    a.maxr = r_max_radix<T>(false);
    double cost = 0;
    for (int m = 2 * n - 1; m <= (5 * (2 * n - 1) + 3) / 4 + 8; ++m) {
      int rad[kRMaxStages];
      const int k = r_radices(m, a.maxr, rad);
      if (k < 2 || (a.k && (double)m * k >= cost)) continue;
      cost = (double)m * k;
      a.m = m;
      a.k = k;
      for (int i = 0; i < k; ++i) a.rad[i] = rad[i];
    }
  }
  if (a.k < 2 && a.maxr < kRPrime) a.k = 0;
  return a;
}

// Program of a pass of kind RL_*.
inline void r_program(const RAxis& a, int kind, RProgram* p) {
  const int k = a.k, *rad = a.rad;
  const bool blue = a.blue();
  p->n = a.n;
  p->m = a.m;
  p->steps = 0;
  p->tw = p->chirp = p->filt = nullptr;
  // transforms run one after the other, every second one with the radices reversed; the last
  // stage of one and the first of the next are one step (two of a radix past 16)
  const bool fused = rad[k - 1] <= 16;
  const int nt = (blue ? 2 : 1) * (kind == RL_CONV ? 2 : 1);
  for (int t = 0; t < nt; ++t) {
    int L = 1;
    for (int i = 0; i < k; ++i) {
      const int r = t % 2 ? rad[k - 1 - i] : rad[i];
      if (t == 0 || i > 0 || !fused) {
        RStep& s = p->st[p->steps++];
        s.rad = (uint8_t)r;
        s.nb = p->m / r;
        s.L = L;
        s.ts = p->m / (L * r);
        const FDiv fn = fdiv_make((uint32_t)s.nb), fl = fdiv_make((uint32_t)L);
        s.mnb = fn.m;
        s.snb = (uint16_t)fn.s;
        s.ml = fl.m;
        s.sl = (uint16_t)fl.s;
        s.in = RI_LDS;
        s.op = RO_NONE;
        s.out = RD_LDS;
        if (t == 0 && i == 0)
          s.in = blue ? (kind == RL_INV ? RI_BLUE_CONJ : RI_BLUE) : (kind == RL_INV ? RI_CONJ : RI_PLAIN);
        if (i == k - 1 && t + 1 < nt)
          s.op = !blue ? RO_PRODUCT : (t % 2 == 0 ? RO_FILTER : RO_BLUE_PRODUCT);
        if (i == k - 1 && t + 1 == nt)
          s.out = blue ? (kind == RL_FWD ? RD_BLUE : RD_BLUE_CONJ) : (kind == RL_FWD ? RD_PLAIN : RD_CONJ);
      }
      L *= r;
    }
  }
}

// ------------------------------------------------------------------ butterflies
// cos and sin of 2 pi k / R at compile time (Taylor series on an eighth of a turn).
template <int R>
struct Roots {
  double c[R], s[R];
  static constexpr double taylor(double x, bool sine) {
    double t = sine ? x : 1.0, acc = t;
    for (int k = sine ? 1 : 0, i = 0; i < 14; ++i, k += 2) {
      t = -t * x * x / ((k + 1) * (k + 2));
      acc += t;
    }
    return acc;
  }
  constexpr Roots() : c(), s() {
    constexpr double q = 0.78539816339744830962;  // pi/4
    for (int k = 0; k < R; ++k) {
      // 2 pi k / R = o pi/4 + x, |x| <= pi/8, with 8k = o R + rem
      int o = 8 * k / R, rem = 8 * k - o * R;
      if (2 * rem > R) {
        ++o;
        rem -= R;
      }
      const double x = q * rem / R, cx = taylor(x, false), sx = taylor(x, true);
      constexpr double h = 0.70710678118654752440;
      double a = cx, b = sx;  // rotated by o eighths
      for (int i = 0; i < o % 2; ++i) {
        const double t = h * (a - b);
        b = h * (a + b);
        a = t;
      }
      for (int i = 0; i < (o % 8) / 2; ++i) {
        const double t = -b;
        b = a;
        a = t;
      }
      c[k] = a;
      s[k] = b;
    }
  }
};

template <typename T, int R>
__device__ __forceinline__ void rdft(cpx<T>* x);

// Odd prime P from the sums and differences of the pairs (s, P - s):
// X_r, X_(P-r) = x_0 + sum_s a_s cos(2 pi r s/P) -+ i sum_s b_s sin(2 pi r s/P).
template <typename T, int P>
__device__ __forceinline__ void rdft_prime(cpx<T>* x) {
  constexpr int H = (P - 1) / 2;
  constexpr Roots<P> W{};
  cpx<T> a[H], b[H];
  cpx<T> x0 = x[0];
#pragma unroll
  for (int s = 1; s <= H; ++s) {
    a[s - 1] = x[s] + x[P - s];
    b[s - 1] = x[s] - x[P - s];
    x[0] = x[0] + a[s - 1];
  }
#pragma unroll
  for (int r = 1; r <= H; ++r) {
    cpx<T> C = x0, S = {0, 0};
#pragma unroll
    for (int s = 1; s <= H; ++s) {
      const T c = (T)W.c[(r * s) % P], n = (T)W.s[(r * s) % P];
      C = C + scl(a[s - 1], c);
      S = S + scl(b[s - 1], n);
    }
    const cpx<T> iS{-S.im, S.re};
    x[r] = C - iS;
    x[P - r] = C + iS;
  }
}

// R = R1 R2: with n = R2 n1 + n2 and k = k1 + R1 k2,
// X_k = sum_n2 W_R2^(n2 k2) W_R^(n2 k1) sum_n1 W_R1^(n1 k1) x_n.
template <typename T, int R1, int R2>
__device__ __forceinline__ void rdft_split(cpx<T>* x) {
  constexpr int R = R1 * R2;
  constexpr Roots<R> W{};
  cpx<T> y[R2][R1];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) y[n2][n1] = x[R2 * n1 + n2];
    rdft<T, R1>(y[n2]);
#pragma unroll
    for (int k1 = 1; k1 < R1; ++k1)
      if (n2 > 0)
        y[n2][k1] = y[n2][k1] * cpx<T>{(T)W.c[n2 * k1], (T)-W.s[n2 * k1]};
  }
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) {
    cpx<T> b[R2];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) b[n2] = y[n2][k1];
    rdft<T, R2>(b);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) x[k1 + R1 * k2] = b[k2];
  }
}

template <typename T, int R>
__device__ __forceinline__ void rdft(cpx<T>* x) {
  if constexpr (R == 2 || R == 3 || R == 4 || R == 5 || R == 8 || R == 16) dft<T, R, false>(x);
  else if constexpr (R == 6) rdft_split<T, 3, 2>(x);
  else if constexpr (R == 9) rdft_split<T, 3, 3>(x);
  else if constexpr (R == 10) rdft_split<T, 5, 2>(x);
  else if constexpr (R == 12) rdft_split<T, 4, 3>(x);
  else if constexpr (R == 14) rdft_split<T, 7, 2>(x);
  else if constexpr (R == 15) rdft_split<T, 5, 3>(x);
  else rdft_prime<T, R>(x);
}

// Butterflies of radix R that a thread holds at once: 10 values, 20 in the strided FP32 tiles
// (whose 16 columns would otherwise need more than a block of threads).
template <typename T, bool STRIDED>
__host__ __device__ constexpr int r_batch(int R) {
  const int q = (sizeof(T) == 4 && STRIDED ? 20 : 10) / R;
  return q < 1 ? 1 : q > 4 ? 4 : q;
}

// Threads for nl lines of an axis: every stage in one batch; a power of two, so that a
// block's waves load the four SIMDs of a CU alike.
template <typename T>
inline int r_threads(const RAxis& a, int nl, bool strided) {
  int t = 64;
  for (int s = 0; s < a.k; ++s) {
    const int q = strided ? r_batch<T, true>(a.rad[s]) : r_batch<T, false>(a.rad[s]);
    const int need = (nl * (a.m / a.rad[s]) + q - 1) / q;
    while (t < need) t *= 2;
  }
  return t;
}

// Threads of a pass of few blocks: doubled while the GPU has room (two waves per SIMD, one
// on a CU's every SIMD for each of 256 blocks) and a stage has a butterfly for each (a prime
// past 16: a few waves for each wave of butterflies), so that a wave issues fewer instructions
// one after the other.
// Waves of one butterfly's threads that pairs of results are dealt to (62x58x68 FP64 96 us a
// step with one; 76 with four, of which grids that fill the GPU keep fewer).
constexpr int kRShares = 4;
template <typename T>
inline int r_spread(const RAxis& a, int nl, int threads, long long blocks) {
  int wide = 0;
  for (int s = 0; s < a.k; ++s) {
    int w = nl * (a.m / a.rad[s]);
    if (a.rad[s] > 16) w = (w + 63) / 64 * 64 * kRShares;
    wide = w > wide ? w : wide;
  }
  // (the FP64 kernels with primes past 16 have half the waves)
  const long long room = sizeof(T) == 8 && a.maxr == kRPrime ? 128 * 1024 : 256 * 1024;
  while (threads < wide && 2 * threads <= r_max_threads<T>() && 2 * threads * blocks <= room)
    threads *= 2;
  return threads;
}

// Lines of a tile in LDS.  NLC > 0: NLC lines, the line index fastest (strided lines: a
// global run of NLC values is an LDS run); NLC = 0: lines apart, one spare value every 8 (the
// butterflies of neighbouring threads write 8 apart).
template <int NLC>
struct RTile {
  int nl;  // lines (NLC = 0)
  int ls;  // LDS values of a line (NLC = 0)
  __device__ __forceinline__ int lines() const { return NLC > 0 ? NLC : nl; }
  __device__ __forceinline__ int at(int l, int e) const {
    return NLC > 0 ? e * NLC + l : l * ls + e + (e >> 3);
  }
  // butterfly u of a stage with nb butterflies a line -> (line, butterfly)
  __device__ __forceinline__ void locate(int u, FDiv fnb, int nb, int* l, int* t) const {
    if constexpr (NLC > 0) {
      *l = u % NLC;
      *t = u / NLC;
    } else {
      *l = (int)fdiv((uint32_t)u, fnb);
      *t = u - *l * nb;
    }
  }
};
__host__ __device__ constexpr int r_line_slots(int n) { return n + (n >> 3) + 1; }

// One step with radix R: butterfly t of line l takes the elements t + k nb, twiddled by
// W_(L R)^(k j), j = t mod L, and leaves the elements (t - j) R + j + k L.  load(l, e),
// product(l, e, v) and store(l, e, v) are the caller's, as is first(), which the first step
// calls once its loads are under way.
// ALIAS: load and store work on buf itself (the last step leaves its results where its
// operands were, so only the first one needs a barrier more).
template <typename T, int R, bool ALIAS, int NLC, typename Load, typename Product,
          typename Store, typename First>
__device__ __forceinline__ void r_step(const RTile<NLC>& tile, const RProgram* __restrict__ p,
                                       const RStep& st, const cpx<T>* tw, cpx<T>* buf, Load load,
                                       Product product, Store store, First first) {
  constexpr int Q = r_batch<T, (NLC > 0)>(R);
  const cpx<T>* __restrict__ ch = reinterpret_cast<const cpx<T>*>(p->chirp);
  const int n = p->n, nb = st.nb, L = st.L, tot = tile.lines() * nb;
  const int tid = threadIdx.x, nt = blockDim.x;
  cpx<T> v[Q][R];
  int ll[Q], tt[Q], jj[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int u = tid + q * nt;
    if (u < tot) {
      int l, t;
      tile.locate(u, st.fnb(), nb, &l, &t);
      ll[q] = l;
      tt[q] = t;
      const int j = t - (int)fdiv((uint32_t)t, st.fl()) * L;
      jj[q] = j;
      if (st.in == RI_LDS) {
#pragma unroll
        for (int k = 0; k < R; ++k) v[q][k] = buf[tile.at(l, t + k * nb)];
#pragma unroll
        for (int k = 1; k < R; ++k) v[q][k] = v[q][k] * tw[k * j * st.ts];
      } else if (st.in <= RI_CONJ) {
#pragma unroll
        for (int k = 0; k < R; ++k) v[q][k] = load(l, t + k * nb);
        if (st.in == RI_CONJ) {
#pragma unroll
          for (int k = 0; k < R; ++k) v[q][k].im = -v[q][k].im;
        }
      } else {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int e = t + k * nb, ec = min(e, n - 1);
          cpx<T> x = load(l, ec);
          if (st.in == RI_BLUE_CONJ) x.im = -x.im;
          x = x * ch[ec];
          v[q][k] = cpx<T>{e < n ? x.re : (T)0, e < n ? x.im : (T)0};
        }
      }
      rdft<T, R>(v[q]);
      if (st.op != RO_NONE) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int e = t + k * nb;
          cpx<T> x = v[q][k];
          if (st.op == RO_PRODUCT) {
            x = product(l, e, x);
          } else if (st.op == RO_FILTER) {
            x = x * reinterpret_cast<const cpx<T>*>(p->filt)[e];
          } else {
            const int ec = min(e, n - 1);
            const cpx<T> c = ch[ec];
            x.im = -x.im;
            x = product(l, ec, x * c);
            // conj(x) c, conjugated once more below with the others
            x = x * conjg(c);
            x = cpx<T>{e < n ? x.re : (T)0, e < n ? x.im : (T)0};
          }
          v[q][k] = conjg(x);
        }
        rdft<T, R>(v[q]);
      }
    }
  }
  if (st.in != RI_LDS) first();
  if (st.out == RD_LDS) {
    if (ALIAS || st.in == RI_LDS) __syncthreads();  // every operand is read
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (tid + q * nt < tot) {
        const int o = st.op != RO_NONE ? tt[q] * R : (tt[q] - jj[q]) * R + jj[q];
        const int d = st.op != RO_NONE ? 1 : L;
#pragma unroll
        for (int k = 0; k < R; ++k) buf[tile.at(ll[q], o + k * d)] = v[q][k];
      }
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (tid + q * nt < tot) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int e = tt[q] + k * nb;  // the last stage: L = nb, j = t
          cpx<T> x = v[q][k];
          if (st.out <= RD_CONJ) {
            if (st.out == RD_CONJ) x.im = -x.im;
            store(ll[q], e, x);
          } else if (e < n) {
            x = conjg(x) * ch[e];
            if (st.out == RD_BLUE_CONJ) x.im = -x.im;
            store(ll[q], e, x);
          }
        }
      }
    }
  }
}

// cos and sin of 2 pi s / P, 0 < s < P / 2, rounded once.
template <typename T, int P>
struct HalfRoots {
  T c[(P - 1) / 2], s[(P - 1) / 2];
  constexpr HalfRoots() : c(), s() {
    constexpr Roots<P> W{};
    for (int k = 0; k < (P - 1) / 2; ++k) {
      c[k] = (T)W.c[k + 1];
      s[k] = (T)W.s[k + 1];
    }
  }
};
template <typename T, int P>
static __constant__ HalfRoots<T, P> r_half_roots = HalfRoots<T, P>{};

// The same with a prime radix past 16.  A thread holds the sums and differences of
// rdft_prime of one butterfly, and each pair of results goes where it belongs as soon as it is
// summed (31 FP64 values and their results together would not fit the registers).  Threads
// past the butterflies take whole waves' shares of the pairs.  The roots come from constant
// memory by scalar loads, once a step (as literals they spilled 358 SGPRs in FP64, and loaded
// pair by pair in a loop they stand in the way of the multiply-adds: 290^3 FP64 1838 us a step,
// 1642 so), rounded once: the twiddle table's, whose arguments are rounded too, leave the
// residue of a constant line behind (Phi of 38 points along z FP64 7.9e-16 against 5.4e-16).
// RO_PRODUCT: the product goes to LDS, conjugated, where the transform back begins.
//
// A butterfly of 31 values is 900 multiply-adds in one thread: what bounds it on large grids,
// and on small ones the few lanes that have one.  A step of 290^3 takes 677 us FP32 and 1642 FP64
// (with Bluestein's algorithm 1544 and 2491), 340x310 37 and 42 (53 and 56), 62x58x68 54 and
// 76 (73 and 68).
template <typename T, int P, bool ALIAS, int NLC, typename Load, typename Product,
          typename Store, typename First>
__device__ __forceinline__ void r_step_prime(const RTile<NLC>& tile, const RStep& st,
                                             const cpx<T>* tw, cpx<T>* buf, Load load,
                                             Product product, Store store, First first) {
  constexpr int H = (P - 1) / 2;
  const int nb = st.nb, L = st.L, tot = tile.lines() * nb;
  // the roots' address is opaque to the compiler, which would make them literals again
  typedef const __attribute__((address_space(4))) T* Roots4;
  uintptr_t wa = (uintptr_t)&r_half_roots<T, P>;
  asm("" : "+s"(wa));
  T wc[H], ws[H];
#pragma unroll
  for (int s = 0; s < H; ++s) {
    wc[s] = ((Roots4)wa)[s];
    ws[s] = ((Roots4)wa)[H + s];
  }
  // shares of the pairs: whole waves (a line read and left in global memory has one)
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int tw_ = (tot + 63) >> 6, nw = (int)blockDim.x >> 6;
  const int shares = st.in != RI_LDS && st.out != RD_LDS ? 1 : nw / tw_;
  const int share = wave / tw_;
  const int u = (int)threadIdx.x - share * tw_ * 64;
  const bool on = share < shares && u < tot;
  int l = 0, t = 0, j = 0;
  cpx<T> x0{0, 0}, a[H], b[H];
  if (on) {
    tile.locate(u, st.fnb(), nb, &l, &t);
    j = t - (int)fdiv((uint32_t)t, st.fl()) * L;
    if (st.in == RI_LDS) {
      x0 = buf[tile.at(l, t)];
#pragma unroll
      for (int s = 1; s <= H; ++s) {
        a[s - 1] = buf[tile.at(l, t + s * nb)];
        b[s - 1] = buf[tile.at(l, t + (P - s) * nb)];
      }
#pragma unroll
      for (int s = 1; s <= H; ++s) {
        a[s - 1] = a[s - 1] * tw[s * j * st.ts];
        b[s - 1] = b[s - 1] * tw[(P - s) * j * st.ts];
      }
    } else {
      x0 = load(l, t);
#pragma unroll
      for (int s = 1; s <= H; ++s) {
        a[s - 1] = load(l, t + s * nb);
        b[s - 1] = load(l, t + (P - s) * nb);
      }
      if (st.in == RI_CONJ) {
        x0 = conjg(x0);
#pragma unroll
        for (int s = 0; s < H; ++s) {
          a[s] = conjg(a[s]);
          b[s] = conjg(b[s]);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < H; ++s) {
      const cpx<T> d = a[s] - b[s];
      a[s] = a[s] + b[s];
      b[s] = d;
    }
  }
  if (st.in != RI_LDS) first();
  // every operand is read, and what first() keeps for the product of a line of one stage is there
  if (ALIAS || (st.out == RD_LDS && (st.in == RI_LDS || st.op != RO_NONE))) __syncthreads();
  if (on) {
    const bool turn = st.op != RO_NONE;
    const int o = turn ? t : (t - j) * P + j, d = turn ? nb : L;
    auto put = [&](int k, cpx<T> v) {
      if (st.out == RD_LDS) {
        if (turn) v = conjg(product(l, t + k * nb, v));
        buf[tile.at(l, o + k * d)] = v;
      } else {
        if (st.out == RD_CONJ) v.im = -v.im;
        store(l, t + k * nb, v);  // the last stage: L = nb, j = t
      }
    };
    if (share == 0) {
      cpx<T> sum = x0;
#pragma unroll
      for (int s = 0; s < H; ++s) sum = sum + a[s];
      put(0, sum);
    }
    int next = share;  // the pairs share, share + shares, ...
#pragma unroll
    for (int r = 1; r <= H; ++r) {
      if (next-- == 0) {
        next = shares - 1;
        cpx<T> C = x0, S = {0, 0};
#pragma unroll
        for (int s = 1; s <= H; ++s) {
          const int k = (r * s) % P;
          const T c = wc[(k <= H ? k : P - k) - 1], n = ws[(k <= H ? k : P - k) - 1];
          C = C + scl(a[s - 1], c);
          S = k <= H ? S + scl(b[s - 1], n) : S - scl(b[s - 1], n);
        }
        const cpx<T> iS{-S.im, S.re};
        put(r, C - iS);
        put(P - r, C + iS);
      }
    }
  }
  if (st.out == RD_LDS) __syncthreads();
}

// The program of a tile's lines.  tw: its twiddles in LDS (the first step reads none, so
// first() may write them); buf: LDS of the tile, free.
template <typename T, int MAXR, bool ALIAS, int NLC, typename Load, typename Product,
          typename Store, typename First>
__device__ __forceinline__ void r_run(const RTile<NLC>& tile, const RProgram* __restrict__ p,
                                      const cpx<T>* tw, cpx<T>* buf, Load load, Product product,
                                      Store store, First first) {
  const int steps = p->steps;
  RStep next = p->st[0];
  for (int s = 0; s < steps; ++s) {
    const RStep st = next;
    next = p->st[min(s + 1, steps - 1)];  // read a step ahead
    switch (st.rad) {
#define GP_R(R)                                                      \
  case R:                                                            \
    if constexpr (R <= MAXR && R <= r_max_radix<T>(true))            \
      r_step<T, R, ALIAS>(tile, p, st, tw, buf, load, product, store, first); \
    break;
      GP_R(2) GP_R(3) GP_R(4) GP_R(5) GP_R(6) GP_R(7) GP_R(8) GP_R(9) GP_R(10) GP_R(11) GP_R(12)
      GP_R(13) GP_R(14) GP_R(15) GP_R(16)
#undef GP_R
#define GP_R(R)                                                      \
  case R:                                                            \
    if constexpr (R <= MAXR) r_step_prime<T, R, ALIAS>(tile, st, tw, buf, load, product, store, first); \
    break;
      GP_R(17) GP_R(19) GP_R(23) GP_R(29) GP_R(31)
#undef GP_R
      default:
        break;
    }
  }
}

// ------------------------------------------------------------------- line passes
// Lines of the half spectrum.  NLC > 0: lines at stride `es` (elements), NLC adjacent columns
// of one plane to a tile (`cols` columns to a plane, plane stride `ps`); NLC = 0: contiguous
// lines, nl to a tile, at LDS stride ls.
struct RLines {
  int nlines, nl, ls;
  int cols;
  unsigned es;
  long long ps;
};

// A copy from global memory to LDS whose loads are issued at once (NU values per thread) and
// whose stores come later.
template <typename X, int NU>
struct Prefetch {
  X v[NU];
  template <typename F>
  __device__ __forceinline__ void load(int n, F f) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = threadIdx.x + u * blockDim.x;
      v[u] = f(t < n ? t : 0);
    }
  }
  template <typename F>
  __device__ __forceinline__ void store(int n, X* dst, F f) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = threadIdx.x + u * blockDim.x;
      if (t < n) dst[t] = v[u];
    }
    for (int t = threadIdx.x + NU * blockDim.x; t < n; t += blockDim.x) dst[t] = f(t);
  }
};

// Kernel value of element e of line l of a convolution: 3D (strided) the quadrant
// ktab[(kx (n2/2+1) + min(e, n2-e)) (n1/2+1) + min(k1, n1-k1)] of line l = kx n1 + k1, 2D
// ktab[l n + e]; a tile's values wait in LDS for the product.  The product is
// U(k) scale^2 / N (the table holds U/N).
template <typename T, int NLC, int MAXR>
__global__ void __launch_bounds__(r_max_threads<T>()) k_rlines(cpx<T>* __restrict__ data, RLines g,
                                                      const RProgram* __restrict__ p,
                                                      const T* __restrict__ ktab,
                                                      const double* __restrict__ scale,
                                                      FoldedFin fin) {
  constexpr unsigned CB = sizeof(cpx<T>);
  extern __shared__ __align__(16) char rfft_raw[];
  if constexpr (NLC == 0) {  // the forward y lines may carry a finalisation's second stage
    if (folded_fin(fin, rfft_raw)) return;
  }
  const int n = p->n, m = p->m;
  const RTile<NLC> tile{g.nl, g.ls};
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(rfft_raw);
  cpx<T>* buf = tw + m;
  T* kt = reinterpret_cast<T*>(buf + (NLC > 0 ? m * NLC : g.nl * g.ls));
  // tiles numbered XCD-contiguously: neighbours share 128-byte lines and an L2
  const int lead = NLC == 0 ? fin.lead : 0;
  const int b = xcd_tile(blockIdx.x - lead, gridDim.x - lead);
  int plane = 0, l0;
  cpx<T>* base;
  unsigned bytes, step;
  if constexpr (NLC > 0) {
    const int tiles = (g.cols + NLC - 1) / NLC;
    plane = b / tiles;
    l0 = (b - plane * tiles) * NLC;
    base = data + (plane * g.ps + l0);
    step = g.es * CB;
    bytes = (unsigned)(n - 1) * step + (unsigned)min(NLC, g.cols - l0) * CB;
  } else {
    l0 = b * g.nl;
    base = data + (long long)l0 * n;
    step = CB;
    bytes = (unsigned)min(g.nl, g.nlines - l0) * (unsigned)n * CB;
  }
  const __amdgpu_buffer_rsrc_t rb = buf_of(base, bytes);
  // lines past the grid: out of the buffer's range (strided lines start past it)
  auto off = [&](int l, int e) -> unsigned {
    if constexpr (NLC > 0)
      return (l0 + l < g.cols ? (unsigned)l * CB : bytes) + (unsigned)e * step;
    else
      return ((unsigned)l * (unsigned)n + (unsigned)e) * CB;
  };
  // the tables are fetched ahead of the first step's operands and kept after it
  const cpx<T>* __restrict__ twg = reinterpret_cast<const cpx<T>*>(p->tw);
  auto tw_of = [&](int t) { return twg[t]; };
  const int nk = ktab == nullptr ? 0 : NLC > 0 ? (n / 2 + 1) * NLC : min(g.nl, g.nlines - l0) * n;
  auto kt_of = [&](int t) {
    if constexpr (NLC > 0) {
      const int k1 = min(l0 + t % NLC, g.cols - 1), h1 = g.cols / 2 + 1;
      return at32(ktab + (size_t)plane * (n / 2 + 1) * h1,
                  (unsigned)(t / NLC * h1 + min(k1, g.cols - k1)));
    } else {
      return at32(ktab + (size_t)l0 * n, (unsigned)t);
    }
  };
  Prefetch<cpx<T>, 1> ptw;
  Prefetch<T, 4> pkt;
  ptw.load(m, tw_of);
  T s2 = 1;
  if (nk > 0) {
    pkt.load(nk, kt_of);
    const double sc = *scale;
    s2 = (T)(sc * sc);
  }
  r_run<T, MAXR, false>(
      tile, p, tw, buf,
      [&](int l, int e) {
        cpx<T> v;
        buf_load(rb, off(l, e), v);
        return v;
      },
      [&](int l, int e, cpx<T> v) {
        T k;
        if constexpr (NLC > 0) k = kt[min(e, n - e) * NLC + l];
        else k = kt[min(l, g.nlines - 1 - l0) * n + e];
        return scl(v, k * s2);
      },
      [&](int l, int e, cpx<T> v) { buf_store(rb, off(l, e), v); },
      [&] {
        ptw.store(m, tw, tw_of);
        if (nk > 0) pkt.store(nk, kt, kt_of);
      });
}

// Keeps a program in device memory.
__global__ inline void k_rprogram(RProgram p, RProgram* __restrict__ dst) {
  static_assert(sizeof(RProgram) % 4 == 0, "copied by words");
  const int* s = reinterpret_cast<const int*>(&p);
  int* d = reinterpret_cast<int*>(dst);
  for (int i = threadIdx.x; i < (int)(sizeof(RProgram) / 4); i += blockDim.x) d[i] = s[i];
}

}  // namespace gpdbec
