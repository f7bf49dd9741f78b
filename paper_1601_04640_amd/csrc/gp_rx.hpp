// Passes along x for run-time-length lines: |psi|^2 with the real-to-complex FFT, and the
// complex-to-real FFT with the nonlinear sub-step and the Crank-Nicolson sweep.
//
// A block takes np pairs of neighbouring x lines of one plane; a pair is one complex line
// (line j real, line j + 1 imaginary) of the FFTs of gp_rfft.hpp, in LDS.  The
// complex-to-real pass keeps going where its transform ends: the thread that reads Phi of
// both lines at a point puts psi after the phase into the same LDS slot (and a second one),
// and the sweep runs from there with the chunks and scans of gp_sweep.hpp, a line's chunks TL
// lanes apart.  So a step reads the spectrum, psi and V once and writes psi once, and Phi is
// never stored.
#pragma once
#include "gp_rfft.hpp"

namespace gpdbec {

// Tile of the x passes: np line pairs per block (a power of two), nbj blocks to a plane.
// fn0, fnp: divisors by n0 and np; ls: LDS values of a line; P: chunks (of S rows) of a line
// in the whole waves that sweep.
struct RXTile {
  int n0, n1, n2, np, nbj, ls, P, S;
  FDiv fn0, fnp;
};


// Sums of NV values over a block of whole waves (at most 16), in a fixed order: each wave's to
// red (NV x 16 doubles), and, a barrier later, total v stored by thread v.
template <int NV>
__device__ __forceinline__ void rx_block_reduce(double (&v)[NV], double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_sum_to_last(v[k]);
  if (lane == 63) {
#pragma unroll
    for (int k = 0; k < NV; ++k) red[k * 16 + wave] = v[k];
  }
}
template <int NV>
__device__ __forceinline__ void rx_block_total(const double* red, double* __restrict__ out) {
  const int nw = blockDim.x >> 6;
  if ((int)threadIdx.x < NV) {
    double acc = red[threadIdx.x * 16];
    for (int w = 1; w < nw; ++w) acc += red[threadIdx.x * 16 + w];
    out[threadIdx.x] = acc;
  }
}

// |psi|^2 of the pairs, FFT, untangled to the half spectrum: A_k = (Z_k + conj Z_(N-k))/2,
// B_k = (Z_k - conj Z_(N-k))/(2i).  part[2b], part[2b+1]: sums of |psi_(i+1) - psi_i|^2 of
// the stored state along x and along axis 1 (from the block's lines to their successors).
// The x neighbour comes from the next lane (the last lane of a wave loads its own).
// fin: the finalisation of the step before (or its first stage), which nothing in this pass
// waits for, in leading blocks (540x600 FP64: 51.7 us a step with a kernel of its own, 48.2
// so; this pass 10.4 and 10.9).
template <typename T, int MAXR>
__global__ void __launch_bounds__(r_max_threads<T>()) k_rr2c(const cpx<T>* __restrict__ psi,
                                                    cpx<T>* __restrict__ spec, RXTile xt,
                                                    const RProgram* __restrict__ p,
                                                    double* __restrict__ part, FoldedFin fin) {
  constexpr unsigned CB = sizeof(cpx<T>);
  constexpr int U = sizeof(T) == 4 ? 4 : 2;  // points of a pair per thread and round
  extern __shared__ __align__(16) char rx_raw[];
  if (folded_fin(fin, rx_raw)) return;
  const int bid = blockIdx.x - fin.lead;
  const int N = xt.n0, n1 = xt.n1, m = p->m, nt = blockDim.x;
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(rx_raw);
  cpx<T>* buf = tw + m;
  const int b = xcd_tile(bid, gridDim.x - fin.lead);
  const int k = b / xt.nbj, j0 = (b - k * xt.nbj) * 2 * xt.np;
  const int lines = min(2 * xt.np, n1 - j0), npairs = (lines + 1) / 2;
  const RTile<0> tile{npairs, xt.ls};
  // the tile's lines and one more; past the plane's last line the buffer ends
  const __amdgpu_buffer_rsrc_t rb =
      buf_of(const_cast<cpx<T>*>(psi) + ((long long)k * n1 + j0) * N,
             (unsigned)min(2 * xt.np + 1, n1 - j0) * (unsigned)N * CB);
  const cpx<T>* __restrict__ twg = reinterpret_cast<const cpx<T>*>(p->tw);
  auto tw_of = [&](int t) { return twg[t]; };
  Prefetch<cpx<T>, 1> ptw;
  ptw.load(m, tw_of);
  const int tot = npairs * N;
  const unsigned line = (unsigned)N * CB;
  const bool last_lane = (threadIdx.x & 63) == 63;
  double s[2] = {0.0, 0.0};
  for (int t0 = 0; t0 < tot; t0 += U * nt) {
    cpx<T> a0[U], a1[U], c1[U], b0[U], b1[U];
    int qq[U], ii[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * nt + (int)threadIdx.x;
      qq[u] = (int)fdiv((uint32_t)t, xt.fn0);
      ii[u] = t - qq[u] * N;
      const unsigned o = ((unsigned)(2 * qq[u]) * (unsigned)N + (unsigned)ii[u]) * CB;
      buf_load(rb, o, a0[u]);
      buf_load(rb, o + line, a1[u]);
      buf_load(rb, o + 2 * line, c1[u]);
      if (last_lane) {
        buf_load(rb, o + CB, b0[u]);
        buf_load(rb, o + line + CB, b1[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const cpx<T> n0 = dpp<DPP_WAVE_SHL1>(a0[u]), n1v = dpp<DPP_WAVE_SHL1>(a1[u]);
      const cpx<T> x0 = csel(last_lane, b0[u], n0), x1 = csel(last_lane, b1[u], n1v);
      const int j = 2 * qq[u];
      if (qq[u] < npairs) {
        // rows past the plane read as zero: their differences do not count
        const bool in = ii[u] + 1 < N, has1 = j + 1 < lines;
        if (in) s[0] += absdiff2_d(x0, a0[u]) + absdiff2_d(x1, a1[u]);
        if (has1) s[1] += absdiff2_d(a1[u], a0[u]);
        if (has1 && j0 + j + 2 < n1) s[1] += absdiff2_d(c1[u], a1[u]);
        buf[tile.at(qq[u], ii[u])] = cpx<T>{a0[u].re * a0[u].re + a0[u].im * a0[u].im,
                                            a1[u].re * a1[u].re + a1[u].im * a1[u].im};
      }
    }
  }
  __syncthreads();
  r_run<T, MAXR, true>(
      tile, p, tw, buf, [&](int l, int e) { return buf[tile.at(l, e)]; },
      [&](int, int, cpx<T> v) { return v; },
      [&](int l, int e, cpx<T> v) { buf[tile.at(l, e)] = v; }, [&] { ptw.store(m, tw, tw_of); });
  __syncthreads();
  const int tot2 = (N / 2 + 1) * xt.np;  // the full tile's indexing; pairs past npairs skipped
  const bool even = (n1 & 1) == 0;       // a pair of spectrum values is one aligned store
  for (int t = threadIdx.x; t < tot2; t += nt) {
    const int kx = (int)fdiv((uint32_t)t, xt.fnp), q = t - kx * xt.np;
    if (q >= npairs) continue;
    const cpx<T> zk = buf[tile.at(q, kx)], zm = buf[tile.at(q, kx == 0 ? 0 : N - kx)];
    const T h = (T)0.5;
    const cpx<T> A{h * (zk.re + zm.re), h * (zk.im - zm.im)};
    const cpx<T> B{h * (zk.im + zm.im), h * (zm.re - zk.re)};
    cpx<T>* o = spec + (((long long)kx * xt.n2 + k) * n1 + j0 + 2 * q);
    if (even) {
      *reinterpret_cast<cpx2<T>*>(o) = cpx2<T>{A, B};
    } else {
      o[0] = A;
      if (2 * q + 1 < lines) o[1] = B;
    }
  }
  __syncthreads();  // the line buffer is free: it holds the reduction
  rx_block_reduce<2>(s, reinterpret_cast<double*>(buf));
  __syncthreads();
  rx_block_total<2>(reinterpret_cast<double*>(buf), part + 2 * (long long)bid);
}

// What the complex-to-real pass works on: psi, V, the scale of psi, the x factors and their
// gains, the step's scalars, the partial sums and (no step) where Phi goes.
template <typename T>
struct RXArgs {
  cpx<T>* psi;
  const T* V;
  const double* scale;
  const cpx<T>* f;
  const cpx<T>* gains;
  double dt, gc, gdd, h0, h1, h2;
  double* part;
  T* phi;
};

// Half spectrum of the pairs (Z_k = A_k + i B_k, Z_(N-k) = conj A_k + i conj B_k), inverse
// FFT: Phi of line j in the real parts, of line j + 1 in the imaginary ones.
// MODE_IMAG / MODE_REAL: psi <- sweep of scale psi exp(-eps dt (V + g_c n + g_dd Phi)), and
// part[7b..] = sums n, V n, n^2, Phi n, x^2 n, y^2 n, z^2 n of scale psi.  MODE_OBSERVE: the
// sums where part is given, Phi where phi is.  S: rows per chunk of the sweep.
//
// LDS bounds the blocks on a CU and the pairs in a block, so it holds what is live: both lines
// of every pair, the twiddles and then, in their place, the sweep's factors.  The scans' gains,
// of which a thread needs its own chunk's once, come from L2 into registers.  With factors and
// gains beside the twiddles 640 points FP64 were 66 KB for one pair (two fit 58 KB now), 1200 110 KB
// (65), 2000 points FP32 132 KB for two pairs (54 for one); a step of 640^3 FP64 took 16.1 ms in
// imaginary and 17.0 in real time (13.6 and 14.2 now), 1200x2400 237 and 250 us (210 and 218),
// 700x3600 208 and 220 (196 and 206), 2000x1500 FP32 95 and 101 (90 and 94).
//
// Four waves per SIMD are asked for (3 or 4 VGPRs spilled in FP64 real time, 1 in FP32 with 16
// rows and primes past 16), two of the FP64 kernels with primes past 16 (202-208 VGPRs).
template <typename T, int MAXR, int MODE, int S>
__global__ void __launch_bounds__(r_max_threads<T>(), (sizeof(T) == 8 && MAXR > 16 ? 2 : 4))
    k_rc2r(const cpx<T>* __restrict__ spec, RXTile xt,
                                                    const RProgram* __restrict__ p,
                                                    RXArgs<T> g) {
  constexpr bool STEP = MODE == MODE_IMAG || MODE == MODE_REAL;
  constexpr bool IMAG_A = MODE == MODE_REAL;
  using GT = typename CnArith<T, IMAG_A>::G;
  constexpr unsigned CB = sizeof(cpx<T>);
  constexpr int U = sizeof(T) == 4 ? 4 : 2;
  extern __shared__ __align__(16) char rx_raw[];
  const int N = xt.n0, n1 = xt.n1, m = p->m, nt = blockDim.x, tid = threadIdx.x;
  const int TL = 2 * xt.np, P = xt.P, nw = P * TL >> 6;  // waves that sweep
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(rx_raw);
  cpx<T>* buf = tw + max(m, P * S);           // line 2q of the tile (Z of the pair before)
  cpx<T>* odd = buf + xt.np * xt.ls;          // line 2q + 1
  cpx<T>* wD = odd + xt.np * xt.ls;           // the sweep: the waves' carries,
  GT* fs = reinterpret_cast<GT*>(tw);  // after the FFT: the factors of P chunks
  GT* gw = reinterpret_cast<GT*>(wD + 2 * nw * TL);  // gains of the waves
  double* red = reinterpret_cast<double*>(wD + 2 * nw * TL + nw);
  const int lg = 31 - __clz(TL), QW = 64 >> lg;      // chunks of a line in a wave
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int k = b / xt.nbj, j0 = (b - k * xt.nbj) * TL;
  const int lines = min(TL, n1 - j0), npairs = (lines + 1) / 2;
  const RTile<0> tile{npairs, xt.ls};
  const cpx<T>* __restrict__ twg = reinterpret_cast<const cpx<T>*>(p->tw);
  auto tw_of = [&](int t) { return twg[t]; };
  auto f_of = [&](int t) { return CnArith<T, IMAG_A>{}.gain(t < N ? g.f[t] : cpx<T>{0, 0}); };
  auto g_of = [&](int t) { return scan_weight<GT>(g.gains + t); };
  Prefetch<cpx<T>, 1> ptw;
  GT wave_gain{};
  ptw.load(m, tw_of);
  if constexpr (STEP) {
    wave_gain = g_of(SG_WAVE * P + min(tid, nw - 1) * QW);
  }
  // the spectrum of the pairs
  {
    const int tot = (N / 2 + 1) * xt.np;  // the full tile's indexing; pairs past npairs skipped
    const bool even = (n1 & 1) == 0;
    for (int t0 = tid; t0 < tot; t0 += U * nt) {
      cpx<T> A[U], B[U];
      int kk[U], qq[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + u * nt;
        kk[u] = (int)fdiv((uint32_t)t, xt.fnp);
        qq[u] = t - kk[u] * xt.np;
        if (t >= tot || qq[u] >= npairs) qq[u] = -1;
        // in-range addresses only; a plane's last line without a successor: B = 0
        const cpx<T>* a =
            spec + (qq[u] >= 0 ? ((long long)kk[u] * xt.n2 + k) * n1 + j0 + 2 * qq[u] : 0);
        if (even) {
          const cpx2<T> v = *reinterpret_cast<const cpx2<T>*>(a);
          A[u] = v.a;
          B[u] = v.b;
        } else {
          const bool has1 = qq[u] >= 0 && 2 * qq[u] + 1 < lines;
          A[u] = a[0];
          B[u] = a[has1 ? 1 : 0];
          B[u] = csel(has1, B[u], cpx<T>{0, 0});
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (qq[u] >= 0) {
          const int kx = kk[u], q = qq[u];
          // the real lines' first and middle values are real
          const bool end = kx == 0 || 2 * kx == N;
          const cpx<T> a{A[u].re, end ? (T)0 : A[u].im}, c{B[u].re, end ? (T)0 : B[u].im};
          buf[tile.at(q, kx)] = cpx<T>{a.re - c.im, a.im + c.re};
          if (!end) buf[tile.at(q, N - kx)] = cpx<T>{a.re + c.im, c.re - a.im};
        }
      }
    }
  }
  __syncthreads();
  r_run<T, MAXR, true>(
      tile, p, tw, buf, [&](int l, int e) { return buf[tile.at(l, e)]; },
      [&](int, int, cpx<T> v) { return v; },
      [&](int l, int e, cpx<T> v) { buf[tile.at(l, e)] = v; },
      [&] {
        ptw.store(m, tw, tw_of);
        if constexpr (STEP) {
          if (tid < nw) gw[tid] = wave_gain;
        }
      });
  __syncthreads();
  const long long row = ((long long)k * n1 + j0) * N;  // first point of the tile
  const unsigned tl = (unsigned)lines * (unsigned)N;
  // the factors, fetched ahead of psi and V (400^3 FP32 1539 us a step, 1523 so; FP64 complex
  // ones after them, for the registers)
  Prefetch<GT, 4> pf;
  constexpr bool EARLY = sizeof(GT) <= 8;
  if constexpr (STEP && EARLY) pf.load(P * S, f_of);
  double s[7] = {0, 0, 0, 0, 0, 0, 0};
  const double z = (k - xt.n2 / 2) * g.h2;
  // both lines of a pair at a point: sums of scale psi, the phase, Phi
  {
    const T ts = g.scale ? (T)(*g.scale) : (T)1;
    const bool sums = STEP || g.part != nullptr;
    const __amdgpu_buffer_rsrc_t rp = buf_of(g.psi + row, sums ? tl * CB : 0u);
    const __amdgpu_buffer_rsrc_t rv =
        buf_of(const_cast<T*>(g.V) + row, sums ? tl * (unsigned)sizeof(T) : 0u);
    const int tot = npairs * N;
    for (int t0 = tid; t0 < tot; t0 += U * nt) {
      cpx<T> pv[U][2];
      T vv[U][2];
      int qq[U], ii[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + u * nt;
        qq[u] = (int)fdiv((uint32_t)t, xt.fn0);
        ii[u] = t - qq[u] * N;
        // lines past the tile are past the buffers: zero
        const unsigned o = (unsigned)(2 * qq[u]) * (unsigned)N + (unsigned)ii[u];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          buf_load(rp, (o + w * (unsigned)N) * CB, pv[u][w]);
          buf_load_real(rv, (o + w * (unsigned)N) * (unsigned)sizeof(T), vv[u][w]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (t0 + u * nt >= tot) continue;
        const int at = tile.at(qq[u], ii[u]);
        const cpx<T> zz = buf[at];
        const double x = (ii[u] - N / 2) * g.h0;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          const int j = j0 + 2 * qq[u] + w;
          const T phi = w ? zz.im : zz.re;
          const cpx<T> ps = scl(pv[u][w], ts);
          const T v = vv[u][w];
          const T n = ps.re * ps.re + ps.im * ps.im;
          if (sums) {
            const double nd = (double)n, y = (j - n1 / 2) * g.h1;
            s[0] += nd;
            s[1] += (double)v * nd;
            s[2] += nd * nd;
            s[3] += (double)phi * nd;
            s[4] += x * x * nd;
            s[5] += y * y * nd;
          }
          if constexpr (STEP) {
            const T th = (T)g.dt * (v + (T)g.gc * n + (T)g.gdd * phi);
            cpx<T> fz;
            if constexpr (MODE == MODE_IMAG) {
              fz = cpx<T>{exp(-th), (T)0};
            } else {
              T sn, cs;
              sincos_phase(th, sn, cs);
              fz = cpx<T>{cs, -sn};
            }
            (w ? odd : buf)[at] = ps * fz;
          } else if (g.phi != nullptr && j < n1) {
            g.phi[row + (2 * qq[u] + w) * (long long)N + ii[u]] = phi;
          }
        }
      }
    }
    s[6] = z * z * s[0];
  }
  // the gains of the sweep's scans: each of the chunk's own once, straight from L2
  GT up[5], up_in{};
  const int q = STEP ? min(tid >> lg, P - 1) : 0;
  if constexpr (STEP) {
    if constexpr (!EARLY) pf.load(P * S, f_of);
#pragma unroll
    for (int st = 0; st < 5; ++st) up[st] = g_of((SG_UP + st) * P + q);
    up_in = g_of(SG_UP_IN * P + q);
  }
  if (STEP || g.part != nullptr) rx_block_reduce<7>(s, red);
  if constexpr (STEP) {
    pf.store(P * S, fs, f_of);  // the FFT is done with the twiddles
    __syncthreads();
    // the sweep: thread (line l, chunk q), as in gp_sweep.hpp with the rows in LDS
    const cpx<T> zero{0, 0};
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // waves past the sweep's repeat its last chunks; neither they nor lines past the tile
    // store anything
    const int l = tid & (TL - 1), lo = q * S;
    const bool act = l < lines && wave < nw;
    cpx<T>* ln = (l & 1 ? odd : buf) + (l < lines ? l >> 1 : 0) * xt.ls;
    auto at = [&](int i) { return i + (i >> 3); };
    cpx<T> pr, r[S], pv[S];
    const GT* fq = fs + lo;
    cpx<T> D = zero;
    {
      // boundary rows and rows past the line as zero
      auto rd = [&](int i) {
        const cpx<T> v = ln[at(min(max(i, 0), N - 1))];
        return csel(i > 0 && i < N - 1, v, zero);
      };
#pragma unroll
      for (int e = 0; e < S; ++e) pv[e] = rd(lo + e);
      pr = rd(lo + S);
      cpx<T> prev = rd(lo - 1);
#pragma unroll
      for (int e = 0; e < S; ++e) {
        const GT gg = fq[e];
        const cpx<T> nx = (e + 1 < S) ? pv[e + 1] : pr;
        const cpx<T> dl{(prev.re + nx.re) - (T)2 * pv[e].re,
                        (prev.im + nx.im) - (T)2 * pv[e].im};
        prev = pv[e];
        r[e] = mulg(gg, dl);
        D = r[e] + mulg(gg, D);
      }
    }
#pragma unroll
    for (int st = 0; st < 5; ++st) {
      const int off = TL << st;
      if (off >= 64) break;
      const cpx<T> Dn = lane_at(D, (lane - off) * 4);
      D = csel(lane >= off, D + mulg(up[st], Dn), D);
    }
    // those down: all at once, or (FP64 complex: the registers) a step ahead
    constexpr int AHEAD = sizeof(GT) == 16 ? 1 : 5;
    GT down[5], down_in;
#pragma unroll
    for (int st = 0; st < AHEAD; ++st) down[st] = g_of((SG_DOWN + st) * P + q);
    if constexpr (AHEAD == 5) down_in = g_of(SG_DOWN_IN * P + q);
    if (lane >= 64 - TL && wave < nw) wD[wave * TL + l] = D;
    const cpx<T> Du = lane_at(D, (lane - TL) * 4);
    __syncthreads();
    cpx<T> C = zero;
    for (int w = 0; w < min(wave, nw); ++w) C = wD[w * TL + l] + mulg(gw[w], C);
    cpx<T> d = csel(lane < TL, C, Du + mulg(up_in, C));
#pragma unroll
    for (int e = 0; e < S; ++e) {
      d = r[e] + mulg(fq[e], d);
      r[e] = d;
    }
    cpx<T> X = zero;
#pragma unroll
    for (int e = S - 1; e >= 0; --e) X = r[e] + mulg(fq[e], X);
#pragma unroll
    for (int st = 0; st < 5; ++st) {
      const int off = TL << st;
      if (off >= 64) break;
      if (st + AHEAD < 5) down[st + AHEAD] = g_of((SG_DOWN + st + AHEAD) * P + q);
      const cpx<T> Xn = lane_at(X, (lane + off) * 4);
      X = csel(lane + off < 64, X + mulg(down[st], Xn), X);
    }
    cpx<T>* wX = wD + nw * TL;
    if constexpr (AHEAD < 5) down_in = g_of(SG_DOWN_IN * P + q);
    if (lane < TL && wave < nw) wX[wave * TL + l] = X;
    const cpx<T> Xd = lane_at(X, (lane + TL) * 4);
    __syncthreads();
    cpx<T> E = zero;
    for (int w = nw - 1; w > wave; --w) E = wX[w * TL + l] + mulg(gw[w], E);
    cpx<T> xv = csel(lane + TL >= 64, E, Xd + mulg(down_in, E));
    // every thread has read its neighbours' rows (two barriers ago)
#pragma unroll
    for (int e = S - 1; e >= 0; --e) {
      xv = r[e] + mulg(fq[e], xv);
      if (act && lo + e < N)
        ln[at(lo + e)] = cpx<T>{pv[e].re + (T)2 * xv.re, pv[e].im + (T)2 * xv.im};
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rp = buf_of(g.psi + row, tl * CB);
    for (unsigned t = tid; t < tl; t += nt) {
      const int ll = (int)fdiv(t, xt.fn0), i = (int)t - ll * N;
      buf_store(rp, t * CB, (ll & 1 ? odd : buf)[(ll >> 1) * xt.ls + at(i)]);
    }
  }
  if (STEP || g.part != nullptr) {
    if constexpr (!STEP) __syncthreads();
    rx_block_total<7>(red, g.part + 7 * (long long)blockIdx.x);
  }
}

}  // namespace gpdbec
