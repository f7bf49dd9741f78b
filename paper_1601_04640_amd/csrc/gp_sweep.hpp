// Crank-Nicolson sweeps along a strided axis (y and z), the line length a kernel argument.
//
// Lines run at stride `es`, TC adjacent columns to a block, and thread (c, q) holds chunk q
// of column c: S consecutive rows, loaded from global memory straight into registers.  With
// the column index fastest across the lanes every load and store is a run of TC values
// (128 bytes for 16 FP32 or 8 FP64 columns), so the lines never pass through LDS: the block
// keeps only its factor table and one carry per wave there, and its occupancy is set by the
// S values of psi and of the recurrence per thread.  The loads and stores are buffer
// accesses: rows past the line and columns past the grid are out of the buffer's range, read
// as zero and are not written, so no element carries a guard or a 64-bit address.
//
// In increment form, with Delta_i = psi_(i-1) + psi_(i+1) - 2 psi_i, the factor table
// f_i = 2 A m_i (m: Thomas factors of (1 + 2A) u_i - A (u_(i-1) + u_(i+1)), zero on the two
// boundary rows), g_i = f_i / 2 and every value halved (exact):
//   forward  h_i = g_i Delta_i + g_i h_(i-1)     backward  k_i = h_i + g_i k_(i+1)
//   u_i = psi_i + 2 k_i.
// Each is run from a zero carry over the chunk, the chunks' affine maps are joined by a scan
// (the chunks of a wave by lane moves TC apart, the waves through LDS), and run again from
// the true carry.  The gains of the scan depend on the factors only and come from a table
// (k_sweep_gains).
#pragma once
#include "gp_device.hpp"
#include "gp_kernels.hpp"  // xcd_tile

namespace gpdbec {

// SWEEP_SOLVE: solve; SWEEP_SUMS: solve, with part[2b] = sum |u|^2 and part[2b+1] = sum
// |u_(i+1) - u_i|^2 along the lines of the block's new values; SWEEP_OBS: those sums of the
// stored values, nothing written.
enum : int { SWEEP_SOLVE = 0, SWEEP_SUMS = 1, SWEEP_OBS = 2 };

// Gains per chunk in the table: the scan steps forward (1, 2, 4, 8, 16 chunks), the carry
// into the wave's chunk, the same backward, and the wave's total (QW <= 32 chunks per wave).
constexpr int kSweepGains = 13;
enum : int { SG_UP = 0, SG_UP_IN = 5, SG_DOWN = 6, SG_DOWN_IN = 11, SG_WAVE = 12 };

// Tables of a sweep, one per factor set (block b: set b): for chunk q (S rows, QW chunks of
// a column per wave) the products of g:
//   [(SG_UP + s) P + q]    over the chunks q, q-1, .. of the wave that step s composes
//   [SG_UP_IN P + q]       over the chunks before q in its wave (1 for the first)
//   [(SG_DOWN + s) P + q]  over q, q+1, ..     [SG_DOWN_IN P + q]  over those after q
//   [SG_WAVE P + q]        over the whole wave
// from the rounded factors, in FP64.  One thread per chunk, P <= kSweepMaxChunks; P counts
// the chunks of whole waves (those past the line have the identity map).
constexpr int kSweepMaxChunks = 256;
struct SweepTables {
  const void* f[3];
  void* w[3];
};
template <typename T>
__global__ void __launch_bounds__(kSweepMaxChunks) k_sweep_gains(SweepTables t, int N, int S,
                                                                 int P, int QW) {
  __shared__ double gr[kSweepMaxChunks], gi[kSweepMaxChunks];
  const cpx<T>* __restrict__ f = reinterpret_cast<const cpx<T>*>(t.f[blockIdx.x]);
  cpx<T>* __restrict__ w = reinterpret_cast<cpx<T>*>(t.w[blockIdx.x]);
  const int q = threadIdx.x;
  auto mul = [](double& ar, double& ai, double br, double bi) {
    const double r = ar * br - ai * bi;
    ai = ar * bi + ai * br;
    ar = r;
  };
  if (q < P) {
    double r = 1.0, i = 0.0;
    for (int a = q * S; a < (q + 1) * S && a < N; ++a)
      mul(r, i, 0.5 * (double)f[a].re, 0.5 * (double)f[a].im);
    gr[q] = r;
    gi[q] = i;
  }
  __syncthreads();
  if (q >= P) return;
  const int first = q / QW * QW, last = first + QW - 1;
  auto over = [&](int a, int b) {  // product over the chunks a..b
    double r = 1.0, i = 0.0;
    for (int c = a; c <= b; ++c) mul(r, i, gr[c], gi[c]);
    return cpx<T>{(T)r, (T)i};
  };
  for (int s = 0; s < 5; ++s) {
    const int n = 1 << s;
    w[(SG_UP + s) * P + q] = over(q - n + 1 > first ? q - n + 1 : first, q);
    w[(SG_DOWN + s) * P + q] = over(q, q + n - 1 < last ? q + n - 1 : last);
  }
  w[SG_UP_IN * P + q] = over(first, q - 1);
  w[SG_DOWN_IN * P + q] = over(q + 1, last);
  w[SG_WAVE * P + q] = over(first, last);
}

// A complex value through a buffer descriptor: `off` in bytes; out of range reads as zero
// and is not written.
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t r, unsigned off, cpx<float>& v) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  const u2 t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
  v = cpx<float>{__uint_as_float(t.x), __uint_as_float(t.y)};
}
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t r, unsigned off, cpx<double>& v) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const u4 t = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
  v = cpx<double>{__hiloint2double((int)t.y, (int)t.x), __hiloint2double((int)t.w, (int)t.z)};
}
__device__ __forceinline__ void buf_load_real(__amdgpu_buffer_rsrc_t r, unsigned off, float& v) {
  v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ void buf_load_real(__amdgpu_buffer_rsrc_t r, unsigned off, double& v) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  const u2 t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
  v = __hiloint2double((int)t.y, (int)t.x);
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, cpx<float> v) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(u2{__float_as_uint(v.re), __float_as_uint(v.im)}, r,
                                        (int)off, 0, 0);
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, cpx<double> v) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_raw_buffer_store_b128(
      u4{(unsigned)__double2loint(v.re), (unsigned)__double2hiint(v.re),
         (unsigned)__double2loint(v.im), (unsigned)__double2hiint(v.im)},
      r, (int)off, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000);
}

// The value of the lane whose index is a4 / 4.
__device__ __forceinline__ float lane_at(float v, int a4) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(a4, __float_as_int(v)));
}
__device__ __forceinline__ double lane_at(double v, int a4) {
  return __hiloint2double(__builtin_amdgcn_ds_bpermute(a4, __double2hiint(v)),
                          __builtin_amdgcn_ds_bpermute(a4, __double2loint(v)));
}
template <typename T>
__device__ __forceinline__ cpx<T> lane_at(cpx<T> v, int a4) {
  return cpx<T>{lane_at(v.re, a4), lane_at(v.im, a4)};
}

// LDS of a sweep block of `waves` waves: the factors of its chunks, the waves' carries and
// the reduction.
template <typename T>
constexpr size_t sweep_lds(int S, int TC, int waves) {
  return sizeof(cpx<T>) * ((size_t)waves * (64 / TC) * (S + kSweepGains) + 2 * (size_t)waves * TC) +
         2 * 16 * sizeof(double);
}

// Grid: (n0 / TC rounded up) tiles of columns times the outer index; block: whole waves over
// TC ceil(N / S) threads.  psi + outer os: the outer index's first column.  lin: tiles in
// dispatch order instead of one contiguous range per XCD.
template <typename T, int S, int TC, bool IMAG_A, int OP, int MAXT, int WPE>
__global__ void __launch_bounds__(MAXT, WPE) k_sweep(cpx<T>* __restrict__ psi,
                                                const cpx<T>* __restrict__ f,
                                                const cpx<T>* __restrict__ gains,
                                                double* __restrict__ part, int N, int n0,
                                                unsigned es, long long os, int lin) {
  using GT = typename CnArith<T, IMAG_A>::G;
  constexpr int QW = 64 / TC;  // chunks of a column in one wave
  constexpr int CB = (int)sizeof(cpx<T>);
  extern __shared__ __align__(16) char sweep_raw[];
  const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = nw * QW;                       // chunks of the block's whole waves
  cpx<T>* wD = reinterpret_cast<cpx<T>*>(sweep_raw);   // carries of the waves, per column
  cpx<T>* wX = wD + nw * TC;
  GT* fs = reinterpret_cast<GT*>(wX + nw * TC);        // g_i, zero past the line
  GT* gs = fs + P * S;                                 // the table of gains
  const int c = tid % TC, q = tid / TC;
  const int tiles = (n0 + TC - 1) / TC;
  const int bid = lin ? blockIdx.x : xcd_tile(blockIdx.x, gridDim.x);
  const int outer = bid / tiles, x0 = (bid - outer * tiles) * TC;
  const bool col = x0 + c < n0;
  const int lo = q * S;
  const unsigned step = es * CB;
  const unsigned top = (unsigned)(N - 1) * step;  // byte offset of the last row
  const __amdgpu_buffer_rsrc_t rb =
      buf_of(psi + (outer * os + x0), top + (unsigned)min(TC, n0 - x0) * CB);
  // byte offset of the chunk's first row; columns past the grid start past the range
  const unsigned v0 = col ? (unsigned)lo * step + (unsigned)c * CB
                          : top + (unsigned)min(TC, n0 - x0) * CB;
  cpx<T> p[S], pl, pr;
#pragma unroll
  for (int e = 0; e < S; ++e) buf_load(rb, v0 + e * step, p[e]);
  buf_load(rb, v0 + S * step, pr);
  if constexpr (OP != SWEEP_OBS) {
    buf_load(rb, col ? v0 - step : v0, pl);  // chunk 0: wraps past the range
    for (int t = tid; t < P * S; t += nt) {
      const cpx<T> v = t < N ? f[t] : cpx<T>{0, 0};
      fs[t] = CnArith<T, IMAG_A>{}.gain(v);
    }
    for (int t = tid; t < P * kSweepGains; t += nt) gs[t] = scan_weight<GT>(gains + t);
  }
  double s0 = 0.0, s1 = 0.0;
  if constexpr (OP == SWEEP_OBS) {
#pragma unroll
    for (int e = 0; e < S; ++e) {
      s0 += abs2_d(p[e]);  // rows past the line are zero
      if (lo + e + 1 < N) s1 += absdiff2_d(e + 1 < S ? p[e + 1] : pr, p[e]);
    }
  } else {
    const cpx<T> zero{0, 0};
    constexpr int NS = QW > 8 ? 4 : QW > 4 ? 3 : QW > 2 ? 2 : 1;  // scan steps in a wave
    // the boundary rows enter as zero
    if (q == 0) p[0] = zero;
    if (lo - 1 == 0) pl = zero;
#pragma unroll
    for (int e = 0; e < S; ++e) p[e] = csel(lo + e == N - 1, zero, p[e]);
    pr = csel(lo + S == N - 1, zero, pr);
    __syncthreads();
    const GT* fq = fs + lo;
    cpx<T> r[S];
    cpx<T> D = zero;
    {
      cpx<T> prev = pl;
#pragma unroll
      for (int e = 0; e < S; ++e) {
        const GT g = fq[e];
        const cpx<T> nx = (e + 1 < S) ? p[e + 1] : pr;
        const cpx<T> dl{(prev.re + nx.re) - (T)2 * p[e].re, (prev.im + nx.im) - (T)2 * p[e].im};
        prev = p[e];
        r[e] = mulg(g, dl);
        D = r[e] + mulg(g, D);
      }
    }
    // inclusive scan of the maps over the wave's chunks of a column, then the waves before
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int off = TC << s;
      const cpx<T> Dn = lane_at(D, (lane - off) * 4);
      D = csel(lane >= off, D + mulg(gs[(SG_UP + s) * P + q], Dn), D);
    }
    if (lane >= 64 - TC) wD[wave * TC + c] = D;
    const cpx<T> Du = lane_at(D, (lane - TC) * 4);
    __syncthreads();
    cpx<T> C = zero;
    for (int w = 0; w < wave; ++w)
      C = wD[w * TC + c] + mulg(gs[SG_WAVE * P + w * QW], C);
    cpx<T> d = csel(lane < TC, C, Du + mulg(gs[SG_UP_IN * P + q], C));
#pragma unroll
    for (int e = 0; e < S; ++e) {
      d = r[e] + mulg(fq[e], d);
      r[e] = d;
    }
    // backward: composed from the right
    cpx<T> X = zero;
#pragma unroll
    for (int e = S - 1; e >= 0; --e) X = r[e] + mulg(fq[e], X);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int off = TC << s;
      const cpx<T> Xn = lane_at(X, (lane + off) * 4);
      X = csel(lane + off < 64, X + mulg(gs[(SG_DOWN + s) * P + q], Xn), X);
    }
    if (lane < TC) wX[wave * TC + c] = X;
    const cpx<T> Xd = lane_at(X, (lane + TC) * 4);
    __syncthreads();
    cpx<T> E = zero;
    for (int w = nw - 1; w > wave; --w)
      E = wX[w * TC + c] + mulg(gs[SG_WAVE * P + w * QW], E);
    cpx<T> x = csel(lane + TC >= 64, E, Xd + mulg(gs[SG_DOWN_IN * P + q], E));
    cpx<T> un{pr.re + (T)2 * x.re, pr.im + (T)2 * x.im};  // the next chunk's first value
#pragma unroll
    for (int e = S - 1; e >= 0; --e) {
      x = r[e] + mulg(fq[e], x);
      // zero on the boundary rows: psi and the factor are
      const cpx<T> u{p[e].re + (T)2 * x.re, p[e].im + (T)2 * x.im};
      buf_store(rb, v0 + e * step, u);
      if constexpr (OP == SWEEP_SUMS) {
        // rows past the line and columns past the grid hold zeros
        s0 += abs2_d(u);
        s1 += absdiff2_d(un, u);
      }
      un = u;
    }
  }
  if constexpr (OP != SWEEP_SOLVE) {
    double* red = reinterpret_cast<double*>(gs + P * kSweepGains);
    s0 = wave_sum_to_last(s0);
    s1 = wave_sum_to_last(s1);
    if (lane == 63) {
      red[wave] = s0;
      red[16 + wave] = s1;
    }
    __syncthreads();
    if (tid < 2) {
      double acc = red[16 * tid];
      for (int w = 1; w < nw; ++w) acc += red[16 * tid + w];
      part[2 * (long long)blockIdx.x + tid] = acc;
    }
  }
}

}  // namespace gpdbec
