// FP64 finalisation of one step's partial sums: totals in a fixed order, the
// observables record of the state the step started from, and the new renormalisation
// factor.  Runs on one block after the step's last pass (one block per instance in the
// batched ensemble).
#pragma once
#include "gp_device.hpp"

namespace gpdbec {

enum : int { FIN_IMAG = 0, FIN_REAL = 1, FIN_OBSERVE = 2, FIN_EKZ = 3 };
constexpr int kRecord = 10;  // norm, mu, energy, e_kin, e_pot, e_int, e_dd, rms x/y/z

struct FinArgs {
  const double* p_x;   // 2 per block: sum |dx psi|^2, sum |d1 psi|^2 (unscaled)
  int nb_x;
  const double* p_nl;  // 7 per block: n, V n, n^2, Phi n, x^2 n, a1^2 n, a2^2 n (scaled)
  int nb_nl;
  const double* p_col; // 2 per block: |u|^2, |d2 u|^2 (new state / unscaled input)
  int nb_col;
  double dV, h0, h1, h2, gc, gdd;
  int geom;            // 0: 3D, 1: XY, 2: XZ
  double* scale;
  double* ekz;         // pending z-kinetic energy of the stored state (3D)
  int* flags;
  double* ring;
  int* ring_pos;
  int ring_cap;
  double* obs;         // FIN_OBSERVE output: the record, then the flags (one copy to the host)
  double* stage;       // two-stage reduction: kStageVals doubles per pre-reduced slice
  int nstage;          // slices (0: the finalize block reads the partials directly)
};

constexpr int kStageVals = 11;   // totals carried per slice (the v[] of finalize_block)
constexpr int kStageMax = 256;   // slices of the two-stage reduction (<= kThreads)

// Sums the partial arrays a block reads, blocks [lo, hi) of each, into v[11] (per
// thread; fixed order).  Each iteration first issues the loads of U blocks of every
// array, then adds them, so a small step's partials arrive in one memory round trip
// (U = 4; U = 1 inside a pass kernel, to stay within the pass's register budget).
template <int U = 4>
__device__ inline void fin_gather(const FinArgs& a, int mode, int slice, int nslice, int tid,
                                  double (&v)[11]) {
  const bool xnl = mode != FIN_EKZ;
  const bool col = mode != FIN_OBSERVE || a.geom == 0;
  auto lo_of = [&](int nb) { return (int)((long long)nb * slice / nslice); };
  auto hi_of = [&](int nb) { return (int)((long long)nb * (slice + 1) / nslice); };
  const int lx = lo_of(a.nb_x), nx = xnl ? hi_of(a.nb_x) - lx : 0;
  const int ln = lo_of(a.nb_nl), nn = xnl ? hi_of(a.nb_nl) - ln : 0;
  const int lc = lo_of(a.nb_col), nc = col ? hi_of(a.nb_col) - lc : 0;
  const int span = nx > nn ? (nx > nc ? nx : nc) : (nn > nc ? nn : nc);
  for (int b0 = tid; b0 < span; b0 += U * kThreads) {
    double t[U][11];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * kThreads;
#pragma unroll
      for (int k = 0; k < 2; ++k) t[u][k] = b < nx ? a.p_x[2 * (size_t)(lx + b) + k] : 0.0;
#pragma unroll
      for (int k = 0; k < 7; ++k) t[u][2 + k] = b < nn ? a.p_nl[7 * (size_t)(ln + b) + k] : 0.0;
#pragma unroll
      for (int k = 0; k < 2; ++k) t[u][9 + k] = b < nc ? a.p_col[2 * (size_t)(lc + b) + k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int k = 0; k < 11; ++k) v[k] += t[u][k];
    }
  }
}

// Totals, in thread 0, of slice `slice` of `nslice` (or, nslice = 0, of the pre-reduced
// slices), summed as kThreads threads in kThreads / 64 waves.  ANY: the block has any number
// of whole waves and each takes its share of those (same sums, bit for bit).  red: LDS for
// 11 kWaves doubles.
template <int U, bool ANY>
__device__ inline void fin_totals(const FinArgs& a, int mode, int slice, int nslice,
                                  double (&v)[11], double* red) {
  const int lane = threadIdx.x & 63;
  const int nw = ANY ? min((int)blockDim.x >> 6, kWaves) : kWaves;
  for (int w = threadIdx.x >> 6; w < kWaves; w += nw) {
    const int tid = w * 64 + lane;
#pragma unroll
    for (int k = 0; k < 11; ++k) v[k] = 0.0;
    if (nslice > 0) {
      fin_gather<U>(a, mode, slice, nslice, tid, v);
    } else if (tid < a.nstage) {  // one slice per thread (nstage <= kStageMax <= kThreads)
#pragma unroll
      for (int k = 0; k < kStageVals; ++k) v[k] = a.stage[tid * kStageVals + k];
    }
#pragma unroll
    for (int k = 0; k < 11; ++k) v[k] = wave_sum_to_last(v[k]);
    if (lane == 63) {
#pragma unroll
      for (int k = 0; k < 11; ++k) red[k * kWaves + w] = v[k];
    }
    if (!ANY) break;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 11; ++k) {
      double acc = red[k * kWaves];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) acc += red[k * kWaves + w];
      v[k] = acc;
    }
  }
}

// First stage of the two-stage reduction: block g writes the totals of slice g.
template <int U, bool ANY>
__device__ inline void prereduce_waves(const FinArgs& a, int mode, int g, double* red) {
  double v[11];
  fin_totals<U, ANY>(a, mode, g, a.nstage, v, red);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kStageVals; ++k) a.stage[g * kStageVals + k] = v[k];
  }
}

// All threads of one block must call this.
template <int U, bool ANY>
__device__ inline void finalize_waves(const FinArgs& a, int mode, double* red) {
  // no multiply-add contraction: the record rounds the same wherever this is inlined (its
  // own kernel, or folded into a pass kernel)
#pragma clang fp contract(off)
  const int tid = threadIdx.x;
  double v[11];
  // the scalars thread 0 needs at the end are fetched before the gather
  double s = 1.0, ekz_in = 0.0;
  int pos = 0;
  if (tid == 0) {
    s = *a.scale;
    if (mode != FIN_EKZ && mode != FIN_OBSERVE && a.geom == 0) ekz_in = *a.ekz;
    if (mode != FIN_EKZ && mode != FIN_OBSERVE) pos = *a.ring_pos;
  }
  fin_totals<U, ANY>(a, mode, 0, a.nstage > 0 ? 0 : 1, v, red);
  if (tid != 0) return;
  const double s2 = s * s;
  if (mode == FIN_EKZ) {
    *a.ekz = 0.5 * s2 * v[10] / (a.h2 * a.h2) * a.dV;
    return;
  }
  const double dV = a.dV;
  double rec[kRecord];
  const double norm = v[2] * dV;
  double ekin = 0.5 * s2 * (v[0] / (a.h0 * a.h0) + v[1] / (a.h1 * a.h1)) * dV;
  if (a.geom == 0) {
    ekin += (mode == FIN_OBSERVE) ? 0.5 * s2 * v[10] / (a.h2 * a.h2) * dV : ekz_in;
  }
  const double epot = v[3] * dV;
  const double eint = 0.5 * a.gc * v[4] * dV;
  const double edd = 0.5 * a.gdd * v[5] * dV;
  rec[0] = norm;
  rec[1] = ekin + epot + 2.0 * eint + 2.0 * edd;
  rec[2] = ekin + epot + eint + edd;
  rec[3] = ekin;
  rec[4] = epot;
  rec[5] = eint;
  rec[6] = edd;
  const double inv = norm > 0.0 ? 1.0 / norm : 0.0;  // rms of a zero state: 0
  const double r0 = sqrt(v[6] * dV * inv), r1 = sqrt(v[7] * dV * inv), r2 = sqrt(v[8] * dV * inv);
  rec[7] = r0;
  rec[8] = (a.geom == 2) ? 0.0 : r1;
  rec[9] = (a.geom == 0) ? r2 : (a.geom == 2 ? r1 : 0.0);
  double* dst;
  if (mode == FIN_OBSERVE) {
    dst = a.obs;
  } else {
    dst = a.ring + (size_t)(pos % a.ring_cap) * kRecord;
    *a.ring_pos = pos + 1;
  }
#pragma unroll
  for (int k = 0; k < kRecord; ++k) dst[k] = rec[k];
  if (!isfinite(norm)) *a.flags |= 1;
  if (mode == FIN_OBSERVE) {
    a.obs[kRecord] = (double)*a.flags;
    return;
  }
  // new state: imaginary time renormalises, real time keeps the physical values
  const double nout = v[9] * dV;
  // imaginary time must renormalise (a zero state cannot be); real time only needs the
  // state to stay finite (zero is a solution)
  if (!isfinite(nout) || (mode == FIN_IMAG && !(nout > 0.0))) {
    *a.flags |= 1;
    *a.scale = 1.0;
    return;
  }
  const double sn = (mode == FIN_IMAG) ? 1.0 / sqrt(nout) : 1.0;
  *a.scale = sn;
  if (a.geom == 0) *a.ekz = 0.5 * sn * sn * v[10] / (a.h2 * a.h2) * dV;
}

// The same for blocks of kThreads threads.
template <int U = 4>
__device__ inline void prereduce_block(const FinArgs& a, int mode, int g) {
  __shared__ double red[11 * kWaves];
  prereduce_waves<U, false>(a, mode, g, red);
}
template <int U = 4>
__device__ inline void finalize_block(const FinArgs& a, int mode) {
  __shared__ double red[11 * kWaves];
  finalize_waves<U, false>(a, mode, red);
}

// A finalisation folded into a pass kernel of any block size: `lead` leading blocks (a
// multiple of the XCDs, so that the tiles keep theirs), of which the first `blocks` work.
// stage: 1, the pre-reduction of a two-stage one; 0, the finalisation itself.
struct FoldedFin {
  FinArgs a;
  int mode, stage, blocks, lead;
};
// True if this is a leading block (its work is done).  lds: kFoldedLds bytes.
constexpr size_t kFoldedLds = 11 * kWaves * sizeof(double);
__device__ inline bool folded_fin(const FoldedFin& f, char* lds) {
  const int b = blockIdx.x;
  if (b >= f.lead) return false;
  if (b < f.blocks) {
    double* red = reinterpret_cast<double*>(lds);
    if (f.stage) prereduce_waves<1, true>(f.a, f.mode, b, red);
    else finalize_waves<1, true>(f.a, f.mode, red);
  }
  return true;
}

}  // namespace gpdbec
