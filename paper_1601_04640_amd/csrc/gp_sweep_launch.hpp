// Host side of the strided Crank-Nicolson sweeps (gp_sweep.hpp): the shape of a sweep, its
// tables and its launch, one instantiation per precision in gp_sweep_inst.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "gp_sweep.hpp"

namespace gpdbec {

// Shape of a sweep of lines of N rows: S rows per chunk, TC columns per block, whole waves
// of threads, tiles in dispatch order (lin) or XCD-contiguous.  S = 0: no such sweep (the
// line is too long, or spans 4 GiB or more).
struct SweepCfg {
  int S = 0, TC = 0, threads = 0, blocks = 0, lin = 0;
  int chunks() const { return threads / TC; }
};

template <typename T>
struct SweepLaunch {
  // lines of N rows at element stride es; n0 adjacent columns, n_outer outer indices
  static SweepCfg cfg(int N, int n0, int n_outer, long long es);
  // values (cpx<T>) of the gain table of a factor set; the tables of the three sets
  static size_t table_len(const SweepCfg& c) { return c.S ? (size_t)kSweepGains * c.chunks() : 0; }
  static hipError_t gains(const SweepCfg& c, hipStream_t st, const SweepTables& t, int N);
  // op: SWEEP_*; imag_a: complex factors (real time, adjoint)
  static hipError_t run(const SweepCfg& c, int op, bool imag_a, hipStream_t st, cpx<T>* psi,
                        const cpx<T>* f, const cpx<T>* w, double* part, int N, int n0,
                        long long es, long long os);
};

template <> SweepCfg SweepLaunch<float>::cfg(int, int, int, long long);
template <> SweepCfg SweepLaunch<double>::cfg(int, int, int, long long);
#define GP_DECLARE_SWEEP(T)                                                                  \
  template <> hipError_t SweepLaunch<T>::gains(const SweepCfg&, hipStream_t,                 \
                                               const SweepTables&, int);                     \
  template <> hipError_t SweepLaunch<T>::run(const SweepCfg&, int, bool, hipStream_t,        \
                                             cpx<T>*, const cpx<T>*, const cpx<T>*, double*, \
                                             int, int, long long, long long);
GP_DECLARE_SWEEP(float)
GP_DECLARE_SWEEP(double)
#undef GP_DECLARE_SWEEP

}  // namespace gpdbec
