// Host side of the run-time-length FFT passes (gp_rfft.hpp), one instantiation per precision
// in gp_rfft_inst.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "gp_rfft.hpp"
#include "gp_rx.hpp"
#include "gp_sweep_launch.hpp"

namespace gpdbec {

// LDS a block may take (of 160 KiB per CU).
constexpr size_t kRLds = 143360;

// Shape of an x pass: its tile, blocks, threads and LDS bytes; blocks = 0: none.
struct RXCfg {
  RXTile xt{};
  int blocks = 0, threads = 0;
  size_t lds = 0;
  // the sweep's shape as the gain tables see it (rows, lines per block, whole waves)
  SweepCfg sweep() const {
    SweepCfg c;
    c.S = blocks ? xt.S : 0;
    c.TC = 2 * xt.np;
    c.threads = c.TC * xt.P;
    return c;
  }
};

template <typename T>
struct RLaunch {
  // raises the kernels' dynamic LDS limit (once per process, outside any capture)
  static hipError_t prepare();
  // keeps the program of a pass in device memory (tables: twiddles, chirp, filter)
  static hipError_t program(hipStream_t st, const RAxis& a, int kind, const void* tw,
                            const void* chirp, const void* filt, RProgram* dst);
  // whether an axis's lines have these passes, contiguous or strided
  static bool contiguous_ok(const RAxis& a);
  static bool strided_ok(const RAxis& a, int cols);
  // the x passes of a grid whose x axis is a: real-to-complex, and complex-to-real with the
  // sub-step and the sweep (gains: its table)
  static RXCfg x_r2c(const RAxis& a, int n1, int n2);
  static RXCfg x_c2r(const RAxis& a, int n1, int n2);
  static hipError_t r2c(hipStream_t st, const RXCfg& c, const RAxis& a, const cpx<T>* psi,
                        cpx<T>* spec, const RProgram* p, double* part, const FoldedFin& fin);
  static hipError_t c2r(hipStream_t st, const RXCfg& c, const RAxis& a, int mode,
                        const cpx<T>* spec, const RProgram* p, const RXArgs<T>& g);
  // contiguous lines of a.n points (nlines of them); scale, ktab: the convolution's
  static hipError_t contiguous(hipStream_t st, cpx<T>* data, int nlines, const RAxis& a,
                               const RProgram* p, const T* ktab, const double* scale,
                               const FoldedFin& fin);
  // lines at stride cols in `planes` planes of a.n x cols values (convolution: the 3D
  // quadrant table)
  static hipError_t strided(hipStream_t st, cpx<T>* data, int cols, int planes, const RAxis& a,
                            const RProgram* p, const T* ktab, const double* scale);
};

#define GP_DECLARE_RFFT(T)                                                                     \
  template <> hipError_t RLaunch<T>::prepare();                                                \
  template <> hipError_t RLaunch<T>::program(hipStream_t, const RAxis&, int, const void*,      \
                                             const void*, const void*, RProgram*);             \
  template <> bool RLaunch<T>::contiguous_ok(const RAxis&);                                    \
  template <> RXCfg RLaunch<T>::x_r2c(const RAxis&, int, int);                                 \
  template <> RXCfg RLaunch<T>::x_c2r(const RAxis&, int, int);                                 \
  template <> hipError_t RLaunch<T>::r2c(hipStream_t, const RXCfg&, const RAxis&,              \
                                         const cpx<T>*, cpx<T>*, const RProgram*, double*,     \
                                         const FoldedFin&);                                    \
  template <> hipError_t RLaunch<T>::c2r(hipStream_t, const RXCfg&, const RAxis&, int,         \
                                         const cpx<T>*, const RProgram*, const RXArgs<T>&);    \
  template <> bool RLaunch<T>::strided_ok(const RAxis&, int);                                  \
  template <> hipError_t RLaunch<T>::contiguous(hipStream_t, cpx<T>*, int, const RAxis&,       \
                                                const RProgram*, const T*, const double*,      \
                                                const FoldedFin&);                             \
  template <> hipError_t RLaunch<T>::strided(hipStream_t, cpx<T>*, int, int, const RAxis&,     \
                                             const RProgram*, const T*, const double*);
GP_DECLARE_RFFT(float)
GP_DECLARE_RFFT(double)
#undef GP_DECLARE_RFFT

}  // namespace gpdbec
