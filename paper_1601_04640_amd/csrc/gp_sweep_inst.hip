// Instantiations and shapes of the strided Crank-Nicolson sweeps for one precision (GP_REAL).
#include "gp_sweep_launch.hpp"

#ifndef GP_REAL
#error "GP_REAL must be float or double"
#endif

namespace gpdbec {
using T = GP_REAL;

namespace {
constexpr bool F32 = sizeof(T) == 4;
// Threads of the largest block and waves per SIMD asked of the compiler: chunks of 16 rows
// take 125 VGPRs in FP32 and 232 in FP64, of 8 rows 72 and 124.
template <int S>
constexpr int max_threads() { return F32 || S == 8 ? 1024 : 512; }
template <int S>
constexpr int waves_per_eu() { return F32 ? (S == 8 ? 7 : 4) : (S == 8 ? 4 : 2); }

SweepCfg shape(int S, int TC, int max_thr, int N, int n0, int n_outer) {
  SweepCfg c;
  const int t = (TC * ((N + S - 1) / S) + 63) / 64 * 64;
  if (t > max_thr) return c;
  c.S = S;
  c.TC = TC;
  c.threads = t;
  c.blocks = (n0 + TC - 1) / TC * n_outer;
  return c;
}
SweepCfg shape8(int TC, int N, int n0, int no) { return shape(8, TC, max_threads<8>(), N, n0, no); }
SweepCfg shape16(int TC, int N, int n0, int no) {
  return shape(16, TC, max_threads<16>(), N, n0, no);
}
}  // namespace

template <>
SweepCfg SweepLaunch<T>::cfg(int N, int n0, int n_outer, long long es) {
  SweepCfg c;
  const long long pitch = (long long)n0 * (long long)sizeof(cpx<T>);
  const double bytes = (double)N * n0 * n_outer * sizeof(cpx<T>);
  // a block's waves fill the 16 wave slots that 4 waves per SIMD leave a CU
  auto fills = [](const SweepCfg& x) { return x.S != 0 && 16 % (x.threads / 64) == 0; };
  if (F32) {
    // 128-byte runs.  Chunks of 16 rows issue least; with few tiles the shorter chain of 8
    // rows, and below one block per CU half the columns.  Measured, FP32: 256^3 43.8 us
    // (16 rows) and 45.6 (8), 400^3 237 and 307, 128x96x80 along y 6.5 and 5.9, 256^2 5.3
    // (16 rows), 5.2 (8) and 4.5 (8 rows, 8 columns).
    c = shape8(16, N, n0, n_outer);
    if (c.S && c.blocks < 256) c = shape8(8, N, n0, n_outer);
    if (!c.S || c.blocks >= 2048) c = shape16(16, N, n0, n_outer);
    if (!c.S || (N > 512 && c.blocks < 256)) c = shape16(8, N, n0, n_outer);
  } else {
    // 16 columns (256-byte runs) where the block's waves fill a CU exactly, else 8.
    // Measured, FP64: 256^3 along z 90 us (16 columns) and 99 (8), 128^3 11.6 and 12.6,
    // but 200^3 48.0 and 44.8, 333x211x150 72 and 58.  Large arrays whose rows do not start
    // on 128-byte lines run fewer blocks per CU with chunks of 16 rows, so that the lines
    // two tiles share are still in L2: 300^3 201 us against 236.  Below one block per CU
    // half the columns: 540x600 7.3 us against 8.5.
    const SweepCfg w = shape8(16, N, n0, n_outer);
    c = shape8(8, N, n0, n_outer);
    if (fills(w) && w.blocks >= 512) c = w;
    if (pitch % 128 && bytes > 268435456.0) {
      const SweepCfg l = shape16(8, N, n0, n_outer);
      if (l.S) c = l;
    }
    if (c.S && c.blocks < 256) {
      const SweepCfg n = shape8(4, N, n0, n_outer);
      if (n.S) c = n;
    }
    if (!c.S) c = shape16(4, N, n0, n_outer);
  }
  if (!c.S) return c;
  // every byte offset the kernel forms, in and out of range, fits 32 bits
  const double span = ((double)c.chunks() * c.S + 2.0 * c.S) * (double)es * sizeof(cpx<T>);
  if (span >= 4294967296.0) return SweepCfg{};
  // One contiguous range of tiles per XCD where neighbouring tiles share 128-byte lines (a
  // ragged pitch: FP32 333x211x150 along z 33 us against 52) and elsewhere (400^3 along z
  // 247 against 277), but not where rows are a multiple of 2 KiB apart: the XCDs would then
  // work the same channels at once (FP64 256^3 along z 90 us against 85).
  c.lin = pitch % 2048 == 0;
  return c;
}

template <>
hipError_t SweepLaunch<T>::gains(const SweepCfg& c, hipStream_t st, const SweepTables& t, int N) {
  const int P = c.S ? c.chunks() : 0;
  if (P < 1 || P > kSweepMaxChunks) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_sweep_gains<T>), dim3(3), dim3(kSweepMaxChunks), 0, st, t, N, c.S, P,
                     64 / c.TC);
  return hipGetLastError();
}

namespace {
template <int S, int TC>
hipError_t launch(const SweepCfg& c, int op, bool imag_a, hipStream_t st, cpx<T>* psi,
                  const cpx<T>* f, const cpx<T>* w, double* part, int N, int n0, unsigned es,
                  long long os) {
  const size_t lds = sweep_lds<T>(S, TC, c.threads / 64);
#define GP_SWEEP(IA, OP)                                                                      \
  hipLaunchKernelGGL((k_sweep<T, S, TC, IA, OP, max_threads<S>(), waves_per_eu<S>()>),         \
                     dim3(c.blocks), dim3(c.threads), lds, st, psi, f, w, part, N, n0, es, os, \
                     c.lin)
  if (op == SWEEP_OBS) GP_SWEEP(true, SWEEP_OBS);
  else if (op == SWEEP_SUMS && imag_a) GP_SWEEP(true, SWEEP_SUMS);
  else if (op == SWEEP_SUMS) GP_SWEEP(false, SWEEP_SUMS);
  else if (op == SWEEP_SOLVE && imag_a) GP_SWEEP(true, SWEEP_SOLVE);
  else if (op == SWEEP_SOLVE) GP_SWEEP(false, SWEEP_SOLVE);
  else return hipErrorInvalidValue;
#undef GP_SWEEP
  return hipGetLastError();
}
}  // namespace

template <>
hipError_t SweepLaunch<T>::run(const SweepCfg& c, int op, bool imag_a, hipStream_t st,
                               cpx<T>* psi, const cpx<T>* f, const cpx<T>* w, double* part,
                               int N, int n0, long long es, long long os) {
#define GP_SHAPE(SV, TCV)                                                                 \
  if (c.S == SV && c.TC == TCV)                                                           \
    return launch<SV, TCV>(c, op, imag_a, st, psi, f, w, part, N, n0, (unsigned)es, os);
  GP_SHAPE(8, 16)
  GP_SHAPE(8, 8)
  GP_SHAPE(16, 8)
#if GP_SWEEP_FP32
  GP_SHAPE(16, 16)
#else
  GP_SHAPE(8, 4)
  GP_SHAPE(16, 4)
#endif
#undef GP_SHAPE
  return hipErrorInvalidValue;
}

}  // namespace gpdbec
