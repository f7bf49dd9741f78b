// Instantiations of the run-time-length FFT passes for one precision (GP_REAL).
#include <mutex>

#include "gp_rfft_launch.hpp"

#ifndef GP_REAL
#error "GP_REAL must be float or double"
#endif

namespace gpdbec {
using T = GP_REAL;

namespace {
constexpr bool F32 = sizeof(T) == 4;
constexpr int kSmall = r_max_radix<T>(false), kBig = r_max_radix<T>(true);

// every (lines per tile, largest radix) instantiated
#if GP_RFFT_FP32
#define GP_FOR_RLINES(X) X(0, kSmall) X(16, kSmall) X(8, kSmall) X(4, kSmall)
#else
#define GP_FOR_RLINES(X) \
  X(0, kSmall) X(8, kSmall) X(4, kSmall) X(2, kSmall) X(0, kBig) X(8, kBig) X(4, kBig) X(2, kBig)
#endif
constexpr int kWide = F32 ? 16 : 8;   // columns of a strided tile: 128-byte runs
constexpr int kNarrow = F32 ? 4 : 2;

// LDS: the twiddles, the lines and the tile's kernel values
size_t lds_strided(const RAxis& a, int nlc) {
  return sizeof(cpx<T>) * (size_t)a.m * (nlc + 1) + sizeof(T) * (size_t)(a.n / 2 + 1) * nlc;
}
size_t lds_contiguous(const RAxis& a, int nl, bool conv) {
  return sizeof(cpx<T>) * ((size_t)a.m + (size_t)nl * r_line_slots(a.m)) +
         (conv ? sizeof(T) * (size_t)nl * a.n : 0);
}
bool fits(const RAxis& a, int nl, size_t lds, bool strided) {
  return a.k > 0 && lds <= kRLds && r_threads<T>(a, nl, strided) <= kRThreads;
}

// Columns of a strided tile: 128-byte runs while the tile's lines leave room for two blocks
// on a CU, then half and a quarter; 0: none fits.
int strided_cols(const RAxis& a) {
  for (int c = kWide; c >= kNarrow; c /= 2)
    if (fits(a, c, lds_strided(a, c), true) && lds_strided(a, c) <= 81920) return c;
  return fits(a, kNarrow, lds_strided(a, kNarrow), true) ? kNarrow : 0;
}

// Lines of a contiguous tile: as many as 256 threads hold in every stage, halved while the
// pass would have fewer than 512 blocks.
int contiguous_lines(const RAxis& a, int nlines) {
  int nl = 1;
  while (nl < 64 && r_threads<T>(a, nl + 1, false) <= 256 &&
         lds_contiguous(a, nl + 1, true) <= 65536)
    ++nl;
  while (nl > 1 && (nlines + nl - 1) / nl < 512) nl /= 2;
  return nl;
}
}  // namespace

template <>
hipError_t RLaunch<T>::prepare() {
  static std::mutex mu;
  static bool done = false;
  std::lock_guard<std::mutex> lock(mu);
  if (done) return hipSuccess;
  const void* ks[] = {
#define X(N, M) reinterpret_cast<const void*>(&k_rlines<T, N, M>),
      GP_FOR_RLINES(X)
#undef X
  };
  for (const void* k : ks) {
    const hipError_t e =
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRLds);
    if (e != hipSuccess) return e;
  }
  done = true;
  return hipSuccess;
}

template <>
hipError_t RLaunch<T>::program(hipStream_t st, const RAxis& a, int kind, const void* tw,
                               const void* chirp, const void* filt, RProgram* dst) {
  if (a.k < 2 || a.k > kRMaxStages) return hipErrorInvalidValue;
  RProgram p{};
  r_program(a, kind, &p);
  p.tw = tw;
  p.chirp = chirp;
  p.filt = filt;
  hipLaunchKernelGGL(k_rprogram, dim3(1), dim3(64), 0, st, p, dst);
  return hipGetLastError();
}

template <>
bool RLaunch<T>::contiguous_ok(const RAxis& a) { return fits(a, 1, lds_contiguous(a, 1, true), false); }

template <>
bool RLaunch<T>::strided_ok(const RAxis& a, int cols) {
  // byte offsets inside a plane, those past its range included, fit 32 bits
  return strided_cols(a) > 0 &&
         (double)a.n * cols * sizeof(cpx<T>) * 2.0 + 4096.0 < 4294967296.0;
}

namespace {
template <int NLC>
hipError_t launch(hipStream_t st, int blocks, int threads, size_t lds, cpx<T>* data,
                  const RLines& g, int maxr, const RProgram* p, const T* ktab,
                  const double* scale) {
  if (maxr == kSmall)
    hipLaunchKernelGGL((k_rlines<T, NLC, kSmall>), dim3(blocks), dim3(threads), lds, st, data, g,
                       p, ktab, scale);
  else
    hipLaunchKernelGGL((k_rlines<T, NLC, kBig>), dim3(blocks), dim3(threads), lds, st, data, g, p,
                       ktab, scale);
  return hipGetLastError();
}
}  // namespace

template <>
hipError_t RLaunch<T>::contiguous(hipStream_t st, cpx<T>* data, int nlines, const RAxis& a,
                                  const RProgram* p, const T* ktab, const double* scale) {
  if (!contiguous_ok(a) || nlines < 1) return hipErrorInvalidValue;
  const int nl = contiguous_lines(a, nlines);
  const RLines g{nlines, nl, r_line_slots(a.m), 0, 1u, 0};
  return launch<0>(st, (nlines + nl - 1) / nl, r_threads<T>(a, nl, false),
                   lds_contiguous(a, nl, ktab != nullptr), data,
                   g, a.maxr, p, ktab, scale);
}

template <>
hipError_t RLaunch<T>::strided(hipStream_t st, cpx<T>* data, int cols, int planes, const RAxis& a,
                               const RProgram* p, const T* ktab, const double* scale) {
  if (!strided_ok(a, cols) || planes < 1) return hipErrorInvalidValue;
  int c = strided_cols(a);
  // few tiles: half the columns (FP32 75x63 planes: 9.1 us, 8.4 with half)
  if (c == kWide && (long long)((cols + c - 1) / c) * planes < 512) c /= 2;
  const RLines g{cols * planes, c, 0, cols, (unsigned)cols, (long long)cols * a.n};
  const int blocks = (cols + c - 1) / c * planes, th = r_threads<T>(a, c, true);
  const size_t lds = lds_strided(a, c);
  switch (c) {
#if GP_RFFT_FP32
    case 16: return launch<16>(st, blocks, th, lds, data, g, a.maxr, p, ktab, scale);
#else
    case 2: return launch<2>(st, blocks, th, lds, data, g, a.maxr, p, ktab, scale);
#endif
    case 8: return launch<8>(st, blocks, th, lds, data, g, a.maxr, p, ktab, scale);
    case 4: return launch<4>(st, blocks, th, lds, data, g, a.maxr, p, ktab, scale);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gpdbec
