// Instantiations of the run-time-length FFT passes for one precision (GP_REAL) and family:
//   GP_FAMILY 0: line passes and programs    1: x passes
//   2 and 3: the kernels of both that hold the prime radices past 16 (compiled apart)
#include <algorithm>
#include <mutex>

#include "gp_rfft_launch.hpp"

#ifndef GP_REAL
#error "GP_REAL must be float or double"
#endif

namespace gpdbec {
using T = GP_REAL;

// Families 2 and 3 define these kernels, 0 and 1 launch them.
#if GP_FAMILY >= 2
#define GP_PRIME_KERNEL template __global__ void
#else
#define GP_PRIME_KERNEL extern template __global__ void
#endif
#if GP_FAMILY % 2 == 0
#define X(NLC)                                                                                \
  GP_PRIME_KERNEL k_rlines<T, NLC, kRPrime>(cpx<T>*, RLines, const RProgram*, const T*,       \
                                            const double*, FoldedFin);
X(0) X(8) X(4)
#if GP_RFFT_FP32
X(16)
#else
X(2)
#endif
#undef X
#else
GP_PRIME_KERNEL k_rr2c<T, kRPrime>(const cpx<T>*, cpx<T>*, RXTile, const RProgram*, double*,
                                   FoldedFin);
#define X(MODE, S)                                                                            \
  GP_PRIME_KERNEL k_rc2r<T, kRPrime, MODE, S>(const cpx<T>*, RXTile, const RProgram*, RXArgs<T>);
X(MODE_IMAG, 8) X(MODE_REAL, 8) X(MODE_OBSERVE, 8)
#if GP_RFFT_FP32
X(MODE_IMAG, 16) X(MODE_REAL, 16)
#endif
#undef X
#endif
#undef GP_PRIME_KERNEL

#if GP_FAMILY < 2
#if GP_FAMILY == 0
hipError_t rx_prepare(T);  // the x passes' LDS limits (family 1)
#endif

namespace {
constexpr bool F32 = sizeof(T) == 4;
constexpr int kSmall = r_max_radix<T>(false), kBig = r_max_radix<T>(true);
constexpr int kWide = F32 ? 16 : 8;   // lines of a tile side by side: 128-byte runs

// Whether the kernels of gp_generic.hpp have written-out butterflies for n points.
bool seven_smooth(int n) {
  for (int p : {2, 3, 5, 7})
    while (n % p == 0) n /= p;
  return n == 1;
}

#if GP_FAMILY == 0
// every (lines per tile, largest radix) instantiated
#if GP_RFFT_FP32
#define GP_FOR_RLINES(X)                                  \
  X(0, kSmall) X(16, kSmall) X(8, kSmall) X(4, kSmall)    \
  X(0, kRPrime) X(16, kRPrime) X(8, kRPrime) X(4, kRPrime)
#else
#define GP_FOR_RLINES(X)                                  \
  X(0, kSmall) X(8, kSmall) X(4, kSmall) X(2, kSmall)     \
  X(0, kBig) X(8, kBig) X(4, kBig) X(2, kBig)             \
  X(0, kRPrime) X(8, kRPrime) X(4, kRPrime) X(2, kRPrime)
#endif
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
  return a.k > 0 && lds <= kRLds && r_threads<T>(a, nl, strided) <= r_max_threads<T>();
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
  const hipError_t e = rx_prepare(T{});
  if (e != hipSuccess) return e;
  done = true;
  return hipSuccess;
}

template <>
hipError_t RLaunch<T>::program(hipStream_t st, const RAxis& a, int kind, const void* tw,
                               const void* chirp, const void* filt, RProgram* dst) {
  if (a.k < 1 || a.k > kRMaxStages) return hipErrorInvalidValue;
  RProgram p{};
  r_program(a, kind, &p);
  p.tw = tw;
  p.chirp = chirp;
  p.filt = filt;
  hipLaunchKernelGGL(k_rprogram, dim3(1), dim3(64), 0, st, p, dst);
  return hipGetLastError();
}

// Where one line takes more than half a CU's LDS, the kernels of gp_generic.hpp, whose lines
// do not share it with the kernel values, are faster if they have the radices (y convolution
// of 2048^2 FP64 50 us, 69 here; 4096^2 FP32 101 and 187; at 3600 FP32, with two blocks on a
// CU, 27.7 and 24.8).
template <>
bool RLaunch<T>::contiguous_ok(const RAxis& a) {
  const size_t lds = lds_contiguous(a, 1, true);
  return fits(a, 1, lds, false) && (lds <= 81920 || !seven_smooth(a.n));
}

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
                  const double* scale, const FoldedFin& fin = {}) {
  blocks += fin.lead;
  if (lds < kFoldedLds) lds = kFoldedLds;
  if (maxr == kSmall)
    hipLaunchKernelGGL((k_rlines<T, NLC, kSmall>), dim3(blocks), dim3(threads), lds, st, data, g,
                       p, ktab, scale, fin);
  else if (maxr == kRPrime)
    hipLaunchKernelGGL((k_rlines<T, NLC, kRPrime>), dim3(blocks), dim3(threads), lds, st, data, g,
                       p, ktab, scale, fin);
  else
    hipLaunchKernelGGL((k_rlines<T, NLC, kBig>), dim3(blocks), dim3(threads), lds, st, data, g, p,
                       ktab, scale, fin);
  return hipGetLastError();
}
}  // namespace

template <>
hipError_t RLaunch<T>::contiguous(hipStream_t st, cpx<T>* data, int nlines, const RAxis& a,
                                  const RProgram* p, const T* ktab, const double* scale,
                                  const FoldedFin& fin) {
  if (!contiguous_ok(a) || nlines < 1) return hipErrorInvalidValue;
  const int nl = contiguous_lines(a, nlines);
  const RLines g{nlines, nl, r_line_slots(a.m), 0, 1u, 0};
  const int blocks = (nlines + nl - 1) / nl;
  return launch<0>(st, blocks, r_spread<T>(a, nl, r_threads<T>(a, nl, false), blocks),
                   lds_contiguous(a, nl, ktab != nullptr), data,
                   g, a.maxr, p, ktab, scale, fin);
}

template <>
hipError_t RLaunch<T>::strided(hipStream_t st, cpx<T>* data, int cols, int planes, const RAxis& a,
                               const RProgram* p, const T* ktab, const double* scale) {
  if (!strided_ok(a, cols) || planes < 1) return hipErrorInvalidValue;
  int c = strided_cols(a);
  // few tiles: half the columns (FP32 75x63 planes: 9.1 us, 8.4 with half)
  if (c == kWide && (long long)((cols + c - 1) / c) * planes < 512) c /= 2;
  const RLines g{cols * planes, c, 0, cols, (unsigned)cols, (long long)cols * a.n};
  const int blocks = (cols + c - 1) / c * planes;
  const int th = r_spread<T>(a, c, r_threads<T>(a, c, true), blocks);
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

#else  // x passes
}  // namespace

hipError_t rx_prepare(T) {
  const void* ks[] = {
#define X(M)                                                       \
  reinterpret_cast<const void*>(&k_rr2c<T, M>),                    \
      reinterpret_cast<const void*>(&k_rc2r<T, M, MODE_IMAG, 8>),  \
      reinterpret_cast<const void*>(&k_rc2r<T, M, MODE_REAL, 8>),  \
      reinterpret_cast<const void*>(&k_rc2r<T, M, MODE_OBSERVE, 8>)
      X(kSmall), X(kRPrime),
#if GP_RFFT_FP32
      reinterpret_cast<const void*>(&k_rc2r<T, kSmall, MODE_IMAG, 16>),
      reinterpret_cast<const void*>(&k_rc2r<T, kSmall, MODE_REAL, 16>),
      reinterpret_cast<const void*>(&k_rc2r<T, kRPrime, MODE_IMAG, 16>),
      reinterpret_cast<const void*>(&k_rc2r<T, kRPrime, MODE_REAL, 16>),
#else
      X(kBig),
#endif
#undef X
  };
  for (const void* k : ks) {
    const hipError_t e =
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

namespace {
// The tile of an x pass: the most line pairs (runs of up to 128 bytes along the spectrum's y)
// that leave room for two blocks on a CU and the grid 256 blocks, else one pair.
template <typename F>
RXCfg x_shape(const RAxis& a, int n1, int n2, F size) {
  RXCfg best;
  if (a.k < 1 || (double)a.n * (kWide + 1) * sizeof(cpx<T>) >= 2147483648.0) return best;
  // Longer lines leave a block one pair: FP32 ones whose radices gp_generic.hpp has written out
  // run its kernels, which were ahead while the sweep's tables stood beside the twiddles (2500^2
  // 36 + 28 + 88 us, 38 + 126 here).  Without them there these passes are ahead to some 4000
  // points (a step of 2500^2 284 us with gp_generic.hpp and 249 here, 3200x1500 157 and 149,
  // 4096^2 590 and 599); the line has not been moved.
  if (a.n > 2048 && seven_smooth(a.n)) return best;
  const int pairs = (n1 + 1) / 2;
  for (int np = kWide / 2; np >= 1; np /= 2) {
    if (np > 1 && np / 2 >= pairs) continue;
    RXCfg c;
    c.xt.n0 = a.n;
    c.xt.n1 = n1;
    c.xt.n2 = n2;
    c.xt.np = np;
    c.xt.nbj = (pairs + np - 1) / np;
    c.xt.ls = r_line_slots(a.m) | 1;
    c.xt.fn0 = fdiv_make((uint32_t)a.n);
    c.xt.fnp = fdiv_make((uint32_t)np);
    const double blocks = (double)c.xt.nbj * n2;
    size(c);
    if (c.threads > r_max_threads<T>() || c.lds > kRLds || blocks > 2147483647.0) continue;
    c.blocks = c.xt.nbj * n2;
    // (where one block fills a CU's LDS anyway, the longer runs)
    if (best.blocks == 0 || c.lds <= 81920) best = c;
    if (c.lds <= 81920 && blocks >= 256) break;
  }
  return best;
}
}  // namespace

template <>
RXCfg RLaunch<T>::x_r2c(const RAxis& a, int n1, int n2) {
  return x_shape(a, n1, n2, [&](RXCfg& c) {
    c.threads = r_spread<T>(a, c.xt.np, r_threads<T>(a, c.xt.np, false),
                            (long long)c.xt.nbj * n2);
    // five blocks of 256 threads share a CU where two of 512 do (85 VGPRs): 400^3 FP32 in
    // 64-byte runs 257 us, 279 in 128-byte ones
    if (F32 && c.xt.np == kWide / 2 && c.threads > 256) c.threads = 1 << 20;  // no such shape
    const size_t lines = sizeof(cpx<T>) * (size_t)c.xt.np * c.xt.ls;
    c.lds = sizeof(cpx<T>) * (size_t)a.m + (lines < 256 ? 256 : lines);
    if (c.lds < kFoldedLds) c.lds = kFoldedLds;
  });
}

template <>
RXCfg RLaunch<T>::x_c2r(const RAxis& a, int n1, int n2) {
  auto with = [&](int rows, int most) {
    return x_shape(a, n1, n2, [&](RXCfg& c) {
      const int tl = 2 * c.xt.np;
      const int sweep = (tl * ((a.n + rows - 1) / rows) + 63) / 64 * 64;
      const int base = r_threads<T>(a, c.xt.np, false);
      int fft = r_spread<T>(a, c.xt.np, base, (long long)c.xt.nbj * n2);
      if (fft > most && base <= most) fft = most;
      c.xt.S = rows;
      c.xt.P = sweep / tl;
      c.threads = sweep > fft ? sweep : fft;
      if (c.threads > most || c.xt.P > kSweepMaxChunks) c.threads = 1 << 20;  // no such shape
      if (rows == 16 && c.xt.np == kWide / 2 && c.threads > 256) c.threads = 1 << 20;
      // the twiddles, then the factors; the lines; the waves' carries and gains; the sums
      const size_t nw = sweep / 64, pre = std::max((size_t)a.m, (size_t)c.xt.P * rows);
      c.lds = sizeof(cpx<T>) * (pre + (size_t)tl * c.xt.ls + 2 * nw * tl + nw) +
              7 * 16 * sizeof(double);
    });
  };
  // FP32 grids that fill the GPU sweep in chunks of 16 rows, 16 lines in a block of up to 256
  // threads or else 8, so that four or more blocks share a CU (a step of 400^3: 1524 us, 1541
  // with 16 lines in 512 threads; 390x90x90: 116.5 us, 130.1 with 8 rows); smaller ones in
  // shorter chains of 8 (101x75x63: 20.0 us against 21.6 for this pass), as long as the gain
  // tables hold that many (to 2048 rows; a step of 2200x512 with 16 rows 61 us, 112 with every
  // pass of gp_generic.hpp).  One-pair tiles keep 8 rows: 2048^2 118 us against 125 with 16,
  // 2000x2048 112 and 118 (of 3D grids 2000x60x50 174 against 168, 2048x100x100 522 against 552).
  const RXCfg c8 = with(8, r_max_threads<T>());
  if (F32) {
    const RXCfg c16 = with(16, 512);
    if ((c16.blocks >= 1024 && c16.xt.np > 1) || c8.blocks == 0) return c16;
  }
  return c8;
}

template <>
hipError_t RLaunch<T>::r2c(hipStream_t st, const RXCfg& c, const RAxis& a, const cpx<T>* psi,
                           cpx<T>* spec, const RProgram* p, double* part, const FoldedFin& fin) {
  if (c.blocks < 1) return hipErrorInvalidValue;
  if (a.maxr == kSmall)
    hipLaunchKernelGGL((k_rr2c<T, kSmall>), dim3(c.blocks + fin.lead), dim3(c.threads), c.lds, st,
                       psi, spec, c.xt, p, part, fin);
  else if (a.maxr == kRPrime)
    hipLaunchKernelGGL((k_rr2c<T, kRPrime>), dim3(c.blocks + fin.lead), dim3(c.threads), c.lds,
                       st, psi, spec, c.xt, p, part, fin);
  else
    hipLaunchKernelGGL((k_rr2c<T, kBig>), dim3(c.blocks + fin.lead), dim3(c.threads), c.lds, st,
                       psi, spec, c.xt, p, part, fin);
  return hipGetLastError();
}

template <>
hipError_t RLaunch<T>::c2r(hipStream_t st, const RXCfg& c, const RAxis& a, int mode,
                           const cpx<T>* spec, const RProgram* p, const RXArgs<T>& g) {
  if (c.blocks < 1) return hipErrorInvalidValue;
#define GP_C2R(R, MD, SV)                                                                    \
  hipLaunchKernelGGL((k_rc2r<T, R, MD, SV>), dim3(c.blocks), dim3(c.threads), c.lds, st, spec, \
                     c.xt, p, g)
#define GP_C2R_MODE(MD)                                            \
  case MD:                                                         \
    if (a.maxr == kRPrime && F32 && c.xt.S == 16) GP_C2R(kRPrime, MD, (F32 ? 16 : 8)); \
    else if (a.maxr == kRPrime) GP_C2R(kRPrime, MD, 8);            \
    else if (a.maxr != kSmall) GP_C2R(kBig, MD, 8);                \
    else if (F32 && c.xt.S == 16) GP_C2R(kSmall, MD, (F32 ? 16 : 8)); \
    else GP_C2R(kSmall, MD, 8);                                    \
    break;
  switch (mode) {
    GP_C2R_MODE(MODE_IMAG)
    GP_C2R_MODE(MODE_REAL)
    case MODE_OBSERVE:
      if (a.maxr == kRPrime) GP_C2R(kRPrime, MODE_OBSERVE, 8);
      else if (a.maxr != kSmall) GP_C2R(kBig, MODE_OBSERVE, 8);
      else GP_C2R(kSmall, MODE_OBSERVE, 8);
      break;
    default:
      return hipErrorInvalidValue;
  }
#undef GP_C2R_MODE
#undef GP_C2R
  return hipGetLastError();
}
#endif  // x passes
#endif  // GP_FAMILY < 2

}  // namespace gpdbec
