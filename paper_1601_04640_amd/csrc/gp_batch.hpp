// Batched ensemble of independent quasi-2D instances (XY or XZ planes) of uneven sizes:
// one launch per pass covers every instance.  Each launch takes a work list of (instance,
// tile) items sorted by decreasing cost: one block per item, or fewer persistent blocks
// that walk it.  The per-instance descriptor points into that instance's own workspace
// region, laid out like a single-grid context, so the tile bodies are the single-grid
// ones.
#pragma once
#include "gp_kernels.hpp"

// Line lengths the batched kernels are specialised for (every axis of every instance);
// the kernel switches below list the same sizes.
#define GP_BATCH_SIZES(X) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(384) X(512)

namespace gpdbec {

// Tile-shape variants per pass and size class (Tiles<T, N, S>), chosen by the autotuner.
constexpr int kBatchShapes = 2;

// Per-instance descriptor.  Arrays are byte offsets from the batch workspace base, which
// the kernels receive as an argument: pointers formed from a kernel argument keep the
// global address space (pointers loaded from memory would fall back to flat accesses with
// 64-bit per-lane addresses).
template <typename T>
struct BDesc {
  size_t psi, V, spec, ktab, tw0, tw1;
  size_t cn0[2];  // x-axis factor tables: [imaginary, real time]
  size_t cn1[2];  // second-axis factor tables
  size_t p_x, p_nl, p_col, scale;
  StepScalars sc;  // step scalars (dt, couplings, spacings)
  int n0, n1;
  FinArgs fa;      // FP64 finalisation of this instance
};

template <typename X>
__device__ __forceinline__ X* bptr(char* base, size_t off) {
  return reinterpret_cast<X*>(base + off);
}

struct WorkItem {
  int inst;
  int tile;
};

enum : int { BP_R2C = 0, BP_CONV = 1, BP_C2R = 2, BP_CN = 3, BP_COUNT = 4 };

// Size classes (<= 256 and 384/512), each with its own work list and kernels: persistent
// blocks over all nine sizes spill, and tile shapes are chosen per class.
#define GP_BATCH_CLASS0(X) X(32) X(48) X(64) X(96) X(128) X(192) X(256)
#define GP_BATCH_CLASS1(X) X(384) X(512)
constexpr int kBatchClasses = 2;
constexpr int kBatchBoth = 2;  // both classes' lists in one launch (shape 0)
__host__ __device__ constexpr int batch_class(int n) { return n > 256 ? 1 : 0; }

// Dynamic LDS: the largest body of the pass and class present is requested at launch.
//
// What bounds these kernels is how many waves a SIMD holds while each tile's load, LDS
// transform and store wait on each other, so registers decide.  c2r and CN take one block
// per work item by default (GP_ITEM_LOOP_KERNELS not defined): nothing stays alive across
// items, the class-1 c2r takes 147 instead of 200 VGPRs, the class-1 CN 140 instead of 201
// (three waves per SIMD instead of two), the class-0 CN 101 instead of 134.  r2c and conv
// walk items blockIdx.x + k gridDim.x with any number of blocks, as the others do when
// gp_batch_set_blocks asks for fewer blocks than items; by default each block has one item,
// so that dispatch balances the load.
//
// Class kBatchBoth covers both classes' lists in one launch, the longer lines first: their
// bodies need about the same registers (c2r 134 and 147) and each pass has one drained tail
// instead of two.  192 FP32 instances of 96^2 to 512^2 points (13.7 M) step in 0.230 ms,
// with 1024 persistent blocks per class and pass in 0.317 (60 instances 0.093 and 0.133, 16
// 0.053 and 0.091; 90 FP64 ones 0.271 and 0.300).
#define GP_CLASS_BODY(AXIS, BODY)                                                      \
  if constexpr (CLS == 0) {                                                            \
    switch (d.AXIS) { GP_BATCH_CLASS0(BODY) default: break; }                          \
  } else if constexpr (CLS == 1) {                                                     \
    switch (d.AXIS) { GP_BATCH_CLASS1(BODY) default: break; }                          \
  } else {                                                                             \
    switch (d.AXIS) { GP_BATCH_CLASS1(BODY) GP_BATCH_CLASS0(BODY) default: break; }    \
  }
// r2c is held to three waves per SIMD in FP32 (168 VGPRs) and two in FP64 (256, four
// spilled: 90 instances 0.271 ms a step, 0.294 with one).
template <typename T>
constexpr int r2c_waves() { return sizeof(T) == 4 ? 3 : 2; }
#ifdef GP_ITEM_LOOP_KERNELS
#define GP_BATCH_KERNEL(NAME, AXIS, BODY, WPE)                                         \
  template <typename T, int MODE, int CLS, int S>                                      \
  __global__ __launch_bounds__(kThreads, WPE) void NAME##_loop(                        \
      char* __restrict__ base, const BDesc<T>* __restrict__ D,                         \
      const WorkItem* __restrict__ work1, int n1, const WorkItem* __restrict__ work0,  \
      int nwork) {                                                                     \
    extern __shared__ __attribute__((aligned(16))) char lds[];                         \
    constexpr int K = (MODE == MODE_REAL) ? 1 : 0;                                     \
    (void)K;                                                                           \
    for (int w = blockIdx.x; w < nwork; w += gridDim.x) {                              \
      const WorkItem item = w < n1 ? work1[w] : work0[w - n1];                         \
      const BDesc<T>& d = D[item.inst];                                                \
      GP_CLASS_BODY(AXIS, BODY)                                                        \
      __syncthreads();                                                                 \
    }                                                                                  \
  }
#else
// Block b takes work1[b], or work0[b - n1] from n1 on.
#define GP_BATCH_KERNEL(NAME, AXIS, BODY, WPE)                                         \
  template <typename T, int MODE, int CLS, int S>                                      \
  __global__ __launch_bounds__(kThreads, WPE) void NAME(                               \
      char* __restrict__ base, const BDesc<T>* __restrict__ D,                         \
      const WorkItem* __restrict__ work1, int n1, const WorkItem* __restrict__ work0) { \
    extern __shared__ __attribute__((aligned(16))) char lds[];                         \
    constexpr int K = (MODE == MODE_REAL) ? 1 : 0;                                     \
    (void)K;                                                                           \
    const int b = blockIdx.x;                                                          \
    const WorkItem item = b < n1 ? work1[b] : work0[b - n1];                           \
    const BDesc<T>& d = D[item.inst];                                                  \
    GP_CLASS_BODY(AXIS, BODY)                                                          \
  }
#endif

#define GP_BODY_R2C(N)                                                                  \
  case N:                                                                               \
    r2c_x_body<T, N, S>(bptr<cpx<T>>(base, d.psi), bptr<cpx<T>>(base, d.spec),           \
                     bptr<cpx<T>>(base, d.tw0), bptr<double>(base, d.p_x), d.n1, 1,      \
                     item.tile, lds);                                                     \
    break;
#define GP_BODY_CONV(N)                                                                 \
  case N:                                                                               \
    conv_line_body<T, N, S>(bptr<cpx<T>>(base, d.spec), bptr<T>(base, d.ktab),           \
                         bptr<double>(base, d.scale), bptr<cpx<T>>(base, d.tw1),         \
                         d.n0 / 2 + 1, item.tile, lds);                                  \
    break;
#define GP_BODY_C2R(N)                                                                  \
  case N:                                                                               \
    c2r_nl_cnx_body<T, N, MODE, S>(bptr<cpx<T>>(base, d.psi), bptr<T>(base, d.V),        \
                                bptr<double>(base, d.scale), bptr<cpx<T>>(base, d.spec), \
                                bptr<cpx<T>>(base, d.tw0), bptr<cpx<T>>(base, d.cn0[K]), \
                                d.sc, bptr<double>(base, d.p_nl), nullptr, d.n1, 1,      \
                                item.tile, lds);                                         \
    break;
#define GP_BODY_CN(N)                                                                   \
  case N:                                                                               \
    cn_col_body<T, N, MODE, true, S>(bptr<cpx<T>>(base, d.psi), bptr<cpx<T>>(base, d.cn1[K]), \
                                  bptr<double>(base, d.p_col), d.n0, (size_t)d.n0,        \
                                  (size_t)d.n0 * d.n1, item.tile, lds);                   \
    break;
GP_BATCH_KERNEL(kb_r2c_x, n0, GP_BODY_R2C, r2c_waves<T>())
GP_BATCH_KERNEL(kb_conv_y, n1, GP_BODY_CONV, 1)
GP_BATCH_KERNEL(kb_c2r_nl_cnx, n0, GP_BODY_C2R, 1)
GP_BATCH_KERNEL(kb_cn_y, n1, GP_BODY_CN, 1)
#undef GP_BODY_R2C
#undef GP_BODY_CONV
#undef GP_BODY_C2R
#undef GP_BODY_CN
#undef GP_BATCH_KERNEL
#undef GP_CLASS_BODY

#ifndef GP_ITEM_LOOP_KERNELS
// One block per instance.
template <typename T>
__global__ __launch_bounds__(kThreads) void kb_finalize(const BDesc<T>* __restrict__ D,
                                                        int mode) {
  finalize_block(D[blockIdx.x].fa, mode);
}
#endif

}  // namespace gpdbec
