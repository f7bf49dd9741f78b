// Multi-instance kernels for one precision (GP_REAL) that walk their work list with any
// number of blocks.  (Item-loop kernels: see thread_idx.)
#define GP_ITEM_LOOP_KERNELS
#include "gp_batch.hpp"
#include "gp_batch_launch.hpp"

#ifndef GP_REAL
#error "GP_REAL must be float or double"
#endif

namespace gpdbec {
using T = GP_REAL;

template <int CLS, int S>
static const void* kernel_of(int pass, int mode) {
  switch (pass) {
    case BP_R2C: return reinterpret_cast<const void*>(kb_r2c_x_loop<T, 0, CLS, S>);
    case BP_CONV: return reinterpret_cast<const void*>(kb_conv_y_loop<T, 0, CLS, S>);
    case BP_C2R:
      if (mode == MODE_IMAG) return reinterpret_cast<const void*>(kb_c2r_nl_cnx_loop<T, MODE_IMAG, CLS, S>);
      if (mode == MODE_REAL) return reinterpret_cast<const void*>(kb_c2r_nl_cnx_loop<T, MODE_REAL, CLS, S>);
      return reinterpret_cast<const void*>(kb_c2r_nl_cnx_loop<T, MODE_OBSERVE, CLS, S>);
    case BP_CN:
      if (mode == MODE_IMAG) return reinterpret_cast<const void*>(kb_cn_y_loop<T, MODE_IMAG, CLS, S>);
      return reinterpret_cast<const void*>(kb_cn_y_loop<T, MODE_REAL, CLS, S>);
    default: return nullptr;
  }
}

template <>
const void* batch_loop_kernel<T>(int pass, int mode, int cls, int shape) {
  if (cls == kBatchBoth)  // (c2r and CN of both classes take a block per item)
    return pass == BP_R2C ? reinterpret_cast<const void*>(kb_r2c_x_loop<T, 0, kBatchBoth, 0>)
                          : reinterpret_cast<const void*>(kb_conv_y_loop<T, 0, kBatchBoth, 0>);
  if (cls == 0) return shape == 0 ? kernel_of<0, 0>(pass, mode) : kernel_of<0, 1>(pass, mode);
  return shape == 0 ? kernel_of<1, 0>(pass, mode) : kernel_of<1, 1>(pass, mode);
}

}  // namespace gpdbec
