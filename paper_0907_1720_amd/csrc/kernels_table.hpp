// Launch entry points of the kernels of one lattice size, one table per
// lattice (kernels_q.hip, built once for each q in 4..7).
#pragma once

#include "device.hpp"

namespace lbm {

struct QKernels {
  hipError_t (*bound)(int D, int prec, void* f, int n, int stride, int layers, int kind, const double* phib,
                      const DevCoef* cf, hipStream_t s);
  hipError_t (*stream)(int code, int prec, const void* fin, void* fout, int n, int stride, const DevCoef* cf,
                       hipStream_t s);
  const void* (*stream_fn)(int prec, int code);
  const void* (*resident_fn)(int prec, int code);
  const void* (*tile_fn)(int prec);
  const void* (*slab_fn)(int prec, int code);
};

// host-side tables (not const: a const table would also be emitted for the
// device, where its host function pointers do not exist)
extern QKernels q_kernels_4, q_kernels_5, q_kernels_6, q_kernels_7;

// register-resident kernels (kernels_reg.hip, built for each q and precision);
// nullptr for variants without one
template <int Q, int PREC>
const void* reg_kernel(int code, bool wide);
template <int Q, int PREC>
const void* seg_kernel(int code, bool wide);
#define LBM_REG_DECL(Q, PREC)                                   \
  template <>                                                   \
  const void* reg_kernel<Q, PREC>(int code, bool wide);         \
  template <>                                                   \
  const void* seg_kernel<Q, PREC>(int code, bool wide);
LBM_REG_DECL(4, 0) LBM_REG_DECL(4, 1) LBM_REG_DECL(4, 2)
LBM_REG_DECL(5, 0) LBM_REG_DECL(5, 1) LBM_REG_DECL(5, 2)
LBM_REG_DECL(6, 0) LBM_REG_DECL(6, 1) LBM_REG_DECL(6, 2)
LBM_REG_DECL(7, 0) LBM_REG_DECL(7, 1) LBM_REG_DECL(7, 2)
#undef LBM_REG_DECL

}  // namespace lbm
