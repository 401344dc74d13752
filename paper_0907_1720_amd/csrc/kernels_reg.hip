// The register-resident kernels of one lattice size and precision, LBM_Q = 4, 5,
// 6 or 7 and LBM_PREC = 0 (double, double), 1 (float, double) or 2 (float,
// float), both set by the build: they take most of the compile time, in twelve
// units.
#include "reg_body.hpp"
#include "kernels_table.hpp"

#if !defined(LBM_Q) || !defined(LBM_PREC)
#error "LBM_Q (the lattice size) and LBM_PREC (the precision) must be defined"
#endif
#if LBM_PREC == 0
#define LBM_TA double, double
#elif LBM_PREC == 1
#define LBM_TA float, double
#else
#define LBM_TA float, float
#endif

namespace lbm {

namespace {
// the kernel of bounded instances, where there is one
template <int D, int P, typename T, typename A>
const void* bound_fn() {
  if constexpr (bound_variant(LBM_Q, D, P, (int)sizeof(A)))
    return (const void*)k_reg<LBM_Q, kSegBound, D, P, T, A, false>;
  else
    return nullptr;
}
}  // namespace

template <>
const void* reg_kernel<LBM_Q, LBM_PREC>(int code, bool wide) {
  switch (code) {
#define LBM_CASE(DD, PP) \
  case DD | (PP << 8):   \
    return wide ? (const void*)k_reg<LBM_Q, kSegRing, DD, PP, LBM_TA, true>  \
                : (const void*)k_reg<LBM_Q, kSegRing, DD, PP, LBM_TA, false>;
    LBM_POLY_CASES
#undef LBM_CASE
#define LBM_CASE(DD, PP)           \
  case DD | (PP << 8) | (1 << 16): \
    return bound_fn<DD, PP, LBM_TA>();
    LBM_POLY_CASES
#undef LBM_CASE
  }
  return nullptr;
}

template <>
const void* seg_kernel<LBM_Q, LBM_PREC>(int code, bool wide) {
  switch (code) {
#define LBM_CASE(DD, PP) \
  case DD | (PP << 8):   \
    return wide ? (const void*)k_seg<LBM_Q, DD, PP, LBM_TA, true> : (const void*)k_seg<LBM_Q, DD, PP, LBM_TA, false>;
    LBM_POLY_CASES
#undef LBM_CASE
  }
  return nullptr;
}

}  // namespace lbm
