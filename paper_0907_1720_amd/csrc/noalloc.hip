// The fixed device scratch of lbm_advance_noalloc: one static array per GPU,
// sized for the tables of one problem and a state that fits one workgroup's
// LDS, so that the entry point allocates nothing.  Host code reaches the array
// only through the device address hipGetSymbolAddress returns for the current
// device (the array's name is a host-side stand-in, not a device address).
#include <mutex>

#include "kernels.hpp"

namespace lbm {

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

__global__ __launch_bounds__(64) void k_zero_ints(int* __restrict__ p, int n) {
  for (int i = threadIdx.x; i < n; i += 64) p[i] = 0;
}

// (one launch in place of three copies from pageable memory and a clear, each of
// which cost as much as a kernel or more: 6 to 8 us)
__global__ __launch_bounds__(256) void k_tables(NoAllocTables t, unsigned char* __restrict__ base, int later) {
  const int i = threadIdx.x;
  if (!later)
    for (int k = i; k < (int)(kNoAllocCoefBytes / 16); k += 256)
      reinterpret_cast<uint4*>(base)[k] = reinterpret_cast<const uint4*>(t.coef)[k];
  if (i == 0) *reinterpret_cast<DevJob*>(base + kNoAllocJobAt) = t.job;
  if (i == 64) *reinterpret_cast<DevItem*>(base + kNoAllocItemAt) = t.item;
  if (i == 128) *reinterpret_cast<DevSeg*>(base + kNoAllocSegAt) = t.seg;
  if (i >= 192 && i < 192 + (later ? 3 : 8)) reinterpret_cast<int*>(base + kNoAllocIntsAt)[i - 192] = 0;
}
}  // namespace

hipError_t launch_tables(const NoAllocTables& t, unsigned char* base, bool later, hipStream_t s) {
  static_assert(sizeof(NoAllocTables) <= 4000, "beyond the arguments of a launch");
  k_tables<<<1, 256, 0, s>>>(t, base, later ? 1 : 0);
  return hipGetLastError();
}

hipError_t noalloc_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_zero_ints(int* p, int n, hipStream_t s) {
  if (n < 0 || n > (1 << 20)) return hipErrorInvalidValue;
  k_zero_ints<<<1, 64, 0, s>>>(p, n);
  return hipGetLastError();
}

}  // namespace lbm
