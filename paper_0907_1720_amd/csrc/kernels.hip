// Read-out kernels and the host launchers of every kernel; the lattice step
// itself is in kernels_body.hpp, instantiated per lattice size by
// kernels_q.hip (tables q_kernels_4 .. q_kernels_7).
//
//  k_read      phi = sum_j f_j  (FP64)
//  k_init_*    f := f_eq(phi)   (initial distribution)
//  k_sum       FP64 sum of phi over a grid, deterministic two-pass
#include <mutex>
#include <unordered_map>

#include "kernels.hpp"
#include "kernels_table.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// read-outs
// ---------------------------------------------------------------------------
// phi may lie in pinned host memory: the values cross to the host as they are
// summed, instead of a read-out buffer and three copies (55 -> 16 us per call
// of 1400 nodes).  With seq > 0 each workgroup that has finished stores words[2 +
// blockIdx] = seq, and the host watches those words: the stream's completion
// signal and its handling took longer than the kernel (a word that the last of
// counted workgroups stores cost another 0.9 of 10.5 us).  The barrier does not
// wait for other waves' stores that are still on their way, so there every value
// goes past the caches (a system-scope store), and every wave waits for its own
// before the barrier that the word's store follows (10.2 us per read of 1400
// nodes; 10.5 with a write-back of the whole cache before the word).  One
// workgroup alone writes only 4 GB/s across the link (8192 nodes: 18 us).
__device__ __forceinline__ void put_word(int* p, int v, bool watched) {
  if (watched)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  else
    *p = v;
}
template <typename T>
__global__ __launch_bounds__(256) void k_read(const T* __restrict__ f, double* __restrict__ phi, int n, int stride,
                                              int q, double phi_rest, const int* __restrict__ status,
                                              int* __restrict__ words, int seq,
                                              const int* __restrict__ bad) {
  const int x = blockIdx.x * 256 + threadIdx.x;
  if (bad && *bad) return;   // phi0 was refused: phi stays as it was
  const bool watched = seq > 0;
  if (x == 0) put_word(words, *status, watched);
  if (x < n) {
    double s = (double)f[x];
    for (int j = 1; j < q; ++j) s += (double)f[(int64_t)j * stride + x];
    s += phi_rest;
    if (watched)
      __hip_atomic_store(phi + x, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    else
      phi[x] = s;
    if (!__builtin_isfinite(s)) put_word(words + 1, 1, watched);   // (every writer stores the same word)
  }
  if (!watched) return;
  wait_vector_memory();
  __syncthreads();
  if (threadIdx.x == 0) put_word(words + 2 + blockIdx.x, seq, true);
}

// ---------------------------------------------------------------------------
// f := f_eq(phi) and the check of a phi that is already on the device
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void init_run(const DevInit& r, int x, const DevCoef* __restrict__ coefs,
                                         int* __restrict__ status) {
  if (x == 0 && r.first) status[r.inst] = 0;
  if (x >= r.len) return;
  const DevCoef* __restrict__ cf = coefs + r.inst;
  T* f = reinterpret_cast<T*>(r.dst);
  const double phi = reinterpret_cast<const double*>(r.src)[x];
  if (cf->gF > 0) {
    for (int j = 0; j < r.q; ++j) f[(int64_t)j * r.stride + x] = (T)general_stored_eq(cf, j, phi);
    return;
  }
  const double p = phi - cf->phi_rest;   // phi_rest = 0 for FP64 storage
  for (int j = 0; j < r.q; ++j) {
    const double* __restrict__ c = cf->init[j];
    double acc = c[r.degree];
    for (int d = r.degree - 1; d >= 0; --d) acc = __builtin_fma(acc, p, c[d]);
    f[(int64_t)j * r.stride + x] = (T)acc;
  }
}

// one launch for all instances of a batch, phi read from pinned host memory
// (one copy, one clear and one launch per instance before: 27 -> 3 us each)
template <typename T>
__global__ __launch_bounds__(256) void k_init_many(const DevInit* __restrict__ recs, const DevCoef* __restrict__ coefs,
                                                   int* __restrict__ status) {
  const DevInit r = recs[blockIdx.y];
  const int x0 = blockIdx.x * 256;
  if (x0 >= r.len) return;
  init_run<T>(r, x0 + threadIdx.x, coefs, status);
}
// `bad` (if given) is set where phi is not finite
template <typename T>
__global__ __launch_bounds__(256) void k_init_one(DevInit r, const DevCoef* __restrict__ coefs,
                                                  int* __restrict__ status, int* __restrict__ bad) {
  const int x = blockIdx.x * 256 + threadIdx.x;
  if (bad && x < r.len && !__builtin_isfinite(reinterpret_cast<const double*>(r.src)[x])) *bad = 1;
  init_run<T>(r, x, coefs, status);
}

__global__ __launch_bounds__(256) void k_check_phi(const double* __restrict__ phi, int n, int* __restrict__ words) {
  bool bad = false, neg = false;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double v = phi[i];
    bad |= !__builtin_isfinite(v);
    neg |= v < 0;
  }
  // (plain stores: every writer of a word stores the same value)
  if (bad) words[0] = 1;
  if (neg) words[1] = 1;
}

__global__ __launch_bounds__(256) void k_sum_partial(const double* __restrict__ v, int n,
                                                     double* __restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) s += v[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
namespace {
const QKernels* table(int q) {
  switch (q) {
    case 4: return &q_kernels_4;
    case 5: return &q_kernels_5;
    case 6: return &q_kernels_6;
    case 7: return &q_kernels_7;
  }
  return nullptr;
}

const void* resident_kernel(int q, int prec, int code) {
  const QKernels* t = table(q);
  return t ? t->resident_fn(prec, code) : nullptr;
}

template <int Q>
const void* reg_or_seg(bool seg, int prec, int code, bool wide) {
  if (prec == 0) return seg ? seg_kernel<Q, 0>(code, wide) : reg_kernel<Q, 0>(code, wide);
  if (prec == 1) return seg ? seg_kernel<Q, 1>(code, wide) : reg_kernel<Q, 1>(code, wide);
  return seg ? seg_kernel<Q, 2>(code, wide) : reg_kernel<Q, 2>(code, wide);
}
const void* reg_or_seg(bool seg, int q, int prec, int code, bool wide) {
  if (q == 4) return reg_or_seg<4>(seg, prec, code, wide);
  if (q == 5) return reg_or_seg<5>(seg, prec, code, wide);
  if (q == 6) return reg_or_seg<6>(seg, prec, code, wide);
  return q == 7 ? reg_or_seg<7>(seg, prec, code, wide) : nullptr;
}

const void* tile_kernel(int q, int prec) {
  const QKernels* t = table(q);
  return t ? t->tile_fn(prec) : nullptr;
}

const void* slab_kernel(int q, int prec, int code) {
  const QKernels* t = table(q);
  return t ? t->slab_fn(prec, code) : nullptr;
}
}  // namespace

hipError_t launch_init_many(bool f32, const DevInit* recs, int count, int longest, const DevCoef* coefs, int* status,
                            hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > 65535) return hipErrorInvalidValue;
  const dim3 grid((longest + 255) / 256, count);
  if (f32)
    k_init_many<float><<<grid, 256, 0, s>>>(recs, coefs, status);
  else
    k_init_many<double><<<grid, 256, 0, s>>>(recs, coefs, status);
  return hipGetLastError();
}

hipError_t launch_init_one(bool f32, const DevInit& rec, const DevCoef* coefs, int* status, int* bad, hipStream_t s) {
  const dim3 grid((rec.len + 255) / 256);
  if (f32)
    k_init_one<float><<<grid, 256, 0, s>>>(rec, coefs, status, bad);
  else
    k_init_one<double><<<grid, 256, 0, s>>>(rec, coefs, status, bad);
  return hipGetLastError();
}

hipError_t launch_check_phi(const double* phi, int n, int* words, hipStream_t s) {
  const int blocks = (n + 255) / 256;
  k_check_phi<<<blocks < 1024 ? blocks : 1024, 256, 0, s>>>(phi, n, words);
  return hipGetLastError();
}

hipError_t launch_bound(int q, int D, int prec, void* f, int n, int stride, int layers, int kind,
                        const double* phib, const DevCoef* cf, hipStream_t s) {
  if (layers < 1 || 2 * layers > 64) return hipErrorInvalidValue;
  const QKernels* t = table(q);
  return t ? t->bound(D, prec, f, n, stride, layers, kind, phib, cf, s) : hipErrorInvalidValue;
}

hipError_t launch_stream(int q, int D, int prec, const void* fin, void* fout, int n, int stride,
                         const DevCoef* cf, hipStream_t s) {
  // D carries the variant code (degree | parity << 8)
  const QKernels* t = table(q);
  return t ? t->stream(D, prec, fin, fout, n, stride, cf, s) : hipErrorInvalidValue;
}

const void* stream_kernel(int q, int code, int prec) {
  const QKernels* t = table(q);
  return t ? t->stream_fn(prec, code) : nullptr;
}

hipError_t launch_resident(int q, int prec, int code, const DevJob* jobs, const DevJobInst* jinst, int njobs,
                           int nchunks, int* counter, int* slots, int* done, const DevCoef* coefs, int* status,
                           long long wait_ticks, int stall_item, int grid, int block, size_t lds, hipStream_t s) {
  const void* fn = resident_kernel(q, prec, code);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  void* args[] = {(void*)&jobs,  (void*)&jinst, (void*)&njobs, (void*)&nchunks,    (void*)&counter,  (void*)&slots,
                  (void*)&done,  (void*)&coefs, (void*)&status, (void*)&wait_ticks, (void*)&stall_item};
  return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, s);
}

hipError_t launch_reg(int q, int prec, int code, bool wide, const DevItem* items, int nitems, const DevJob* jobs,
                      const DevSeg* segs, int* counter, int* done, const DevCoef* coefs, int* status,
                      long long wait_ticks, int stall_item, int grid, int block, size_t lds, hipStream_t s) {
  const void* fn = reg_or_seg(false, q, prec, code, wide);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  void* args[] = {(void*)&items, (void*)&nitems, (void*)&jobs,   (void*)&segs,       (void*)&counter,
                  (void*)&done,  (void*)&coefs,  (void*)&status, (void*)&wait_ticks, (void*)&stall_item};
  return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, s);
}

hipError_t reg_occupancy(int q, int prec, int code, bool wide, int block, size_t lds, int* blocks_per_cu) {
  const void* fn = reg_or_seg(false, q, prec, code, wide);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, block, lds);
}

hipError_t launch_seg(int q, int prec, int code, bool wide, const DevSeg* segs, int nsegs, int nodes, int s_per, int sx,
                      bool tile, int launch, void* xbuf, unsigned tag, const DevCoef* coefs, int* status,
                      long long wait_ticks, int mute_seg, int block, size_t lds, hipStream_t s) {
  const void* fn = reg_or_seg(true, q, prec, code, wide);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int as_tile = tile ? 1 : 0;
  void* args[] = {(void*)&segs, (void*)&nodes, (void*)&s_per, (void*)&sx,     (void*)&as_tile,    (void*)&launch,
                  (void*)&xbuf, (void*)&tag,   (void*)&coefs, (void*)&status, (void*)&wait_ticks, (void*)&mute_seg};
  return hipLaunchKernel(fn, dim3(nsegs), dim3(block), args, lds, s);
}

hipError_t seg_occupancy(int q, int prec, int code, bool wide, int block, size_t lds, int* blocks_per_cu) {
  const void* fn = reg_or_seg(true, q, prec, code, wide);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, block, lds);
}

namespace {
// kernel attributes, queried once per kernel (the planner asks per instance)
bool kernel_attributes(const void* fn, hipFuncAttributes* out) {
  static std::mutex mu;
  static std::unordered_map<const void*, hipFuncAttributes> cache;
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(fn);
  if (it == cache.end()) {
    hipFuncAttributes a;
    if (hipFuncGetAttributes(&a, fn) != hipSuccess) return false;
    it = cache.emplace(fn, a).first;
  }
  *out = it->second;
  return true;
}
}  // namespace

int resident_vgprs(int q, int prec, int code) {
  hipFuncAttributes a;
  const void* fn = resident_kernel(q, prec, code);
  if (!fn || !kernel_attributes(fn, &a) || a.numRegs <= 0) return 128;
  return a.numRegs;
}

size_t resident_static_lds(int q, int prec, int code) {
  hipFuncAttributes a;
  const void* fn = resident_kernel(q, prec, code);
  if (!fn) return 0;
  if (!kernel_attributes(fn, &a)) return 1024;
  return a.sharedSizeBytes;
}

hipError_t launch_tile(int q, int prec, const DevTile* tiles, int ntiles, const DevTileInst* tinsts, void* buf0,
                       void* buf1, int launch, int s_per, int halo, const DevCoef* coefs, int* status, int block,
                       size_t lds, hipStream_t s) {
  const void* fn = tile_kernel(q, prec);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  void* args[] = {(void*)&tiles, (void*)&tinsts, (void*)&buf0, (void*)&buf1, (void*)&launch, (void*)&s_per,
                  (void*)&halo,  (void*)&coefs,  (void*)&status};
  return hipLaunchKernel(fn, dim3(ntiles), dim3(block), args, lds, s);
}

hipError_t launch_slab(int q, int prec, int code, const DevSlab* slabs, int nslabs, const DevTileInst* tinsts, void* buf0,
                       void* buf1, int s_per, int halo, void* xbuf, int* flags, const DevCoef* coefs, int* status,
                       long long wait_ticks, int mute_slab, int block, size_t lds, hipStream_t s) {
  const void* fn = slab_kernel(q, prec, code);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  void* args[] = {(void*)&slabs, (void*)&tinsts, (void*)&buf0,  (void*)&buf1,   (void*)&s_per,
                  (void*)&halo,  (void*)&xbuf,   (void*)&flags, (void*)&coefs,  (void*)&status,
                  (void*)&wait_ticks, (void*)&mute_slab};
  return hipLaunchKernel(fn, dim3(nslabs), dim3(block), args, lds, s);
}

hipError_t slab_occupancy(int q, int prec, int code, int block, size_t lds, int* blocks_per_cu) {
  const void* fn = slab_kernel(q, prec, code);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, block, lds);
}

hipError_t resident_occupancy(int q, int prec, int code, int block, size_t lds, int* blocks_per_cu) {
  const void* fn = resident_kernel(q, prec, code);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, block, lds);
}

hipError_t launch_read(bool f32, const void* f, double* phi, int n, int stride, int q, double phi_rest,
                       const int* status, int* words, int seq, const int* bad, hipStream_t s) {
  const dim3 grid((n + 255) / 256);
  if (f32)
    k_read<float><<<grid, 256, 0, s>>>((const float*)f, phi, n, stride, q, phi_rest, status, words, seq, bad);
  else
    k_read<double><<<grid, 256, 0, s>>>((const double*)f, phi, n, stride, q, phi_rest, status, words, seq, bad);
  return hipGetLastError();
}

hipError_t launch_sum(const double* v, int n, double* part, int nparts, hipStream_t s) {
  k_sum_partial<<<nparts, 256, 0, s>>>(v, n, part);
  return hipGetLastError();
}

}  // namespace lbm
