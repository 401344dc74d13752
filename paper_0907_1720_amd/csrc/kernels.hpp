// Launchers of the HIP kernels (defined in kernels.hip; the kernels are in
// kernels_body.hpp, one instantiation per lattice size in kernels_q.hip).  All
// take device pointers.
#pragma once

#include <cstddef>

#include "device.hpp"

// Kernel variants of the relaxation polynomial: (padded degree D, parity P).
// Dense (P = 0): D1Q5 KdV/KS/K(2,2) 5, cubic Pi 13, quartic Pi_1 up to 13;
// D1Q7 Kawahara 7, cubic Pi 13, quartic Pi_1 19.  Odd (P = 1): mKdV 9.  Power
// sums with real exponents (P = 2): degree 2, 5, 7 or 11 of each class's
// polynomial in phi^step (its strided layout); P = 3: the same for exactly the
// classes phi^0 and phi^(1/2), degree 2 or 5.
#define LBM_POLY_CASES \
  LBM_CASE(5, 0)       \
  LBM_CASE(7, 0)       \
  LBM_CASE(9, 0)       \
  LBM_CASE(13, 0)      \
  LBM_CASE(19, 0)      \
  LBM_CASE(5, 1)       \
  LBM_CASE(9, 1)       \
  LBM_CASE(13, 1)      \
  LBM_CASE(19, 1)
#define LBM_POWER_CASES \
  LBM_CASE(2, 2)        \
  LBM_CASE(5, 2)        \
  LBM_CASE(7, 2)        \
  LBM_CASE(11, 2)       \
  LBM_CASE(2, 3)        \
  LBM_CASE(5, 3)
#define LBM_VARIANT_CASES LBM_POLY_CASES LBM_POWER_CASES

// dense degrees available to the boundary kernel
#define LBM_INIT_CASES \
  LBM_CASE(5)          \
  LBM_CASE(7)          \
  LBM_CASE(9)          \
  LBM_CASE(13)         \
  LBM_CASE(19)

namespace lbm {

// smallest kernel degree >= D of the given parity (0 if none); parity 2 =
// power sums with real exponents
inline int padded_degree(int D, int parity) {
  const int dense[] = {5, 7, 9, 13, 19};
  const int odd[] = {5, 9, 13, 19};
  const int power_sum[] = {2, 5, 7, 11};
  const int half_powers[] = {2, 5};
  if (parity == 0) {
    for (int v : dense)
      if (v >= D) return v;
  } else if (parity == 2) {
    for (int v : power_sum)
      if (v >= D) return v;
  } else if (parity == 3) {
    for (int v : half_powers)
      if (v >= D) return v;
  } else {
    for (int v : odd)
      if (v >= D) return v;
  }
  return 0;
}
inline int variant_code(int D, int parity) { return D | (parity << 8); }

// prec: 0 = FP64 storage and arithmetic; 1 = FP32 deviation storage, FP64
// relaxation; 2 = FP32 deviation storage, FP32 relaxation.
// f := f_eq(phi) for `count` runs of nodes (records in device or pinned host
// memory, all of one storage), the longest of `longest` nodes; or for one run,
// by value
hipError_t launch_init_many(bool f32, const DevInit* recs, int count, int longest, const DevCoef* coefs, int* status,
                            hipStream_t s);
hipError_t launch_init_one(bool f32, const DevInit& rec, const DevCoef* coefs, int* status, int* bad, hipStream_t s);
// words[0] := 1 if any phi is not finite, words[1] := 1 if any is negative (two
// words in device or pinned host memory, left alone otherwise)
hipError_t launch_check_phi(const double* phi, int n, int* words, hipStream_t s);
// slabs: one launch no larger than the GPU holds at once, one workgroup per
// slab; flags[0 .. nslabs) start at 0; xbuf holds 4 Q halo values per slab;
// a halo wait gives up after wait_ticks ticks of the wall clock (status bit
// 2); slab mute_slab (-1: none) never raises its flag (test hook)
hipError_t launch_slab(int q, int prec, int code, const DevSlab* slabs, int nslabs, const DevTileInst* tinsts,
                       void* buf0, void* buf1, int s_per, int halo, void* xbuf, int* flags, const DevCoef* coefs,
                       int* status, long long wait_ticks, int mute_slab, int block, size_t lds, hipStream_t s);
hipError_t slab_occupancy(int q, int prec, int code, int block, size_t lds, int* blocks_per_cu);
// bounded domains: reset `layers` (1..32) nodes at each end from phib[0 .. 2 layers)
// (kind 1 equilibrium, 2 non-equilibrium extrapolation); D = init degree
hipError_t launch_bound(int q, int D, int prec, void* f, int n, int stride, int layers, int kind,
                        const double* phib, const DevCoef* cf, hipStream_t s);
// `code` = variant_code(D, parity) of the relaxation polynomial
hipError_t launch_stream(int q, int code, int prec, const void* fin, void* fout, int n, int stride,
                         const DevCoef* cf, hipStream_t s);
// the fused collide+stream kernel of variant `code` (arguments: const T* fin,
// T* fout, int n, int stride, const DevCoef* cf; 256 threads per block), for
// graph nodes; nullptr for an unknown variant
const void* stream_kernel(int q, int code, int prec);
// persistent launch over `njobs` jobs (bin-packed instances of one variant
// `code`), each split into `nchunks` step chunks; done[0..njobs) starts at 0.
// code | (1 << 16) selects the kernel of bounded jobs (boundary layers reset
// in LDS after every step).  A chunk's wait for its predecessor gives up after
// wait_ticks ticks of the wall clock (status bit 4); queue item stall_item
// (-1: none) is taken but never run (test hook)
hipError_t launch_resident(int q, int prec, int code, const DevJob* jobs, const DevJobInst* jinst, int njobs,
                           int nchunks, int* counter, int* slots, int* done, const DevCoef* coefs, int* status,
                           long long wait_ticks, int stall_item, int grid, int block, size_t lds, hipStream_t s);
// Register-resident kernels (polynomial variants, parity < 2): nodes per lane.
// The narrow kernels fit 128 registers (four waves per SIMD), the wide ones 256
// (two); the i-th width of either, 0 past the last.  (Multiples of four on D1Q4
// and D1Q5 cost the narrow kernels a register move for every sixth operation;
// large tables, which few problems use, are built for fewer widths; without three
// nodes per lane 512 D1Q7 grids of 1000 nodes with cubic fluxes, FP32 arithmetic,
// took 1.2 times the LDS kernels' time.)
constexpr int kRegWidths = 6;
constexpr int reg_width(int q, int elem, int degree, int parity, bool wide, int i) {
  constexpr int w[8][2][kRegWidths] = {{{1, 2, 3, 5, 6}, {5, 8, 10, 12, 14, 17}},   // D1Q4 / D1Q5, FP64
                                       {{2, 3, 4}, {1, 2, 3, 4, 6, 8}},             // D1Q6 / D1Q7, FP64
                                       {{1, 2, 3, 5, 8}, {5, 8, 10, 12, 14, 17}},   // D1Q4 / D1Q5, FP32 storage
                                       {{2, 3, 6}, {1, 3, 6, 8, 10, 12}},           // D1Q6 / D1Q7, FP32 storage
                                       {{3, 6}, {1, 6, 10, 17}},                    // the same, large tables
                                       {{2, 3, 4}, {1, 4, 8}},
                                       {{3, 6}, {1, 6, 10, 17}},
                                       {{2, 3, 4}, {1, 4, 8, 12}}};
  const bool large = parity == 0 ? degree >= 9 : degree >= 13;
  return w[(large ? 4 : 0) + (elem == 8 ? 0 : 2) + (q >= 6 ? 1 : 0)][wide ? 1 : 0][i];
}
// coefficients per population; whether those below the leading one fit the scalar
// registers; or else, with few nodes per lane, the vector registers of a wide kernel
constexpr int reg_coefs(int degree, int parity) { return parity == 0 ? degree + 1 : (degree + 1) / 2; }
constexpr bool reg_pinned(int q, int degree, int parity, int arith) {
  return q * (reg_coefs(degree, parity) - 1) * arith / 4 <= 52;
}
constexpr bool reg_held(int q, int degree, int parity, int elem, int arith, bool wide, int R) {
  return wide && R <= 2 && !reg_pinned(q, degree, parity, arith) &&
         q * (reg_coefs(degree, parity) * arith + R * (elem + arith)) / 4 <= 224;
}
// Bounded instances: two nodes per lane and four steps between exchanges, with
// tables in scalar registers; the lanes that compute the layers are one wave's.
constexpr int kBoundWidth = 2, kBoundSteps = 4;
constexpr int kBoundValues = 32;                     // layers x populations of an end, at most
// LDS elements of a wave besides its strips (slots outside the layers read up to
// seven places beyond the last)
constexpr int bound_lds(int elem) { return (4 * kBoundValues + 64) * 8 / elem; }
constexpr bool bound_variant(int q, int degree, int parity, int arith) {
  return q <= 5 && parity < 2 && reg_pinned(q, degree, parity, arith);
}
constexpr int reg_waves(bool wide) { return wide ? 8 : 16; }   // most waves of a workgroup: a CU's
inline bool reg_variant(int code) { return ((code >> 8) & 0xff) < 2; }
// persistent launch over `nitems` parts of jobs of ring segments; done[job] and
// the counter start at 0; waits and stall_item as launch_resident
hipError_t launch_reg(int q, int prec, int code, bool wide, const DevItem* items, int nitems, const DevJob* jobs,
                      const DevSeg* segs, int* counter, int* done, const DevCoef* coefs, int* status,
                      long long wait_ticks, int stall_item, int grid, int block, size_t lds, hipStream_t s);
hipError_t reg_occupancy(int q, int prec, int code, bool wide, int block, size_t lds, int* blocks_per_cu);
// one segment per workgroup (polynomial variants): slabs of one launch, or tiles
// (`launch`-th block of sx steps); xbuf holds 4 (hg + 1) R q words per
// segment for each 32 bits of a value, none of them tagged `tag` or above;
// segment mute_seg (-1: none) never publishes
hipError_t launch_seg(int q, int prec, int code, bool wide, const DevSeg* segs, int nsegs, int nodes, int s_per, int sx,
                      bool tile, int launch, void* xbuf, unsigned tag, const DevCoef* coefs, int* status,
                      long long wait_ticks, int mute_seg, int block, size_t lds, hipStream_t s);
hipError_t seg_occupancy(int q, int prec, int code, bool wide, int block, size_t lds, int* blocks_per_cu);
// VGPRs per thread of the resident kernel of variant `code`
int resident_vgprs(int q, int prec, int code);
// static LDS bytes of the resident kernel (0 by construction)
size_t resident_static_lds(int q, int prec, int code);
// phi = sum_j f_j into device or pinned host memory; words[0] := *status,
// words[1] := 1 if any value is not finite (left alone otherwise).  With
// seq > 0, at most 256 kReadWords nodes: words[2 + k] := seq at system scope once
// the k-th 256 values are there.  Nothing is written where *bad (if given) is set.
constexpr int kReadWords = 60;
hipError_t launch_read(bool f32, const void* f, double* phi, int n, int stride, int q, double phi_rest,
                       const int* status, int* words, int seq, const int* bad, hipStream_t s);
hipError_t launch_sum(const double* v, int n, double* part, int nparts, hipStream_t s);
hipError_t resident_occupancy(int q, int prec, int code, int block, size_t lds, int* blocks_per_cu);
// lbm_advance_noalloc: the fixed per-device scratch (tables at offset 0, the
// state from kNoAllocTableBytes on) and its device address on the current
// device (looked up once per device); a fill kernel that zeroes n ints
constexpr size_t kNoAllocTableBytes = size_t(16) << 10;
constexpr size_t kNoAllocStateBytes = size_t(256) << 10;
constexpr size_t kNoAllocScratchBytes = kNoAllocTableBytes + kNoAllocStateBytes;
hipError_t noalloc_scratch(void** out);
hipError_t launch_zero_ints(int* p, int n, hipStream_t s);
// The tables of a register-resident call, carried to the scratch `base` by the
// kernel's own arguments: the polynomial part of DevCoef, one job of one segment,
// and words that start at zero.  `later`: the next launch of the same call (job,
// item and the first three words only).
constexpr size_t kNoAllocCoefBytes = (offsetof(DevCoef, groots) + 15) / 16 * 16;
constexpr size_t kNoAllocJobAt = 12288, kNoAllocItemAt = kNoAllocJobAt + 128, kNoAllocSegAt = kNoAllocJobAt + 256,
                 kNoAllocIntsAt = kNoAllocJobAt + 512;
struct alignas(16) NoAllocTables {
  unsigned char coef[kNoAllocCoefBytes];
  DevJob job;
  DevItem item;
  DevSeg seg;
};
hipError_t launch_tables(const NoAllocTables& t, unsigned char* base, bool later, hipStream_t s);
// temporal blocking: launch `launch` of an advance, s_per steps per launch
hipError_t launch_tile(int q, int prec, const DevTile* tiles, int ntiles, const DevTileInst* tinsts, void* buf0,
                       void* buf1, int launch, int s_per, int halo, const DevCoef* coefs, int* status, int block,
                       size_t lds, hipStream_t s);

}  // namespace lbm
