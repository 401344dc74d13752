// Register-resident time steps for gfx950: a wave holds 64 R consecutive nodes
// of a periodic instance in vector registers, lane l the nodes l R .. l R + R-1
// (all q populations), and advances `s_per` steps between exchanges.
//
// Streaming is the alternating (AA) pattern of the LDS kernels with registers
// for slots: an even step relaxes each node and swaps opposite populations in
// place; an odd step gathers from the neighbouring nodes' slots and scatters
// back to them.  Within a lane both are a renaming of registers; the sum_j
// |e_j| values that cross a lane edge move with wave-shift DPP moves, twice per
// odd step.  What crosses a wave edge is not moved at all: a wave carries
// `halo` = s_per max|e_j| extra nodes on each side, the exact region shrinks by
// max|e_j| nodes per step, and after s_per steps the waves of an instance
// publish the outer `halo` nodes of their cores in LDS, meet at one workgroup
// barrier and refill their halos (two strip buffers alternate, so one barrier
// suffices).  The per-node arithmetic is the Relaxer's, in its order: results
// are bitwise those of every other kernel.
//
// Bound: VALU issue.  Per KdV node update in FP64 the step loop issues 34
// arithmetic operations and 0.7 to 4 lane-edge moves (17 to 3 nodes per lane);
// the LDS-resident loop before it issued 37.7 and, with one 160 KB instance set
// per CU, kept VALU busy 0.54 of the time (LDS latency, one barrier per step).
// On one MI355X the loop alone reaches 1.0e12 node updates/s in FP64 (issue
// peak at 2.4 GHz: 1.1e12) and 8.5e11 in FP32 storage, whose ten conversions
// per node stay; with halos and exchanges 9.3e11 and 8.2e11 (8 to 17 nodes per
// lane).  Batches, LDS-resident before -> now: 4096 KdV/mKdV grids of 256..4096
// nodes 5.4e11 -> 8.3e11 (FP64) and 6.0e11 -> 6.8e11 (FP32 storage) node
// updates/s; 512 Kuramoto-Sivashinsky grids of 1024 nodes 8.1 -> 5.8 ms per 8000
// steps; one KdV grid of 800 nodes 0.53 -> 0.34 us per step.
#pragma once

#include <utility>

#include "kernels.hpp"

namespace lbm {

// Relaxation of R nodes held in registers, in place, with opposite populations
// swapped: f[r][opp(j)] = f*_j(r).  Same operations in the same order per node
// as Relaxer<Q, D, P, T, A>; nodes advance together a population pair at a
// time, so that a coefficient is read once for all of them.
template <int Q, int D, int P, typename T, typename A, bool Held>
struct RegRelaxer {
  static_assert(P < 2, "polynomial equilibria");
  static constexpr int K = reg_coefs(D, P);   // coefficients per population
  static constexpr bool kRest = (sizeof(T) == 4 && sizeof(A) == 8);
  // coefficients below the leading one: held in scalar registers for the whole
  // launch when they fit, in vector registers (Held) where a lane has few nodes,
  // else read from the constant cache at every step.  That read takes about 150
  // cycles per group of eight FP64 coefficients whatever the nodes, so that a
  // lone wave of one node per lane spent 2500 cycles on a degree-13 D1Q7 step of
  // 450 issue cycles.
  static constexpr bool kPin = reg_pinned(Q, D, P, (int)sizeof(A)) || Held;
  using CT = const __attribute__((address_space(4))) A*;
  CT c;
  A top[Q];
  A low[kPin ? Q : 1][kPin ? K - 1 : 1];
  A add[kRest && P == 1 ? Q : 1];
  A w0;
  double s0;

  __device__ __forceinline__ void init(const DevCoef* __restrict__ cf) {
    c = (CT)Relax<T, A>::coef(cf);
    const CT coef = c;
    w0 = *(CT)Relax<T, A>::w0p(cf);
    s0 = *(const __attribute__((address_space(4))) double*)&cf->s0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      top[j] = coef[j * kRow + K - 1];
      asm volatile("" : "+v"(top[j]));
    }
    if constexpr (kPin) {
#pragma unroll
      for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int d = 0; d < K - 1; ++d) {
          low[j][d] = coef[j * kRow + d];
#if defined(__HIP_DEVICE_COMPILE__)
          if constexpr (Held)
            asm volatile("" : "+v"(low[j][d]));
          else
            asm volatile("" : "+s"(low[j][d]));
#endif
        }
    }
    if constexpr (kRest && P == 1) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        add[j] = (A) * (const __attribute__((address_space(4))) double*)&cf->cst[j];
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+s"(add[j]));
#endif
      }
    }
  }
  __device__ __forceinline__ A finish(int j, A acc, A p, A f) const {
    if constexpr (P == 1) {
      if constexpr (kRest)
        acc = fma_a(acc, p, add[j]);
      else
        acc = fma_a(acc, p, (A)0);
    }
    return fma_a(w0, f, acc);
  }

  // the nodes R0 .. R0 + B - 1 of the R
  template <int R, int R0, int B>
  __device__ __forceinline__ void relax_nodes(T (&f)[R][Q]) const {
    A p[R], u[R];
#pragma unroll
    for (int r = R0; r < R0 + B; ++r) {
      double s = (double)f[r][0];
      if constexpr (kRest && P == 1) s = s0 + s;
#pragma unroll
      for (int j = 1; j < Q; ++j) s += (double)f[r][j];
      p[r] = (A)s;
      u[r] = P == 0 ? p[r] : p[r] * p[r];
    }
    // tables outside registers: a group of kGroup coefficients is loaded while
    // the one before is evaluated, and no earlier (two pointers the compiler
    // must treat as new after every other group), so that at most two are held
    CT pt[2] = {c, c};
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (!kPin) asm volatile("" : "+s"(pt[0]), "+s"(pt[1]) : "v"(p[R0 + B - 1]));
#endif
    int used = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int o = opposite<Q>(j);
      if (o < j) continue;
      A a[R], b[R];
      horner<R, R0, B>(j, a, u, pt, used);
      if (o != j) horner<R, R0, B>(o, b, u, pt, used);
#pragma unroll
      for (int r = R0; r < R0 + B; ++r) {
        const T x = (T)finish(j, a[r], p[r], (A)f[r][j]);
        if (o != j) {
          const T y = (T)finish(o, b[r], p[r], (A)f[r][o]);
          f[r][j] = y;
        }
        f[r][o] = x;
      }
    }
  }
  static constexpr int kGroup = 32 / (int)sizeof(A) * 2;
  template <int R, int R0, int B>
  __device__ __forceinline__ void horner(int j, A (&a)[R], const A (&u)[R], CT (&pt)[2], int& used) const {
#pragma unroll
    for (int r = R0; r < R0 + B; ++r) a[r] = top[j];
#pragma unroll
    for (int d = K - 2; d >= 0; --d, ++used) {
      const A cd = kPin ? low[kPin ? j : 0][kPin ? d : 0] : pt[(used / kGroup) & 1][j * kRow + d];
#pragma unroll
      for (int r = R0; r < R0 + B; ++r) a[r] = fma_a(a[r], u[r], cd);
#if defined(__HIP_DEVICE_COMPILE__)
      if constexpr (!kPin)
        if (used % kGroup == kGroup - 1) asm volatile("" : "+s"(pt[(used / kGroup) & 1]) : "v"(a[R0]));
#endif
    }
  }
  // all R nodes, B at a time
  template <int B, int R, int R0 = 0>
  __device__ __forceinline__ void relax_swap(T (&f)[R][Q]) const {
    constexpr int N = B < R - R0 ? B : R - R0;
    relax_nodes<R, R0, N>(f);
    if constexpr (R0 + N < R) {
      __builtin_amdgcn_sched_barrier(0);
      relax_swap<B, R, R0 + N>(f);
    }
  }
};

// value of lane l - 1 (up) or l + 1 (down), `By` lanes away; lanes beyond the
// wave read zero (their nodes are outside the exact region)
template <int Ctrl>
__device__ __forceinline__ int dpp_move(int v) {
  return __builtin_amdgcn_update_dpp(0, v, Ctrl, 0xf, 0xf, true);
}
template <int By>
__device__ __forceinline__ int lane_shift(int v) {
  if constexpr (By > 0)
    return lane_shift<By - 1>(dpp_move<0x138>(v));   // wave_shr:1
  else if constexpr (By < 0)
    return lane_shift<By + 1>(dpp_move<0x130>(v));   // wave_shl:1
  else
    return v;
}
template <int By>
__device__ __forceinline__ float lane_shift(float v) {
  return __int_as_float(lane_shift<By>(__float_as_int(v)));
}
template <int By>
__device__ __forceinline__ double lane_shift(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = lane_shift<By>((int)(unsigned)(b & 0xffffffffll));
  const int hi = lane_shift<By>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

constexpr int floor_div(int a, int b) { return a >= 0 ? a / b : -((b - 1 - a) / b); }

// n[r][j] = the value at node (lane R + r) - e_j, population opp(j): what node r
// reads in an odd step
template <int Q, int R, typename T>
__device__ __forceinline__ void reg_gather(const T (&f)[R][Q], T (&n)[R][Q]) {
  auto each = [&]<int r, int j>() {
    constexpr int at = r - velocity<Q>(j);
    constexpr int off = floor_div(at, R);   // lane offset of the source
    n[r][j] = lane_shift<-off>(f[at - off * R][opposite<Q>(j)]);
  };
  [&]<int... i>(std::integer_sequence<int, i...>) { (each.template operator()<i / Q, i % Q>(), ...); }
  (std::make_integer_sequence<int, R * Q>{});
}
// the inverse: n[r][j] goes to node (lane R + r) - e_j, population opp(j)
template <int Q, int R, typename T>
__device__ __forceinline__ void reg_scatter(const T (&n)[R][Q], T (&f)[R][Q]) {
  auto each = [&]<int r, int j>() {
    constexpr int at = r - velocity<Q>(j);
    constexpr int off = floor_div(at, R);
    f[at - off * R][opposite<Q>(j)] = lane_shift<off>(n[r][j]);
  };
  [&]<int... i>(std::integer_sequence<int, i...>) { (each.template operator()<i / Q, i % Q>(), ...); }
  (std::make_integer_sequence<int, R * Q>{});
}

template <int Q, int R, int B, typename T, typename X>
__device__ __forceinline__ void reg_even(T (&f)[R][Q], X& relax) {
  relax.template relax_swap<B>(f);
}
template <int Q, int R, int B, typename T, typename X>
__device__ __forceinline__ void reg_odd(T (&f)[R][Q], X& relax) {
  T n[R][Q];
  reg_gather<Q, R>(f, n);
  relax.template relax_swap<B>(n);
  reg_scatter<Q, R>(n, f);
}

// LDS stores of this wave's lanes come before the loads that follow by others of
// them: a wave's LDS operations complete in order, and the fence keeps the
// compiler from moving them across (it costs no instruction).
__device__ __forceinline__ void wave_lds_order() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#endif
}

template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_agent(const T* p) {
  return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the sign-free word that holds the exponent: not below infinity's for NaN and Inf
__device__ __forceinline__ unsigned exponent_word(float v) { return (unsigned)__float_as_int(v) & 0x7fffffffu; }
__device__ __forceinline__ unsigned exponent_word(double v) { return (unsigned)__double2hiint(v) & 0x7fffffffu; }

// What the segments of a slab launch share.
struct SegLinks {
  int sx;                    // steps between exchanges with the neighbours (a multiple of s_per)
  uint64_t* xbuf;            // strips: [segment][buffer][side][node of a lane][population][half][hg + 1 lanes]
  unsigned tag;              // block b's words carry tag + b
  int me;                    // this segment
  bool mute;                 // never publishes (test hook)
  long long wait_ticks;
};

// 32 bits of a value with the tag of their block, moved as one word: a strip word
// tells by itself whether it has arrived, so an exchange is one store on its way
// and one load that finds it -- no wait for stores before a flag, no flag before
// the loads (2.1 -> 1.2 us per exchange).
__device__ __forceinline__ uint64_t tagged(unsigned tag, unsigned bits) { return ((uint64_t)tag << 32) | bits; }
__device__ __forceinline__ unsigned value_bits(float v, int) { return (unsigned)__float_as_int(v); }
__device__ __forceinline__ unsigned value_bits(double v, int half) {
  return (unsigned)(half ? __double2hiint(v) : __double2loint(v));
}
__device__ __forceinline__ void value_of(float* v, const unsigned (&b)[1]) { *v = __int_as_float((int)b[0]); }
__device__ __forceinline__ void value_of(double* v, const unsigned (&b)[2]) { *v = __hiloint2double((int)b[1], (int)b[0]); }

// LDS elements of one wave: its exchange strips, or one row of its nodes on the
// way between memory order and lane order
constexpr int reg_lds(int q, int R, int hl) {
  const int strips = 4 * (hl + 1) * R * q;
  return strips > 64 * R ? strips : 64 * R;
}

// The value of lane l, the same in all lanes.
__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

// The reset of a bounded instance's outer layers after a step, by the wave that
// holds them (the first wave the left ones, the last the right ones), with the
// arithmetic of k_bound: f_j := f_eq_j(phi*), for kind 2 plus the
// non-equilibrium part of the first interior node.  The equilibria of four steps
// are computed ahead, lane c population c % Q of layer c / Q, and wait in LDS.
// The interior node's populations are read from their lanes, lane j evaluates
// its population's polynomial, and the differences are read back.  Odd: an odd
// number of steps is done, so f_j(x) lies at node x - e_j, population opp(j).
// The boundary waves' steps bound the instance, by latency: 0.60 us per step of
// 801 nodes with equilibrium layers, 0.69 with extrapolation, 0.40 without any;
// with the interior node's part exchanged through LDS it was 0.82, and 1.14 with
// the state in LDS.
template <int Q, int D, typename T>
struct RegBound {
  double* eq;            // [4 steps][layers][Q]
  double row[D + 1];     // of population lane % Q
  double rest;
  int layers, kind;
  bool comp;             // this lane computes
  bool near;             // this lane holds slots of the layers
  int inner;             // the first interior node, counted from the wave's first (uniform)
  int at;                // this lane's first node, relative to the first layer

  // the interior node's populations; its place in a lane is M
  template <bool Odd, int R, int M>
  __device__ __forceinline__ void populations(const T (&f)[R][Q], T (&g)[Q]) const {
    auto one = [&]<int j>() {
      constexpr int y = M - (Odd ? velocity<Q>(j) : 0);
      constexpr int off = floor_div(y, R);
      g[j] = lane_value(f[y - off * R][Odd ? opposite<Q>(j) : j], inner / R + off);
    };
    [&]<int... j>(std::integer_sequence<int, j...>) { (one.template operator()<j>(), ...); }
    (std::make_integer_sequence<int, Q>{});
  }
  template <bool Odd, int R, int U>
  __device__ __forceinline__ void reset(T (&f)[R][Q]) const {
    static_assert(R == 2, "a place for each parity");
    // (what decides for each slot is computed anew: held, it spilled registers;
    // slots outside the layers read whatever lies there)
    int b0 = at;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(b0));
#endif
    const double* p = eq + (near ? (U * layers + b0) * Q : 0);
    double v[R][Q];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int j = Odd ? opposite<Q>(k) : k;
        const int b = r + (Odd ? velocity<Q>(j) : 0);
        v[r][k] = p[b * Q + j];
      }
    double neq[Q] = {};
    if (kind == 2) {
      T g[Q];
      if (inner & 1)
        populations<Odd, R, 1>(f, g);
      else
        populations<Odd, R, 0>(f, g);
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < Q; ++k) s += (double)g[k];
      const double h = horner(s);
#pragma unroll
      for (int k = 0; k < Q; ++k) neq[k] = (double)g[k] - lane_value(h, k);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int j = Odd ? opposite<Q>(k) : k;
        const int b = b0 + r + (Odd ? velocity<Q>(j) : 0);
        const T x = (T)(v[r][k] + neq[j]);
        f[r][k] = (unsigned)b < (unsigned)layers ? x : f[r][k];
      }
  }
  __device__ __forceinline__ double horner(double p) const {
    double acc = row[D];
#pragma unroll
    for (int d = D - 1; d >= 0; --d) acc = __builtin_fma(acc, p, row[d]);
    return acc;
  }
};

// Advance of one segment by the waves that hold it.  `sg` is the segment, `w`
// this wave's number in it; waves without a segment (act false) only meet the
// barriers.
//  Ring: the whole instance; the outer halos of the first and last waves are
//   each other's.
//  Slab: part of an instance, one workgroup each, all of a launch resident
//   together.  A segment carries `extra` lanes more at each end, so that its
//   ends stay exact for `sx` steps; then its first and last waves publish the
//   outer owned lanes in global memory and refill their outer halos from their
//   neighbours', reading until every word carries the block's tag.  Words move
//   with device-scope relaxed atomics (coherent across the XCDs' L2 caches
//   without whole-cache write-back).  Strips alternate between two buffers by
//   block; a wave overwrites one only after it has the neighbour's next block,
//   which the neighbour publishes after it has read this one.  Tags grow from
//   launch to launch, so that nothing is cleared in between.  A wait that outlasts `wait_ticks` ticks of the constant-rate
//   wall clock marks the instance (status bit 2) and is the wave's last: it runs
//   on without waiting, so that every kernel ends.
//  Bounded: the whole instance, no ring; after every step the outer layers are
//   reset from the exact solution (RegBound::reset).
//  (A tile is a slab of at most `sx` steps, which meets no exchange with
//   neighbours.)
// State moves between memory order and lane order through a row of LDS per wave,
// so that both sides are coalesced.
// Bounded by VALU issue where the waves fill the SIMDs, by the exchange (1.2 us)
// and the latency of a lone wave's step where one instance is spread thin.
// Against the LDS-resident slabs and tiles (two to four workgroup barriers and Q
// LDS accesses per node and step): one 4096-node FP32 KS solve 4.03 -> 0.93 ms
// per 4000 steps, 128 x 8192 KS FP64 x 2000 4.46 -> 3.2 ms, 96 Kawahara FP64 of
// 2048..16384 nodes x 2000 10.8 -> 4.6 ms, a 3,000,017-node KdV grid x 64 0.65 ->
// 0.34 ms; one 800-node KdV grid, one workgroup before, 0.34 -> 0.25 us per step.
template <int Q, int R, int B, int Kind, int D, int P, typename T, typename A, bool Held>
__device__ __forceinline__ void reg_segment(T* __restrict__ L, int steps, int s_per, const DevSeg& sg, int w, bool act,
                                            const DevCoef* __restrict__ cf, int* __restrict__ status,
                                            const SegLinks& lk, [[maybe_unused]] int from) {
  constexpr int H = Q / 2;
  using GT = __attribute__((address_space(1))) T;   // global memory
  const int lane = threadIdx.x & 63;
  const int hl = (s_per * H + R - 1) / R;   // halo lanes at each end of a wave
  if (!act) {
    __syncthreads();
    for (int done = s_per; done < steps; done += s_per) __syncthreads();
    __syncthreads();
    return;
  }
  RegRelaxer<Q, D, P, T, A, Held> relax;
  relax.init(cf);
  const int W = sg.waves, n = sg.n;
  // lanes of nodes advanced by this wave, among the segment's `lanes`
  const int b0 = (int)((int64_t)w * sg.lanes / W), b1 = (int)((int64_t)(w + 1) * sg.lanes / W);
  const int cl = b1 - b0;
  constexpr bool ring = Kind == kSegRing;
  // strips: [buffer][side][(hl + 1) R nodes][Q] of each wave
  const int strip = (hl + 1) * R * Q, per_wave = reg_lds(Q, R, hl) + (Kind == kSegBound ? bound_lds((int)sizeof(T)) : 0);
  int pub = -1, ref = -1;
  {
    const int i = lane - hl;
    if (i >= 0 && i <= hl)
      pub = w * per_wave + i * R * Q;
    else if (i < cl && i >= cl - 1 - hl)
      pub = w * per_wave + strip + (i - (cl - 1 - hl)) * R * Q;
    if (lane < hl) {
      if (w > 0)
        ref = (w - 1) * per_wave + strip + (lane + 1) * R * Q;
      else if (ring)
        ref = (W - 1) * per_wave + strip + ((lane + 1) * R - sg.over) * Q;
    } else if (i >= cl && i < cl + hl) {
      if (w < W - 1)
        ref = (w + 1) * per_wave + (i - cl) * R * Q;
      else if (ring)
        ref = ((i - cl) * R + sg.over) * Q;
    }
  }
  T* S = L + sg.lds_off;
  T* row = S + w * per_wave;   // this wave's, for one row of its nodes
  T f[R][Q];
  const int first = (b0 - hl - sg.extra) * R;   // the wave's first node, relative to x0
  {
    const GT* g = (const GT*)(uintptr_t)sg.in;
    int base = (sg.x0 + first) % n;
    base += base < 0 ? n : 0;
    const bool once = n >= 64 * R;   // the wave's nodes pass the ring's end once at most
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      T v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        int x = base + r * 64 + lane;
        x = once ? x - (x >= n ? n : 0) : x % n;
        v[r] = g[(int64_t)j * sg.stride + x];
      }
#pragma unroll
      for (int r = 0; r < R; ++r) row[r * 64 + lane] = v[r];
      wave_lds_order();
#pragma unroll
      for (int r = 0; r < R; ++r) f[r][j] = row[lane * R + r];
      wave_lds_order();
    }
  }
  // in == out for rings: every wave has loaded before the first one stores
  // (calls of at most s_per steps meet no other barrier); and no wave publishes
  // into another's row
  wait_vector_memory();
  __syncthreads();
  // slab: this lane's part in the exchange with the neighbours (element offsets, -1 none)
  int gpub = -1, gref = -1, gshift = 0, kx = 0;
  bool ends = false, waits = true;
  [[maybe_unused]] int gstrip = 0, glanes = 0;
  [[maybe_unused]] unsigned tag = lk.tag, gbuf = 0;
  constexpr int Halves = (int)sizeof(T) / 4;
  if constexpr (Kind == kSegSlab) {
    const int hg = hl + sg.extra, owned = sg.lanes - 2 * sg.extra;
    const int o = b0 - hl + lane - sg.extra;   // among the owned lanes
    glanes = hg + 1;
    gstrip = glanes * R * Q * Halves;
    const bool left_end = w == 0, right_end = w == W - 1;
    ends = left_end || right_end;
    kx = lk.sx;
    const bool core = lane >= hl && lane < hl + cl;
    if (left_end && core && o >= 0 && o <= hg)
      gpub = lk.me * 4 * gstrip + o;
    else if (right_end && core && o < owned && o >= owned - 1 - hg)
      gpub = lk.me * 4 * gstrip + gstrip + o - (owned - 1 - hg);
    // the ring's end may lie inside a lane: the neighbour's nodes are `gshift` off
    if (left_end && o >= -hg && o < 0) {
      gshift = sg.over_left ? R - sg.over_left : 0;
      gref = sg.left * 4 * gstrip + gstrip + o + hg + 1 - (sg.over_left ? 1 : 0);
    } else if (right_end && o >= owned && o < owned + hg) {
      gshift = sg.over;
      gref = sg.right * 4 * gstrip + o - owned;
    }
    if (lk.mute) gpub = -1;
  }
  if constexpr (Kind == kSegBound) {
    // exchanges every four steps; the exact solution is loaded four steps ahead
    const bool right = w == W - 1, edge = w == 0 || right;   // (two waves or more)
    const int nl = sg.layers;
    RegBound<Q, D, T> bound;
    bound.eq = reinterpret_cast<double*>(S + w * per_wave + reg_lds(Q, R, hl));
    bound.rest = cf->phi_rest;
    bound.layers = nl;
    bound.kind = sg.kind;
    bound.comp = edge && lane < nl * Q;
    bound.inner = (right ? n - 1 - nl : nl) - first;
    bound.at = first + lane * R - (right ? n - nl : 0);
    bound.near = edge && bound.at + R - 1 + H >= 0 && bound.at - H < nl;
    const double* rows = (const double*)(uintptr_t)sg.rows + (right ? nl : 0) + (edge ? lane / Q : 0);
#pragma unroll
    for (int d = 0; d <= D; ++d) bound.row[d] = edge ? cf->init[lane % Q][d] : 0.0;
    double next[4] = {};
    if (bound.comp) {
#pragma unroll
      for (int u = 0; u < 4; ++u) next[u] = u < steps ? rows[(int64_t)(from + u) * 2 * nl] : 0.0;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    // the row has arrived: no step waits for it, and with it for the loads ahead
#pragma unroll
    for (int d = 0; d <= D; ++d) asm volatile("" : "+v"(bound.row[d]));
#endif
    int buf = 0;
    for (int left = steps, at = from + 4;; left -= 4, at += 4) {
      if (bound.comp) {
#pragma unroll
        for (int u = 0; u < 4; ++u) bound.eq[u * nl * Q + lane] = bound.horner(next[u] - bound.rest);
#pragma unroll
        for (int u = 0; u < 4; ++u) next[u] = 4 + u < left ? rows[(int64_t)(at + u) * 2 * nl] : 0.0;
      }
      wave_lds_order();
      reg_even<Q, R, B>(f, relax);
      if (edge) bound.template reset<true, R, 0>(f);
      if (left == 1) break;
      reg_odd<Q, R, B>(f, relax);
      if (edge) bound.template reset<false, R, 1>(f);
      if (left == 2) break;
      reg_even<Q, R, B>(f, relax);
      if (edge) bound.template reset<true, R, 2>(f);
      if (left == 3) break;
      reg_odd<Q, R, B>(f, relax);
      if (edge) bound.template reset<false, R, 3>(f);
      if (left <= 4) break;
      if (pub >= 0) {
        T* p = S + pub + buf;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < Q; ++j) p[r * Q + j] = f[r][j];
      }
      __syncthreads();
      if (ref >= 0) {
        const T* p = S + ref + buf;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < Q; ++j) f[r][j] = p[r * Q + j];
      }
      buf = 2 * strip - buf;
    }
  }
  int pairs = Kind == kSegBound ? 0 : steps >> 1, k = s_per >> 1, buf = 0;
  if (pairs > 0) do {
      reg_even<Q, R, B>(f, relax);
      reg_odd<Q, R, B>(f, relax);
      if (--k == 0 && (pairs > 1 || (steps & 1))) {   // more steps to come: exchange
        k = s_per >> 1;
        bool across = false;   // this exchange is with the neighbours too
        if constexpr (Kind == kSegSlab) {
          kx -= s_per;
          across = kx == 0;
          if (across) {
            kx = lk.sx;
            if (gpub >= 0) {
              uint64_t* p = lk.xbuf + gbuf + gpub;
#pragma unroll
              for (int r = 0; r < R; ++r)
#pragma unroll
                for (int j = 0; j < Q; ++j)
#pragma unroll
                  for (int h = 0; h < Halves; ++h)
                    store_agent(p + ((r * Q + j) * Halves + h) * glanes, tagged(tag, value_bits(f[r][j], h)));
            }
          }
        }
        if (pub >= 0) {
          T* p = S + pub + buf;
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < Q; ++j) p[r * Q + j] = f[r][j];
        }
        __syncthreads();
        if (ref >= 0) {
          const T* p = S + ref + buf;
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < Q; ++j) f[r][j] = p[r * Q + j];
        }
        buf = 2 * strip - buf;
        if constexpr (Kind == kSegSlab) {
          if (across) {
            if (ends) {
              // a few nodes of a lane at a time: twice their registers are in flight
              constexpr int C = sizeof(T) == 4 ? (R < 4 ? R : 4) : (R < 2 ? R : 2);
              const uint64_t* p = lk.xbuf + gbuf + gref;
              const long long t0 = wall_clock64();
#pragma unroll
              for (int c = 0; c < R; c += C) {
                bool here;
                do {
                  here = true;
                  if (gref >= 0) {
#pragma unroll
                    for (int r = c; r < c + C && r < R; ++r) {
                      const int at = r + gshift >= R ? (r + gshift - R) * Q * Halves * glanes + 1
                                                     : (r + gshift) * Q * Halves * glanes;
#pragma unroll
                      for (int j = 0; j < Q; ++j) {
                        unsigned b[Halves];
#pragma unroll
                        for (int h = 0; h < Halves; ++h) {
                          const uint64_t v = load_agent(p + at + (j * Halves + h) * glanes);
                          here &= (unsigned)(v >> 32) == tag;
                          b[h] = (unsigned)v;
                        }
                        value_of(&f[r][j], b);
                      }
                    }
                  }
                  here = __all(here);
                  if (!here && waits && wall_clock64() - t0 >= lk.wait_ticks) {
                    waits = false;
                    if (lane == 0) atomicOr(status + sg.inst, 2);
                  }
                } while (!here && waits);
              }
            }
            ++tag;
            gbuf = 2 * gstrip - gbuf;
          }
        }
      }
    } while (--pairs > 0);
  if (steps & 1) {   // the last step: relax, then stream to the natural layout
    T t[R][Q];
    if constexpr (Kind != kSegBound) reg_even<Q, R, B>(f, relax);
    reg_gather<Q, R>(f, t);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < Q; ++j) f[r][j] = t[r][j];
  }
  GT* out = (GT*)(uintptr_t)sg.out;
  // the largest exponent of the lane's owned nodes, as an unsigned word
  unsigned top = 0;
  const bool core = lane >= hl && lane < hl + cl;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int x = first + lane * R + r;
    const bool own = core && x >= 0 && x < sg.len;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const unsigned e = own ? exponent_word(f[r][j]) : 0u;
      top = top > e ? top : e;
    }
  }
  if (top >= exponent_word((T)__builtin_inf())) atomicOr(status + sg.inst, 1);
  __syncthreads();   // the strips have been read: rows may go over them
  const int lo = hl * R > -first ? hl * R : -first;   // owned nodes of the wave, in memory order
  const int hi = (hl + cl) * R < sg.len - first ? (hl + cl) * R : sg.len - first;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
#pragma unroll
    for (int r = 0; r < R; ++r) row[lane * R + r] = f[r][j];
    wave_lds_order();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int x = r * 64 + lane;
      const T v = row[x];
      if (x >= lo && x < hi) out[(int64_t)j * sg.stride + sg.x0 + first + x] = v;
    }
    wave_lds_order();
  }
}

// Nodes relaxed together: all of a lane's where each coefficient is loaded once
// for them; else few, since more would only hold more temporaries.
constexpr int reg_together(bool pin, int R) { return !pin ? R : R <= 3 ? R : R == 5 ? 3 : 2; }

// the width of this job
template <int Q, int Kind, int D, int P, typename T, typename A, bool Wide, int I>
__device__ __forceinline__ void reg_widths(int nodes, T* __restrict__ L, int steps, int s_per, const DevSeg& sg, int w,
                                           bool act, const DevCoef* __restrict__ cf, int* __restrict__ status,
                                           const SegLinks& lk, int from) {
  constexpr int R = Kind == kSegBound ? (I == 0 ? kBoundWidth : 0) : reg_width(Q, (int)sizeof(T), D, P, Wide, I);
  if constexpr (R > 0) {
    constexpr bool held = reg_held(Q, D, P, (int)sizeof(T), (int)sizeof(A), Wide, R);
    constexpr int B = reg_together(held || reg_pinned(Q, D, P, (int)sizeof(A)), R);
    if (nodes == R)
      reg_segment<Q, R, B, Kind, D, P, T, A, held>(L, steps, s_per, sg, w, act, cf, status, lk, from);
    else if constexpr (I + 1 < kRegWidths)
      reg_widths<Q, Kind, D, P, T, A, Wide, I + 1>(nodes, L, steps, s_per, sg, w, act, cf, status, lk, from);
  }
}

// One segment per workgroup: the slabs of co-resident workgroups (a launch no
// larger than the GPU holds at once), or, with `tile`, tiles: launch `launch` of
// an advance reads one state buffer and writes the other, `sx` steps each.
template <int Q, int D, int P, typename T, typename A, bool Wide>
__global__ __launch_bounds__(64 * reg_waves(Wide)) __attribute__((amdgpu_waves_per_eu(Wide ? 2 : 4))) void k_seg(
    const DevSeg* __restrict__ segs, int nodes, int s_per, int sx, int tile, int launch, uint64_t* xbuf,
    unsigned tag, const DevCoef* __restrict__ coefs, int* __restrict__ status, long long wait_ticks,
    int mute_seg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int me = blockIdx.x;
  DevSeg sg = segs[me];
  int steps = sg.steps;
  if (tile) {
    steps -= launch * sx;
    if (steps <= 0) return;
    if (steps > sx) steps = sx;
    if (launch & 1) {
      const uint64_t t = sg.in;
      sg.in = sg.out;
      sg.out = t;
    }
  }
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SegLinks lk{sx, xbuf, tag, me, me == mute_seg, wait_ticks};
  reg_widths<Q, kSegSlab, D, P, T, A, Wide, 0>(nodes, reinterpret_cast<T*>(smem_raw), steps, s_per, sg, w, w < sg.waves,
                                               coefs + sg.inst, status, lk, 0);
}

// Persistent kernel over the parts of jobs (a job: ring segments of one variant
// and one width, all the waves of a workgroup).  A workgroup takes the next item
// of the list until it is empty; the list holds part p of a job before part
// p + 1, so a part that waits for its predecessor (done[job]) waits for a
// workgroup that is running.  The wait is bounded: after `wait_ticks` ticks of
// the constant-rate wall clock the part marks its instances (status bit 4), is
// skipped and published, so that a scheduling fault ends the kernel.
// `stall_item` (-1 normally) names an item that is taken but never run nor
// published -- a test hook that makes the next part's wait give up.
template <int Q, int Kind, int D, int P, typename T, typename A, bool Wide>
__global__ __launch_bounds__(64 * reg_waves(Wide)) __attribute__((amdgpu_waves_per_eu(Wide ? 2 : 4))) void k_reg(
    const DevItem* __restrict__ items, int nitems, const DevJob* __restrict__ jobs, const DevSeg* __restrict__ segs,
    int* __restrict__ counter, int* __restrict__ done, const DevCoef* __restrict__ coefs, int* __restrict__ status,
    long long wait_ticks, int stall_item) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* L = reinterpret_cast<T*>(smem_raw);
  __shared__ int slot;   // the queue item, then whether a wait gave up
  const int tid = threadIdx.x;
  int pub_job = -1, pub_val = 0;
  for (;;) {
    if (tid == 0) {
      if (pub_job >= 0) __hip_atomic_store(done + pub_job, pub_val, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      slot = atomicAdd(counter, 1);
    }
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(slot);
    __syncthreads();
    if (item >= nitems) break;
    pub_job = -1;
    if (item == stall_item) continue;
    const DevItem it = items[item];
    const DevJob jb = jobs[it.job];
    if (it.steps > 0) {
      if (it.part > 0) {
        if (tid == 0) {
          const long long t0 = wall_clock64();
          int seen;
          while ((seen = __hip_atomic_load(done + it.job, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < it.part &&
                 wall_clock64() - t0 < wait_ticks)
            __builtin_amdgcn_s_sleep(8);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          slot = seen < it.part ? 1 : 0;
        }
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int gave_up = __builtin_amdgcn_readfirstlane(slot);
        if (gave_up) {
          if (tid < jb.count) atomicOr(status + segs[jb.first + tid].inst, 4);
          __syncthreads();
          if (it.more) {
            pub_job = it.job;
            pub_val = it.part + 1;
          }
          continue;
        }
      }
      // the segment of this wave
      const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      int mine = -1;
      for (int k = 0; k < jb.count; ++k)
        if (wave >= segs[jb.first + k].w0 && wave < segs[jb.first + k].w0 + segs[jb.first + k].waves) mine = k;
      mine = __builtin_amdgcn_readfirstlane(mine);
      const bool act = mine >= 0;
      DevSeg sg{};
      if (act) sg = segs[jb.first + mine];
      const DevCoef* cf = coefs + (act ? sg.inst : 0);
      const int w = wave - sg.w0;
      reg_widths<Q, Kind, D, P, T, A, Wide, 0>(jb.nodes, L, it.steps, jb.s_per, sg, w, act, cf, status, SegLinks{},
                                               it.from);
      __syncthreads();   // strips are read before the next item's are written
      if (it.more) {
        __threadfence();   // this thread's write-back is visible to every CU
        __syncthreads();
        pub_job = it.job;
        pub_val = it.part + 1;
      }
    }
  }
}

}  // namespace lbm
