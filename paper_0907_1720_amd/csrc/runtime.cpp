// C-ABI runtime: problem and batch handles, device memory, the planner that
// chooses between the LDS-resident, slab, temporal-blocking and HBM streaming
// kernels, bounded advances, the server, the autotuner and the read-outs.
// Host code only; the kernels live in kernels_body.hpp (instantiated per
// lattice by kernels_q.hip) and their launchers in kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <new>
#include <vector>

#include "coeffs.hpp"
#include "kernels.hpp"
#include "wave.hpp"
#include "lbmhpde.h"

using namespace lbm;

#define LBM_HIP(call)                                \
  do {                                               \
    hipError_t e_ = (call);                          \
    if (e_ != hipSuccess) return LBM_ERR_DEVICE;     \
  } while (0)

namespace {

constexpr int kBlock = 256;
constexpr int kMaxSlabs = 2048;       // workgroups of one slab launch
constexpr int kUnevenNodes = 256;     // smallest power-sum grid split where its group is uneven
constexpr int kSplitNodes = 1024;     // smallest power-sum grid split into slabs when the GPU is mostly idle
constexpr int kMaxResidentGrid = 256 * 8;
constexpr int kMaxResident = 64;      // LDS-resident launches per advance pass (one per lattice, precision, variant)
constexpr int kAuxStreams = 16;       // concurrent lanes (resident launches, tiled groups, slab launches)
constexpr uint64_t kMagic = 0x4c424d4850444531ull;   // "LBMHPDE1"

struct HostInst {
  lbm_desc desc;
  Model mdl;
  int q = 5;
  int D = 5;        // variant code of the relaxation polynomial (padded degree | parity << 8)
  int Dinit = 5;    // padded dense degree of the initialisation polynomial
  int n = 0;
  int stride = 0;
  bool f32 = false;  // FP32 deviation storage
  int prec = 0;      // lbm_precision
  int64_t off = 0;  // element offset in its precision's state arrays
  int cur = 0;      // which of the two state buffers is current
  int64_t steps_done = 0;
};

// A block of kStepBlock fused collide+stream launches of one instance as a
// HIP graph (the streaming path is launch bound for small grids): replayed
// whole, it advances the instance kStepBlock steps and, kStepBlock being even,
// leaves its state in the buffer it started from.
constexpr int kStepBlock = 64;
struct StepGraph {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  const void* fin = nullptr;    // what the graph was built for
  const void* fout = nullptr;
  const void* cf = nullptr;
  int n = 0, stride = 0, code = -1, q = 0, prec = -1;
};

void release_graph(StepGraph* g) {
  if (g->exec) hipGraphExecDestroy(g->exec);
  if (g->graph) hipGraphDestroy(g->graph);
  *g = StepGraph{};
}

struct DeviceLimits {
  int cus = 0;
  size_t lds_max = 0;
  double wall_ticks_per_us = 100.0;   // constant-rate device clock (wall_clock64)
  bool ok = false;
};

DeviceLimits query_limits() {
  DeviceLimits L;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return L;
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return L;
  L.cus = v;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return L;
  L.lds_max = (size_t)v;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeWallClockRate, dev) == hipSuccess && v > 0)
    L.wall_ticks_per_us = v / 1000.0;   // kHz
  L.ok = true;
  return L;
}

// Slab workgroups of all batches of this process on one GPU.  A slab launch ends
// only if all its workgroups get a place; two launches that each hold places the
// other waits for would not.  So the launches in flight together never count more
// workgroups than the GPU has CUs: a workgroup that waits for a place then has an
// empty CU, or one whose kernel waits for no slab.  A launch that would exceed
// that waits, on the device, for the other batches' before it.
//
// The places are those of an XCD's 32 CUs: a launch hands its workgroups to the
// XCDs in turn, whether they have room or not, and begins at any of them (of 108
// and 148 workgroups side by side that take a CU each, three had to wait).
constexpr int kXcdCus = 32;
int xcd_count(int cus) { return std::max(1, cus / kXcdCus); }
// a launch's workgroups, as many to each XCD as to the one that gets the most
int64_t even_places(int64_t workgroups, int cus) {
  const int x = xcd_count(cus);
  return (workgroups + x - 1) / x * x;
}
//
// That kernel may be another batch's whole instances for many steps, while part of
// a slab launch has its places and waits: the gate also knows how many, so that the
// slabs' waits are given as much longer (passes beyond kLongPass; a shorter one
// takes less than a second, and leaves its CUs to slabs when it ends).
constexpr int64_t kLongPass = 1 << 15;
struct SlabGate {
  struct Flight {
    const lbm_batch_s* owner;
    hipEvent_t done;
    int need;          // workgroups (even_places), 0 once seen over
    int64_t ahead;     // steps of whole instances, 0 once seen over
  };
  std::mutex mu;
  std::vector<Flight> flight;   // one per batch that has launched slabs or a long pass
};
SlabGate& slab_gate() {
  static SlabGate gates[64];
  int dev = 0;
  (void)hipGetDevice(&dev);
  return gates[dev & 63];
}

struct PlanMemo;

}  // namespace

struct lbm_batch_s {
  hipStream_t stream = nullptr;
  std::vector<HostInst> inst;
  DeviceLimits lim;
  int path = 0;
  // state: two buffers per precision (current / other for the streaming path)
  double* f64[2] = {nullptr, nullptr};
  float* f32[2] = {nullptr, nullptr};
  size_t n64 = 0, n32 = 0;            // elements per buffer
  bool own_state = true;
  void* arena[2] = {nullptr, nullptr};  // serving: both state buffers carved from two arenas
  DevCoef* coefs = nullptr;
  int* status = nullptr;              // per instance: 1 = non-finite seen
  int* slots = nullptr;               // per-workgroup queue slot of the resident kernel
  // The tables of a pass (queue words that start at zero, jobs, segments, slabs,
  // tiles ...), laid out anew for each and uploaded in one copy: two slots of
  // tables_cap bytes, used in turn, and their pinned mirror.
  unsigned char* tables = nullptr;
  unsigned char* tables_host = nullptr;
  size_t tables_cap = 0;
  std::vector<DevJobInst> hitems;     // of the pass being planned
  std::vector<DevJob> hjobs;
  std::vector<DevSeg> hsegs;
  SlabGate* gate = nullptr;           // entered with gate_done
  hipEvent_t gate_done = nullptr;
  std::shared_ptr<PlanMemo> memo;
  hipEvent_t items_done[2] = {nullptr, nullptr};
  int slot = 0;
  double* scratch = nullptr;          // phi read-out of grids beyond the stage; partial sums
  size_t scratch_elems = 0;
  // Pinned host memory that kernels read phi0 from and write phi to: kStageHead
  // bytes of status words, then data.  Every call that uses it synchronises the
  // stream before it returns.
  unsigned char* stage = nullptr;
  int read_seq = 0;                   // read-outs watched so far
  size_t stage_bytes = 0;             // data bytes
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  // halo strips of register slabs: words tagged below strip_tag (0: never written)
  uint64_t* strips = nullptr;
  size_t strips_cap = 0;
  uint32_t strip_tag = 1;
  void* xbuf = nullptr;               // halo strips of the slab path
  size_t xbuf_bytes = 0;
  int* sflags = nullptr;              // per-slab block flags
  int sflags_cap = 0;
  int tile_steps = 0;                 // steps per tiled launch (0 = automatic)
  int tile_wgs = 0;                   // tiled workgroups per CU the LDS budget is split for (0 = automatic)
  int res_grid = 0;                   // cap on the resident grid (0 = automatic)
  int res_chunks = 0;                 // step chunks per resident job (0 = automatic)
  int lanes = 0;                      // streams a pass spreads its launches over (0 = automatic)
  hipStream_t aux[kAuxStreams] = {};
  hipEvent_t fork = nullptr;
  hipEvent_t join[kAuxStreams] = {};
  float last_ms = 0.0f;
  std::vector<StepGraph> step_graphs;   // per instance and current-buffer parity
  double* bound = nullptr;              // boundary values of bounded problems (device)
  size_t bound_cap = 0;                 // doubles
  // a bounded advance in progress: phi* rows per instance (device address, 0
  // for periodic instances) and the layers reset at each end
  bool bnd_active = false;
  int bnd_layers = 0;
  std::vector<uint64_t> bnd_ptr;
  // bounded device waits (test hook lbm_batch_test_stall): limit in us (0 =
  // automatic) and the wait to force to give up (0 none, 1 resident, 2 slab)
  int64_t test_wait_us = 0;
  int test_stall = 0;
};

struct lbm_problem_s {
  lbm_batch_s* b = nullptr;
};

namespace {

void fill_devcoef(const HostInst& h, DevCoef* c) {
  std::memset(c, 0, sizeof(*c));
  const Model& m = h.mdl;
  const int parity = h.D >> 8;
  c->w0 = m.w0;
  c->w0f = (float)m.w0;
  if (m.gF > 0) {
    // power sums: omega * G and G per class; FP32 deviations relax in phi
    // = phi_rest + sum_j g_j and add -omega f_rest
    c->gF = m.gF;
    c->groots = 1;
    for (int cl = 1; cl < m.gF; ++cl)
      if (m.gnu[cl] != 0.5 && m.gnu[cl] != 0.25 && m.gnu[cl] != 0.75) c->groots = 0;
    for (int cl = 0; cl < m.gF; ++cl) {
      c->gnu[cl] = m.gnu[cl];
      c->gd0[cl] = m.gd0[cl];
      c->gstep[cl] = m.gstep[cl];
      for (int j = 0; j < m.q; ++j) {
        for (int d = 0; d <= kGDeg && d < kGRow; ++d) c->ginit[cl][j][d] = m.gG[cl][j][d];
        for (int i = 0; i < m.gK[cl] && i < kGRow; ++i) c->gwc[cl][j][i] = m.gwG[cl][j][m.gd0[cl] + m.gstep[cl] * i];
      }
    }
    if (h.f32) {
      c->phi_rest = m.phi_rest;
      c->s0 = m.phi_rest;
      for (int j = 0; j < m.q; ++j) {
        c->cst[j] = -m.wfrest[j];
        c->grest[j] = m.f_rest[j];
      }
    }
    return;
  }
  // FP64 relaxation table: omega * G over the kept degrees
  for (int j = 0; j < m.q; ++j) {
    if (parity == 0) {
      for (int d = 0; d <= m.D; ++d) c->wc[j][d] = m.wG[j][d];
    } else {
      for (int d = 1, k = 0; d <= m.D; d += 2, ++k) c->wc[j][k] = m.wG[j][d];
    }
  }
  if (h.f32) {
    c->phi_rest = m.phi_rest;
    for (int j = 0; j < m.q; ++j) {
      for (int d = 0; d <= m.D; ++d) {
        c->init[j][d] = m.H[j][d];
        c->wHf[j][d] = (float)m.wH[j][d];
      }
    }
    if (h.prec == LBM_F32_DEV) {
      // odd tables: Horner in phi = phi_rest + delta, then -omega f_rest;
      // dense tables: omega * H, the Taylor shift to the rest state, in delta
      // itself (no cancellation against f_rest, one add less per node)
      c->s0 = m.phi_rest;
      for (int j = 0; j < m.q; ++j) {
        c->cst[j] = -m.wfrest[j];
        if (parity == 0)
          for (int d = 0; d <= m.D; ++d) c->wc[j][d] = m.wH[j][d];
      }
    }
  } else {
    for (int j = 0; j < m.q; ++j)
      for (int d = 0; d <= m.D; ++d) c->init[j][d] = m.G[j][d];
  }
}

size_t elem_size(const HostInst& h) { return h.f32 ? sizeof(float) : sizeof(double); }

void destroy_batch(lbm_batch_s* b) {
  if (!b) return;
  hipStreamSynchronize(b->stream);
  if (b->gate) {
    std::lock_guard<std::mutex> hold(b->gate->mu);
    auto& fl = b->gate->flight;
    fl.erase(std::find_if(fl.begin(), fl.end(), [&](const SlabGate::Flight& f) { return f.owner == b; }));
    hipEventDestroy(b->gate_done);
  }
  if (b->arena[0]) {
    hipFree(b->arena[0]);
    hipFree(b->arena[1]);
  } else {
    if (b->own_state) {
      hipFree(b->f64[0]);
      hipFree(b->f32[0]);
    }
    hipFree(b->f64[1]);
    hipFree(b->f32[1]);
  }
  hipFree(b->coefs);
  hipFree(b->status);
  hipFree(b->slots);
  for (StepGraph& g : b->step_graphs) release_graph(&g);
  hipFree(b->bound);
  hipFree(b->tables);
  if (b->tables_host) hipHostFree(b->tables_host);
  for (int k = 0; k < 2; ++k)
    if (b->items_done[k]) hipEventDestroy(b->items_done[k]);
  hipFree(b->scratch);
  if (b->stage) hipHostFree(b->stage);
  hipFree(b->strips);
  hipFree(b->xbuf);
  hipFree(b->sflags);
  if (b->ev0) hipEventDestroy(b->ev0);
  if (b->ev1) hipEventDestroy(b->ev1);
  for (int k = 0; k < kAuxStreams; ++k) {
    if (b->aux[k]) hipStreamDestroy(b->aux[k]);
    if (b->join[k]) hipEventDestroy(b->join[k]);
  }
  if (b->fork) hipEventDestroy(b->fork);
  delete b;
}

lbm_status prepare_one(const lbm_desc& d, HostInst* hp) {
  HostInst& h = *hp;
  h = HostInst();
  h.desc = d;
  lbm_status s = build_model(d, &h.mdl);
  if (s != LBM_OK) return s;
  h.q = h.mdl.q;
  h.prec = d.prec;
  h.f32 = h.prec != LBM_F64;
  // odd equilibria (every degree with a nonzero coefficient is odd) evaluate in phi^2;
  // the FP32 relaxation uses the shifted (dense) table
  bool odd = h.prec != LBM_F32_DEV_ARITH32 && h.mdl.gF == 0;
  for (int j = 0; j < h.mdl.q && odd; ++j)
    for (int p = 0; p <= h.mdl.D; p += 2)
      if (h.mdl.G[j][p] != 0.0) odd = false;
  int parity = h.mdl.gF > 0 ? 2 : (odd ? 1 : 0);
  int kmax = 1;   // power sums: the longest strided class
  for (int c = 0; c < h.mdl.gF; ++c) kmax = std::max(kmax, h.mdl.gK[c]);
  int kd = padded_degree(h.mdl.gF > 0 ? kmax - 1 : h.mdl.D, parity);
  // exactly the classes phi^0 and phi^(1/2): the specialised variant, if its degree fits
  if (parity == 2 && h.mdl.gF == 2 && h.mdl.gnu[1] == 0.5 && padded_degree(kmax - 1, 3) > 0) {
    parity = 3;
    kd = padded_degree(kmax - 1, 3);
  }
  // power sums initialise through their own tables; any init variant serves
  h.Dinit = h.mdl.gF > 0 ? padded_degree(1, 0) : padded_degree(h.mdl.D, 0);
  if (kd == 0 || h.Dinit == 0) return LBM_ERR_UNSUPPORTED;
  h.D = variant_code(kd, parity);
  h.n = (int)d.n;
  h.stride = (int)lbm_row_stride(d.n);
  return LBM_OK;
}

lbm_status prepare_instances(const lbm_desc* descs, int count, std::vector<HostInst>* out) {
  out->resize(count);
  for (int i = 0; i < count; ++i) {
    lbm_status s = prepare_one(descs[i], &(*out)[i]);
    if (s != LBM_OK) return s;
  }
  return LBM_OK;
}

constexpr int kReadWatchUs = 60;
constexpr size_t kStageHead = 256, kStageLeast = size_t(16) << 10, kStageMost = size_t(8) << 20;
// stage bytes of `len` nodes of an instance (phi, its record, its coefficients)
size_t stage_need(int64_t len, bool coefs) {
  return (size_t)len * sizeof(double) + sizeof(DevInit) + (coefs ? sizeof(DevCoef) : 0) + 64;
}

lbm_status alloc_tables(lbm_batch_s* b, size_t maxn, size_t stage_want);

// (each allocation of pinned memory takes about 40 us)
lbm_status alloc_pass_tables(lbm_batch_s* b, size_t cap) {
  cap = (cap + 255) / 256 * 256;
  if (b->tables_cap) {
    LBM_HIP(hipStreamSynchronize(b->stream));   // earlier passes must be done with them
    hipFree(b->tables);
    hipHostFree(b->tables_host);
    b->tables = b->tables_host = nullptr;
    b->tables_cap = 0;
  }
  if (hipMalloc(&b->tables, 2 * cap) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
  if (hipHostMalloc((void**)&b->tables_host, 2 * cap, hipHostMallocDefault) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
  b->tables_cap = cap;
  return LBM_OK;
}

lbm_status alloc_batch(lbm_batch_s* b, void* dev_buf, size_t buf_bytes) {
  size_t n64 = 0, n32 = 0, maxn = 0, stage = 0;
  for (HostInst& h : b->inst) {
    stage += stage_need(h.n, h.f32);
    size_t e = (size_t)h.q * h.stride;
    if (h.f32) {
      h.off = (int64_t)n32;
      n32 += e;
    } else {
      h.off = (int64_t)n64;
      n64 += e;
    }
    maxn = std::max(maxn, (size_t)h.n);
  }
  b->n64 = n64;
  b->n32 = n32;
  if (dev_buf) {
    // caller-owned memory holds the current state buffer of the single problem
    size_t need = n64 * sizeof(double) + n32 * sizeof(float);
    if (buf_bytes < need) return LBM_ERR_OUT_OF_MEMORY;
    b->own_state = false;
    if (n64) b->f64[0] = (double*)dev_buf;
    if (n32) b->f32[0] = (float*)dev_buf;
  } else {
    if (n64 && hipMalloc(&b->f64[0], n64 * sizeof(double)) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
    if (n32 && hipMalloc(&b->f32[0], n32 * sizeof(float)) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
  }
  return alloc_tables(b, maxn, stage);
}

// Per-instance tables, queues, streams and events for `b->inst.size()` slots;
// read-out scratch for grids of up to maxn nodes, a stage of up to stage_want bytes.
lbm_status alloc_tables(lbm_batch_s* b, size_t maxn, size_t stage_want) {
  const int count = (int)b->inst.size();
  if (hipMalloc(&b->coefs, sizeof(DevCoef) * count) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
  if (hipMalloc(&b->status, sizeof(int) * count) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
  // one queue slot per workgroup of each resident launch
  if (hipMalloc(&b->slots, sizeof(int) * kMaxResidentGrid * 2 * kMaxResident) != hipSuccess)
    return LBM_ERR_OUT_OF_MEMORY;
  for (int k = 0; k < kAuxStreams; ++k) {
    LBM_HIP(hipStreamCreateWithFlags(&b->aux[k], hipStreamNonBlocking));
    LBM_HIP(hipEventCreateWithFlags(&b->join[k], hipEventDisableTiming));
  }
  LBM_HIP(hipEventCreateWithFlags(&b->fork, hipEventDisableTiming));
  // (a job, its instance and segment, and two queue items of each instance)
  const lbm_status ts = alloc_pass_tables(
      b, 4096 + (size_t)count * (sizeof(int) + sizeof(DevJob) + sizeof(DevJobInst) + sizeof(DevSeg) + 2 * sizeof(DevItem)));
  if (ts != LBM_OK) return ts;
  for (int k = 0; k < 2; ++k) LBM_HIP(hipEventCreateWithFlags(&b->items_done[k], hipEventDisableTiming));
  b->scratch_elems = maxn + 64;
  if (hipMalloc(&b->scratch, sizeof(double) * b->scratch_elems) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
  b->stage_bytes = std::min(kStageMost, std::max(kStageLeast, stage_want));
  if (hipHostMalloc((void**)&b->stage, kStageHead + b->stage_bytes, hipHostMallocDefault) != hipSuccess)
    return LBM_ERR_OUT_OF_MEMORY;
  LBM_HIP(hipMemsetAsync(b->status, 0, sizeof(int) * count, b->stream));
  LBM_HIP(hipEventCreate(&b->ev0));
  LBM_HIP(hipEventCreate(&b->ev1));
  return LBM_OK;
}

// every instance's coefficients, through the stage
lbm_status upload_coefs(lbm_batch_s* b) {
  DevCoef* hc = reinterpret_cast<DevCoef*>(b->stage + kStageHead);
  const int most = (int)(b->stage_bytes / sizeof(DevCoef)), count = (int)b->inst.size();
  for (int i = 0; i < count; i += most) {
    const int n = std::min(most, count - i);
    for (int k = 0; k < n; ++k) fill_devcoef(b->inst[i + k], hc + k);
    LBM_HIP(hipMemcpyAsync(b->coefs + i, hc, sizeof(DevCoef) * (size_t)n, hipMemcpyHostToDevice, b->stream));
    LBM_HIP(hipStreamSynchronize(b->stream));
  }
  return LBM_OK;
}

lbm_status create_batch(const lbm_desc* descs, int count, void* stream, void* dev_buf, size_t buf_bytes,
                        lbm_batch_s** out) {
  if (!descs || count <= 0 || !out) return LBM_ERR_INVALID_ARG;
  std::vector<HostInst> inst;
  lbm_status s = prepare_instances(descs, count, &inst);
  if (s != LBM_OK) return s;
  lbm_batch_s* b = new (std::nothrow) lbm_batch_s();
  if (!b) return LBM_ERR_OUT_OF_MEMORY;
  b->stream = (hipStream_t)stream;
  b->inst = std::move(inst);
  b->lim = query_limits();
  if (!b->lim.ok) {
    delete b;
    return LBM_ERR_DEVICE;
  }
  s = alloc_batch(b, dev_buf, buf_bytes);
  if (s == LBM_OK) s = upload_coefs(b);
  if (s != LBM_OK) {
    destroy_batch(b);
    return s;
  }
  *out = b;
  return LBM_OK;
}

double* f64_cur(lbm_batch_s* b, const HostInst& h) { return b->f64[h.cur] + h.off; }
float* f32_cur(lbm_batch_s* b, const HostInst& h) { return b->f32[h.cur] + h.off; }
void* state_cur(lbm_batch_s* b, const HostInst& h) {
  return h.f32 ? (void*)f32_cur(b, h) : (void*)f64_cur(b, h);
}
void* state_at(lbm_batch_s* b, const HostInst& h, int buf) {
  return h.f32 ? (void*)(b->f32[buf] + h.off) : (void*)(b->f64[buf] + h.off);
}
void* state_other(lbm_batch_s* b, const HostInst& h) {
  return h.f32 ? (void*)(b->f32[1 - h.cur] + h.off) : (void*)(b->f64[1 - h.cur] + h.off);
}

lbm_status ensure_second_buffer(lbm_batch_s* b, bool f32) {
  if (f32) {
    if (!b->f32[1] && b->n32 && hipMalloc(&b->f32[1], b->n32 * sizeof(float)) != hipSuccess)
      return LBM_ERR_OUT_OF_MEMORY;
  } else {
    if (!b->f64[1] && b->n64 && hipMalloc(&b->f64[1], b->n64 * sizeof(double)) != hipSuccess)
      return LBM_ERR_OUT_OF_MEMORY;
  }
  return LBM_OK;
}

// The checks of an initial state and, for FP32 storage, its rest state (the mean
// of phi0, conserved on a periodic grid).
lbm_status check_phi(const HostInst& h, const double* phi) {
  bool bad = false, neg = false;
  for (int x = 0; x < h.n; ++x) {
    bad |= !std::isfinite(phi[x]);
    neg |= phi[x] < 0;
  }
  // real (non-integer) powers of phi need phi >= 0
  return bad || (neg && h.mdl.gF > 1) ? LBM_ERR_INVALID_ARG : LBM_OK;
}
void rest_from(HostInst* h, const double* phi) {
  long double s = 0;
  for (int x = 0; x < h->n; ++x) s += phi[x];
  set_rest_state(&h->mdl, (double)(s / h->n));
}

// f := f_eq(phi) of instances idx[k] from host arrays phi[k], already checked.
// phi0 and the records go through the pinned stage, as many instances at a time
// as it holds (or a piece of one that is larger), and one launch per storage
// reads them there; coefficients are copied where they changed (FP32 storage:
// the rest state; `fresh`: new models).  Synchronises the stream.
lbm_status load_many(lbm_batch_s* b, const int* idx, const double* const* phi, int count, bool fresh) {
  unsigned char* base = b->stage + kStageHead;
  struct Piece { int inst; const double* phi; int64_t x0, len; };
  int64_t x0 = 0;   // nodes of instance k already sent
  for (int k = 0; k < count;) {
    std::vector<Piece> pieces;
    size_t need = 0;
    while (k < count) {
      const HostInst& h = b->inst[idx[k]];
      const bool coefs = x0 == 0 && (h.f32 || fresh);
      if (need + stage_need(h.n - x0, coefs) > b->stage_bytes) break;
      need += stage_need(h.n - x0, coefs);
      pieces.push_back({idx[k], phi[k] + x0, x0, h.n - x0});
      x0 = 0;
      ++k;
    }
    if (pieces.empty()) {   // larger than the stage
      const HostInst& h = b->inst[idx[k]];
      const int64_t len = (int64_t)(b->stage_bytes - stage_need(0, x0 == 0)) / (int64_t)sizeof(double);
      pieces.push_back({idx[k], phi[k] + x0, x0, std::min<int64_t>(len, h.n - x0)});
      x0 += pieces[0].len;
    }
    // coefficients, in runs of consecutive instances
    DevCoef* hc = reinterpret_cast<DevCoef*>(base);
    int nc = 0;
    std::vector<int> coef_inst;
    for (const Piece& pc : pieces) {
      HostInst& h = b->inst[pc.inst];
      if (pc.x0 != 0) continue;
      h.cur = 0;
      h.steps_done = 0;
      if (h.f32) rest_from(&h, pc.phi);
      if (!h.f32 && !fresh) continue;
      fill_devcoef(h, hc + nc++);
      coef_inst.push_back(pc.inst);
    }
    for (int c = 0; c < nc;) {
      int e = c + 1;
      while (e < nc && coef_inst[e] == coef_inst[e - 1] + 1) ++e;
      LBM_HIP(hipMemcpyAsync(b->coefs + coef_inst[c], hc + c, sizeof(DevCoef) * (size_t)(e - c), hipMemcpyHostToDevice,
                             b->stream));
      c = e;
    }
    // records (FP64 storage, then FP32) and phi0
    DevInit* rec = reinterpret_cast<DevInit*>(base + sizeof(DevCoef) * (size_t)nc);
    double* data = reinterpret_cast<double*>(rec + pieces.size());
    int at = 0;
    for (int f32 = 0; f32 < 2; ++f32) {
      const int first = at;
      int64_t longest = 0;
      for (const Piece& pc : pieces) {
        const HostInst& h = b->inst[pc.inst];
        if (h.f32 != (f32 != 0)) continue;
        std::memcpy(data, pc.phi, sizeof(double) * (size_t)pc.len);
        DevInit r{};
        r.src = (uint64_t)(uintptr_t)data;
        r.dst = (uint64_t)(uintptr_t)state_cur(b, h) + (uint64_t)pc.x0 * elem_size(h);
        r.len = (int32_t)pc.len;
        r.stride = h.stride;
        r.inst = pc.inst;
        r.q = h.q;
        r.degree = h.Dinit;
        r.first = pc.x0 == 0;
        rec[at++] = r;
        data += pc.len;
        longest = std::max(longest, pc.len);
      }
      for (int c = first; c < at; c += 65535)
        LBM_HIP(launch_init_many(f32 != 0, rec + c, std::min(at - c, 65535), (int)longest, b->coefs, b->status, b->stream));
    }
    LBM_HIP(hipStreamSynchronize(b->stream));   // the stage is free again
  }
  return LBM_OK;
}

// Whether kernels may use a caller's array in place: it is this GPU's memory.
// Another GPU's, which need not be mapped here, and host memory, which a caller
// may name as well, go by copies.
bool on_this_gpu(const void* p) {
  hipPointerAttribute_t at;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();   // (memory the runtime does not know)
    return false;
  }
  return at.type == hipMemoryTypeDevice && at.device == dev;
}

// f := f_eq(phi) of instance i from device memory
lbm_status load_device(lbm_batch_s* b, int i, const double* phi) {
  HostInst& h = b->inst[i];
  if (h.f32 || !on_this_gpu(phi)) {   // the rest state is summed on the host
    std::vector<double> host(h.n);
    LBM_HIP(hipMemcpyAsync(host.data(), phi, sizeof(double) * h.n, hipMemcpyDeviceToHost, b->stream));
    LBM_HIP(hipStreamSynchronize(b->stream));
    lbm_status s = check_phi(h, host.data());
    const double* from = host.data();
    return s == LBM_OK ? load_many(b, &i, &from, 1, false) : s;
  }
  volatile int* words = reinterpret_cast<volatile int*>(b->stage);
  words[0] = words[1] = 0;
  LBM_HIP(launch_check_phi(phi, h.n, reinterpret_cast<int*>(b->stage), b->stream));
  LBM_HIP(hipStreamSynchronize(b->stream));
  if (words[0] || (words[1] && h.mdl.gF > 1)) return LBM_ERR_INVALID_ARG;
  h.cur = 0;
  h.steps_done = 0;
  DevInit r{};
  r.src = (uint64_t)(uintptr_t)phi;
  r.dst = (uint64_t)(uintptr_t)state_cur(b, h);
  r.len = h.n;
  r.stride = h.stride;
  r.inst = i;
  r.q = h.q;
  r.degree = h.Dinit;
  r.first = 1;
  LBM_HIP(launch_init_one(false, r, b->coefs, b->status, nullptr, b->stream));
  LBM_HIP(hipStreamSynchronize(b->stream));   // phi may be reused by the caller
  return LBM_OK;
}

bool fits_resident(const lbm_batch_s* b, const HostInst& h) {
  return (size_t)lds_stride(h.q) * h.n * elem_size(h) + resident_static_lds(h.q, h.prec, h.D) <= b->lim.lds_max;
}



// The step-block graph of instance i for its current buffer, built on first use
// and rebuilt when the instance's buffers, coefficients or shape changed.
lbm_status step_graph(lbm_batch_s* b, int i, StepGraph** out) {
  const HostInst& h = b->inst[i];
  if (b->step_graphs.size() < 2 * b->inst.size()) b->step_graphs.resize(2 * b->inst.size());
  StepGraph* g = &b->step_graphs[2 * i + h.cur];
  const void* fin = state_cur(b, h);
  const void* fout = state_other(b, h);
  const void* cf = b->coefs + i;
  if (g->exec && g->fin == fin && g->fout == fout && g->cf == cf && g->n == h.n && g->stride == h.stride &&
      g->code == h.D && g->q == h.q && g->prec == h.prec) {
    *out = g;
    return LBM_OK;
  }
  if (g->exec) LBM_HIP(hipStreamSynchronize(b->stream));   // a replay of the stale graph may be in flight
  release_graph(g);
  const void* fn = stream_kernel(h.q, h.D, h.prec);
  if (!fn) return LBM_ERR_UNSUPPORTED;
  struct Args { const void* in; void* out; int n; int stride; const void* cf; };
  std::vector<Args> args(kStepBlock);
  std::vector<void*> ptrs(5 * kStepBlock);
  LBM_HIP(hipGraphCreate(&g->graph, 0));
  hipGraphNode_t prev = nullptr;
  for (int k = 0; k < kStepBlock; ++k) {
    Args& a = args[k];
    a.in = (k & 1) ? fout : fin;
    a.out = const_cast<void*>((k & 1) ? fin : fout);
    a.n = h.n;
    a.stride = h.stride;
    a.cf = cf;
    void** p = &ptrs[5 * k];
    p[0] = &a.in;
    p[1] = &a.out;
    p[2] = &a.n;
    p[3] = &a.stride;
    p[4] = &a.cf;
    hipKernelNodeParams kp{};
    kp.func = const_cast<void*>(fn);
    kp.gridDim = dim3((h.n + 255) / 256);
    kp.blockDim = dim3(256);
    kp.sharedMemBytes = 0;
    kp.kernelParams = p;
    kp.extra = nullptr;
    hipGraphNode_t node;
    LBM_HIP(hipGraphAddKernelNode(&node, g->graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp));
    prev = node;
  }
  LBM_HIP(hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0));
  g->fin = fin;
  g->fout = fout;
  g->cf = cf;
  g->n = h.n;
  g->stride = h.stride;
  g->code = h.D;
  g->q = h.q;
  g->prec = h.prec;
  *out = g;
  return LBM_OK;
}

constexpr int64_t kMaxStepsPerLaunch = int64_t(1) << 30;
constexpr int kNoAllocMaxNodes = 8192;   // lbm_advance_noalloc: the largest grid one LDS holds

// Limit of a device wait for a cooperating workgroup that has `steps` steps of
// work to finish first: 10 s plus 20 us per step (a node sweep takes well
// under 10 us on every path), in ticks of the device wall clock.
long long wait_ticks(const lbm_batch_s* b, int64_t steps) {
  const double us = b->test_wait_us > 0 ? (double)b->test_wait_us : 1e7 + 20.0 * (double)steps;
  return (long long)(us * b->lim.wall_ticks_per_us);
}

constexpr int kChunkItems = 16;        // queue items per workgroup when jobs outnumber workgroups
constexpr int64_t kMinChunkSteps = 256;
constexpr int kMaxChunks = 64;
constexpr int64_t kSlabLaunchSteps = 16;
constexpr int kMaxSlabChunks = 8;
constexpr int64_t kMinSlabChunk = 256;   // steps of one chunk of a slab launch

// Lanes a pass spreads its launches over.  HIP runs a process's streams on
// GPU_MAX_HW_QUEUES hardware queues (4 unless that variable is set) and new
// streams go to the least used queue; kernels on streams that share a queue
// run one after another, so more lanes than queues only chain launches
// behind each other in creation order.
int hw_lanes() {
  static const int lanes = [] {
    const char* v = std::getenv("GPU_MAX_HW_QUEUES");
    const int n = v ? std::atoi(v) : 0;
    return n > 0 ? std::min(n, kAuxStreams) : std::min(4, kAuxStreams);
  }();
  return lanes;
}

// Register-resident path: how an instance of n nodes lies in waves of R nodes
// per lane.  A wave's 64 lanes hold its core and `halo` lanes at each end
// (s max|e| nodes for s steps between exchanges).  A grid shorter than a wave's
// smallest core is held as several periods of itself.
struct RegFit {
  int R = 0;       // nodes per lane
  int s = 0;       // steps between wave exchanges
  bool wide = false;
  int lanes = 0;   // lanes of owned nodes (all periods)
  int over = 0;    // nodes by which they exceed the periods
  int waves = 0;
  double cost = 0.0;   // of one wave and step, in VALU operations
  double lag = 0.0;    // what a lone wave waits for its coefficients beside (many nodes hide it)
};
// A step of `waves` waves that share a SIMD: one takes about 1.25 times, two
// about 1.05 times its operations' time each, unless the wait for coefficients is
// longer; with one node per lane nothing hides that wait.
double reg_step(const RegFit& f, int waves) {
  const double slow = waves == 1 ? 1.25 : waves == 2 ? 1.05 : 1.0;
  if (f.R == 1) return slow * waves * f.cost + f.lag;
  return std::max(slow * waves * f.cost, 1.25 * f.cost + f.lag);
}
// What a group of whole instances takes on `cus` CUs, in VALU operations of a wave
// times steps, when they are packed into jobs of at most `share` waves: whole
// instances of one width and step count to a job, `full` waves to a CU.  `beside`:
// the jobs of a CU at once.
struct RegClass {
  int64_t steps = 0;
  RegFit f;
  int64_t count[17] = {};   // instances of so many waves
  int least = 16, most = 1; // the waves there are
};
double reg_group(const std::vector<RegClass>& classes, int share, int full, double cus, int* beside) {
  // jobs by the waves they hold: first fit, decreasing
  struct Jobs { const RegClass* c; int waves; int64_t count; };
  std::vector<Jobs> jobs;
  int64_t total = 0;
  for (const RegClass& c : classes) {
    int64_t room[17] = {};   // jobs with so much room left
    for (int w = c.most; w >= c.least; --w) {
      int64_t left = c.count[w];
      for (int r = w; r <= share && left > 0; ++r) {
        const int each = r / w;   // of them a job with this room takes
        const int64_t filled = std::min(room[r], left / each);
        room[r] -= filled;
        room[r - each * w] += filled;
        left -= filled * each;
        if (room[r] > 0 && left > 0 && left < each) {
          --room[r];
          room[r - (int)left * w] += 1;
          left = 0;
        }
      }
      if (left > 0) {
        const int each = share / w;
        room[share - each * w] += left / each;
        if (left % each) room[share - (int)(left % each) * w] += 1;
      }
    }
    for (int r = 0; r < share; ++r)
      if (room[r] > 0) {
        jobs.push_back({&c, share - r, room[r]});
        total += room[r];
      }
  }
  // jobs side by side on a CU, as many as end the group sooner; more than that
  // follow one another, laid end to end
  double best = 0.0;
  for (int b = 1; b <= std::max(1, full / share); ++b) {
    double longest = 0.0, sum = 0.0;
    for (const Jobs& j : jobs) {
      // (the waves of one workgroup spread evenly over the SIMDs, those of several
      // need not: two of two waves each took as long as two waves on one SIMD; and
      // 600 grids of 2400 nodes, one to a job, two jobs to a CU, took a quarter
      // more than two to a job)
      const int per_simd = j.waves == 1 || j.waves == 3 ? (b * j.waves + 3) / 4 : b * ((j.waves + 3) / 4);
      const double t = (b > 1 ? 1.1 : 1.0) * (double)j.c->steps * reg_step(j.c->f, per_simd);
      longest = std::max(longest, t);
      sum += t * j.count / b;
    }
    const double t = total <= b * cus ? longest : std::max(longest, 1.02 * sum / cus);
    if (b == 1 || t < best) {
      best = t;
      *beside = b;
    }
    if (total <= b * cus) break;
  }
  return best;
}
int reg_halo(int q, int R, int s) { return (s * (q / 2) + R - 1) / R; }
// LDS elements of one wave: its exchange strips, or a row of its nodes
int reg_strip(int q, int R, int s) { return std::max(4 * (reg_halo(q, R, s) + 1) * R * q, 64 * R); }
void reg_place(int q, int n, RegFit* f) {
  const int hl = reg_halo(q, f->R, f->s), least = 2 * (hl + 1), cap = 64 - 2 * hl;
  const int periods = std::max(1, (least * f->R + n - 1) / n);
  f->lanes = (periods * n + f->R - 1) / f->R;
  f->over = f->lanes * f->R - periods * n;
  f->waves = (f->lanes + cap - 1) / cap;
}
// The widths of a variant's kernels, ascending, each with its steps between
// exchanges: those with the least cost per core node.  Cost of a wave's step:
// the nodes' operations, the lane-edge moves (2 sum|e| per two steps, two
// registers each in FP64), and 1/s of an exchange, which took about 5 R q
// (FP64) or 2 R q (FP32) operations' time.
int reg_menu(int q, int prec, int code, bool wide, RegFit* out) {
  const bool f32 = prec != 0;
  const int D = code & 0xff, K = (code >> 8) == 0 ? D + 1 : (D + 1) / 2 + 1;
  const int elem = f32 ? 4 : 8, arith = prec == 2 ? 4 : 8;
  const int conv = f32 ? (prec == 2 ? q + 2 : 2 * q) : 0;
  const int cross = (q <= 5 ? 6 : 12) * (f32 ? 1 : 2);
  int count = 0;
  for (int k = 0; k < kRegWidths; ++k) {
    const int R = reg_width(q, elem, D, code >> 8, wide, k);
    if (R == 0) break;
    RegFit best;
    double least = 0.0;
    for (int s = 2; s <= 16; s += 2) {
      const int hl = reg_halo(q, R, s), cap = 64 - 2 * hl;
      if (cap < 4 * (hl + 1)) break;   // the strips of a wave's two ends stay apart
      const double c = R * (q * (K + 1) + q - 1.0 + conv) + cross + ((f32 ? 2.0 : 5.0) * R * q + 40.0) / s;
      if (least == 0.0 || c / cap < least) {
        least = c / cap;
        best.R = R;
        best.s = s;
        best.wide = wide;
        best.cost = c;
        best.lag = reg_pinned(q, D, code >> 8, arith) || reg_held(q, D, code >> 8, elem, arith, wide, R)
                       ? 0.0
                       : 37.0 * q * (K - 1) * arith / 64 * std::min(1.0, 2.0 / R);
      }
    }
    if (best.R) out[count++] = best;
  }
  if (wide) {   // the largest grids of one LDS need the widest kernel at its least halo
    out[count] = out[count - 1];
    out[count].s = 4;
    out[count].cost *= 1.1;
    ++count;
  }
  return count;
}

// The same width with the narrowest halo, and as many steps between exchanges as
// that holds: more exchanges, but an instance may need a wave less.
RegFit reg_tight(int q, int prec, RegFit f) {
  const int hl = reg_halo(q, f.R, 2), s = std::min(16, hl * f.R / (q / 2) / 2 * 2);
  f.cost += ((prec != 0 ? 2.0 : 5.0) * f.R * q + 40.0) * (1.0 / s - 1.0 / f.s);
  f.s = s;
  return f;
}

// bounded instances: one width
RegFit bound_fit() {
  RegFit f;
  f.R = kBoundWidth;
  f.s = kBoundSteps;
  f.cost = 250.0;   // of the waves with layers
  return f;
}

// Slabs and tiles of the register path: an instance cut into segments of about
// equal lanes, one workgroup each, whose ends stay exact for sx steps.
struct SegPlan {
  RegFit f;
  int sx = 0;          // steps between exchanges with the neighbours, or of a tile's launch
  int extra = 0;       // outer halo lanes beside a wave's own
  int most = 0;        // owned lanes of a segment, at most
  int waves = 0;       // of the largest segment
  int per_cu = 1;      // workgroups a CU is meant to hold
  double est = 0.0;    // of a step of the whole group, in VALU operations of a wave
};
// An exchange between workgroups, in VALU operations of a wave (about 1.67 ns):
// 1.2 us, and 2.2 us more for each further workgroup that shares the CU
// (2000-step batches of 128 KS and 96 Kawahara grids, 1 to 6 a CU).
constexpr double kLinkCost = 700.0, kLinkShare = 1300.0;
// Segments of an instance of n nodes; 0: they cannot be cut as planned.  A
// slab's outer owned lanes, which its neighbour reads, lie in its first and
// last wave, and a wave's strips apart; a tile only needs the latter.
int seg_count(const SegPlan& p, int q, int n, bool tile) {
  const int hl = reg_halo(q, p.f.R, p.f.s), cap = 64 - 2 * hl, hg = hl + p.extra;
  const int all = (n + p.f.R - 1) / p.f.R, k = (all + p.most - 1) / p.most;
  const int lanes = all / k + 2 * p.extra, waves = (lanes + cap - 1) / cap;   // of the smallest
  if (waves > 1 && lanes / waves < 2 * (hl + 1)) return 0;
  if (tile) return k;
  if (waves == 1 ? all / k < 2 * (hg + 1) : lanes / waves < p.extra + hg + 1) return 0;
  // the largest may take a wave more
  const int top = (all + k - 1) / k + 2 * p.extra, more = (top + cap - 1) / cap;
  return top / more < p.extra + hg + 1 || top / more < 2 * (hl + 1) ? 0 : k;
}
// Whether the slab kernel's registers do not hold a lane's R nodes beside what it
// keeps for its neighbours: the widest lanes of FP64 storage on D1Q5 and of D1Q4
// tables past degree 5, and with FP32 storage and FP64 arithmetic the widest of
// the larger tables.  Measured against the step such widths are priced at: 1.4 to
// 3.4 times in FP64 (128 K(2,2) grids of 16384 nodes, 2500 steps: 13.0 ms with 17
// nodes per lane, 7.4 ms with 14 or fewer), 1.2 to 1.5 in FP32 storage; the others
// 0.9 to 1.15.  Whole instances (k_reg) have no such widths.
bool seg_spills(int q, int prec, int code, int R) {
  const int D = code & 0xff;
  const bool dense = (code >> 8) == 0;
  if (R < (q <= 5 ? 17 : 12) || prec == 2) return false;
  if (prec == 0) return q == 5 || (dense && D > 5);
  return q == 7 || (q > 4 && dense && D > 7);
}
// The cheapest plan of a group (sizes: node count, instances of it) on `cus`
// CUs: a step of the waves that share a SIMD, and 1/sx of an exchange or of a
// tile's way from and to HBM.
// `want`: steps asked for (0: free); `wgs`: workgroups per CU asked for (0: free);
// `chunks`: step chunks that the group's steps can be cut into.
bool seg_plan(int q, int prec, int code, const std::map<int, int>& sizes, int cus, int want, int wgs, bool tile,
              int chunks, SegPlan* out) {
  const int H = q / 2;
  int64_t nodes = 0;
  for (const auto& [n, times] : sizes) nodes += (int64_t)n * times;
  bool found = false;
  // (what is likely good first: the rest is then passed over by its bounds)
  const bool much = nodes > (int64_t)cus * 1024;
  for (int c = 0; c < 2; ++c) {
    const int cls = much ? 1 - c : c;
    RegFit menu[kRegWidths + 1];
    const int widths = reg_menu(q, prec, code, cls != 0, menu), full = reg_waves(cls != 0);
    for (int m = 0; m < widths; ++m) {
      const int k = much ? widths - 1 - m : m;
      if (seg_spills(q, prec, code, menu[k].R)) continue;
      const double least = std::max(reg_step(menu[k], 1), nodes / (256.0 * menu[k].R * cus) * menu[k].cost);
      if (found && least >= out->est) continue;
      for (int pick = 0; pick < 7; ++pick) {
        SegPlan p;
        p.f = menu[k];
        if (want > 0) {
          if (pick > 0) break;
          while (p.f.s > 2 && want % p.f.s != 0) p.f.s -= 2;
          p.sx = want;
        } else {
          p.sx = (((pick & 1 ? 12 : 8) << pick / 2) + p.f.s - 1) / p.f.s * p.f.s;
        }
        const int hl = reg_halo(q, p.f.R, p.f.s), cap = 64 - 2 * hl;
        p.extra = std::max(0, (p.sx * H + p.f.R - 1) / p.f.R - hl);
        if (found && !tile && least + kLinkCost / p.sx >= out->est) continue;
        for (int w = 1; w <= (wgs > 0 ? std::max(1, full / wgs) : full); w = w < 4 ? w + 1 : w + 2) {
          p.waves = w;
          p.most = w * cap - 2 * p.extra;
          if (p.most < 1) continue;
          const int hold = full / w;   // workgroups a CU holds
          // (a launch holds whole instances of `count` segments, or of them on average)
          auto price = [&](int64_t total, double count) {
            p.per_cu = (int)std::min<int64_t>(hold, (total + cus - 1) / cus);
            const int per_simd = (p.per_cu * w + 3) / 4;
            const int64_t places = (int64_t)p.per_cu * cus;
            const double held = sizes.size() == 1 ? places - places % (int64_t)count : places - 0.5 * (count - 1.0);
            double rounds = total <= places ? 1.0 : tile ? std::ceil((double)total / places) : 1e30;
            for (int c = 1; c <= chunks && !tile && total > places; ++c)
              rounds = std::min(rounds, (c > 1 ? 1.02 : 1.0) * std::ceil(c * (total / held) - 1e-9) / c);
            const double link = tile ? 3000.0 + 0.4 * (p.per_cu * p.most * p.f.R) * q
                                     : kLinkCost + kLinkShare * (p.per_cu - 1) + (prec != 0 ? 2.0 : 5.0) * p.f.R * q;
            p.est = rounds * (reg_step(p.f, per_simd) + link / p.sx);
          };
          price(std::max<int64_t>(1, nodes / ((int64_t)p.most * p.f.R)), 1.0);   // as few segments as there can be
          if (found && p.est >= out->est) continue;
          int64_t total = 0, instances = 0;
          bool ok = true;
          for (const auto& [n, times] : sizes) {
            instances += times;
            const int c = seg_count(p, q, n, tile);
            ok = c > 0 && (tile || c <= cus);
            if (!ok) break;
            total += (int64_t)c * times;
          }
          if (!ok) continue;
          price(total, (double)total / instances);
          if (!found || p.est < out->est) {
            *out = p;
            found = true;
          }
        }
      }
    }
  }
  return found;
}

// A step of one instance alone on a CU, in VALU operations of a wave; `share`: of
// the CU's time in a full GPU, at least.
double ring_step(int q, int prec, int code, int n, double* share = nullptr) {
  double least = 1e30, part = 1e30;
  for (int cls = 0; cls < 2; ++cls) {
    RegFit menu[kRegWidths + 1];
    const int widths = reg_menu(q, prec, code, cls != 0, menu);
    for (int k = 0; k < widths; ++k) {
      reg_place(q, n, &menu[k]);
      if (menu[k].waves > reg_waves(cls != 0)) continue;
      least = std::min(least, reg_step(menu[k], (menu[k].waves + 3) / 4));
      // (as many whole instances as a CU's waves hold)
      const int hold = reg_waves(cls != 0) / menu[k].waves;
      part = std::min(part, reg_step(menu[k], (hold * menu[k].waves + 3) / 4) / hold);
    }
  }
  if (share) *share = part;
  return least;
}

// Step chunks of a slab group that needs more workgroups than a launch holds.
// The (instance, chunk) items fill the launches in chunk order, whole instances
// at a time; a launch is closed before an item that exceeds `fill` workgroups and
// before a second item of an instance (one of fewer steps than chunks leaves the
// later chunks smaller), so that an instance's chunk c + 1 always lies in a later
// launch than its chunk c.
struct SlabChunks {
  int chunks = 1;
  int64_t fill = 0;   // workgroups a launch is filled to
};
int64_t chunk_steps(int64_t steps, int chunks, int c) { return steps / chunks + (c < steps % chunks ? 1 : 0); }
// Launches of `chunks` chunks filled to `fill`; `time`: their longest items' steps,
// added up (a launch lasts about its longest item's steps, whatever its fill).
// mem: (workgroups, steps) of each instance.
int slab_launches(const std::vector<std::pair<int, int64_t>>& mem, int chunks, int64_t fill, int64_t* time) {
  int launches = 0, at = 0;
  int64_t count = 0, longest = 0;
  std::vector<int> in(mem.size(), 0);   // the launch of an instance's last item
  *time = 0;
  for (int c = 0; c < chunks; ++c)
    for (size_t m = 0; m < mem.size(); ++m) {
      const int64_t st = chunk_steps(mem[m].second, chunks, c);
      if (st == 0) continue;
      if (at == 0 || count + mem[m].first > fill || in[m] == at) {
        at = ++launches;
        *time += longest;
        count = longest = 0;
      }
      in[m] = at;
      count += mem[m].first;
      longest = std::max(longest, st);
    }
  *time += longest;
  return launches;
}
// The chunks, each of kMinSlabChunk steps or more, with the least time (a launch
// of its own takes about as long as kSlabLaunchSteps steps: its states' way in and
// out); and the least fill that needs no more launches, so that none is a short
// tail that costs a whole launch's time (512 Kawahara and K(2,2) grids, FP32
// storage, counted in workgroups instead of whole instances: 255, 255, 255 and 3,
// 65.9 ms; counted as they are filled 58.5 ms).
SlabChunks slab_chunks(const std::vector<std::pair<int, int64_t>>& mem, int64_t capacity) {
  SlabChunks out;
  out.fill = capacity;
  int64_t total = 0, longest = 0, most = 0;
  for (const auto& [slabs, steps] : mem) {
    total += slabs;
    longest = std::max(longest, steps);
    most = std::max<int64_t>(most, slabs);
  }
  if (total <= capacity) return out;
  int64_t time = 0, least = INT64_MAX;
  int launches = 0;
  for (int c = 1; c <= kMaxSlabChunks && (c == 1 || longest / c >= kMinSlabChunk); ++c) {
    int64_t t;
    const int l = slab_launches(mem, c, capacity, &t);
    if (t + l * kSlabLaunchSteps >= least) continue;
    least = t + l * kSlabLaunchSteps;
    out.chunks = c;
    launches = l;
    time = t;
  }
  for (int64_t lo = most, hi = capacity; lo < hi;) {
    const int64_t mid = (lo + hi) / 2;
    int64_t t;
    if (slab_launches(mem, out.chunks, mid, &t) <= launches && t <= time)
      out.fill = hi = mid;
    else
      lo = mid + 1;
  }
  return out;
}

// The GPU's CUs over launches side by side, in whole CUs of every XCD (even_places):
// each next one to the launch that would end last, none beyond its `most`
// workgroups.  Empty: more launches than an XCD has CUs.
std::vector<int> cu_shares(const std::vector<double>& work, const std::vector<int>& most, int cus) {
  const int unit = xcd_count(cus), units = cus / unit;
  if ((int)work.size() > units) return {};
  std::vector<int> share(work.size(), unit);
  for (int u = (int)work.size(); u < units; ++u) {
    size_t top = work.size();
    for (size_t k = 0; k < work.size(); ++k)
      if (share[k] < most[k] && (top == work.size() || work[k] / share[k] > work[top] / share[top])) top = k;
    if (top == work.size()) break;
    share[top] += unit;
  }
  return share;
}

// waits of b's stream before slab launches of `need` workgroups (gate held); ahead:
// the steps of other batches' whole instances in flight
lbm_status pass_gate(SlabGate& gate, lbm_batch_s* b, int need, int64_t* ahead) {
  int sum = 0;
  *ahead = 0;
  for (SlabGate::Flight& f : gate.flight) {
    // (b's own earlier passes come before on its stream)
    if ((f.need == 0 && f.ahead == 0) || (f.owner == b && f.need <= need && f.ahead == 0)) continue;
    if (hipEventQuery(f.done) == hipSuccess) {
      f.need = 0;
      f.ahead = 0;
    } else {
      (void)hipGetLastError();   // (not ready is no error)
    }
    if (f.owner == b) continue;
    sum += f.need;
    *ahead += f.ahead;
  }
  if (need == 0) return LBM_OK;
  for (const SlabGate::Flight& f : gate.flight) {
    if (sum + need <= b->lim.cus) break;
    if (f.owner == b || f.need == 0) continue;
    LBM_HIP(hipStreamWaitEvent(b->stream, f.done, 0));
    sum -= f.need;
  }
  return LBM_OK;
}
// b's launches have been issued; until they are over, its entry counts the most of
// the workgroups of them and of b's earlier ones, and all their steps
lbm_status enter_gate(SlabGate& gate, lbm_batch_s* b, int need, int64_t ahead) {
  if (!b->gate) {
    LBM_HIP(hipEventCreateWithFlags(&b->gate_done, hipEventDisableTiming));
    gate.flight.push_back({b, b->gate_done, 0, 0});
    b->gate = &gate;
  }
  LBM_HIP(hipEventRecord(b->gate_done, b->stream));
  for (SlabGate::Flight& f : gate.flight)
    if (f.owner == b) {
      f.need = std::max(f.need, need);
      f.ahead += ahead;
    }
  return LBM_OK;
}

// Plans depend on sizes and step counts alone, and a program that advances a few
// steps at a time asks for the same ones again: 300 sizes beyond one LDS cost 160
// us of planning for 130 us of steps.  A batch keeps the latest, by everything
// they were made from.
struct RingPlan {
  std::vector<RegFit> fit;
  int job_waves = 4, jobs_per_cu = 1;
  bool wide = false, found = false;
};
struct PlanMemo {
  std::map<std::vector<int64_t>, std::pair<bool, SegPlan>> segs;
  std::map<std::vector<int64_t>, RingPlan> rings;
  size_t ring_instances = 0;   // of all of them
  std::map<std::tuple<int, int, int, int>, std::pair<double, double>> ring_steps;   // by (q, prec, code, nodes)
  // whether a (q, prec, variant, nodes) instance on so many CUs advances sooner in slabs
  std::map<std::tuple<int, int, int, int, int>, bool> sooner;
};

// Nodes per lane: few spend more on halos and lane edges, many leave more of
// an instance's last lanes empty and give fewer waves to share the SIMDs.
// Each instance takes the width with the least wave time among one kernel's
// (narrow or wide: one launch per group, since a pass's launches run side by
// side only while there are hardware queues) up to a bound, or all of them the
// same one; kernel, widths and waves per job are those for which the group,
// packed, is estimated to end first.  (By its waves alone, 512 grids of 1000
// nodes took nine waves each, one to a job of sixteen.)
bool plan_rings(const lbm_batch_s* b, int q, int pr, int code, const std::vector<int>& g, const int64_t* steps, double cus,
                RingPlan* out) {
  std::vector<RegFit>& fit = out->fit;
  fit.resize(g.size());
  std::vector<RegFit> trial(g.size());
  const bool bounded = (code >> 16) != 0;
  double best = 0.0;
  std::vector<RegClass> classes;
  std::map<int64_t, int> step_ids;   // of the group's step counts
  std::vector<int> step_id, class_of;
  std::vector<RegFit> placed;   // each instance by each width
  for (int i : g) step_id.push_back(step_ids.insert({steps[i], (int)step_ids.size()}).first->second);
  for (int cls = 0; cls < 2; ++cls) {
    RegFit menu[kRegWidths + 1];
    const int full = reg_waves(cls != 0);
    int widths = 0;
    if (!bounded) {
      widths = reg_menu(q, pr, code, cls != 0, menu);
    } else if (cls == 0) {
      menu[0] = bound_fit();
      widths = 1;
    }
    if (widths == 0) continue;
    // wave time of an instance: that of whole rounds over the SIMDs where no
    // other has room beside it
    auto load = [&](const RegFit& f) { return (2 * f.waves > full ? (f.waves + 3) / 4 * 4 : f.waves) * f.cost; };
    placed.resize(g.size() * widths);
    for (size_t u = 0; u < g.size(); ++u) {
      RegFit* at = &placed[u * widths];
      const int n = b->inst[g[u]].n;
      if (u > 0 && n == b->inst[g[u - 1]].n) {
        std::copy(at - widths, at, at);
        continue;
      }
      for (int w = 0; w < widths; ++w) {
        at[w] = menu[w];
        reg_place(q, n, &at[w]);
        if (bounded) continue;
        RegFit f = reg_tight(q, pr, menu[w]);
        reg_place(q, n, &f);
        if (load(f) < load(at[w])) at[w] = f;
      }
    }
    for (int pick = 2 * widths - 1; pick >= 0; --pick) {
      const int most = pick / 2, from = pick % 2 ? most : 0;
      if (from == most && most == 0 && pick % 2) continue;
      int64_t waves = 0;
      int top = 1;
      bool ok = true;
      classes.clear();
      class_of.assign(step_ids.size() * widths * 2, -1);
      for (size_t u = 0; u < g.size() && ok; ++u) {
        double least = 0.0;
        int taken = 0;
        for (int w = from; w <= most; ++w) {
          const RegFit& f = placed[u * widths + w];
          if (f.waves > full) continue;
          if (least == 0.0 || load(f) < least) {
            trial[u] = f;
            taken = 2 * w + (f.s != menu[w].s);
            least = load(f);
          }
        }
        ok = least > 0.0;
        if (!ok) break;
        waves += trial[u].waves;
        top = std::max(top, trial[u].waves);
        int& at = class_of[step_id[u] * widths * 2 + taken];
        if (at < 0) {
          at = (int)classes.size();
          classes.emplace_back();
          classes[at].steps = steps[g[u]];
          classes[at].f = trial[u];
        }
        RegClass& c = classes[at];
        ++c.count[trial[u].waves];
        c.least = std::min(c.least, trial[u].waves);
        c.most = std::max(c.most, trial[u].waves);
      }
      if (!ok) continue;
      // waves of a job: as many as the waves make for each CU, all a CU holds,
      // and (few classes) what lies between
      const int even = std::max(top, (int)std::min<double>(full, std::ceil(waves / cus)));
      for (int share = top; share <= full; ++share) {
        if (share != full && share != even && classes.size() > 64) continue;
        int beside = 1;
        const double est = reg_group(classes, share, full, cus, &beside);
        if (best == 0.0 || est < best) {
          best = est;
          fit = trial;
          out->job_waves = share;
          out->jobs_per_cu = beside;
          out->wide = cls != 0;
        }
      }
    }
  }
  return best > 0.0;
}

// One pass: every instance advances by steps[i] <= kMaxStepsPerLaunch.
lbm_status advance_pass(lbm_batch_s* b, const int64_t* steps) {
  const int count = (int)b->inst.size();
  if (!b->memo) b->memo = std::make_shared<PlanMemo>();
  PlanMemo& memo = *b->memo;
  // resident groups by (q, precision, variant); the rest streams through HBM
  // (q, prec, variant code, bounded)
  std::map<std::tuple<int, int, int, int>, std::vector<int>> res;
  // register-resident, by (q, prec, variant): whole instances, slabs, tiles
  // (bounded instances among the first: variant | 1 << 16)
  std::map<std::tuple<int, int, int>, std::vector<int>> reg, spread, rtile;
  std::vector<int> str;          // one launch per step (the plain path)
  std::vector<int> til[8][3];    // temporal blocking, by (q, prec)
  // slabs, by (q, prec, variant, workgroups per CU)
  std::map<std::tuple<int, int, int, int>, std::vector<int>> slb;
  // A pass whose resident instances fill less than a quarter of the GPU's LDS
  // leaves most CUs idle; its step time is that of its largest instances, one
  // CU each.  There, instances of kSplitNodes nodes or more are split into
  // narrow slabs (an eighth of an LDS) spread over otherwise idle CUs.
  // The same holds for instances beyond one LDS when all the pass's state is
  // that small (a serving round): their slabs are narrow too.
  size_t res_bytes = 0, all_bytes = 0;
  for (int i = 0; i < count; ++i) {
    if (!steps[i] || b->path != 0) continue;
    const size_t by = (size_t)lds_stride(b->inst[i].q) * b->inst[i].n * elem_size(b->inst[i]);
    all_bytes += by;
    if (fits_resident(b, b->inst[i])) res_bytes += by;
  }
  const size_t lds_all = (size_t)b->lim.cus * b->lim.lds_max;
  const bool latency = b->path == 0 && b->res_grid == 0 && 4 * res_bytes < lds_all;
  // Polynomial instances there go by estimate: over their share of the CUs, or
  // whole on one, whichever ends a step sooner.
  int sharing = 0;
  for (int i = 0; i < count; ++i) sharing += latency && steps[i] > 0;
  auto spread_sooner = [&](const HostInst& h) {
    const int cus = b->lim.cus / std::max(1, sharing);
    const auto key = std::make_tuple(h.q, h.prec, h.D, h.n, cus);
    const auto it = memo.sooner.find(key);
    if (it != memo.sooner.end()) return it->second;
    if (memo.sooner.size() >= 4096) memo.sooner.clear();
    SegPlan p;
    const bool yes = cus > 1 && seg_plan(h.q, h.prec, h.D, {{h.n, 1}}, cus, 0, 0, false, 1, &p) &&
                     p.est < 0.95 * ring_step(h.q, h.prec, h.D, h.n);
    return memo.sooner[key] = yes;
  };
  // Power sums in LDS: an instance is one CU's work, so that a group ends with its
  // largest one.  Where that takes more than one and a half times the even share
  // of the CUs, the group goes in slabs of a quarter of an LDS (256 grids of 256
  // to 4096 nodes, 2.9 times: 4.80 -> 2.49 ms per 1000 steps; half-LDS slabs
  // 4.11, an eighth 2.62; 1024 such grids, 0.7 times, stay whole).  Over ranges of
  // sizes, powers and step counts with shares of 1.9 to 4 the slabs took 0.52 to
  // 0.70 of the whole instances' time in FP64 and 0.62 to 0.9 in FP32 storage; 300
  // grids of 128 to 1024 nodes, 2.0 times, the same time.
  std::map<std::tuple<int, int, int>, std::pair<int64_t, int64_t>> loads;   // steps x nodes: all, largest
  for (int i = 0; i < count; ++i) {
    const HostInst& h = b->inst[i];
    if (reg_variant(h.D) || h.desc.bc != LBM_BC_PERIODIC || steps[i] == 0) continue;
    auto& l = loads[std::make_tuple(h.q, h.prec, h.D)];
    l.first += steps[i] * h.n;
    l.second = std::max<int64_t>(l.second, steps[i] * h.n);
  }
  auto uneven = [&](const HostInst& h) {
    const auto& l = loads[std::make_tuple(h.q, h.prec, h.D)];
    return b->path == 0 && b->res_grid == 0 && b->res_chunks == 0 && b->tile_wgs == 0 && 2.0 * b->lim.cus * l.second > 3.0 * l.first;
  };
  // (an instance that fits a CU stays whole where there is no memory for the second
  // state buffer that slabs write to)
  int room[2] = {-1, -1};
  auto has_room = [&](bool f32) {
    if (room[f32] < 0) {
      room[f32] = ensure_second_buffer(b, f32) == LBM_OK;
      if (!room[f32]) (void)hipGetLastError();   // (no error of the launches to come)
    }
    return room[f32] == 1;
  };
  const int slab_wgs = b->tile_wgs > 0 ? b->tile_wgs : latency && 4 * all_bytes < lds_all ? 8 : 2;
  for (int i = 0; i < count; ++i) {
    if (steps[i] == 0) continue;
    const HostInst& h = b->inst[i];
    const bool fits = fits_resident(b, h);
    const bool in_reg = reg_variant(h.D) && h.desc.bc == LBM_BC_PERIODIC;
    if (h.desc.bc != LBM_BC_PERIODIC) {
      // bounded instances advance only in a bounded call, on the resident path
      if (!b->bnd_active) return LBM_ERR_INVALID_ARG;
      if (!fits || (b->path != 0 && b->path != 2)) return LBM_ERR_UNSUPPORTED;
      // two nodes per lane on the register path where two waves or more, of one
      // CU, hold them and a wave's lanes the layers' values (801 nodes: 1.14 -> 0.69 us
      // per step); in LDS otherwise
      RegFit f = bound_fit();
      reg_place(h.q, h.n, &f);
      if (bound_variant(h.q, h.D & 0xff, (h.D >> 8) & 0xff, h.prec == 2 ? 4 : 8) && f.waves >= 2 &&
          f.waves <= reg_waves(false) && b->bnd_layers * h.q <= kBoundValues)
        reg[std::make_tuple(h.q, h.prec, h.D | (1 << 16))].push_back(i);
      else
        res[std::make_tuple(h.q, h.prec, h.D, 1)].push_back(i);
      continue;
    }
    if (b->path == 2 && !fits) return LBM_ERR_UNSUPPORTED;
    if (b->path == 1)
      str.push_back(i);
    else if (b->path == 3 && in_reg)
      rtile[std::make_tuple(h.q, h.prec, h.D)].push_back(i);
    else if (b->path == 3)
      til[h.q][h.prec].push_back(i);
    else if (in_reg && (b->path == 4 || !fits || (latency && spread_sooner(h) && has_room(h.f32))))
      spread[std::make_tuple(h.q, h.prec, h.D)].push_back(i);
    else if (b->path == 4 || !fits)
      slb[std::make_tuple(h.q, h.prec, h.D, slab_wgs)].push_back(i);
    else if (!in_reg && latency && h.n >= kSplitNodes)
      slb[std::make_tuple(h.q, h.prec, h.D, 8)].push_back(i);
    else if (!in_reg && !latency && h.n >= kUnevenNodes && uneven(h) && has_room(h.f32))
      slb[std::make_tuple(h.q, h.prec, h.D, 4)].push_back(i);
    else if (in_reg)
      reg[std::make_tuple(h.q, h.prec, h.D)].push_back(i);
    else
      res[std::make_tuple(h.q, h.prec, h.D, 0)].push_back(i);
  }
  // item records of this call go to slot `k`; wait until the copy issued from
  // the same slot two calls ago has been consumed
  const int k = b->slot;
  b->slot ^= 1;
  LBM_HIP(hipEventSynchronize(b->items_done[k]));
  std::vector<DevJobInst>& hitems = b->hitems;
  std::vector<DevJob>& hjobs = b->hjobs;
  std::vector<DevSeg>& hsegs = b->hsegs;
  hitems.clear();
  hjobs.clear();
  hsegs.clear();
  // est_max / est_sum: the longest job's and all jobs' duration estimates
  struct Launch { int q; int prec; int code; int first, count; size_t lds; int block; int64_t maxsteps; double est_max, est_sum; bool reg, wide; int per_cu, grid, part0, parts; int64_t partsteps; double issue; };
  std::vector<Launch> launches;
  int used = 0, njobs = 0, nsegs = 0;
  constexpr int kMaxJobInstances = 16;   // instances per job (one wave each at least)
  for (const auto& group : res) {
    {
      const int pr = std::get<1>(group.first);
      const int bnd = std::get<3>(group.first);
      // the kernel: the variant, and whether its jobs reset boundary layers
      const int code = std::get<2>(group.first) | (bnd << 16);
      std::vector<int> g = group.second;
      const size_t es = pr ? sizeof(float) : sizeof(double);
      const int q = std::get<0>(group.first);
      auto bytes_of = [&](int i) { return ((size_t)lds_stride(q) * b->inst[i].n * es + 15) / 16 * 16; };
      // a workgroup's LDS share: half the LDS, or the largest instance
      size_t cap = b->lim.lds_max / 2;
      for (int i : g) cap = std::max(cap, bytes_of(i));
      // jobs: first-fit decreasing bin packing of equal-step instances into the
      // LDS share; jobs hold instances of one variant and one step count
      std::stable_sort(g.begin(), g.end(), [&](int a, int c) {
        if (steps[a] != steps[c]) return steps[a] > steps[c];
        if (b->inst[a].D != b->inst[c].D) return b->inst[a].D < b->inst[c].D;
        return bytes_of(a) > bytes_of(c);
      });
      // waves per job: the waves a CU can hold at this kernel's register use,
      // shared by the jobs whose LDS fits on one CU
      const int vgprs = std::max(1, resident_vgprs(q, pr, code));
      const int cu_waves = 4 * std::max(1, std::min(8, 512 / vgprs));
      const int jobs_per_cu = std::max<int>(1, (int)(b->lim.lds_max / cap));
      // waves per job: the CU's waves shared by the jobs it holds at once -- in
      // the latency regime (one job per instance) with no more instances than
      // CUs, one job per CU (a 256-tau sweep of bounded instances gets twice the
      // waves).  (bounded kernels are compiled for workgroups of at most 512
      // threads)
      const int cu_jobs = latency && (int)g.size() <= b->lim.cus ? 1 : jobs_per_cu;
      const int kJobWaves = std::max(1, std::min(bnd ? 8 : 16, cu_waves / cu_jobs));
      // a pass that leaves most CUs idle (latency regime) gives every instance a
      // job of its own and up to a wave per 64 nodes: its steps end sooner
      const int kNodesPerWave = latency ? 64 : 128;
      // Passes per step of a full job: a job's waves sweep its nodes 64 per
      // pass, and a member of n nodes needs ceil(n / (64 passes)) waves to end
      // its sweep within that many passes.  Packed by bytes alone, a job's
      // members can need more waves than the job has, so some waves take a
      // pass more than the rest and every step waits for them.  Where two jobs
      // share each CU (eight waves per SIMD: the step is bound by VALU issue) a
      // job therefore admits a member only while the members' waves at that
      // pass count fit.  One job per CU is bound by the step's latency instead,
      // and fuller jobs pay there.  (Measured on 4096 KdV and mKdV grids while
      // those ran in LDS: FP32 storage 46.5 -> 45.3 ms, FP64 1.5% slower.)
      const bool wave_budget = !latency && jobs_per_cu >= 2;
      const int full_passes = std::max<int>(
          std::max(1, kNodesPerWave / 64),
          (int)((cap / ((size_t)lds_stride(q) * es) + 64 * (size_t)kJobWaves - 1) / (64 * (size_t)kJobWaves)));
      auto waves_at = [&](int i) {
        return wave_budget ? (b->inst[i].n + 64 * full_passes - 1) / (64 * full_passes) : 0;
      };
      struct Bin { int64_t steps; int variant; size_t bytes; int waves; std::vector<int> members; };
      std::vector<Bin> bins;
      auto pack = [&](int max_inst) {
        bins.clear();
        size_t open_from = 0;   // bins before this index have another step count or variant
        for (int i : g) {
          if (!bins.empty() && (bins.back().steps != steps[i] || bins.back().variant != b->inst[i].D))
            open_from = bins.size();
          bool placed = false;
          for (size_t u = open_from; u < bins.size() && !placed; ++u) {
            Bin& bn = bins[u];
            if (bn.bytes + bytes_of(i) <= cap && (int)bn.members.size() < max_inst &&
                bn.waves + waves_at(i) <= kJobWaves) {
              bn.bytes += bytes_of(i);
              bn.waves += waves_at(i);
              bn.members.push_back(i);
              placed = true;
            }
          }
          if (!placed) bins.push_back(Bin{steps[i], b->inst[i].D, bytes_of(i), waves_at(i), {i}});
        }
      };
      pack(latency ? 1 : std::min(kMaxJobInstances, kJobWaves));
      // fewer jobs than the GPU holds at once (jobs_per_cu per CU) leave CUs
      // idle for the whole pass: cap the instances per job so that there are
      // enough (1024 instances of 1024 FP32 D1Q5 nodes would otherwise make
      // 256 half-LDS jobs for 512 slots)
      const int slots = jobs_per_cu * b->lim.cus;
      if (!latency && (int)bins.size() < slots && (int)g.size() > (int)bins.size())
        pack(std::max(1, ((int)g.size() + slots - 1) / slots));
      Launch L{q, pr, code, njobs, 0, 0, 64, 0, 0.0, 0.0, false, false, 0, 0, 0, 0, 0, 0.0};
      struct Planned { const Bin* bin; std::vector<int> waves; double est; };
      std::vector<Planned> plan;
      for (const Bin& bn : bins) {
        // waves: one each, then one more at a time to the member with the most
        // nodes per wave (at most one wave per kNodesPerWave nodes)
        const int m = (int)bn.members.size();
        std::vector<int> wv(m, 1);
        int total = m;
        while (total < kJobWaves) {
          int best = -1;
          double load = 0.0;
          for (int u = 0; u < m; ++u) {
            const int n = b->inst[bn.members[u]].n;
            if (wv[u] >= (n + kNodesPerWave - 1) / kNodesPerWave) continue;
            const double l = (double)n / wv[u];
            if (l > load) {
              load = l;
              best = u;
            }
          }
          if (best < 0) break;
          ++wv[best];
          ++total;
        }
        // duration estimate: steps x nodes of the busiest thread x arithmetic per node
        int npt = 1;
        for (int u = 0; u < m; ++u) npt = std::max(npt, (b->inst[bn.members[u]].n + 64 * wv[u] - 1) / (64 * wv[u]));
        const int dd = b->inst[bn.members[0]].D & 0xff;
        plan.push_back(Planned{&bn, wv, (double)bn.steps * npt * (q * (dd + 3))});
      }
      // longest job first (longest-processing-time order for the queue)
      std::stable_sort(plan.begin(), plan.end(), [](const Planned& a, const Planned& c) { return a.est > c.est; });
      for (const Planned& pl : plan) {
        const Bin& bn = *pl.bin;
        const std::vector<int>& wv = pl.waves;
        const int m = (int)bn.members.size();
        L.maxsteps = std::max<int64_t>(L.maxsteps, bn.steps);
        L.est_max = std::max(L.est_max, pl.est);
        L.est_sum += pl.est;
        DevJob& jb = (++njobs, hjobs.emplace_back());
        jb.first = used;
        jb.count = m;
        jb.steps = (int)bn.steps;
        jb.degree = bn.variant;
        jb.bounded = bnd;
        jb.pad_ = 0;
        int t0 = 0, off = 0;
        for (int u = 0; u < m; ++u) {
          const int i = bn.members[u];
          const HostInst& h = b->inst[i];
          DevJobInst& it = (++used, hitems.emplace_back());
          it.addr = (uint64_t)(uintptr_t)state_cur(b, h);
          it.n = h.n;
          it.stride = h.stride;
          it.degree = h.D;
          it.inst = i;
          it.lds_off = off;
          it.t0 = t0;
          it.nt = 64 * wv[u];
          it.phib = bnd ? b->bnd_ptr[i] : 0;
          it.bkind = bnd ? (h.desc.bc == LBM_BC_DIRICHLET_EQ ? 1 : 2) : 0;
          it.layers = bnd ? b->bnd_layers : 0;
          it.pad_ = 0;
          t0 += it.nt;
          off += (int)(bytes_of(i) / es);
        }
        L.lds = std::max(L.lds, (size_t)off * es);
        L.block = std::max(L.block, t0);
      }
      L.count = njobs - L.first;
      if ((int)launches.size() >= kMaxResident) return LBM_ERR_UNSUPPORTED;
      launches.push_back(L);
    }
  }
  // Register-resident slabs and tiles.  Groups go side by side, each by its plan
  // for the whole GPU or for its share of the CUs, where every workgroup of all of
  // them finds a CU; else one after another, each over the whole GPU.  What cannot
  // be cut into slabs is advanced tile by tile.
  struct SegLaunch { int q; int prec; int code; SegPlan p; bool tile; int first, count, launches; size_t lds, at; int64_t blocks; double est; };
  std::vector<SegLaunch> segs;
  std::vector<DevSeg> xsv;
  std::vector<std::pair<int, int>> flips;   // (instance, buffer exchanges)
  size_t strips_need = 0;  // words
  int slab_cus = 0;        // workgroups of all slab launches (even_places)
  double all_work = 1.0;   // node updates x operations of all register groups
  auto work_of = [&](const std::tuple<int, int, int>& key, const std::vector<int>& g) {
    double w = 0.0;
    for (int i : g) w += (double)steps[i] * b->inst[i].n;
    return w * (std::get<0>(key) * ((std::get<2>(key) & 0xff) + 3));
  };
  for (const auto* part : {&reg, &spread})
    for (const auto& group : *part) all_work += work_of(group.first, group.second);
  // One group's launches: slabs, or tiles.  `together`: the workgroups of all slab
  // groups find a CU at once, so that the group is one launch beside the others;
  // else it has the GPU to itself, in as many launches as that takes.
  bool in_chunks = false;   // a group's steps are cut into chunks: its launches must keep their order
  bool beside = true;       // slabs leave CUs to whole instances, rather than taking the GPU after them
  auto add_segs = [&](const std::tuple<int, int, int>& key, const std::vector<int>& g, const SegPlan& p, bool together,
                      bool tile) -> lbm_status {
    const int q = std::get<0>(key), pr = std::get<1>(key), code = std::get<2>(key), R = p.f.R;
    const size_t es = pr != 0 ? 4 : 8;
    const int hg = reg_halo(q, R, p.f.s) + p.extra;
    SegLaunch L{q, pr, code, p, tile, (int)xsv.size(), 0, 1, (size_t)p.waves * reg_strip(q, R, p.f.s) * es, 0, 0, 0.0};
    int per_cu = 0;
    LBM_HIP(seg_occupancy(q, pr, code, p.f.wide, 64 * p.waves, L.lds, &per_cu));
    if (per_cu < 1) return LBM_ERR_UNSUPPORTED;
    const int64_t capacity = together ? b->lim.cus : (int64_t)std::min(per_cu, p.per_cu) * b->lim.cus;
    SlabChunks cut;
    if (!tile) {
      std::vector<std::pair<int, int64_t>> mem;
      for (int i : g) mem.push_back({seg_count(p, q, b->inst[i].n, false), steps[i]});
      cut = slab_chunks(mem, capacity);
      in_chunks |= cut.chunks > 1;
    }
    auto close = [&] {
      if (L.count == 0) return;
      if (!tile) {
        L.at = strips_need;
        strips_need += (size_t)L.count * 4 * (hg + 1) * R * q * (es / 4);
        slab_cus += (int)even_places(L.count, b->lim.cus);
      }
      segs.push_back(L);
      L.first = (int)xsv.size();
      L.count = 0;
      L.blocks = 0;
      L.est = 0.0;
    };
    const int wave_nodes = (p.per_cu * p.waves + 3) / 4;
    std::vector<size_t> in_launch(b->inst.size(), SIZE_MAX);   // the launch of an instance's last item
    for (int c = 0; c < cut.chunks; ++c)
      for (int i : g) {
        const HostInst& h = b->inst[i];
        const int64_t st = chunk_steps(steps[i], cut.chunks, c);
        if (st == 0) continue;
        const int ks = seg_count(p, q, h.n, tile), all = (h.n + R - 1) / R;
        if (!tile && (L.count + ks > cut.fill || in_launch[i] == segs.size())) close();
        in_launch[i] = segs.size();
        L.est = std::max(L.est, (double)st * wave_nodes * p.f.cost);
        L.blocks = std::max<int64_t>(L.blocks, (st + p.sx - 1) / p.sx);
        const int from = h.cur ^ (c & 1);   // each earlier chunk flipped the buffer once
        for (int m = 0; m < ks; ++m) {
          const int l0 = (int)((int64_t)all * m / ks), l1 = (int)((int64_t)all * (m + 1) / ks);
          DevSeg sg{};
          sg.in = (uint64_t)(uintptr_t)state_at(b, h, from);
          sg.out = (uint64_t)(uintptr_t)state_at(b, h, 1 - from);
          sg.n = h.n;
          sg.stride = h.stride;
          sg.inst = i;
          sg.x0 = l0 * R;
          sg.len = std::min(l1 * R, h.n) - sg.x0;
          sg.lanes = l1 - l0 + 2 * p.extra;
          sg.extra = p.extra;
          sg.over = m + 1 == ks ? all * R - h.n : 0;
          sg.over_left = m == 0 ? all * R - h.n : 0;
          const int cap = 64 - 2 * reg_halo(q, R, p.f.s);
          sg.waves = (sg.lanes + cap - 1) / cap;
          sg.steps = (int)st;
          sg.left = L.count + (m + ks - 1) % ks;
          sg.right = L.count + (m + 1) % ks;
          xsv.push_back(sg);
        }
        L.count += ks;
        const int turns = tile ? (int)((st + p.sx - 1) / p.sx) : 1;
        L.launches = std::max(L.launches, turns);
        flips.push_back({i, turns});
      }
    close();
    return LBM_OK;
  };
  if (!spread.empty() || !rtile.empty()) {
    const int slab_steps = b->tile_steps > 0 ? (b->tile_steps + 1) / 2 * 2 : 0;   // even: strips in natural layout
    auto sizes_of = [&](const std::vector<int>& g) {
      std::map<int, int> sizes;
      for (int i : g) ++sizes[b->inst[i].n];
      return sizes;
    };
    auto chunks_of = [&](const std::vector<int>& g) {
      int64_t longest = 0;
      for (int i : g) longest = std::max(longest, steps[i]);
      return (int)std::max<int64_t>(1, std::min<int64_t>(kMaxSlabChunks, longest / kMinSlabChunk));
    };
    auto plan = [&](const std::tuple<int, int, int>& key, const std::map<int, int>& sizes, int cus, int want, bool tile,
                    int chunks, SegPlan* p) {
      std::vector<int64_t> from{std::get<0>(key), std::get<1>(key), std::get<2>(key), cus, want, b->tile_wgs, tile, chunks};
      for (const auto& [n, times] : sizes) {
        from.push_back(n);
        from.push_back(times);
      }
      const auto it = memo.segs.find(from);
      if (it == memo.segs.end()) {
        // (steps asked for that no segment's halos hold are halved)
        bool found;
        while (!(found = seg_plan(std::get<0>(key), std::get<1>(key), std::get<2>(key), sizes, cus, want, b->tile_wgs, tile,
                                  chunks, p)) &&
               want > (tile ? 1 : 2))
          want = tile ? want / 2 : want / 4 * 2;
        if (memo.segs.size() >= 256) memo.segs.clear();
        memo.segs[std::move(from)] = {found, *p};
        return found;
      }
      *p = it->second.second;
      return it->second.first;
    };
    auto ring_time = [&](const std::tuple<int, int, int>& key, int n, double* step) {
      const auto of = std::make_tuple(std::get<0>(key), std::get<1>(key), std::get<2>(key), n);
      auto it = memo.ring_steps.find(of);
      if (it == memo.ring_steps.end()) {
        if (memo.ring_steps.size() >= 4096) memo.ring_steps.clear();
        std::pair<double, double> t;
        t.first = ring_step(std::get<0>(key), std::get<1>(key), std::get<2>(key), n, &t.second);
        it = memo.ring_steps.insert({of, t}).first;
      }
      *step = it->second.second;
      return it->second.first;
    };
    // Whole instances instead where enough of them fill the GPU: the group's
    // waves over the CUs, no exchange between workgroups and no rounds of
    // launches.
    for (auto it = spread.begin(); it != spread.end();) {
      const auto& key = it->first;
      double longest = 0.0, sum = 0.0;
      for (int i : it->second) {
        double step = 0.0;
        const double one = ring_time(key, b->inst[i].n, &step);
        longest = std::max(longest, one);
        sum += step / b->lim.cus;
      }
      SegPlan p;
      const bool whole = b->path == 0 && longest < 1e29 && b->tile_steps == 0 && b->tile_wgs == 0 &&
                         (!plan(key, sizes_of(it->second), b->lim.cus, slab_steps, false, chunks_of(it->second), &p) ||
                          std::max(longest, sum) < p.est);
      if (whole) {
        std::vector<int>& to = reg[key];
        to.insert(to.end(), it->second.begin(), it->second.end());
      }
      it = whole ? spread.erase(it) : std::next(it);
    }
    // what no slab plan takes goes by tiles
    std::vector<SegPlan> plans;     // over the whole GPU, then those taken
    for (auto it = spread.begin(); it != spread.end();) {
      const auto& key = it->first;
      std::vector<int>& g = it->second;
      SegPlan p;
      if (!plan(key, sizes_of(g), b->lim.cus, slab_steps, false, chunks_of(g), &p)) {
        std::map<int, bool> cuts;
        for (int i : g) {
          const int n = b->inst[i].n;
          if (!cuts.count(n)) cuts[n] = plan(key, {{n, 1}}, b->lim.cus, slab_steps, false, 1, &p);
        }
        std::vector<int> keep;
        for (int i : g) {
          if (cuts[b->inst[i].n])
            keep.push_back(i);
          else
            rtile[key].push_back(i);
        }
        g.swap(keep);
        if (!g.empty() && !plan(key, sizes_of(g), b->lim.cus, slab_steps, false, chunks_of(g), &p)) {
          for (int i : g) rtile[key].push_back(i);
          g.clear();
        }
      }
      if (!g.empty()) plans.push_back(p);
      it = g.empty() ? spread.erase(it) : std::next(it);
    }
    for (const auto* part : {&spread, &rtile})
      for (const auto& group : *part) {
        lbm_status st = ensure_second_buffer(b, std::get<1>(group.first) != 0);
        if (st != LBM_OK) return st;
      }
    // Several groups: each by its plan for the whole GPU if all their
    // workgroups find a CU there, else by its share, else one after another.
    auto places_of = [&](const std::vector<SegPlan>& ps) {
      int64_t total = 0;
      size_t at = 0;
      for (const auto& [key, g] : spread) {
        int64_t wgs = 0;
        for (int i : g) wgs += seg_count(ps[at], std::get<0>(key), b->inst[i].n, false);
        total += even_places(wgs, b->lim.cus);
        ++at;
      }
      return total;
    };
    bool together = places_of(plans) <= b->lim.cus;
    if (spread.size() > 1 && !together) {
      // (shares in whole CUs of every XCD, the largest cut while they exceed the GPU)
      const int unit = xcd_count(b->lim.cus);
      std::vector<SegPlan> shared;
      std::vector<int> share, least;
      int sum = 0;
      for (const auto& [key, g] : spread) {
        least.push_back((int)even_places(g.size(), b->lim.cus));
        const double part = b->lim.cus * work_of(key, g) / all_work / unit;
        share.push_back(std::max(least.back(), unit * (int)std::lround(part)));
        sum += share.back();
      }
      while (sum > b->lim.cus) {
        size_t top = share.size();
        for (size_t k = 0; k < share.size(); ++k)
          if (share[k] > least[k] && (top == share.size() || share[k] > share[top])) top = k;
        if (top == share.size()) break;
        share[top] -= unit;
        sum -= unit;
      }
      bool ok = sum <= b->lim.cus;
      for (const auto& [key, g] : spread) {
        SegPlan p;
        ok = ok && plan(key, sizes_of(g), share[shared.size()], slab_steps, false, 1, &p);
        shared.push_back(p);
      }
      if (ok && places_of(shared) <= b->lim.cus) {
        plans.swap(shared);
        together = true;
      }
    }
    beside = together;
    size_t at = 0;
    for (const auto& [key, g] : spread) {
      lbm_status st = add_segs(key, g, plans[at], together, false);
      if (st != LBM_OK) return st;
      ++at;
    }
    for (const auto& [key, g] : rtile) {
      SegPlan p;
      if (!plan(key, sizes_of(g), b->lim.cus, b->tile_steps, true, 1, &p)) return LBM_ERR_UNSUPPORTED;
      lbm_status st = add_segs(key, g, p, false, true);
      if (st != LBM_OK) return st;
    }
  }
  // Register-resident jobs: whole instances of one variant, step count and width,
  // bin-packed by waves.  They share the GPU with slabs only where those leave it:
  // slab launches that fill it start when the whole instances have ended (512
  // Kawahara and K(2,2) grids, FP32 storage, 5000 steps: the 2048-node half took
  // 15.5 ms on a third of the CUs with slabs waiting, 9.8 ms on all of them; the
  // pass 58.5 -> 52.7 ms).
  if (!beside) {
    all_work = 1.0;
    for (const auto& group : reg) all_work += work_of(group.first, group.second);
  }
  std::vector<double> reg_job_est;
  double reg_est = 0.0;    // estimated CU time of all register launches
  int64_t reg_jobs = 0;
  for (const auto& group : reg) {
    const int q = std::get<0>(group.first), pr = std::get<1>(group.first), code = std::get<2>(group.first);
    const std::vector<int>& g = group.second;
    const int es = pr != 0 ? 4 : 8;
    const bool bounded = (code >> 16) != 0;
    // the CUs that are this group's by its share of the pass's work
    const double cus = std::max(1.0, b->lim.cus * work_of(group.first, group.second) / all_work);
    std::vector<int64_t> from{q, pr, code, (int64_t)std::lround(64.0 * cus)};
    for (int i : g) {
      from.push_back(b->inst[i].n);
      from.push_back(steps[i]);
    }
    if (memo.ring_instances > 65536) {
      memo.rings.clear();
      memo.ring_instances = 0;
    }
    memo.ring_instances += g.size();
    RingPlan& ring = memo.rings[std::move(from)];
    if (!ring.found) ring.found = plan_rings(b, q, pr, code, g, steps, cus, &ring);
    if (!ring.found) return LBM_ERR_UNSUPPORTED;
    const std::vector<RegFit>& fit = ring.fit;
    std::vector<int> order(g.size());
    for (size_t u = 0; u < g.size(); ++u) order[u] = (int)u;
    std::stable_sort(order.begin(), order.end(), [&](int a, int c) {
      if (steps[g[a]] != steps[g[c]]) return steps[g[a]] > steps[g[c]];
      if (fit[a].R != fit[c].R) return fit[a].R > fit[c].R;
      if (fit[a].s != fit[c].s) return fit[a].s > fit[c].s;
      return fit[a].waves > fit[c].waves;
    });
    // first fit, decreasing; `open` holds the first bin of this width with room
    // for a given number of waves
    struct Bin { int waves; std::vector<int> members; };
    std::vector<Bin> bins;
    size_t open[17] = {};
    for (size_t o = 0; o < order.size(); ++o) {
      const int u = order[o], w = fit[u].waves;
      if (o == 0 || steps[g[u]] != steps[g[order[o - 1]]] || fit[u].R != fit[order[o - 1]].R ||
          fit[u].s != fit[order[o - 1]].s)
        for (size_t& v : open) v = bins.size();
      size_t& v = open[w];
      while (v < bins.size() && bins[v].waves + w > ring.job_waves) ++v;
      if (v == bins.size()) bins.push_back(Bin{0, {}});
      bins[v].waves += w;
      bins[v].members.push_back(u);
    }
    auto job_est = [&](const Bin& bn) {
      return (double)steps[g[bn.members[0]]] * ((bn.waves + 3) / 4) * fit[bn.members[0]].cost;
    };
    std::stable_sort(bins.begin(), bins.end(), [&](const Bin& a, const Bin& c) { return job_est(a) > job_est(c); });
    Launch L{q, pr, code, njobs, 0, 0, 64, 0, 0.0, 0.0, true, ring.wide, ring.jobs_per_cu, 0, 0, 0, 0, 0.0};
    for (const Bin& bn : bins) {
      const RegFit& f0 = fit[bn.members[0]];
      const int64_t st = steps[g[bn.members[0]]];
      const double est = job_est(bn);
      L.maxsteps = std::max<int64_t>(L.maxsteps, st);
      L.est_max = std::max(L.est_max, est);
      L.est_sum += est;
      L.issue += (double)st * bn.waves * (f0.cost - f0.R * q);
      DevJob& jb = (++njobs, hjobs.emplace_back());
      jb = DevJob{};
      jb.first = nsegs;
      jb.count = (int)bn.members.size();
      jb.steps = (int)st;
      jb.degree = code;
      jb.nodes = f0.R;
      jb.s_per = f0.s;
      int w0 = 0, off = 0;
      for (int u : bn.members) {
        const int i = g[u];
        const HostInst& h = b->inst[i];
        DevSeg& sg = (++nsegs, hsegs.emplace_back());
        sg = DevSeg{};
        sg.in = sg.out = (uint64_t)(uintptr_t)state_cur(b, h);
        sg.n = sg.len = h.n;
        sg.stride = h.stride;
        sg.inst = i;
        sg.lanes = fit[u].lanes;
        sg.over = fit[u].over;
        sg.w0 = w0;
        sg.waves = fit[u].waves;
        sg.lds_off = off;
        if (bounded) {
          sg.layers = b->bnd_layers;
          sg.kind = h.desc.bc == LBM_BC_DIRICHLET_EQ ? 1 : 2;
          sg.rows = b->bnd_ptr[i];
        }
        w0 += fit[u].waves;
        off += fit[u].waves * (reg_strip(q, f0.R, f0.s) + (bounded ? bound_lds(es) : 0));
      }
      L.lds = std::max(L.lds, (size_t)off * es);
      L.block = std::max(L.block, 64 * w0);
    }
    L.count = njobs - L.first;
    reg_est += L.est_sum;
    reg_jobs += L.count;
    launches.push_back(L);
    for (const Bin& bn : bins) reg_job_est.push_back(job_est(bn));
  }
  // Queue items of the register launches.  Where the jobs of all launches
  // outnumber the CUs, a launch takes the share of the workgroups that is its
  // share of the work, and its jobs are laid end to end over them: each
  // workgroup gets the same time, and the job that crosses from one to the next
  // is split -- its first steps open the next workgroup's time, its last close
  // the previous one's, so that the second part has the first one's result
  // before it starts (preemptive scheduling on identical machines, McNaughton
  // 1959; fixed step chunks, with a queue barely longer than the workgroups,
  // spent a third of the time waiting for the chunk before).  Items are taken
  // in the order of their planned start.
  // The work by which launches share the CUs is the operations their waves issue: a
  // step is priced with q operations more per node (a population's update is two
  // operations, issued as one FMA), which is a larger part of a small table's (4096
  // KdV and mKdV grids, FP32 arithmetic: 48.5 ms shared by price, 45.3 by issue).
  std::vector<DevItem> parts;
  std::vector<double> issue;
  std::vector<int> most;
  for (Launch& L : launches) {
    if (!L.reg) continue;
    int per_cu = 0;
    LBM_HIP(reg_occupancy(L.q, L.prec, L.code, L.wide, L.block, L.lds, &per_cu));
    if (per_cu < 1) return LBM_ERR_UNSUPPORTED;
    L.per_cu = std::min(per_cu, L.per_cu);
    issue.push_back(L.issue);
    most.push_back((L.count + L.per_cu - 1) / L.per_cu);
  }
  const std::vector<int> shares = cu_shares(issue, most, b->lim.cus);
  size_t job0 = 0, nth = 0;
  for (Launch& L : launches) {
    if (!L.reg) continue;
    const double* est = &reg_job_est[job0];
    job0 += L.count;
    const int per_cu = L.per_cu;
    L.grid = std::min<int>(L.count, per_cu * b->lim.cus);
    if (reg_jobs > b->lim.cus)
      L.grid = std::max(1, std::min(L.grid, shares.empty() ? (int)std::lround(per_cu * b->lim.cus * L.est_sum / reg_est)
                                                           : per_cu * shares[nth]));
    ++nth;
    if (b->res_grid > 0) L.grid = std::min(L.grid, b->res_grid);
    L.part0 = (int)parts.size();
    const DevJob* jobs = hjobs.data() + L.first;
    if (b->res_chunks > 0) {   // chunks as asked, chunk by chunk
      for (int c = 0; c < b->res_chunks; ++c)
        for (int k = 0; k < L.count; ++k) {
          const int base = jobs[k].steps / b->res_chunks, rem = jobs[k].steps % b->res_chunks;
          const int st = base + (c < rem ? 1 : 0);
          if (st == 0 && c > 0) continue;
          const int next = base + (c + 1 < rem ? 1 : 0);
          parts.push_back(DevItem{k, c, st, c * base + std::min(c, rem), c + 1 < b->res_chunks && next > 0 ? 1 : 0});
        }
    } else if (L.grid >= L.count) {
      for (int k = 0; k < L.count; ++k) parts.push_back(DevItem{k, 0, jobs[k].steps, 0, 0});
    } else {
      // (a job is not split for a few steps, and what that wastes of the even
      // share must not pile up behind the last workgroup: 300 equal jobs on 256
      // took two rounds.  So the share is raised until all of them end by it.)
      struct Planned { double start; DevItem item; };
      std::vector<Planned> plan, trial;
      double least = 0.0;
      for (int slack = 0; slack <= 16; ++slack) {
        const double span = std::max(L.est_sum / L.grid, L.est_max) * (1.0 + 0.01 * slack);
        double t = 0.0, end = 0.0;   // of the current workgroup's last item; of the latest so far
        int used_wgs = 1;
        trial.clear();
        for (int k = 0; k < L.count; ++k) {
          const int st = jobs[k].steps;
          int second = st;   // steps that stay with this workgroup, at its end
          if (t + est[k] > span * (1.0 + 1e-9) && used_wgs < L.grid) {
            second = (int)(st * ((span - t) / est[k]));
            if (second < st / 32 || second < 8) second = 0;
            if (st - second < st / 32 || st - second < 8) second = st;
          }
          const int first = st - second;
          if (second > 0) {
            trial.push_back({t, DevItem{k, first > 0 ? 1 : 0, second, first, 0}});
            t += est[k] * second / st;
            end = std::max(end, t);
          }
          if (first > 0) {
            trial.push_back({0.0, DevItem{k, 0, first, 0, second > 0 ? 1 : 0}});
            t = est[k] * first / st;
            end = std::max(end, t);
            ++used_wgs;
          }
        }
        if (slack == 0 || end < least) {
          least = end;
          plan.swap(trial);
        }
        if (end <= span * (1.0 + 1e-9)) break;
      }
      std::stable_sort(plan.begin(), plan.end(), [](const Planned& x, const Planned& y) {
        return x.start != y.start ? x.start < y.start : x.item.part < y.item.part;
      });
      for (const Planned& pl : plan) parts.push_back(pl.item);
    }
    L.parts = (int)parts.size() - L.part0;
    for (int k = L.part0; k < (int)parts.size(); ++k) L.partsteps = std::max<int64_t>(L.partsteps, parts[k].steps);
  }
  // temporal blocking plan per (q, prec) group
  struct TileGroup { int q; int prec; int first, ntiles, tfirst, tcount, s, halo, launches, block; size_t lds; double est; };
  std::vector<TileGroup> tgroups;
  std::vector<DevTile> tvec;
  // tile-instance records of this pass (the tiled path: one per instance; the
  // slab path: one per instance and step chunk), copied to slot k below
  std::vector<DevTileInst> htin;
  int tin_used = 0;
  // slab plan per (q, prec): cooperative launches of at most `capacity` slabs
  // (every workgroup of a launch resident at once), run one after another on
  // one lane; an instance whose slabs exceed one launch, or whose slabs would
  // be narrower than a halo, goes to temporal blocking instead.  What needs
  // several launches goes in step chunks (slab_chunks).
  struct SlabLaunch { int q; int prec; int code; int first, count, cap, s, halo, block; size_t lds; size_t xoff; int foff; double est; };
  std::vector<SlabLaunch> slaunch;
  std::vector<DevSlab> svec;
  size_t xbuf_need = 0;
  int flags_need = 0;
  int min_per_cu = 1 << 30;
  const int tin_slab0 = tin_used;
  std::vector<int> slab_insts;
  for (const auto& group : slb) {
    {
      const int qq = std::get<0>(group.first), pr = std::get<1>(group.first), code = std::get<2>(group.first);
      const int wgs = std::get<3>(group.first);
      const std::vector<int>& g = group.second;
      const int q = qq, H = q / 2;
      const size_t es = pr ? sizeof(float) : sizeof(double);
      const int W = (int)((b->lim.lds_max / (size_t)wgs - 16) / (lds_stride(q) * es));
      int sp = b->tile_steps > 0 ? (b->tile_steps + 1) / 2 * 2 : 16;   // even: strips in natural layout
      while (sp > 2 && W - 2 * sp * H < 2 * sp * H) sp -= 2;
      const int halo = sp * H;
      const int cmax = W - 2 * halo;
      // two or more nodes per thread; if the kernel's registers do not let
      // `wgs` workgroups of that size share a CU (its LDS is cut for wgs), take
      // the largest smaller workgroup (a multiple of one wave, not below 256
      // threads) that lets them, so no part of the LDS stays unused
      int block = std::min(1024, std::max(64, (W / 2 + 63) / 64 * 64));
      const size_t lds = (size_t)W * lds_stride(q) * es + 16;
      int per_cu = 0;
      if (cmax < halo || slab_occupancy(q, pr, code, block, lds, &per_cu) != hipSuccess) per_cu = 0;
      for (int nb = block - 64; per_cu > 0 && per_cu < wgs && nb >= 256; nb -= 64) {
        int pc = 0;
        if (slab_occupancy(q, pr, code, nb, lds, &pc) != hipSuccess) break;
        if (pc > per_cu) {
          block = nb;
          per_cu = pc;
        }
      }
      const int capacity = std::min(per_cu * b->lim.cus, kMaxSlabs);
      if (per_cu > 0) min_per_cu = std::min(min_per_cu, per_cu);
      SlabLaunch L{q, pr, code, (int)svec.size(), 0, capacity, sp, halo, block, lds, 0, 0, 0.0};
      // the instances that take slabs, their slab counts and core widths
      std::vector<std::pair<int, int>> mem;   // (instance, slabs)
      for (int i : g) {
        const HostInst& h = b->inst[i];
        const int ks = cmax > 0 ? (h.n + cmax - 1) / cmax : 0;
        const int core = ks > 0 ? (h.n + ks - 1) / ks : 0;
        if (ks < 1 || ks > capacity || core < halo || h.n - (ks - 1) * core < halo) {
          til[qq][pr].push_back(i);
          continue;
        }
        mem.push_back({i, ks});
      }
      std::vector<std::pair<int, int64_t>> cost;
      for (const auto& [i, ks] : mem) cost.push_back({ks, steps[i]});
      const SlabChunks cut = slab_chunks(cost, capacity);
      std::vector<size_t> in_launch(b->inst.size(), SIZE_MAX);   // the launch of an instance's last item
      for (int c = 0; c < cut.chunks; ++c) {
        for (const auto& [i, ks] : mem) {
          const HostInst& h = b->inst[i];
          const int64_t st = chunk_steps(steps[i], cut.chunks, c);
          if (st == 0) continue;
          const int core = (h.n + ks - 1) / ks;
          if (L.count + ks > cut.fill || in_launch[i] == slaunch.size()) {
            slaunch.push_back(L);
            L.first = (int)svec.size();
            L.count = 0;
            L.est = 0.0;
          }
          in_launch[i] = slaunch.size();
          // duration estimate, in the unit of the resident jobs' (steps x nodes
          // of the busiest thread x arithmetic per node)
          L.est = std::max(L.est, (double)st * ((core + 2 * halo + block - 1) / block) * (q * ((h.D & 0xff) + 3)));
          DevTileInst ti{};
          ti.off = h.off;
          ti.n = h.n;
          ti.stride = h.stride;
          ti.steps = (int)st;
          ti.cur0 = h.cur ^ (c & 1);   // each earlier chunk flipped the buffer once
          ti.degree = h.D;
          ti.inst = i;
          htin.push_back(ti);
          for (int m = 0; m < ks; ++m) {
            DevSlab sl;
            sl.ti = tin_used;
            sl.x0 = m * core;
            sl.core = std::min(core, h.n - m * core);
            sl.left = L.count + (m + ks - 1) % ks;
            sl.right = L.count + (m + 1) % ks;
            sl.pad_ = 0;
            svec.push_back(sl);
          }
          L.count += ks;
          ++tin_used;
          if (c == 0) slab_insts.push_back(i);
        }
      }
      if (L.count) slaunch.push_back(L);
    }
  }
  // every launch its own strip and flag region (launches may run side by side)
  for (SlabLaunch& S : slaunch) {
    S.xoff = xbuf_need;
    S.foff = flags_need;
    xbuf_need += ((size_t)S.count * 4 * S.q * S.halo * (S.prec ? sizeof(float) : sizeof(double)) + 255) / 256 * 256;
    flags_need += S.count;
  }
  // side by side only while all their workgroups fit the GPU twice over;
  // otherwise one after another (each launch alone fits by construction)
  int64_t total_slabs = 0, total_places = 0, total_cap = 0;
  for (const SlabLaunch& S : slaunch) {
    total_slabs += S.count;
    total_places += even_places(S.count, b->lim.cus);
    total_cap += S.cap;
  }
  bool slab_side_by_side =
      segs.empty() && slaunch.size() > 1 && 2 * total_slabs <= (int64_t)min_per_cu * b->lim.cus &&
      total_places <= (int64_t)min_per_cu * b->lim.cus;
  // A small pass (a serving round) whose slab launches would run one after
  // another, each less than half full on average, is bound by that sequence of
  // mostly idle launches; temporal blocking has no co-residency condition, so
  // its groups run side by side: those instances take it instead (results are
  // the same bit for bit).  Launches that fill the GPU keep their slabs.
  if (latency && slaunch.size() > 1 && !slab_side_by_side && 2 * total_slabs < total_cap) {
    for (int i : slab_insts) til[b->inst[i].q][b->inst[i].prec].push_back(i);
    tin_used = tin_slab0;
    htin.resize(tin_slab0);
    svec.clear();
    slaunch.clear();
    xbuf_need = 0;
    flags_need = 0;
    slab_side_by_side = false;
  }
  if (!svec.empty() || !xsv.empty()) {
    if (xbuf_need > b->xbuf_bytes || flags_need > b->sflags_cap || strips_need > b->strips_cap) {
      // grow the exchange buffers; earlier passes must be done with them
      LBM_HIP(hipStreamSynchronize(b->stream));
      if (strips_need > b->strips_cap) {
        hipFree(b->strips);
        b->strips = nullptr;
        b->strips_cap = 0;
        if (hipMalloc(&b->strips, sizeof(uint64_t) * strips_need) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
        b->strips_cap = strips_need;
        b->strip_tag = UINT32_MAX;   // to be cleared
      }
      if (xbuf_need > b->xbuf_bytes) {
        hipFree(b->xbuf);
        b->xbuf = nullptr;
        b->xbuf_bytes = 0;
        if (hipMalloc(&b->xbuf, xbuf_need) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
        b->xbuf_bytes = xbuf_need;
      }
      if (flags_need > b->sflags_cap) {
        hipFree(b->sflags);
        b->sflags = nullptr;
        b->sflags_cap = 0;
        if (hipMalloc(&b->sflags, sizeof(int) * flags_need) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
        b->sflags_cap = flags_need;
      }
    }
    for (const auto& group : slb) {
      lbm_status st = ensure_second_buffer(b, std::get<1>(group.first) != 0);
      if (st != LBM_OK) return st;
    }
  }
  for (int qq = 4; qq < 8; ++qq) {
    for (int pr = 0; pr < 3; ++pr) {
      const std::vector<int>& g = til[qq][pr];
      if (g.empty()) continue;
      const int q = qq, H = q / 2;
      const size_t es = pr ? sizeof(float) : sizeof(double);
      const int wgs = b->tile_wgs > 0 ? b->tile_wgs : 2;
      const int W = (int)(b->lim.lds_max / (size_t)wgs / (lds_stride(q) * es));
      // tile core: as wide as the LDS share allows, but narrow enough that the
      // group yields about 4 tiles per CU (a few large instances would otherwise
      // leave most CUs idle); halo / core kept below 1/4
      int64_t nodes = 0;
      for (int i : g) nodes += b->inst[i].n;
      const int want = (int)std::max<int64_t>(256, nodes / (4 * (int64_t)b->lim.cus));
      int sp = b->tile_steps > 0 ? b->tile_steps : 32;
      while (sp > 1 && (W - 2 * sp * H < 2 * sp * H || (b->tile_steps == 0 && 8 * sp * H > want))) sp /= 2;
      const int halo = sp * H;
      const int core = std::max(1, std::min(W - 2 * halo, want));
      TileGroup G{q, pr, (int)tvec.size(), 0, tin_used, 0, sp, halo, 0, kBlock, 0, 0.0};
      int64_t maxsteps = 0;
      int maxcore = 1, maxd = 0;
      for (int i : g) {
        const HostInst& h = b->inst[i];
        htin.emplace_back();
        DevTileInst& ti = htin.back();
        ti.off = h.off;
        ti.n = h.n;
        ti.stride = h.stride;
        ti.steps = (int)steps[i];
        ti.cur0 = h.cur;
        ti.degree = h.D;
        ti.inst = i;
        const int c = std::min(core, h.n);
        for (int x0 = 0; x0 < h.n; x0 += c) {
          DevTile t{tin_used, x0, std::min(c, h.n - x0), 0};
          tvec.push_back(t);
        }
        maxcore = std::max(maxcore, c);
        maxd = std::max(maxd, h.D & 0xff);
        maxsteps = std::max<int64_t>(maxsteps, steps[i]);
        ++tin_used;
      }
      G.ntiles = (int)tvec.size() - G.first;
      G.tcount = tin_used - G.tfirst;
      G.launches = (int)((maxsteps + sp - 1) / sp);
      G.lds = (size_t)lds_stride(q) * (maxcore + 2 * halo) * es;
      // two or more nodes per thread
      G.block = std::min(kBlock, std::max(64, ((maxcore + 2 * halo) / 2 + 63) / 64 * 64));
      // duration estimate (as the resident jobs'): the launches' steps x nodes of
      // the busiest thread x arithmetic per node x rounds of tiles over the CUs
      G.est = (double)G.launches * sp * ((maxcore + 2 * halo + G.block - 1) / G.block) * (q * (maxd + 3)) *
              ((G.ntiles + 2 * b->lim.cus - 1) / (2 * b->lim.cus));
      tgroups.push_back(G);
    }
  }
  if (!tvec.empty()) {
    for (int qq = 4; qq < 8; ++qq)
      for (int pr = 0; pr < 3; ++pr) {
        lbm_status st = til[qq][pr].empty() ? LBM_OK : ensure_second_buffer(b, pr != 0);
        if (st != LBM_OK) return st;
      }
  }

  // every table of the pass in one copy (five copies and clears took 10 us more)
  size_t need = 0;
  auto place = [&](size_t bytes) {
    const size_t at = need;
    need += (bytes + 15) / 16 * 16;
    return at;
  };
  const size_t words = launches.size() + (size_t)njobs;   // a counter of each launch, parts done of each job
  const size_t words_at = place(sizeof(int) * words), jobs_at = place(sizeof(DevJob) * hjobs.size());
  const size_t items_at = place(sizeof(DevJobInst) * hitems.size()), segs_at = place(sizeof(DevSeg) * hsegs.size());
  const size_t parts_at = place(sizeof(DevItem) * parts.size()), xsegs_at = place(sizeof(DevSeg) * xsv.size());
  const size_t slabs_at = place(sizeof(DevSlab) * svec.size()), tiles_at = place(sizeof(DevTile) * tvec.size());
  const size_t tinsts_at = place(sizeof(DevTileInst) * htin.size());
  if (need > b->tables_cap) {
    const lbm_status ts = alloc_pass_tables(b, 2 * need);
    if (ts != LBM_OK) return ts;
  }
  unsigned char* th = b->tables_host + (size_t)k * b->tables_cap;
  unsigned char* td = b->tables + (size_t)k * b->tables_cap;
  auto fill = [&](size_t at, const auto& v) {
    if (!v.empty()) std::memcpy(th + at, v.data(), sizeof(v[0]) * v.size());
  };
  std::memset(th + words_at, 0, sizeof(int) * words);
  fill(jobs_at, hjobs);
  fill(items_at, hitems);
  fill(segs_at, hsegs);
  fill(parts_at, parts);
  fill(xsegs_at, xsv);
  fill(slabs_at, svec);
  fill(tiles_at, tvec);
  fill(tinsts_at, htin);
  LBM_HIP(hipEventRecord(b->ev0, b->stream));
  if (need > 0) LBM_HIP(hipMemcpyAsync(td, th, need, hipMemcpyHostToDevice, b->stream));
  int* counters = reinterpret_cast<int*>(td + words_at);
  int* done_all = counters + launches.size();
  const DevJob* djobs = reinterpret_cast<const DevJob*>(td + jobs_at);
  const DevJobInst* ditems = reinterpret_cast<const DevJobInst*>(td + items_at);
  const DevSeg* dsegs = reinterpret_cast<const DevSeg*>(td + segs_at);
  const DevItem* dparts = reinterpret_cast<const DevItem*>(td + parts_at);
  const DevSeg* dxsegs = reinterpret_cast<const DevSeg*>(td + xsegs_at);
  const DevSlab* ds = reinterpret_cast<const DevSlab*>(td + slabs_at);
  const DevTile* dtiles = reinterpret_cast<const DevTile*>(td + tiles_at);
  const DevTileInst* dti_all = reinterpret_cast<const DevTileInst*>(td + tinsts_at);
  // Lanes: every resident launch, every tiled group and every slab launch (or
  // the chain of slab launches, when they cannot run side by side) is one
  // item; with more items than lanes, each item in order of its duration
  // estimate, longest first, goes to the lane with the least estimated work
  // so far (longest-processing-time scheduling).  With no more items than
  // lanes each has a lane of its own, issued in plan order (launches that each
  // fill the GPU take its CUs in that order: the 4096-instance KdV/mKdV pass
  // ran 1% longer with the longer mKdV launch first).  The fork is recorded
  // after all table uploads above.
  // slab launches: each needs all its workgroups resident at once.  Each fits
  // the GPU alone, and the other lanes' kernels never wait on it, so its
  // workgroups all get CUs once those kernels retire; two slab launches side
  // by side could each hold CUs the other waits for, so they share a lane, in
  // order, unless all of them fit the GPU twice over
  // (register slabs plan a place for every workgroup: side by side as long as
  // there is a CU for each of all their workgroups -- one that waits for a place
  // then has an empty CU, or a CU whose kernel waits for no slab -- and no group
  // is cut into step chunks, which read what the chunk before them wrote)
  // kind 0 resident, 1 tiled, 2 slab (-1: the chain), 3 register slab or tile
  struct LaneItem { int kind; int idx; double est; };
  std::vector<LaneItem> items;
  const bool segs_side_by_side = slaunch.empty() && !in_chunks && slab_cus <= b->lim.cus;
  double chain_est = 0.0;
  bool chain = false;
  for (size_t l = 0; l < segs.size(); ++l) {
    if (segs[l].tile || segs_side_by_side) {
      items.push_back({3, (int)l, segs[l].est});
    } else {
      chain_est += segs[l].est;
      chain = true;
    }
  }
  for (size_t l = 0; l < launches.size(); ++l) {
    const Launch& L = launches[l];
    items.push_back({0, (int)l, std::max(L.est_max, L.est_sum / b->lim.cus)});
  }
  for (size_t g = 0; g < tgroups.size(); ++g) items.push_back({1, (int)g, tgroups[g].est});
  if (slab_side_by_side) {
    for (size_t l = 0; l < slaunch.size(); ++l) items.push_back({2, (int)l, slaunch[l].est});
  } else if (!slaunch.empty()) {
    for (const SlabLaunch& S : slaunch) chain_est += S.est;
    chain = true;
  }
  if (chain) items.push_back({2, -1, chain_est});
  const bool fork = items.size() > 1;
  // Workgroups of launches side by side that can have a CU each shall have one: a
  // launch begins with the same CUs of an XCD as the one before it, as long as its
  // workgroups fit beside that one's (108 and 148 small ones left 30 to 42 CUs idle;
  // 4096 KdV and mKdV grids with FP32 arithmetic took 55 ms on shared CUs, 48.5 ms
  // on their own).  None fits beside one with more than half of the LDS.
  int64_t side = segs_side_by_side ? slab_cus : 0;
  for (const Launch& L : launches) side += even_places(L.reg ? L.grid : L.count, b->lim.cus);
  for (const SegLaunch& L : segs) side += L.tile ? even_places(L.count, b->lim.cus) : 0;
  for (const TileGroup& G : tgroups) side += even_places(G.ntiles, b->lim.cus);
  for (const SlabLaunch& S : slaunch) side += even_places(S.count, b->lim.cus);
  if (fork && side <= b->lim.cus)
    for (Launch& L : launches)
      if (L.reg) L.lds = std::max(L.lds, b->lim.lds_max / 2 + 16);
  const int nlanes = std::min<int>((int)items.size(), b->lanes > 0 ? b->lanes : hw_lanes());
  if ((int)items.size() > nlanes)
    std::stable_sort(items.begin(), items.end(), [](const LaneItem& x, const LaneItem& y) { return x.est > y.est; });
  std::vector<double> lane_load(nlanes, 0.0);
  std::vector<char> lane_forked(nlanes, 0);
  SlabGate& gate = slab_gate();
  std::unique_lock<std::mutex> gate_lock;
  int gate_need = 0;
  for (const SegLaunch& L : segs)
    if (!L.tile) gate_need = segs_side_by_side ? slab_cus : std::max(gate_need, (int)even_places(L.count, b->lim.cus));
  for (const SlabLaunch& L : slaunch) gate_need += (int)even_places(L.count, b->lim.cus);
  gate_need = std::min(gate_need, b->lim.cus);
  // Steps that whole instances may keep CUs from a slab launch, part of which waits
  // for the rest meanwhile (10 s of them passed for a time-out): this pass's, and
  // those of other batches' passes in flight.
  int64_t ahead = 0, others = 0;
  for (const Launch& L : launches)
    ahead += L.reg ? (L.parts + L.grid - 1) / L.grid * L.partsteps : (L.count + b->lim.cus - 1) / b->lim.cus * L.maxsteps;
  const bool gated = gate_need > 0 || ahead > kLongPass;
  if (gated) {
    gate_lock = std::unique_lock<std::mutex>(gate.mu);
    lbm_status gs = pass_gate(gate, b, gate_need, &others);
    if (gs != LBM_OK) return gs;
  }
  const int64_t slab_ahead = ahead + others;
  // Tags of this pass: its launches have strips of their own, so that all of them
  // count from the same tag.
  int64_t strip_tags = 0;
  for (const SegLaunch& L : segs) strip_tags = std::max(strip_tags, L.tile ? 0 : L.blocks);
  if (strips_need > 0 && b->strip_tag + strip_tags >= UINT32_MAX) {
    LBM_HIP(hipMemsetAsync(b->strips, 0, sizeof(uint64_t) * b->strips_cap, b->stream));
    b->strip_tag = 1;
  }
  const uint32_t tag = b->strip_tag;
  b->strip_tag += (uint32_t)strip_tags;
  if (fork) LBM_HIP(hipEventRecord(b->fork, b->stream));
  auto issue_slab = [&](size_t l, hipStream_t st) -> lbm_status {
    const SlabLaunch& L = slaunch[l];
    void* b0 = L.prec ? (void*)b->f32[0] : (void*)b->f64[0];
    void* b1 = L.prec ? (void*)b->f32[1] : (void*)b->f64[1];
    int* flags = b->sflags + L.foff;
    LBM_HIP(hipMemsetAsync(flags, 0, sizeof(int) * L.count, st));
    const int mute = (b->test_stall == 2 && l == 0) ? 0 : -1;
    LBM_HIP(launch_slab(L.q, L.prec, L.code, ds + L.first, L.count, dti_all, b0, b1, L.s, L.halo,
                        (unsigned char*)b->xbuf + L.xoff, flags, b->coefs, b->status, wait_ticks(b, L.s + slab_ahead), mute,
                        L.block, L.lds, st));
    return LBM_OK;
  };
  auto issue_seg = [&](size_t l, hipStream_t st) -> lbm_status {
    const SegLaunch& L = segs[l];
    const int mute = (b->test_stall == 2 && l == 0) ? 0 : -1;
    for (int r = 0; r < L.launches; ++r)
      LBM_HIP(launch_seg(L.q, L.prec, L.code, L.p.f.wide, dxsegs + L.first, L.count, L.p.f.R, L.p.f.s, L.p.sx, L.tile, r,
                         b->strips + L.at, tag, b->coefs, b->status, wait_ticks(b, L.p.sx + slab_ahead), mute, 64 * L.p.waves, L.lds, st));
    return LBM_OK;
  };
  for (size_t ii = 0; ii < items.size(); ++ii) {
    const LaneItem& it = items[ii];
    hipStream_t st = b->stream;
    if (fork) {
      const int ln = (int)items.size() <= nlanes
                         ? (int)ii
                         : (int)(std::min_element(lane_load.begin(), lane_load.end()) - lane_load.begin());
      lane_load[ln] += it.est;
      st = b->aux[ln];
      if (!lane_forked[ln]) {
        LBM_HIP(hipStreamWaitEvent(st, b->fork, 0));
        lane_forked[ln] = 1;
      }
    }
    if (it.kind == 0) {
      const int l = it.idx;
      const Launch& L = launches[l];
      int* done = done_all + L.first;
      if (L.reg) {
        const int stall = (b->test_stall == 1 && l == 0 && L.parts > L.count) ? 0 : -1;
        LBM_HIP(launch_reg(L.q, L.prec, L.code, L.wide, dparts + L.part0, L.parts, djobs + L.first, dsegs, counters + l,
                           done, b->coefs, b->status, wait_ticks(b, L.partsteps), stall, L.grid, L.block, L.lds, st));
        continue;
      }
      int per_cu = 0;
      LBM_HIP(resident_occupancy(L.q, L.prec, L.code, L.block, L.lds, &per_cu));
      if (per_cu < 1) return LBM_ERR_UNSUPPORTED;
      int grid = std::min<int>(std::min<int>(L.count, per_cu * b->lim.cus), kMaxResidentGrid);
      if (b->res_grid > 0) grid = std::min(grid, b->res_grid);
      // more jobs than workgroups: split the steps into chunks so that each
      // workgroup takes about kChunkItems items and the launch ends evenly;
      // chunks keep at least kMinChunkSteps steps (a chunk reloads its state)
      int nchunks = 1;
      if (L.count > grid) {
        nchunks = (int)std::min<int64_t>((kChunkItems * (int64_t)grid + L.count - 1) / L.count,
                                         std::max<int64_t>(1, L.maxsteps / kMinChunkSteps));
        nchunks = std::max(1, std::min(nchunks, kMaxChunks));
      }
      if (b->res_chunks > 0) nchunks = b->res_chunks;
      // (the LDS-resident launches come first in the list)
      int* slots = b->slots + (size_t)(k * kMaxResident + l) * kMaxResidentGrid;
      const long long ticks = wait_ticks(b, L.maxsteps / nchunks + 1);
      const int stall = (b->test_stall == 1 && l == 0 && nchunks > 1) ? 0 : -1;
      LBM_HIP(launch_resident(L.q, L.prec, L.code, djobs + L.first, ditems, L.count, nchunks, counters + l, slots, done,
                              b->coefs, b->status, ticks, stall, grid, L.block, L.lds, st));
    } else if (it.kind == 1) {
      const TileGroup& G = tgroups[it.idx];
      const DevTile* dt = dtiles + G.first;
      void* b0 = G.prec ? (void*)b->f32[0] : (void*)b->f64[0];
      void* b1 = G.prec ? (void*)b->f32[1] : (void*)b->f64[1];
      for (int l = 0; l < G.launches; ++l)
        LBM_HIP(launch_tile(G.q, G.prec, dt, G.ntiles, dti_all, b0, b1, l, G.s, G.halo, b->coefs, b->status, G.block,
                            G.lds, st));
      for (int t = G.tfirst; t < G.tfirst + G.tcount; ++t) {
        HostInst& h = b->inst[htin[t].inst];
        const int L = (int)((htin[t].steps + G.s - 1) / G.s);
        h.cur = htin[t].cur0 ^ (L & 1);
      }
    } else if (it.kind == 3) {
      lbm_status s = issue_seg((size_t)it.idx, st);
      if (s != LBM_OK) return s;
    } else if (it.idx >= 0) {
      lbm_status s = issue_slab((size_t)it.idx, st);
      if (s != LBM_OK) return s;
    } else {
      for (size_t l = 0; l < segs.size(); ++l) {
        if (segs[l].tile || segs_side_by_side) continue;
        lbm_status s = issue_seg(l, st);
        if (s != LBM_OK) return s;
      }
      for (size_t l = 0; l < slaunch.size(); ++l) {
        lbm_status s = issue_slab(l, st);
        if (s != LBM_OK) return s;
      }
    }
  }
  for (const auto& [i, turns] : flips) b->inst[i].cur ^= turns & 1;
  if (!slaunch.empty())
    for (const DevSlab& sl : svec)
      if (sl.x0 == 0) b->inst[htin[sl.ti].inst].cur ^= 1;   // one flip per instance: output in the other buffer
  if (fork) {
    for (int a = 0; a < nlanes; ++a) {
      if (!lane_forked[a]) continue;
      LBM_HIP(hipEventRecord(b->join[a], b->aux[a]));
      LBM_HIP(hipStreamWaitEvent(b->stream, b->join[a], 0));
    }
  }
  LBM_HIP(hipEventRecord(b->items_done[k], b->stream));
  if (gated) {
    lbm_status gs = enter_gate(gate, b, gate_need, ahead > kLongPass ? ahead : 0);
    if (gs != LBM_OK) return gs;
    gate_lock.unlock();
  }
  // streaming instances: one fused collide+stream launch per step, whole
  // blocks of kStepBlock steps replayed from a graph
  for (int i : str) {
    HostInst& h = b->inst[i];
    lbm_status s = ensure_second_buffer(b, h.f32);
    if (s != LBM_OK) return s;
    int64_t t = 0;
    if (steps[i] >= 2 * kStepBlock) {
      StepGraph* g = nullptr;
      s = step_graph(b, i, &g);
      if (s != LBM_OK) return s;
      for (; t + kStepBlock <= steps[i]; t += kStepBlock) LBM_HIP(hipGraphLaunch(g->exec, b->stream));
    }
    for (; t < steps[i]; ++t) {
      LBM_HIP(launch_stream(h.q, h.D, h.prec, state_cur(b, h), state_other(b, h), h.n, h.stride, b->coefs + i,
                            b->stream));
      h.cur = 1 - h.cur;
    }
  }
  LBM_HIP(hipEventRecord(b->ev1, b->stream));
  for (int i = 0; i < count; ++i) b->inst[i].steps_done += steps[i];
  return LBM_OK;
}

lbm_status advance(lbm_batch_s* b, const int64_t* steps) {
  const int count = (int)b->inst.size();
  std::vector<int64_t> left(steps, steps + count);
  for (int64_t v : left)
    if (v < 0) return LBM_ERR_INVALID_ARG;
  for (;;) {
    std::vector<int64_t> now(count);
    bool any = false;
    for (int i = 0; i < count; ++i) {
      now[i] = std::min(left[i], kMaxStepsPerLaunch);
      left[i] -= now[i];
      any |= now[i] > 0;
    }
    if (!any) return LBM_OK;
    lbm_status s = advance_pass(b, now.data());
    if (s != LBM_OK) return s;
  }
}

// phi of instance i, and its status.  Grids up to the stage are summed straight
// into it (or into this GPU's memory); larger ones, and other memory, go by the
// scratch buffer.
lbm_status read_phi(lbm_batch_s* b, int i, double* out, int on_device, lbm_status* inst_status) {
  HostInst& h = b->inst[i];
  const double rest = h.f32 ? h.mdl.phi_rest : 0.0;
  int* words = reinterpret_cast<int*>(b->stage);
  volatile int* seen = words;
  seen[0] = seen[1] = 0;
  const bool staged = !on_device && sizeof(double) * (size_t)h.n <= b->stage_bytes;
  const bool direct = on_device && on_this_gpu(out);
  double* to = direct ? out : staged ? reinterpret_cast<double*>(b->stage + kStageHead) : b->scratch;
  if (staged && h.n <= 256 * kReadWords) {
    // watched for as long as an idle stream takes; behind an advance that is
    // still running (and on errors) the stream is waited for
    static_assert(sizeof(int) * (2 + kReadWords) <= kStageHead, "the stage's words");
    const int blocks = (h.n + 255) / 256;
    const int seq = b->read_seq = b->read_seq % 0x7fffffff + 1;
    for (int k = 0; k < blocks; ++k) seen[2 + k] = 0;
    LBM_HIP(launch_read(h.f32, state_cur(b, h), to, h.n, h.stride, h.q, rest, b->status + i, words, seq, nullptr,
                        b->stream));
    const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(kReadWatchUs);
    int here = 0;
    do {
      for (int k = 0; k < 64 && here < blocks; ++k)
        while (here < blocks && __atomic_load_n(words + 2 + here, __ATOMIC_ACQUIRE) == seq) ++here;
    } while (here < blocks && std::chrono::steady_clock::now() < until);
    const bool there = here == blocks;
    if (!there) LBM_HIP(hipStreamSynchronize(b->stream));
  } else {
    LBM_HIP(launch_read(h.f32, state_cur(b, h), to, h.n, h.stride, h.q, rest, b->status + i, words, 0, nullptr, b->stream));
    if (!direct && !staged)
      LBM_HIP(hipMemcpyAsync(out, to, sizeof(double) * h.n, on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                             b->stream));
    LBM_HIP(hipStreamSynchronize(b->stream));
  }
  if (staged) std::memcpy(out, to, sizeof(double) * h.n);
  // status bit 1: a non-finite value; bits 2 and 4: a device wait for a
  // cooperating workgroup gave up, so the state was not advanced as asked
  const int flags = seen[0], bad = seen[1];
  lbm_status s = (flags & 6) ? LBM_ERR_TIMEOUT : (bad || flags) ? LBM_ERR_NONFINITE : LBM_OK;
  if (inst_status) *inst_status = s;
  return s;
}

// ---------------------------------------------------------------------------
// Autotuning: time candidate planner settings on a copy of the batch (same
// descriptors, coefficients and state) and keep the fastest.  The planner's
// choices it covers: the tile shape and steps per launch of the temporal-
// blocking path (instances that do not fit one workgroup's LDS), the step
// chunking of the resident path, and -- for small batches -- the LDS-resident
// vs HBM-streaming choice itself.
// ---------------------------------------------------------------------------
struct Knobs {
  int path, tile_steps, tile_wgs, res_grid, res_chunks;
};
constexpr double kTuneMargin = 0.97;

Knobs knobs_of(const lbm_batch_s* b) { return Knobs{b->path, b->tile_steps, b->tile_wgs, b->res_grid, b->res_chunks}; }

void set_knobs(lbm_batch_s* b, const Knobs& k) {
  b->path = k.path;
  b->tile_steps = k.tile_steps;
  b->tile_wgs = k.tile_wgs;
  b->res_grid = k.res_grid;
  b->res_chunks = k.res_chunks;
}

lbm_status clone_for_tuning(lbm_batch_s* b, lbm_batch_s** out) {
  const int count = (int)b->inst.size();
  std::vector<lbm_desc> d(count);
  for (int i = 0; i < count; ++i) d[i] = b->inst[i].desc;
  lbm_batch_s* c = nullptr;
  lbm_status s = create_batch(d.data(), count, b->stream, nullptr, 0, &c);
  if (s != LBM_OK) return s;
  // same descriptors in the same order: same layout; copy coefficients and state
  for (int i = 0; i < count && s == LBM_OK; ++i) {
    c->inst[i].mdl = b->inst[i].mdl;
    c->inst[i].cur = b->inst[i].cur;
  }
  auto copy = [&](void* dst, const void* src, size_t bytes) -> lbm_status {
    if (!bytes) return LBM_OK;
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, b->stream) == hipSuccess ? LBM_OK
                                                                                           : LBM_ERR_DEVICE;
  };
  if (s == LBM_OK) s = copy(c->coefs, b->coefs, sizeof(DevCoef) * count);
  for (int k = 0; k < 2 && s == LBM_OK; ++k) {
    if (b->f64[k]) {
      if (k == 1) s = ensure_second_buffer(c, false);
      if (s == LBM_OK) s = copy(c->f64[k], b->f64[k], sizeof(double) * b->n64);
    }
    if (b->f32[k] && s == LBM_OK) {
      if (k == 1) s = ensure_second_buffer(c, true);
      if (s == LBM_OK) s = copy(c->f32[k], b->f32[k], sizeof(float) * b->n32);
    }
  }
  if (s == LBM_OK && hipStreamSynchronize(b->stream) != hipSuccess) s = LBM_ERR_DEVICE;
  if (s != LBM_OK) {
    destroy_batch(c);
    return s;
  }
  *out = c;
  return LBM_OK;
}

// device time (ms) of one pass of `probe` steps with knobs k: best of two after a warm-up pass
lbm_status time_knobs(lbm_batch_s* c, const Knobs& k, int64_t probe, double* ms) {
  set_knobs(c, k);
  std::vector<int64_t> st(c->inst.size(), probe);
  double best = 1e300;
  for (int r = 0; r < 3; ++r) {
    lbm_status s = advance(c, st.data());
    if (s != LBM_OK) return s;
    LBM_HIP(hipEventSynchronize(c->ev1));
    float t = 0.0f;
    LBM_HIP(hipEventElapsedTime(&t, c->ev0, c->ev1));
    if (r > 0) best = std::min(best, (double)t);
  }
  *ms = best;
  return LBM_OK;
}

lbm_status autotune(lbm_batch_s* b, int64_t probe, lbm_tuning* out) {
  const int count = (int)b->inst.size();
  bool any_fit = false, any_big = false;
  double nodes = 0.0;
  int64_t minn = INT64_MAX;
  for (const HostInst& h : b->inst) {
    const bool f = fits_resident(b, h);
    any_fit |= f;
    any_big |= !f;
    nodes += h.n;
    minn = std::min<int64_t>(minn, h.n);
  }
  lbm_batch_s* c = nullptr;
  lbm_status s = clone_for_tuning(b, &c);
  if (s != LBM_OK) return s;
  int tried = 0;
  Knobs best{0, 0, 0, 0, 0};
  double best_ms = 0.0, default_ms = 0.0;
  s = time_knobs(c, best, probe, &default_ms);
  best_ms = default_ms;
  ++tried;
  auto consider = [&](const Knobs& k) {
    if (s != LBM_OK) return;
    double ms = 0.0;
    s = time_knobs(c, k, probe, &ms);
    ++tried;
    if (s == LBM_OK && ms < kTuneMargin * best_ms) {   // clear wins only, not timing noise
      best_ms = ms;
      best = k;
    }
  };
  // 1. temporal blocking: steps per launch x workgroups per CU
  if (any_big || minn >= 1024) {
    static const int kTiles[][2] = {{8, 2}, {16, 2}, {32, 2}, {64, 2}, {16, 1}, {32, 1}, {64, 1}};
    const int path = any_big ? best.path : 3;   // instances that fit: try them tiled as well
    for (const auto& t : kTiles) consider(Knobs{path, t[0], t[1], 0, 0});
    if (!any_big) consider(Knobs{3, 0, 0, 0, 0});
  }
  // 2. resident step chunks
  if (any_fit && best.path != 3) {
    static const int kChunks[] = {1, 4, 8, 16, 32};
    const Knobs base = best;
    for (int ch : kChunks) consider(Knobs{base.path, base.tile_steps, base.tile_wgs, 0, ch});
  }
  // 3. HBM streaming, one launch per step: only for a few instances
  if (count <= 16 && nodes * (double)probe <= 2.5e8) consider(Knobs{1, 0, 0, 0, 0});
  destroy_batch(c);
  if (s != LBM_OK) return s;
  set_knobs(b, best);
  if (out) {
    out->path = best.path;
    out->tile_steps = best.tile_steps;
    out->tile_wgs = best.tile_wgs;
    out->res_chunks = best.res_chunks;
    out->candidates = tried;
    out->pad_ = 0;
    out->best_node_updates_per_s = nodes * (double)probe / (best_ms * 1e-3);
    out->default_node_updates_per_s = nodes * (double)probe / (default_ms * 1e-3);
  }
  return LBM_OK;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* lbm_status_str(lbm_status s) {
  switch (s) {
    case LBM_OK: return "ok";
    case LBM_ERR_INVALID_ARG: return "invalid argument";
    case LBM_ERR_UNSUPPORTED: return "unsupported";
    case LBM_ERR_SINGULAR_TAU: return "singular relaxation polynomial tau_k";
    case LBM_ERR_OUT_OF_MEMORY: return "out of device memory";
    case LBM_ERR_DEVICE: return "HIP runtime error";
    case LBM_ERR_NONFINITE: return "non-finite state";
    case LBM_ERR_BUSY: return "busy";
    case LBM_ERR_TIMEOUT: return "device wait timed out";
  }
  return "unknown status";
}

const char* lbm_version(void) { return "lbmhpde 0.1 gfx950"; }

int64_t lbm_row_stride(int64_t n) { return (n + 63) / 64 * 64; }

lbm_status lbm_validate(const lbm_desc* d) {
  if (!d) return LBM_ERR_INVALID_ARG;
  Model m;
  return build_model(*d, &m);
}

lbm_status lbm_coefficients(const lbm_desc* d, double* G, int32_t cap, int32_t* q_out, int32_t* degree_out) {
  if (!d || !G || !q_out || !degree_out) return LBM_ERR_INVALID_ARG;
  Model m;
  lbm_status s = build_model(*d, &m);
  if (s != LBM_OK) return s;
  if (m.gF > 0) return LBM_ERR_UNSUPPORTED;   // not a polynomial in phi
  if (cap < m.q * (m.D + 1)) return LBM_ERR_INVALID_ARG;
  for (int j = 0; j < m.q; ++j)
    for (int p = 0; p <= m.D; ++p) G[j * (m.D + 1) + p] = m.G[j][p];
  *q_out = m.q;
  *degree_out = m.D;
  return LBM_OK;
}

lbm_status lbm_coefficients_general(const lbm_desc* d, double* nu, double* G, int32_t cap, int32_t* classes_out,
                                    int32_t* q_out, int32_t* degree_out) {
  if (!d || !nu || !G || !classes_out || !q_out || !degree_out) return LBM_ERR_INVALID_ARG;
  Model m;
  lbm_status s = build_model(*d, &m);
  if (s != LBM_OK) return s;
  const int F = m.gF > 0 ? m.gF : 1;
  if (cap < F * m.q * (m.D + 1)) return LBM_ERR_INVALID_ARG;
  for (int c = 0; c < F; ++c) {
    nu[c] = m.gF > 0 ? m.gnu[c] : 0.0;
    for (int j = 0; j < m.q; ++j)
      for (int p = 0; p <= m.D; ++p) G[(c * m.q + j) * (m.D + 1) + p] = m.gF > 0 ? m.gG[c][j][p] : m.G[j][p];
  }
  *classes_out = F;
  *q_out = m.q;
  *degree_out = m.D;
  return LBM_OK;
}

lbm_status lbm_stability(const lbm_desc* d, double phi_min, double phi_max, int64_t steps,
                         double* growth_per_step, double* amplification) {
  if (!d || !growth_per_step || steps < 0 || !(phi_min <= phi_max) || !std::isfinite(phi_min) ||
      !std::isfinite(phi_max))
    return LBM_ERR_INVALID_ARG;
  Model m;
  lbm_status s = build_model(*d, &m);
  if (s != LBM_OK) return s;
  if (m.gF > 1 && phi_min <= 0) return LBM_ERR_INVALID_ARG;   // real powers: phi > 0 only
  const double g = stability_growth(m, phi_min, phi_max);
  *growth_per_step = g;
  if (amplification) *amplification = std::pow(g, (double)steps);
  return LBM_OK;
}

lbm_status lbm_required_bytes(const lbm_desc* d, size_t* bytes) {
  if (!d || !bytes) return LBM_ERR_INVALID_ARG;
  Model m;
  lbm_status s = build_model(*d, &m);
  if (s != LBM_OK) return s;
  size_t es = d->prec == LBM_F64 ? sizeof(double) : sizeof(float);
  *bytes = (size_t)m.q * (size_t)lbm_row_stride(d->n) * es;
  return LBM_OK;
}

lbm_status lbm_create(const lbm_desc* d, void* stream, void* dev_buf, size_t buf_bytes, lbm_problem* out) {
  if (!d || !out) return LBM_ERR_INVALID_ARG;
  lbm_batch_s* b = nullptr;
  lbm_status s = create_batch(d, 1, stream, dev_buf, buf_bytes, &b);
  if (s != LBM_OK) return s;
  lbm_problem_s* p = new (std::nothrow) lbm_problem_s();
  if (!p) {
    destroy_batch(b);
    return LBM_ERR_OUT_OF_MEMORY;
  }
  p->b = b;
  *out = p;
  return LBM_OK;
}

lbm_status lbm_load_phi(lbm_problem h, const double* phi, int phi_on_device) {
  if (!h || !phi) return LBM_ERR_INVALID_ARG;
  if (phi_on_device) return load_device(h->b, 0, phi);
  const lbm_status s = check_phi(h->b->inst[0], phi);
  if (s != LBM_OK) return s;
  const int i = 0;
  return load_many(h->b, &i, &phi, 1, false);
}

lbm_status lbm_advance(lbm_problem h, int64_t steps) {
  if (!h || steps < 0) return LBM_ERR_INVALID_ARG;
  return advance(h->b, &steps);
}

// lbm_create + lbm_load_phi + lbm_advance + lbm_read_phi of one periodic
// problem whose state fits one workgroup's LDS, with every device buffer in
// the fixed per-device scratch (noalloc.hip): the same kernels (k_init_one, one
// resident launch per 2^30 steps, k_read), so the result is bitwise that of the
// handle path.  Host-side buffers live on this call's stack.
//
// Short calls are bound by their launches, copies and waits: 257 nodes and 101
// steps took 118 us, of which the steps are 25.  A polynomial FP64 call is four
// launches, one copy (the flags) and one wait; phi0 is checked where it is.
lbm_status lbm_advance_noalloc(const lbm_desc* d, const double* phi0, int64_t steps, double* phi, void* stream) {
  if (!d || !phi0 || !phi || steps < 0 || d->n < 1 || d->n > kNoAllocMaxNodes) return LBM_ERR_INVALID_ARG;
  if (d->bc != LBM_BC_PERIODIC) return LBM_ERR_INVALID_ARG;
  const hipStream_t st = (hipStream_t)stream;
  HostInst h;
  lbm_status s = prepare_one(*d, &h);
  if (s != LBM_OK) return s;
  const DeviceLimits lim = query_limits();
  if (!lim.ok) return LBM_ERR_DEVICE;
  const size_t es = elem_size(h);
  const size_t lds = ((size_t)lds_stride(h.q) * h.n * es + 15) / 16 * 16;
  if ((size_t)h.q * h.stride * es > kNoAllocStateBytes || lds + resident_static_lds(h.q, h.prec, h.D) > lim.lds_max)
    return LBM_ERR_INVALID_ARG;
  void* base = nullptr;
  LBM_HIP(noalloc_scratch(&base));
  // tables at the start of the scratch, the state after them
  static_assert(sizeof(DevCoef) <= kNoAllocJobAt, "coefficient table outgrew its scratch region");
  static_assert(sizeof(DevJob) <= 128 && sizeof(DevItem) <= 128 && sizeof(DevSeg) <= 256 && sizeof(DevJobInst) <= 256,
                "job record outgrew its scratch region");
  unsigned char* bytes = (unsigned char*)base;
  DevCoef* dcoef = (DevCoef*)bytes;
  DevJob* djob = (DevJob*)(bytes + kNoAllocJobAt);
  DevItem* ditem = (DevItem*)(bytes + kNoAllocItemAt);
  DevSeg* dseg = (DevSeg*)(bytes + kNoAllocSegAt);
  DevJobInst* dji = (DevJobInst*)(bytes + kNoAllocSegAt);   // the LDS path's record, in its place
  int* ints = (int*)(bytes + kNoAllocIntsAt);   // queue counter, slot, done, status, read-out words, phi0 refused
  void* f = bytes + kNoAllocTableBytes;
  const bool in_reg = reg_variant(h.D);
  if (h.f32 || !in_reg) {
    // phi0 on the host: the checks of lbm_load_phi and the rest state (mean of phi0)
    double host[kNoAllocMaxNodes];
    LBM_HIP(hipMemcpyAsync(host, phi0, sizeof(double) * h.n, hipMemcpyDeviceToHost, st));
    LBM_HIP(hipStreamSynchronize(st));
    if (check_phi(h, host) != LBM_OK) return LBM_ERR_INVALID_ARG;
    if (h.f32) rest_from(&h, host);
  }
  DevCoef cf;
  fill_devcoef(h, &cf);
  // one job of one instance: in registers the way its step is shortest, else a
  // wave per 64 nodes, at most 16
  NoAllocTables tables{};
  RegFit fit;
  DevJob& jb = tables.job;
  jb.count = 1;
  jb.degree = h.D;
  DevJobInst ji{};
  if (in_reg) {
    for (int cls = 0; cls < 2; ++cls) {
      RegFit menu[kRegWidths + 1];
      const int widths = reg_menu(h.q, h.prec, h.D, cls != 0, menu);
      for (int k = 0; k < widths; ++k) {
        reg_place(h.q, h.n, &menu[k]);
        if (menu[k].waves <= reg_waves(cls != 0) &&
            (fit.waves == 0 || reg_step(menu[k], (menu[k].waves + 3) / 4) < reg_step(fit, (fit.waves + 3) / 4)))
          fit = menu[k];
      }
    }
    if (fit.waves == 0) return LBM_ERR_INVALID_ARG;
    jb.nodes = fit.R;
    jb.s_per = fit.s;
    DevSeg& sg = tables.seg;
    sg.in = sg.out = (uint64_t)(uintptr_t)f;
    sg.n = sg.len = h.n;
    sg.stride = h.stride;
    sg.lanes = fit.lanes;
    sg.over = fit.over;
    sg.waves = fit.waves;
    std::memcpy(tables.coef, &cf, kNoAllocCoefBytes);
  } else {
    ji.addr = (uint64_t)(uintptr_t)f;
    ji.n = h.n;
    ji.stride = h.stride;
    ji.degree = h.D;
    ji.nt = 64 * std::max(1, std::min(16, (h.n + 63) / 64));
    LBM_HIP(hipMemcpyAsync(dcoef, &cf, sizeof(cf), hipMemcpyHostToDevice, st));
    LBM_HIP(hipMemcpyAsync(dji, &ji, sizeof(ji), hipMemcpyHostToDevice, st));
    LBM_HIP(launch_zero_ints(ints, 8, st));
  }
  DevInit init{};
  init.src = (uint64_t)(uintptr_t)phi0;
  init.dst = (uint64_t)(uintptr_t)f;
  init.len = h.n;
  init.stride = h.stride;
  init.q = h.q;
  init.degree = h.Dinit;
  init.first = 1;
  bool first = true;
  for (int64_t left = steps; left > 0 || first;) {
    const int64_t now = std::min(left, kMaxStepsPerLaunch);
    left -= now;
    jb.steps = (int)now;
    tables.item = DevItem{0, 0, (int)now, 0, 0};
    if (in_reg) LBM_HIP(launch_tables(tables, bytes, !first, st));
    if (first) LBM_HIP(launch_init_one(h.f32, init, dcoef, ints + 3, in_reg ? ints + 6 : nullptr, st));
    first = false;
    if (now == 0) break;
    if (in_reg) {
      LBM_HIP(launch_reg(h.q, h.prec, h.D, fit.wide, ditem, 1, djob, dseg, ints, ints + 2, dcoef, ints + 3, 0, -1, 1,
                         64 * fit.waves, (size_t)fit.waves * reg_strip(h.q, fit.R, fit.s) * es, st));
    } else {
      LBM_HIP(hipMemcpyAsync(djob, &jb, sizeof(jb), hipMemcpyHostToDevice, st));
      LBM_HIP(hipStreamSynchronize(st));   // jb is reused by the next launch
      LBM_HIP(launch_zero_ints(ints, 3, st));
      LBM_HIP(launch_resident(h.q, h.prec, h.D, djob, dji, 1, 1, ints, ints + 1, ints + 2, dcoef, ints + 3, 0, -1, 1,
                              ji.nt, lds, st));
    }
  }
  LBM_HIP(launch_read(h.f32, f, phi, h.n, h.stride, h.q, h.f32 ? h.mdl.phi_rest : 0.0, ints + 3, ints + 4, 0, ints + 6,
                      st));
  int flags[3] = {0, 0, 0};
  LBM_HIP(hipMemcpyAsync(flags, ints + 4, sizeof(flags), hipMemcpyDeviceToHost, st));
  LBM_HIP(hipStreamSynchronize(st));
  if (flags[2]) return LBM_ERR_INVALID_ARG;
  if (flags[0] & 6) return LBM_ERR_TIMEOUT;
  return (flags[0] || flags[1]) ? LBM_ERR_NONFINITE : LBM_OK;
}

}  // extern "C"

namespace {
// Where the boundary rows of a bounded call come from: host arrays (copied),
// or travelling waves evaluated on the device.
struct RowSource {
  const double* const* host = nullptr;   // per instance
  const lbm_wave* waves = nullptr;       // per instance
};

bool valid_wave(const lbm_wave* w) {
  if (!w) return false;
  if (w->shape < LBM_WAVE_SECH || w->shape > LBM_WAVE_COS) return false;
  const double v[] = {w->a, w->b, w->p, w->d, w->r, w->k, w->xc, w->c, w->x_first, w->t0};
  for (double x : v)
    if (!std::isfinite(x)) return false;
  if (w->p < 0.0 || w->r < 0.0) return false;
  // tanh may be negative: integer exponents only
  if (w->shape == LBM_WAVE_TANH && (w->p != std::floor(w->p) || w->r != std::floor(w->r))) return false;
  return true;
}

// Bounded instances of a batch advance `steps` (<= kMaxStepsPerLaunch) steps on
// the resident path, their boundary layers reset in LDS after every step;
// rows [steps][2 layers] of bounded instance i from `src`.
lbm_status advance_bounded_resident(lbm_batch_s* b, int64_t steps, const RowSource& src, int layers) {
  const int count = (int)b->inst.size();
  int nb = 0;
  for (int i = 0; i < count; ++i) nb += b->inst[i].desc.bc != LBM_BC_PERIODIC;
  const size_t rows = (size_t)steps * 2 * layers;
  const size_t need = rows * (size_t)nb;
  // a synchronous copy: earlier launches have read the buffer by the time it lands
  LBM_HIP(hipStreamSynchronize(b->stream));
  if (need > b->bound_cap) {
    hipFree(b->bound);
    b->bound = nullptr;
    b->bound_cap = 0;
    if (hipMalloc(&b->bound, sizeof(double) * need) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
    b->bound_cap = need;
  }
  b->bnd_ptr.assign(count, 0);
  std::vector<WaveRows> waves;
  for (int i = 0, k = 0; i < count; ++i) {
    const HostInst& h = b->inst[i];
    if (h.desc.bc == LBM_BC_PERIODIC) continue;
    double* dst = b->bound + (size_t)k++ * rows;
    if (src.host)
      LBM_HIP(hipMemcpy(dst, src.host[i], sizeof(double) * rows, hipMemcpyHostToDevice));
    else
      waves.push_back(wave_rows(dst, h.n, h.desc.dx, h.desc.dt, src.waves[i]));
    b->bnd_ptr[i] = (uint64_t)(uintptr_t)dst;
  }
  LBM_HIP(launch_wave_rows(waves.data(), (int)waves.size(), steps, layers, b->stream));
  b->bnd_active = true;
  b->bnd_layers = layers;
  std::vector<int64_t> st(count, steps);
  lbm_status s = advance_pass(b, st.data());
  b->bnd_active = false;
  return s;
}
lbm_status batch_advance_bounded(lbm_batch_s* b, int64_t steps, const RowSource& src, int layers) {
  if (steps < 0 || steps > kMaxStepsPerLaunch) return LBM_ERR_INVALID_ARG;
  int hmax = 0;
  for (const HostInst& h : b->inst)
    if (h.desc.bc != LBM_BC_PERIODIC) hmax = std::max(hmax, h.q / 2);
  if (layers == 0) layers = hmax;
  if (layers < hmax || layers > 32) return LBM_ERR_INVALID_ARG;
  for (size_t i = 0; i < b->inst.size(); ++i) {
    const HostInst& h = b->inst[i];
    if (h.desc.bc == LBM_BC_PERIODIC) continue;
    if (src.host && steps > 0 && !src.host[i]) return LBM_ERR_INVALID_ARG;
    if (src.waves && !valid_wave(&src.waves[i])) return LBM_ERR_INVALID_ARG;
    if (h.n < 2 * layers + 2) return LBM_ERR_INVALID_ARG;
  }
  if (steps == 0) return LBM_OK;
  return advance_bounded_resident(b, steps, src, layers);
}

// device rows buffer of at least steps * 2 layers doubles (b->bound), no
// earlier launch still reading it
lbm_status bound_rows_buffer(lbm_batch_s* b, size_t need) {
  LBM_HIP(hipStreamSynchronize(b->stream));
  if (need > b->bound_cap) {
    hipFree(b->bound);
    b->bound = nullptr;
    b->bound_cap = 0;
    if (hipMalloc(&b->bound, sizeof(double) * need) != hipSuccess) return LBM_ERR_OUT_OF_MEMORY;
    b->bound_cap = need;
  }
  return LBM_OK;
}

// single bounded problem: `layers` resolved and checked against the problem
lbm_status bounded_layers(const HostInst& in, int32_t* layers) {
  if (in.desc.bc != LBM_BC_DIRICHLET_EQ && in.desc.bc != LBM_BC_DIRICHLET_NEE) return LBM_ERR_INVALID_ARG;
  const int H = in.q / 2;
  if (*layers == 0) *layers = H;
  if (*layers < H || *layers > 32 || in.n < 2 * *layers + 2) return LBM_ERR_INVALID_ARG;
  return LBM_OK;
}

lbm_status advance_bounded_one(lbm_batch_s* b, int64_t steps, const RowSource& src, int32_t layers) {
  HostInst& in = b->inst[0];
  lbm_status s = bounded_layers(in, &layers);
  if (s != LBM_OK) return s;
  if (src.waves && !valid_wave(src.waves)) return LBM_ERR_INVALID_ARG;
  if (steps == 0) return LBM_OK;
  // LDS-resident unless the streaming path is asked for or the state does not fit
  if ((b->path == 0 || b->path == 2) && fits_resident(b, in) && steps <= kMaxStepsPerLaunch)
    return advance_bounded_resident(b, steps, src, layers);
  s = ensure_second_buffer(b, in.f32);
  if (s != LBM_OK) return s;
  const size_t need = (size_t)steps * 2 * layers;
  s = bound_rows_buffer(b, need);
  if (s != LBM_OK) return s;
  if (src.host) {
    LBM_HIP(hipMemcpy(b->bound, src.host[0], sizeof(double) * need, hipMemcpyHostToDevice));
  } else {
    const WaveRows wr = wave_rows(b->bound, in.n, in.desc.dx, in.desc.dt, src.waves[0]);
    LBM_HIP(launch_wave_rows(&wr, 1, steps, layers, b->stream));
  }
  const int kind = in.desc.bc == LBM_BC_DIRICHLET_EQ ? 1 : 2;
  LBM_HIP(hipEventRecord(b->ev0, b->stream));
  for (int64_t t = 0; t < steps; ++t) {
    LBM_HIP(launch_stream(in.q, in.D, in.prec, state_cur(b, in), state_other(b, in), in.n, in.stride, b->coefs,
                          b->stream));
    in.cur = 1 - in.cur;
    LBM_HIP(launch_bound(in.q, in.Dinit, in.prec, state_cur(b, in), in.n, in.stride, layers, kind,
                         b->bound + (size_t)t * 2 * layers, b->coefs, b->stream));
  }
  LBM_HIP(hipEventRecord(b->ev1, b->stream));
  in.steps_done += steps;
  return LBM_OK;
}
}  // namespace

extern "C" {

lbm_status lbm_batch_advance_bounded(lbm_batch b, int64_t steps, const double* const* phib, int32_t layers) {
  if (!b) return LBM_ERR_INVALID_ARG;
  for (const HostInst& h : b->inst)
    if (h.desc.bc != LBM_BC_PERIODIC && steps > 0 && !phib) return LBM_ERR_INVALID_ARG;
  RowSource src;
  src.host = phib;
  return batch_advance_bounded(b, steps, src, layers);
}

lbm_status lbm_batch_advance_bounded_wave(lbm_batch b, int64_t steps, const lbm_wave* waves, int32_t layers) {
  if (!b || !waves) return LBM_ERR_INVALID_ARG;
  RowSource src;
  src.waves = waves;
  return batch_advance_bounded(b, steps, src, layers);
}

lbm_status lbm_advance_bounded(lbm_problem h, int64_t steps, const double* phib, int32_t layers) {
  if (!h || steps < 0 || (steps > 0 && !phib)) return LBM_ERR_INVALID_ARG;
  const double* rows[1] = {phib};
  RowSource src;
  src.host = rows;
  return advance_bounded_one(h->b, steps, src, layers);
}

lbm_status lbm_advance_bounded_wave(lbm_problem h, int64_t steps, const lbm_wave* w, int32_t layers) {
  if (!h || steps < 0 || !w) return LBM_ERR_INVALID_ARG;
  RowSource src;
  src.waves = w;
  return advance_bounded_one(h->b, steps, src, layers);
}

lbm_status lbm_wave_rows(lbm_problem h, int64_t steps, const lbm_wave* w, int32_t layers, double* out) {
  if (!h || steps < 0 || !w || (steps > 0 && !out) || !valid_wave(w)) return LBM_ERR_INVALID_ARG;
  lbm_batch_s* b = h->b;
  lbm_status s = bounded_layers(b->inst[0], &layers);
  if (s != LBM_OK) return s;
  if (steps == 0) return LBM_OK;
  const size_t need = (size_t)steps * 2 * layers;
  s = bound_rows_buffer(b, need);
  if (s != LBM_OK) return s;
  const HostInst& in = b->inst[0];
  const WaveRows wr = wave_rows(b->bound, in.n, in.desc.dx, in.desc.dt, *w);
  LBM_HIP(launch_wave_rows(&wr, 1, steps, layers, b->stream));
  LBM_HIP(hipStreamSynchronize(b->stream));
  LBM_HIP(hipMemcpy(out, b->bound, sizeof(double) * need, hipMemcpyDeviceToHost));
  return LBM_OK;
}

lbm_status lbm_read_phi(lbm_problem h, double* out, int out_on_device) {
  if (!h || !out) return LBM_ERR_INVALID_ARG;
  return read_phi(h->b, 0, out, out_on_device, nullptr);
}

lbm_status lbm_sum_phi(lbm_problem h, double* total) {
  if (!h || !total) return LBM_ERR_INVALID_ARG;
  lbm_batch_s* b = h->b;
  HostInst& hi = b->inst[0];
  int* words = reinterpret_cast<int*>(b->stage);
  LBM_HIP(launch_read(hi.f32, state_cur(b, hi), b->scratch, hi.n, hi.stride, hi.q, hi.f32 ? hi.mdl.phi_rest : 0.0,
                      b->status, words, 0, nullptr, b->stream));
  // deterministic FP64 reduction: fixed partition on the device, fixed order on the host
  const int parts = 64;
  double* part = b->scratch + hi.n;
  LBM_HIP(launch_sum(b->scratch, hi.n, part, parts, b->stream));
  double hp[parts];
  LBM_HIP(hipMemcpyAsync(hp, part, sizeof(hp), hipMemcpyDeviceToHost, b->stream));
  LBM_HIP(hipStreamSynchronize(b->stream));
  double t = 0.0;
  for (int i = 0; i < parts; ++i) t += hp[i];
  *total = t;
  return std::isfinite(t) ? LBM_OK : LBM_ERR_NONFINITE;
}

lbm_status lbm_state_bytes(lbm_problem h, size_t* bytes) {
  if (!h || !bytes) return LBM_ERR_INVALID_ARG;
  const HostInst& hi = h->b->inst[0];
  *bytes = 32 + (size_t)hi.q * hi.n * elem_size(hi);
  return LBM_OK;
}

lbm_status lbm_save_f(lbm_problem h, void* host_buf, size_t bytes) {
  if (!h || !host_buf) return LBM_ERR_INVALID_ARG;
  lbm_batch_s* b = h->b;
  HostInst& hi = b->inst[0];
  size_t need = 0;
  lbm_state_bytes(h, &need);
  if (bytes < need) return LBM_ERR_INVALID_ARG;
  unsigned char* p = (unsigned char*)host_buf;
  uint64_t hdr[4] = {kMagic, (uint64_t)hi.steps_done, (uint64_t)hi.q | ((uint64_t)hi.f32 << 32), (uint64_t)hi.n};
  std::memcpy(p, hdr, 32);
  const size_t row = (size_t)hi.n * elem_size(hi);
  for (int j = 0; j < hi.q; ++j) {
    const void* src = hi.f32 ? (const void*)(f32_cur(b, hi) + (size_t)j * hi.stride)
                             : (const void*)(f64_cur(b, hi) + (size_t)j * hi.stride);
    LBM_HIP(hipMemcpyAsync(p + 32 + j * row, src, row, hipMemcpyDeviceToHost, b->stream));
  }
  LBM_HIP(hipStreamSynchronize(b->stream));
  return LBM_OK;
}

lbm_status lbm_load_f(lbm_problem h, const void* host_buf, size_t bytes) {
  if (!h || !host_buf) return LBM_ERR_INVALID_ARG;
  lbm_batch_s* b = h->b;
  HostInst& hi = b->inst[0];
  size_t need = 0;
  lbm_state_bytes(h, &need);
  if (bytes < need) return LBM_ERR_INVALID_ARG;
  const unsigned char* p = (const unsigned char*)host_buf;
  uint64_t hdr[4];
  std::memcpy(hdr, p, 32);
  if (hdr[0] != kMagic || hdr[2] != ((uint64_t)hi.q | ((uint64_t)hi.f32 << 32)) || hdr[3] != (uint64_t)hi.n)
    return LBM_ERR_INVALID_ARG;
  const size_t row = (size_t)hi.n * elem_size(hi);
  for (int j = 0; j < hi.q; ++j) {
    void* dst = hi.f32 ? (void*)(f32_cur(b, hi) + (size_t)j * hi.stride)
                       : (void*)(f64_cur(b, hi) + (size_t)j * hi.stride);
    LBM_HIP(hipMemcpyAsync(dst, p + 32 + j * row, row, hipMemcpyHostToDevice, b->stream));
  }
  LBM_HIP(hipMemsetAsync(b->status, 0, sizeof(int), b->stream));
  LBM_HIP(hipStreamSynchronize(b->stream));
  hi.steps_done = (int64_t)hdr[1];
  return LBM_OK;
}

lbm_status lbm_set_path(lbm_problem h, int32_t path) {
  if (!h || path < 0 || path > 4) return LBM_ERR_INVALID_ARG;
  h->b->path = path;
  return LBM_OK;
}

lbm_status lbm_last_advance_ms(lbm_problem h, float* ms) {
  if (!h || !ms) return LBM_ERR_INVALID_ARG;
  return lbm_batch_last_advance_ms(h->b, ms);
}

lbm_status lbm_destroy(lbm_problem h) {
  if (!h) return LBM_ERR_INVALID_ARG;
  destroy_batch(h->b);
  delete h;
  return LBM_OK;
}

lbm_status lbm_batch_create(const lbm_desc* descs, int32_t count, void* stream, lbm_batch* out) {
  return create_batch(descs, count, stream, nullptr, 0, out);
}

lbm_status lbm_batch_load_phi(lbm_batch b, const double* const* phi0) {
  if (!b || !phi0) return LBM_ERR_INVALID_ARG;
  for (size_t i = 0; i < b->inst.size(); ++i)
    if (!phi0[i]) return LBM_ERR_INVALID_ARG;
  std::vector<int> idx(b->inst.size());
  for (size_t i = 0; i < b->inst.size(); ++i) {
    lbm_status s = check_phi(b->inst[i], phi0[i]);
    if (s != LBM_OK) return s;
    idx[i] = (int)i;
  }
  return load_many(b, idx.data(), phi0, (int)idx.size(), false);
}

lbm_status lbm_batch_advance(lbm_batch b, const int64_t* steps) {
  if (!b) return LBM_ERR_INVALID_ARG;
  if (!steps) return LBM_OK;
  return advance(b, steps);
}

lbm_status lbm_batch_read_phi(lbm_batch b, int32_t i, double* out, lbm_status* inst_status) {
  if (!b || !out || i < 0 || i >= (int32_t)b->inst.size()) return LBM_ERR_INVALID_ARG;
  lbm_status s = read_phi(b, i, out, 0, inst_status);
  return (s == LBM_ERR_NONFINITE || s == LBM_ERR_TIMEOUT) ? LBM_OK : s;
}

lbm_status lbm_batch_last_advance_ms(lbm_batch b, float* ms) {
  if (!b || !ms) return LBM_ERR_INVALID_ARG;
  LBM_HIP(hipEventSynchronize(b->ev1));
  LBM_HIP(hipEventElapsedTime(ms, b->ev0, b->ev1));
  return LBM_OK;
}

lbm_status lbm_batch_set_path(lbm_batch b, int32_t path) {
  if (!b || path < 0 || path > 4) return LBM_ERR_INVALID_ARG;
  b->path = path;
  return LBM_OK;
}

lbm_status lbm_batch_set_tiling(lbm_batch b, int32_t steps_per_launch, int32_t wgs_per_cu) {
  if (!b || steps_per_launch < 0 || steps_per_launch > 4096 || wgs_per_cu < 0 || wgs_per_cu > 8)
    return LBM_ERR_INVALID_ARG;
  b->tile_steps = steps_per_launch;
  b->tile_wgs = wgs_per_cu;
  return LBM_OK;
}

lbm_status lbm_batch_autotune(lbm_batch b, int64_t probe_steps, lbm_tuning* out) {
  if (!b || probe_steps < 1 || probe_steps > kMaxStepsPerLaunch) return LBM_ERR_INVALID_ARG;
  if (b->arena[0]) return LBM_ERR_UNSUPPORTED;   // server-owned batches re-plan every block
  return autotune(b, probe_steps, out);
}

lbm_status lbm_batch_set_resident(lbm_batch b, int32_t max_workgroups, int32_t chunks) {
  if (!b || max_workgroups < 0 || max_workgroups > kMaxResidentGrid || chunks < 0 || chunks > kMaxChunks)
    return LBM_ERR_INVALID_ARG;
  b->res_grid = max_workgroups;
  b->res_chunks = chunks;
  return LBM_OK;
}

lbm_status lbm_batch_set_lanes(lbm_batch b, int32_t lanes) {
  if (!b || lanes < 0 || lanes > kAuxStreams) return LBM_ERR_INVALID_ARG;
  b->lanes = lanes;
  return LBM_OK;
}

lbm_status lbm_batch_test_stall(lbm_batch b, int32_t what, int64_t wait_us) {
  if (!b || what < 0 || what > 2 || wait_us < 0 || wait_us > (int64_t(1) << 40)) return LBM_ERR_INVALID_ARG;
  b->test_stall = what;
  b->test_wait_us = wait_us;
  return LBM_OK;
}

lbm_status lbm_set_tiling(lbm_problem h, int32_t steps_per_launch, int32_t wgs_per_cu) {
  if (!h) return LBM_ERR_INVALID_ARG;
  return lbm_batch_set_tiling(h->b, steps_per_launch, wgs_per_cu);
}

lbm_status lbm_batch_destroy(lbm_batch b) {
  if (!b) return LBM_ERR_INVALID_ARG;
  destroy_batch(b);
  return LBM_OK;
}

}  // extern "C"

// ===========================================================================
// Serving: continuous batching of solve requests
// ===========================================================================
namespace {

// first-fit allocator over [0, size) in 256-byte units
struct Arena {
  struct Block { size_t off, len; };
  std::vector<Block> free;
  size_t size = 0;
  void init(size_t bytes) {
    size = bytes / 256 * 256;
    free.assign(1, Block{0, size});
  }
  bool alloc(size_t bytes, size_t* off) {
    bytes = (bytes + 255) / 256 * 256;
    for (size_t i = 0; i < free.size(); ++i) {
      if (free[i].len >= bytes) {
        *off = free[i].off;
        free[i].off += bytes;
        free[i].len -= bytes;
        if (free[i].len == 0) free.erase(free.begin() + i);
        return true;
      }
    }
    return false;
  }
  void release(size_t off, size_t bytes) {
    bytes = (bytes + 255) / 256 * 256;
    size_t i = 0;
    while (i < free.size() && free[i].off < off) ++i;
    free.insert(free.begin() + i, Block{off, bytes});
    if (i + 1 < free.size() && free[i].off + free[i].len == free[i + 1].off) {
      free[i].len += free[i + 1].len;
      free.erase(free.begin() + i + 1);
    }
    if (i > 0 && free[i - 1].off + free[i - 1].len == free[i].off) {
      free[i - 1].len += free[i].len;
      free.erase(free.begin() + i);
    }
  }
  size_t available() const {
    size_t t = 0;
    for (const Block& b : free) t += b.len;
    return t;
  }
};

double now_s() {
  return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

struct Request {
  int64_t id;
  lbm_desc desc;
  std::vector<double> phi0;
  int64_t steps;
};

struct Slot {
  bool active = false;
  int64_t id = -1;
  int64_t remaining = 0;
  size_t off = 0, bytes = 0;
};

struct Result {
  std::vector<double> phi;
  lbm_status status;
  double t_submit = 0.0, t_admit = 0.0, t_retire = 0.0;   // host steady clock
};

size_t state_bytes_of(const lbm_desc& d) {
  const int q = resolved_lattice(d);
  const size_t es = d.prec == LBM_F64 ? sizeof(double) : sizeof(float);
  return (size_t)q * (size_t)lbm_row_stride(d.n) * es;
}

}  // namespace

struct lbm_server_s {
  lbm_batch_s* b = nullptr;
  Arena arena;
  int block = 1000;
  int64_t max_n = 0;
  int64_t next_id = 1;
  std::vector<Request> queue;        // FIFO
  std::vector<Slot> slots;
  std::vector<Result> results;       // indexed by id - 1 (kept until polled)
  std::vector<char> done;
  std::vector<int64_t> steps_buf;
  double node_updates = 0.0;
  double device_ms = 0.0;
  // a round launched and not yet retired (lbm_server_pump): its node updates
  bool inflight = false;
  bool inflight_empty = false;   // the round advanced nothing (only zero-step requests)
  double inflight_nu = 0.0;
};

extern "C" {

lbm_status lbm_server_create(void* stream, size_t budget_bytes, int32_t max_slots, int64_t max_n,
                             int32_t block_steps, lbm_server* out) {
  if (!out || max_slots <= 0 || max_slots > 65536 || max_n < 5 || max_n > (int64_t(1) << 30) ||
      block_steps <= 0 || budget_bytes < 4096)
    return LBM_ERR_INVALID_ARG;
  lbm_server_s* sv = new (std::nothrow) lbm_server_s();
  if (!sv) return LBM_ERR_OUT_OF_MEMORY;
  lbm_batch_s* b = new (std::nothrow) lbm_batch_s();
  if (!b) {
    delete sv;
    return LBM_ERR_OUT_OF_MEMORY;
  }
  sv->b = b;
  b->stream = (hipStream_t)stream;
  b->lim = query_limits();
  b->inst.resize(max_slots);
  lbm_status s = b->lim.ok ? LBM_OK : LBM_ERR_DEVICE;
  // two mirrored arenas: the current state and the other buffer of the tiled path
  sv->arena.init(budget_bytes);
  for (int k = 0; k < 2 && s == LBM_OK; ++k)
    if (hipMalloc(&b->arena[k], sv->arena.size) != hipSuccess) s = LBM_ERR_OUT_OF_MEMORY;
  if (s == LBM_OK) {
    b->f64[0] = (double*)b->arena[0];
    b->f32[0] = (float*)b->arena[0];
    b->f64[1] = (double*)b->arena[1];
    b->f32[1] = (float*)b->arena[1];
    b->n64 = sv->arena.size / sizeof(double);
    b->n32 = sv->arena.size / sizeof(float);
    s = alloc_tables(b, (size_t)max_n, (size_t)2 << 20);
  }
  if (s != LBM_OK) {
    destroy_batch(b);
    delete sv;
    return s;
  }
  sv->block = block_steps;
  sv->max_n = max_n;
  sv->slots.resize(max_slots);
  sv->steps_buf.assign(max_slots, 0);
  *out = sv;
  return LBM_OK;
}

lbm_status lbm_server_submit(lbm_server sv, const lbm_desc* d, const double* phi0, int64_t steps, int64_t* id) {
  if (!sv || !d || !phi0 || !id || steps < 0) return LBM_ERR_INVALID_ARG;
  // the checks admission repeats: the model, its kernel variant and phi0
  HostInst probe;
  lbm_status s = prepare_one(*d, &probe);
  if (s != LBM_OK) return s;
  if (d->n > sv->max_n) return LBM_ERR_INVALID_ARG;
  if (d->bc != LBM_BC_PERIODIC) return LBM_ERR_UNSUPPORTED;   // requests carry no boundary data
  if (state_bytes_of(*d) > sv->arena.size) return LBM_ERR_OUT_OF_MEMORY;
  for (int64_t i = 0; i < d->n; ++i)
    if (!std::isfinite(phi0[i]) || (probe.mdl.gF > 1 && phi0[i] < 0)) return LBM_ERR_INVALID_ARG;
  Request r;
  r.id = sv->next_id++;
  r.desc = *d;
  r.phi0.assign(phi0, phi0 + d->n);
  r.steps = steps;
  sv->queue.push_back(std::move(r));
  sv->results.emplace_back();
  sv->results.back().t_submit = now_s();
  sv->done.push_back(0);
  *id = sv->queue.back().id;
  return LBM_OK;
}

}  // extern "C"

namespace {

// retires the request in `slot`, which could not be started, with status s
void server_drop(lbm_server_s* sv, int slot, lbm_status s) {
  Slot& sl = sv->slots[slot];
  Result& res = sv->results[sl.id - 1];
  sv->arena.release(sl.off, sl.bytes);
  sv->b->inst[slot] = HostInst();
  res.status = s;
  res.t_admit = res.t_retire = now_s();
  sv->done[sl.id - 1] = 1;
  sl = Slot();
}

// Admission: queued requests in arrival order while a slot and arena space
// are free (f := f_eq(phi0) on the stream, which it synchronises).
void server_admit(lbm_server_s* sv) {
  lbm_batch_s* b = sv->b;
  std::vector<int> idx;
  std::vector<const double*> phi;
  size_t qi = 0;
  for (; qi < sv->queue.size(); ++qi) {
    Request& r = sv->queue[qi];
    int slot = -1;
    for (size_t k = 0; k < sv->slots.size(); ++k)
      if (!sv->slots[k].active) {
        slot = (int)k;
        break;
      }
    if (slot < 0) break;
    const size_t bytes = state_bytes_of(r.desc);
    size_t off = 0;
    if (!sv->arena.alloc(bytes, &off)) break;   // FIFO: wait for space
    HostInst& h = b->inst[slot];
    const lbm_status s = prepare_one(r.desc, &h);
    Slot& sl = sv->slots[slot];
    sl.active = true;
    sl.id = r.id;
    sl.remaining = r.steps;
    sl.off = off;
    sl.bytes = bytes;
    if (s == LBM_OK) {
      h.off = (int64_t)(off / (h.f32 ? sizeof(float) : sizeof(double)));
      idx.push_back(slot);
      phi.push_back(r.phi0.data());
    } else {
      server_drop(sv, slot, s);
    }
  }
  // one load for all; submission ran the same checks, so a failure is a device
  // error: its requests retire with it (no phi) and the queue moves on
  if (!idx.empty()) {
    const lbm_status s = load_many(b, idx.data(), phi.data(), (int)idx.size(), true);
    for (int slot : idx) {
      sv->results[sv->slots[slot].id - 1].t_admit = now_s();
      if (s != LBM_OK) server_drop(sv, slot, s);
    }
  }
  sv->queue.erase(sv->queue.begin(), sv->queue.begin() + qi);
}

// One block for every active request in one planner pass (asynchronous on
// the stream).  A round lasts as long as its slowest request's block;
// requests whose steps take less time take proportionally more steps in the
// same round, up to 8 blocks.  A step's time is estimated as its arithmetic
// per node (lattice size x polynomial degree) times the node sweeps of one
// workgroup (1024 threads; larger grids are spread over several).
lbm_status server_launch(lbm_server_s* sv, int* act_out) {
  lbm_batch_s* b = sv->b;
  auto step_cost = [&](size_t k) {
    const HostInst& h = b->inst[k];
    const int sweeps = (std::min(h.n, 4096) + 1023) / 1024;
    return (double)h.q * ((h.D & 0xff) + 3) * sweeps;
  };
  double cmax = 0.0;
  for (size_t k = 0; k < sv->slots.size(); ++k)
    if (sv->slots[k].active) cmax = std::max(cmax, step_cost(k));
  int act = 0;
  double nu = 0.0;
  for (size_t k = 0; k < sv->slots.size(); ++k) {
    const Slot& sl = sv->slots[k];
    const double scale = sl.active ? std::min(8.0, std::max(1.0, cmax / step_cost(k))) : 1.0;
    sv->steps_buf[k] = sl.active ? std::min<int64_t>(sl.remaining, (int64_t)(sv->block * scale)) : 0;
    if (sl.active) {
      ++act;
      nu += (double)sv->steps_buf[k] * b->inst[k].n;
    }
  }
  *act_out = act;
  if (!act) return LBM_OK;
  sv->inflight_empty = nu == 0.0;
  if (!sv->inflight_empty) {
    lbm_status s = advance(b, sv->steps_buf.data());
    if (s != LBM_OK) return s;
  }
  sv->inflight = true;
  sv->inflight_nu = nu;
  return LBM_OK;
}

// The launched round has finished on the device: account for it, retire the
// requests it completed (phi read out, space released).
lbm_status server_finish(lbm_server_s* sv, int* retired) {
  lbm_batch_s* b = sv->b;
  if (!sv->inflight_empty) {
    float ms = 0.0f;
    LBM_HIP(hipEventSynchronize(b->ev1));
    if (hipEventElapsedTime(&ms, b->ev0, b->ev1) == hipSuccess) sv->device_ms += ms;
  }
  sv->node_updates += sv->inflight_nu;
  sv->inflight = false;
  sv->inflight_nu = 0.0;
  int ret = 0;
  for (size_t k = 0; k < sv->slots.size(); ++k) {
    Slot& sl = sv->slots[k];
    if (!sl.active) continue;
    sl.remaining -= sv->steps_buf[k];
    sv->steps_buf[k] = 0;
    if (sl.remaining > 0) continue;
    Result& res = sv->results[sl.id - 1];
    res.phi.resize(b->inst[k].n);
    lbm_status st = LBM_OK;
    lbm_status s = read_phi(b, (int)k, res.phi.data(), 0, &st);
    if (s != LBM_OK && s != LBM_ERR_NONFINITE && s != LBM_ERR_TIMEOUT) return s;
    res.status = st;
    res.t_retire = now_s();
    sv->done[sl.id - 1] = 1;
    sv->arena.release(sl.off, sl.bytes);
    sl = Slot();
    ++ret;
  }
  *retired = ret;
  return LBM_OK;
}

void server_counts(const lbm_server_s* sv, int32_t* active, int32_t* queued) {
  int act = 0;
  for (const Slot& sl : sv->slots) act += sl.active ? 1 : 0;
  if (active) *active = act;
  if (queued) *queued = (int32_t)sv->queue.size();
}

}  // namespace

extern "C" {

// One synchronous scheduling round: finish a round a pump left running,
// admit, advance every active request by one block (all concurrent on the
// device), wait, retire.
lbm_status lbm_server_step(lbm_server sv, int32_t* active, int32_t* queued, int32_t* retired) {
  if (!sv) return LBM_ERR_INVALID_ARG;
  int ret = 0, r = 0, act = 0;
  if (sv->inflight) {
    lbm_status s = server_finish(sv, &r);
    if (s != LBM_OK) return s;
    ret += r;
  }
  server_admit(sv);
  lbm_status s = server_launch(sv, &act);
  if (s != LBM_OK) return s;
  if (sv->inflight) {
    s = server_finish(sv, &r);
    if (s != LBM_OK) return s;
    ret += r;
  }
  server_counts(sv, active, queued);
  if (retired) *retired = ret;
  return LBM_OK;
}

// Continuous batching without blocking the caller: while a round runs on the
// device, return at once (*running = 1); once it has finished, retire what it
// completed, admit queued requests and launch the next round.
lbm_status lbm_server_pump(lbm_server sv, int32_t* running, int32_t* active, int32_t* queued, int32_t* retired) {
  if (!sv) return LBM_ERR_INVALID_ARG;
  int ret = 0, act = 0;
  if (sv->inflight && !sv->inflight_empty) {
    const hipError_t q = hipEventQuery(sv->b->ev1);
    if (q == hipErrorNotReady) {
      if (running) *running = 1;
      server_counts(sv, active, queued);
      if (retired) *retired = 0;
      return LBM_OK;
    }
    if (q != hipSuccess) return LBM_ERR_DEVICE;
  }
  if (sv->inflight) {
    lbm_status s = server_finish(sv, &ret);
    if (s != LBM_OK) return s;
  }
  server_admit(sv);
  lbm_status s = server_launch(sv, &act);
  if (s != LBM_OK) return s;
  if (running) *running = sv->inflight ? 1 : 0;
  server_counts(sv, active, queued);
  if (retired) *retired = ret;
  return LBM_OK;
}

lbm_status lbm_server_timing(lbm_server sv, int64_t id, double* queue_s, double* service_s) {
  if (!sv || id < 1 || id >= sv->next_id) return LBM_ERR_INVALID_ARG;
  if (sv->done[id - 1] == 0) return LBM_ERR_BUSY;
  const Result& r = sv->results[id - 1];
  if (queue_s) *queue_s = r.t_admit - r.t_submit;
  if (service_s) *service_s = r.t_retire - r.t_admit;
  return LBM_OK;
}

lbm_status lbm_server_poll(lbm_server sv, int64_t id, double* out, int64_t n, lbm_status* inst_status) {
  if (!sv || id < 1 || id >= sv->next_id) return LBM_ERR_INVALID_ARG;
  if (sv->done[id - 1] != 1) return sv->done[id - 1] == 2 ? LBM_ERR_INVALID_ARG : LBM_ERR_BUSY;
  Result& r = sv->results[id - 1];
  if (!out || n < (int64_t)r.phi.size()) return LBM_ERR_INVALID_ARG;
  std::memcpy(out, r.phi.data(), sizeof(double) * r.phi.size());
  if (inst_status) *inst_status = r.status;
  r.phi.clear();
  r.phi.shrink_to_fit();
  sv->done[id - 1] = 2;   // delivered
  return LBM_OK;
}

lbm_status lbm_server_stats(lbm_server sv, double* node_updates, double* device_ms, size_t* free_bytes) {
  if (!sv) return LBM_ERR_INVALID_ARG;
  if (node_updates) *node_updates = sv->node_updates;
  if (device_ms) *device_ms = sv->device_ms;
  if (free_bytes) *free_bytes = sv->arena.available();
  return LBM_OK;
}

lbm_status lbm_server_destroy(lbm_server sv) {
  if (!sv) return LBM_ERR_INVALID_ARG;
  destroy_batch(sv->b);
  delete sv;
  return LBM_OK;
}

}  // extern "C"
