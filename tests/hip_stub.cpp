// A stand-in for the HIP runtime and the kernel launchers, so that the whole host
// runtime (runtime.cpp, coeffs.cpp) runs without a GPU.  Device memory is host
// memory; a launch does no arithmetic but records what it would read and write:
//  * a state buffer holds the number of steps done to it, which a read-out
//    returns as phi, so that a lost, repeated or misplaced step shows;
//  * streams, events and host waits are kept as sets of launches that are over
//    before the next one starts; two launches that touch one buffer, one of them
//    writing, without such an order are a fault, as is a launch that holds two
//    step chunks of one instance, or a kernel given memory that is not on the GPU.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "kernels.hpp"
#include "wave.hpp"

using namespace lbm;

namespace {

using Clock = std::vector<bool>;
void join(Clock* a, const Clock& b) {
  if (a->size() < b.size()) a->resize(b.size());
  for (size_t k = 0; k < b.size(); ++k)
    if (b[k]) (*a)[k] = true;
}
bool has(const Clock& a, int k) { return k < (int)a.size() && a[k]; }

struct Access { int launch; bool write; };
struct Record { int64_t kind, stream, groups, steps, tag, blocks, width, jobs; };
// A slab launch: the workgroups that an XCD gets at most (a launch hands them to
// the eight XCDs of 32 CUs in turn, from any of them on), and what is over before
// it starts.
struct SlabRun { int launch; int64_t wgs; Clock before; };
bool ordered(const SlabRun& a, const SlabRun& b) { return has(a.before, b.launch) || has(b.before, a.launch); }
enum { kReg = 0, kSlabs = 1, kTiles = 2, kLds = 3, kLdsSlabs = 4, kLdsTiles = 5, kStream = 6, kRead = 7, kInit = 8 };

struct World {
  std::map<hipStream_t, Clock> streams;
  std::map<hipEvent_t, Clock> events;
  Clock host;
  int launches = 0;
  std::map<uint64_t, std::vector<Access>> access;   // by the address of row 0
  std::map<uint64_t, int64_t> done;                 // steps done to a state
  std::map<uint64_t, size_t> device, pinned, foreign;
  size_t used = 0, limit = ~size_t(0);
  std::vector<Record> log;
  std::vector<SlabRun> slabs;
  int copies = 0;
  long long slab_wait = 0;                  // ticks, of the latest slab launch
  int faults = 0;
  std::string first;
};
World w;

void fault(const char* fmt, ...) {
  char buf[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  if (w.faults++ == 0) w.first = buf;
}
bool inside(const std::map<uint64_t, size_t>& m, uint64_t p, size_t bytes) {
  auto it = m.upper_bound(p);
  if (it == m.begin()) return false;
  --it;
  return p + bytes <= it->first + it->second;
}
void reachable(const void* p, size_t bytes, const char* what) {
  const uint64_t a = (uint64_t)(uintptr_t)p;
  if (!inside(w.device, a, bytes) && !inside(w.pinned, a, bytes)) fault("%s: a kernel given memory that is not on the GPU", what);
}

// the most slab workgroups that launches of `from` have on an XCD together, no two of
// which are kept apart by an order; `taken`: of those chosen so far
void in_flight(const std::vector<const SlabRun*>& from, int64_t taken, int64_t* most) {
  *most = std::max(*most, taken);
  int64_t left = taken;
  for (const SlabRun* r : from) left += r->wgs;
  if (left <= *most) return;
  std::vector<const SlabRun*> rest(from.begin() + 1, from.end()), beside;
  for (const SlabRun* r : rest)
    if (!ordered(*from[0], *r)) beside.push_back(r);
  in_flight(beside, taken + from[0]->wgs, most);
  if (beside.size() < rest.size()) in_flight(rest, taken, most);
}
// one launch on `s` that reads and writes the states at these addresses
struct Touch { uint64_t at; bool write; };
void launch(hipStream_t s, const std::vector<Touch>& what, Record r) {
  Clock before = w.streams[s];
  join(&before, w.host);
  const int me = w.launches++;
  for (const Touch& t : what) {
    for (const Access& a : w.access[t.at])
      if (a.launch != me && (a.write || t.write) && !has(before, a.launch))
        fault("launches %d and %d touch the state at %llx in no order", a.launch, me, (unsigned long long)t.at);
    w.access[t.at].push_back({me, t.write});
  }
  if (r.kind == kSlabs) {   // (a launch alone may hold several workgroups of a CU, launches together may not)
    w.slabs.erase(std::remove_if(w.slabs.begin(), w.slabs.end(), [](const SlabRun& o) { return has(w.host, o.launch); }),
                  w.slabs.end());
    w.slabs.push_back({me, (r.groups + 7) / 8, before});
    const SlabRun& run = w.slabs.back();
    std::vector<const SlabRun*> beside;
    for (const SlabRun& o : w.slabs)
      if (o.launch != me && !ordered(o, run)) beside.push_back(&o);
    int64_t most = 0;
    in_flight(beside, run.wgs, &most);
    if (most > 32 && most > run.wgs) fault("%lld slab workgroups in flight together on an XCD", (long long)most);
  }
  before.resize(me + 1);
  before[me] = true;
  w.streams[s] = before;
  int id = 0;
  for (const auto& [st, c] : w.streams) {
    if (st == s) break;
    ++id;
  }
  r.stream = id;
  w.log.push_back(r);
}
uint64_t word(const void* p) { return (uint64_t)(uintptr_t)p; }

}  // namespace

// ---------------------------------------------------------------- test access
extern "C" {
// forgets the launches so far (states keep their step counts)
void stub_reset() {
  w.log.clear();
  w.access.clear();
  w.faults = w.copies = 0;
  w.first.clear();
}
int stub_faults(char* text, int cap) {
  if (text && cap > 0) snprintf(text, cap, "%s", w.first.c_str());
  return w.faults;
}
int stub_copies() { return w.copies; }   // and clears, on a stream
long long stub_slab_wait() { return w.slab_wait; }
int stub_launches() { return (int)w.log.size(); }
void stub_launch(int k, int64_t* out) { std::memcpy(out, &w.log[k], sizeof(Record)); }
// device memory that may be allocated from now on
void stub_limit(size_t more) { w.limit = more == ~size_t(0) ? more : w.used + more; }
int stub_pinned() { return (int)w.pinned.size(); }   // allocations
// memory of another GPU
void* stub_foreign(size_t bytes) {
  void* p = calloc(1, bytes);
  w.foreign[word(p)] = bytes;
  return p;
}
void* stub_device(size_t bytes) {
  void* p = nullptr;
  return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
}

// ------------------------------------------------------------------- runtime
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 163840 : 100000;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  if (w.used + n > w.limit) return hipErrorOutOfMemory;
  *p = calloc(1, n ? n : 1);
  w.device[word(*p)] = n;
  w.used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  const size_t n = w.device[word(p)];
  w.used -= n;
  w.device.erase(word(p));
  w.access.erase(w.access.lower_bound(word(p)), w.access.lower_bound(word(p) + n));
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n ? n : 1);
  w.pinned[word(*p)] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  w.pinned.erase(word(p));
  free(p);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof(*a));
  const bool here = inside(w.device, word(p), 1), there = inside(w.foreign, word(p), 1);
  if (!here && !there && !inside(w.pinned, word(p), 1)) return hipErrorInvalidValue;
  a->type = here || there ? hipMemoryTypeDevice : hipMemoryTypeHost;
  a->device = there ? 1 : 0;
  a->devicePointer = const_cast<void*>(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  ++w.copies;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  ++w.copies;
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)calloc(1, 8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { w.streams.erase(s); free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { join(&w.host, w.streams[s]); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { join(&w.streams[s], w.events[e]); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)calloc(1, 8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { w.events.erase(e); free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { w.events[e] = w.streams[s]; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { join(&w.host, w.events[e]); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) {   // over as far as the host has waited for it
  const Clock& c = w.events[e];
  for (size_t k = 0; k < c.size(); ++k)
    if (c[k] && !has(w.host, (int)k)) return hipErrorNotReady;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
// (a graph is the chain of fused steps of one instance: the first one's input, and their number)
struct StubGraph { const void* in = nullptr; const void* out = nullptr; int nodes = 0; };
hipError_t hipGraphCreate(hipGraph_t* g, unsigned) { *g = (hipGraph_t) new StubGraph; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { delete (StubGraph*)g; return hipSuccess; }
hipError_t hipGraphAddKernelNode(hipGraphNode_t* n, hipGraph_t g, const hipGraphNode_t*, size_t, const hipKernelNodeParams* p) {
  StubGraph* sg = (StubGraph*)g;
  if (sg->nodes++ == 0) {
    sg->in = *(const void**)p->kernelParams[0];
    sg->out = *(const void**)p->kernelParams[1];
  }
  *n = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t) new StubGraph(*(StubGraph*)g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete (StubGraph*)e; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  const StubGraph* g = (const StubGraph*)e;
  launch(s, {{word(g->in), true}, {word(g->out), true}}, {kStream, 0, 0, g->nodes, 0, 0, 0, 0});
  w.done[word(g->in)] += g->nodes;
  return hipSuccess;
}
}  // extern "C"

// ------------------------------------------------------------------ launchers
namespace lbm {

hipError_t launch_init_many(bool, const DevInit* recs, int count, int, const DevCoef*, int* status, hipStream_t s) {
  std::vector<Touch> what;
  for (int k = 0; k < count; ++k) {
    reachable((const void*)(uintptr_t)recs[k].src, sizeof(double) * recs[k].len, "phi0");
    if (!recs[k].first) continue;
    what.push_back({recs[k].dst, true});
    w.done[recs[k].dst] = 0;
    status[recs[k].inst] = 0;
  }
  launch(s, what, {kInit, 0, count, 0, 0, 0, 0, 0});
  return hipSuccess;
}
hipError_t launch_init_one(bool f32, const DevInit& r, const DevCoef* c, int* status, int*, hipStream_t s) {
  return launch_init_many(f32, &r, 1, r.len, c, status, s);
}
hipError_t launch_check_phi(const double* phi, int n, int* words, hipStream_t) {
  reachable(phi, sizeof(double) * n, "phi0");
  reachable(words, 2 * sizeof(int), "words");
  return hipSuccess;
}
hipError_t launch_read(bool, const void* f, double* phi, int n, int, int, double, const int* status, int* words, int seq,
                       const int*, hipStream_t s) {
  reachable(phi, sizeof(double) * n, "phi");
  launch(s, {{word(f), false}}, {kRead, 0, 0, 0, 0, 0, 0, 0});
  words[0] = *status;
  if (inside(w.device, word(phi), 8) || inside(w.pinned, word(phi), 8))
    for (int k = 0; k < n; ++k) phi[k] = (double)w.done[word(f)];
  for (int k = 0; seq && k < (n + 255) / 256; ++k) words[2 + k] = seq;
  return hipSuccess;
}
hipError_t launch_sum(const double*, int, double*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_bound(int, int, int, void*, int, int, int, int, const double*, const DevCoef*, hipStream_t) { return hipSuccess; }
hipError_t launch_stream(int, int, int, const void* in, void* out, int, int, const DevCoef*, hipStream_t s) {
  launch(s, {{word(in), false}, {word(out), true}}, {kStream, 0, 0, 1, 0, 0, 0, 0});
  w.done[word(out)] = w.done[word(in)] + 1;
  return hipSuccess;
}
const void* stream_kernel(int, int, int) { return &w; }
hipError_t launch_resident(int, int, int, const DevJob* jobs, const DevJobInst* inst, int njobs, int, int*, int*, int*,
                           const DevCoef*, int*, long long, int, int grid, int, size_t, hipStream_t s) {
  std::vector<Touch> what;
  std::set<uint64_t> seen;
  for (int k = 0; k < njobs; ++k)
    for (int u = jobs[k].first; u < jobs[k].first + jobs[k].count; ++u) {
      if (!seen.insert(inst[u].addr).second) fault("instance %d twice in one launch", inst[u].inst);
      what.push_back({inst[u].addr, true});
      w.done[inst[u].addr] += jobs[k].steps;
    }
  launch(s, what, {kLds, 0, grid, 0, 0, 0, 0, 0});
  return hipSuccess;
}
hipError_t launch_reg(int, int, int, bool wide, const DevItem* items, int nitems, const DevJob* jobs, const DevSeg* segs, int*,
                      int*, const DevCoef*, int*, long long, int, int grid, int block, size_t lds, hipStream_t s) {
  std::vector<Touch> what;
  std::set<int> seen;
  int64_t width = 0;   // the widest job's nodes per lane
  for (int k = 0; k < nitems; ++k) {
    const DevJob& j = jobs[items[k].job];
    seen.insert(items[k].job);
    width = width > j.nodes ? width : j.nodes;
    for (int u = j.first; u < j.first + j.count; ++u) {
      what.push_back({segs[u].in, true});
      w.done[segs[u].in] += items[k].steps;
    }
  }
  // the launch's length in steps of jobs of equal steps' cost: items in the list's
  // order to the workgroup that is free first, a job's second part after its first
  std::vector<int64_t> free(grid, 0);
  std::map<int, int64_t> over;
  int64_t end = 0;
  for (int k = 0; k < nitems; ++k) {
    auto at = std::min_element(free.begin(), free.end());
    if (items[k].part > 0) *at = std::max(*at, over[items[k].job]);
    *at += items[k].steps;
    over[items[k].job] = *at;
    end = std::max(end, *at);
  }
  // the part of a CU's waves that jobs of this size fill, in percent
  const int waves = block / 64, filled = 100 * (reg_waves(wide) / waves * waves) / reg_waves(wide);
  launch(s, what, {kReg, 0, grid, end, filled, (int64_t)lds, width, (int64_t)seen.size()});
  return hipSuccess;
}
hipError_t launch_seg(int, int, int, bool, const DevSeg* segs, int nsegs, int width, int, int sx, bool tile, int turn, void*,
                      unsigned tag, const DevCoef*, int*, long long wait, int, int, size_t, hipStream_t s) {
  w.slab_wait = wait;
  std::vector<Touch> what;
  std::map<int, std::pair<DevSeg, int64_t>> seen;   // first segment of an instance, nodes so far
  int64_t most = 0, blocks = 0;
  for (int k = 0; k < nsegs; ++k) {
    const DevSeg& sg = segs[k];
    auto [it, fresh] = seen.insert({sg.inst, {sg, 0}});
    const DevSeg& a = it->second.first;
    if (!fresh && (a.in != sg.in || a.out != sg.out || a.steps != sg.steps)) fault("instance %d twice in one launch", sg.inst);
    it->second.second += sg.len;
  }
  for (const auto& [inst, v] : seen) {
    const DevSeg& sg = v.first;
    if (v.second != sg.n) fault("instance %d: segments hold %lld of %d nodes", inst, (long long)v.second, sg.n);
    int64_t st = sg.steps;
    uint64_t in = sg.in, out = sg.out;
    if (tile) {
      st = st - (int64_t)turn * sx < sx ? st - (int64_t)turn * sx : sx;
      if (st <= 0) continue;
      if (turn & 1) std::swap(in, out);
    }
    what.push_back({in, false});
    what.push_back({out, true});
    w.done[out] = w.done[in] + st;
    most = most > st ? most : st;
    blocks = (most + sx - 1) / sx;
  }
  launch(s, what, {tile ? kTiles : kSlabs, 0, nsegs, most, tag, blocks, width, 0});
  return hipSuccess;
}
hipError_t launch_slab(int, int prec, int, const DevSlab* slabs, int nslabs, const DevTileInst* ti, void* b0, void* b1, int,
                       int, void*, int*, const DevCoef*, int*, long long wait, int, int, size_t, hipStream_t s) {
  w.slab_wait = wait;
  const size_t es = prec ? 4 : 8;
  std::vector<Touch> what;
  std::map<int, int> seen;   // the step chunk of an instance
  int64_t most = 0;
  for (int k = 0; k < nslabs; ++k) {
    const DevTileInst& t = ti[slabs[k].ti];
    auto [it, fresh] = seen.insert({t.inst, slabs[k].ti});
    if (!fresh && it->second != slabs[k].ti) fault("instance %d twice in one launch", t.inst);
    if (!fresh) continue;
    const uint64_t p0 = word(b0) + t.off * es, p1 = word(b1) + t.off * es;
    const uint64_t in = t.cur0 ? p1 : p0, out = t.cur0 ? p0 : p1;
    what.push_back({in, false});
    what.push_back({out, true});
    w.done[out] = w.done[in] + t.steps;
    most = most > t.steps ? most : t.steps;
  }
  launch(s, what, {kLdsSlabs, 0, nslabs, most, 0, 0, 0, 0});
  return hipSuccess;
}
hipError_t launch_tile(int, int prec, const DevTile* tiles, int ntiles, const DevTileInst* ti, void* b0, void* b1, int turn,
                       int sp, int, const DevCoef*, int*, int, size_t, hipStream_t s) {
  const size_t es = prec ? 4 : 8;
  std::vector<Touch> what;
  std::set<int> seen;
  for (int k = 0; k < ntiles; ++k) {
    const DevTileInst& t = ti[tiles[k].ti];
    if (!seen.insert(tiles[k].ti).second) continue;
    int64_t st = t.steps - (int64_t)turn * sp;
    st = st < sp ? st : sp;
    if (st <= 0) continue;
    const uint64_t p0 = word(b0) + t.off * es, p1 = word(b1) + t.off * es;
    const bool second = (t.cur0 ^ (turn & 1)) != 0;
    const uint64_t in = second ? p1 : p0, out = second ? p0 : p1;
    what.push_back({in, false});
    what.push_back({out, true});
    w.done[out] = w.done[in] + st;
  }
  launch(s, what, {kLdsTiles, 0, ntiles, 0, 0, 0, 0, 0});
  return hipSuccess;
}
hipError_t launch_zero_ints(int* p, int n, hipStream_t) { std::memset(p, 0, sizeof(int) * n); return hipSuccess; }
hipError_t launch_tables(const NoAllocTables&, unsigned char*, bool, hipStream_t) { return hipSuccess; }
hipError_t noalloc_scratch(void** out) {
  static void* p = stub_device(kNoAllocScratchBytes);
  *out = p;
  return hipSuccess;
}
WaveRows wave_rows(double* rows, int n, double dx, double dt, const lbm_wave& wv) { return WaveRows{rows, dx, dt, wv, n, -1, -1}; }
hipError_t launch_wave_rows(const WaveRows*, int, int64_t, int, hipStream_t) { return hipSuccess; }

// workgroups of a CU: its waves (by the kernel's registers) and its LDS
hipError_t reg_occupancy(int, int, int, bool wide, int block, size_t lds, int* n) {
  const int by_lds = lds ? (int)(163840 / lds) : 64, by_waves = 64 * reg_waves(wide) / block;
  *n = by_lds < by_waves ? by_lds : by_waves;
  return hipSuccess;
}
hipError_t seg_occupancy(int q, int prec, int code, bool wide, int block, size_t lds, int* n) {
  return reg_occupancy(q, prec, code, wide, block, lds, n);
}
hipError_t resident_occupancy(int, int, int, int block, size_t lds, int* n) {
  const int by_lds = lds ? (int)(163840 / lds) : 64, by_waves = 1024 / block;
  *n = by_lds < by_waves ? by_lds : by_waves;
  return hipSuccess;
}
hipError_t slab_occupancy(int q, int prec, int code, int block, size_t lds, int* n) {
  return resident_occupancy(q, prec, code, block, lds, n);
}
int resident_vgprs(int, int, int) { return 64; }
size_t resident_static_lds(int, int, int) { return 0; }

}  // namespace lbm
