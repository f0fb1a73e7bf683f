// Stand-ins for the HIP calls and the kernel launchers of libh2gemv, on the
// CPU: the library's host sources (h2_*.cpp, h2_noalloc.hip) linked against
// this file run their whole call sequences under the sanitizers, with device
// memory in ordinary heap allocations.
//
// Work is deferred.  A launch, copy or event record becomes an operation with
// the dependencies that streams and events give it, and runs only when
// something waits for it; among the operations that may run, a seeded choice
// picks the next one.  A missing wait between streams therefore shows as a
// result that changes with the seed, a buffer that is freed or reused too
// early as a sanitizer report, a wrong handle as an abort with its name.
// Device memory can be limited (h2_standin_limit), and launches are counted by
// name (h2_standin_count).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "h2_compress.h"
#include "h2_internal.h"

namespace {

[[noreturn]] void die(const char* what) {
  std::fprintf(stderr, "STANDIN FAIL: %s\n", what);
  std::fflush(stderr);
  std::abort();
}

struct Op;
using OpP = std::shared_ptr<Op>;
struct Op {
  std::vector<OpP> deps;
  std::function<void()> fn;
  bool done = false;
};

struct Graph {
  std::vector<OpP> nodes;
};
struct GraphExec {
  std::vector<std::vector<size_t>> deps;
  std::vector<std::function<void()>> fns;
  OpP last;  // of the last launch
};
struct Stream {
  OpP tail, before;  // last operation; the last one before the capture
  std::vector<OpP> waits;
  std::shared_ptr<Graph> cap;  // capturing into
};
struct Event {
  OpP op;
  std::shared_ptr<Graph> cap;
  bool recorded = false;
  double t = 0.0;
};

std::recursive_mutex g_mu;
std::set<Stream*> g_streams;
std::set<Event*> g_events;
std::set<GraphExec*> g_execs;
std::vector<OpP> g_pending;
std::map<void*, size_t> g_mem;
size_t g_used = 0, g_peak = 0, g_limit = size_t(1) << 34;
int g_hide_free = 0;
uint64_t g_seed = 1;
std::map<std::string, int64_t> g_count;
Stream g_null;
double g_clock = 0.0;
using Lock = std::lock_guard<std::recursive_mutex>;

uint64_t rnd() {
  uint64_t z = (g_seed += 0x9e3779b97f4a7c15ull);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

bool ready(const OpP& o) {
  for (const OpP& d : o->deps)
    if (!d->done) return false;
  return true;
}

// Runs pending operations, picked at random among the ready ones, until `until` is done (null: all).
void run(const OpP& until) {
  while (until ? !until->done : !g_pending.empty()) {
    std::vector<size_t> r;
    for (size_t i = 0; i < g_pending.size(); ++i)
      if (ready(g_pending[i])) r.push_back(i);
    if (r.empty()) die("operations wait for each other");
    const size_t i = r[rnd() % r.size()];
    OpP o = g_pending[i];
    g_pending.erase(g_pending.begin() + (long)i);
    if (o->fn) o->fn();
    o->fn = nullptr;
    o->done = true;
    o->deps.clear();
  }
}

Stream* stream_of(hipStream_t s) {
  if (!s) return &g_null;
  Stream* p = reinterpret_cast<Stream*>(s);
  if (!g_streams.count(p)) die("a stream that does not exist");
  return p;
}
Event* event_of(hipEvent_t e) {
  Event* p = reinterpret_cast<Event*>(e);
  if (!g_events.count(p)) die("an event that does not exist");
  return p;
}

OpP enqueue(hipStream_t s, const char* name, std::function<void()> fn) {
  Lock l(g_mu);
  Stream* st = stream_of(s);
  if (name) ++g_count[name];
  OpP o = std::make_shared<Op>();
  if (st->tail) o->deps.push_back(st->tail);
  for (OpP& w : st->waits) o->deps.push_back(w);
  st->waits.clear();
  o->fn = std::move(fn);
  st->tail = o;
  if (st->cap) st->cap->nodes.push_back(o);
  else g_pending.push_back(o);
  return o;
}

template <class F>
hipError_t launch(hipStream_t s, const char* name, F f) {
  enqueue(s, name, std::function<void()>(f));
  return hipSuccess;
}

void sync_stream(Stream* st) {
  if (st->cap) die("a synchronization of a stream under capture");
  if (st->tail) run(st->tail);
  for (OpP& w : st->waits) run(w);
}

void no_capture(const char* what) {
  for (Stream* s : g_streams)
    if (s->cap) die(what);
}

hipError_t do_malloc(void** p, size_t n) {
  Lock l(g_mu);
  no_capture("an allocation under capture");
  *p = nullptr;
  if (g_used + n > g_limit) return hipErrorOutOfMemory;
  void* q = std::malloc(std::max<size_t>(n, 1));
  std::memset(q, 0xa5, n);
  g_mem[q] = n;
  g_used += n;
  g_peak = std::max(g_peak, g_used);
  *p = q;
  return hipSuccess;
}

}  // namespace

// ---- controls of the harness
extern "C" {
void h2_standin_seed(uint64_t s) { Lock l(g_mu); g_seed = s; }
void h2_standin_limit(int64_t free_bytes) {  // free device memory from now on (negative: ample)
  Lock l(g_mu);
  g_limit = free_bytes < 0 ? size_t(1) << 34 : g_used + (size_t)free_bytes;
}
// hipMemGetInfo tells the truth (0), that nothing is free (1), that all of it is (2)
void h2_standin_hide_free(int hide) { Lock l(g_mu); g_hide_free = hide; }
int64_t h2_standin_peak() {  // largest memory held beyond the present since the last call
  Lock l(g_mu);
  const int64_t p = (int64_t)g_peak - (int64_t)g_used;
  g_peak = g_used;
  return p;
}
int64_t h2_standin_count(const char* name) { Lock l(g_mu); return g_count[name]; }
int64_t h2_standin_live() { Lock l(g_mu); return (int64_t)(g_streams.size() + g_events.size() + g_execs.size() + g_mem.size()); }
}

// ---- HIP
extern "C" {
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  Lock l(g_mu);
  *f = g_hide_free == 1 ? 0 : g_hide_free == 2 ? g_limit : g_limit - g_used;
  *t = g_limit;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* sym) { *p = const_cast<void*>(sym); return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return do_malloc(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return do_malloc(p, n); }
hipError_t hipFree(void* p) {
  Lock l(g_mu);
  if (!p) return hipSuccess;
  no_capture("a release under capture");
  auto it = g_mem.find(p);
  if (it == g_mem.end()) die("hipFree of something else");
  run(nullptr);  // waits for the device
  g_used -= it->second;
  g_mem.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipDeviceSynchronize(void) {
  Lock l(g_mu);
  no_capture("a device synchronization under capture");
  run(nullptr);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { Lock l(g_mu); sync_stream(stream_of(s)); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) {
  Lock l(g_mu);
  if (f != hipStreamNonBlocking) die("a blocking stream");
  Stream* p = new Stream();
  g_streams.insert(p);
  *s = reinterpret_cast<hipStream_t>(p);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  Lock l(g_mu);
  Stream* p = stream_of(s);
  if (p == &g_null) die("the null stream destroyed");
  if (p->cap) die("a stream destroyed under capture");
  g_streams.erase(p);
  delete p;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Lock l(g_mu);
  Stream* st = stream_of(s);
  Event* ev = event_of(e);
  if (!ev->recorded) die("a wait for an event that was never recorded");
  if (ev->cap) {
    if (!st->cap) {
      if (!st->waits.empty()) die("a stream with waits joins a capture");
      st->cap = ev->cap;
      st->before = st->tail;
      st->tail = nullptr;
    } else if (st->cap != ev->cap) {
      die("a wait across captures");
    }
  } else if (st->cap) {
    die("a stream under capture waits for an event from outside");
  }
  if (ev->op) st->waits.push_back(ev->op);
  return hipSuccess;
}
static hipError_t event_create(hipEvent_t* e) {
  Lock l(g_mu);
  Event* p = new Event();
  g_events.insert(p);
  *e = reinterpret_cast<hipEvent_t>(p);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return event_create(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return event_create(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  Lock l(g_mu);
  Event* p = event_of(e);
  g_events.erase(p);
  delete p;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Lock l(g_mu);
  Event* ev = event_of(e);
  ev->op = enqueue(s, nullptr, nullptr);
  ev->cap = stream_of(s)->cap;
  ev->recorded = true;
  ev->t = g_clock += 0.25;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Lock l(g_mu);
  Event* ev = event_of(e);
  if (ev->cap) die("a synchronization on a captured event");
  if (ev->op) run(ev->op);
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  Lock l(g_mu);
  Event* ev = event_of(e);
  if (ev->op && !ev->op->done) {
    if (rnd() % 4) return hipErrorNotReady;
    run(ev->op);
  }
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  Lock l(g_mu);
  *ms = (float)(event_of(b)->t - event_of(a)->t + (double)(rnd() % 64) / 64.0);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  return launch(st, "memcpy", [=] { std::memmove(d, s, n); });
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
  Lock l(g_mu);
  no_capture("a synchronous copy under capture");
  OpP o = enqueue(nullptr, "memcpy", [=] { std::memmove(d, s, n); });
  if (k != hipMemcpyDeviceToDevice) run(o);  // device to device does not wait
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t s) {
  { Lock l(g_mu); if (stream_of(s)->cap) die("a memset under capture"); }
  return launch(s, "memset", [=] { std::memset(d, v, n); });
}
hipError_t hipMemset(void* d, int v, size_t n) { return hipMemsetAsync(d, v, n, nullptr); }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  Lock l(g_mu);
  Stream* st = stream_of(s);
  if (st == &g_null || st->cap) die("a capture of this stream");
  if (!st->waits.empty()) enqueue(s, nullptr, nullptr);
  st->cap = std::make_shared<Graph>();
  st->before = st->tail;
  st->tail = nullptr;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  Lock l(g_mu);
  Stream* st = stream_of(s);
  if (!st->cap) die("the end of a capture that did not begin");
  std::shared_ptr<Graph> gr = st->cap;
  // every forked stream's work must be joined back
  std::set<Op*> seen;
  std::vector<OpP> todo;
  if (st->tail) todo.push_back(st->tail);
  for (OpP& w : st->waits) todo.push_back(w);
  while (!todo.empty()) {
    OpP o = todo.back();
    todo.pop_back();
    if (!seen.insert(o.get()).second) continue;
    for (OpP& d : o->deps) todo.push_back(d);
  }
  for (OpP& o : gr->nodes)
    if (o->fn && !seen.count(o.get())) die("captured work that is not joined back");
  for (Stream* x : g_streams)
    if (x->cap == gr) {
      x->cap = nullptr;
      x->tail = x->before;
      x->before = nullptr;
      x->waits.clear();
    }
  *g = reinterpret_cast<hipGraph_t>(new Graph(*gr));
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  Lock l(g_mu);
  Graph* gr = reinterpret_cast<Graph*>(g);
  GraphExec* x = new GraphExec();
  std::map<Op*, size_t> at;
  for (size_t i = 0; i < gr->nodes.size(); ++i) at[gr->nodes[i].get()] = i;
  for (OpP& o : gr->nodes) {
    x->fns.push_back(o->fn);
    x->deps.emplace_back();
    for (OpP& d : o->deps)
      if (at.count(d.get())) x->deps.back().push_back(at[d.get()]);
  }
  g_execs.insert(x);
  *e = reinterpret_cast<hipGraphExec_t>(x);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete reinterpret_cast<Graph*>(g); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  Lock l(g_mu);
  GraphExec* x = reinterpret_cast<GraphExec*>(e);
  if (!g_execs.count(x)) die("a graph that does not exist");
  OpP root = enqueue(s, "graph", nullptr);
  if (x->last && !x->last->done) root->deps.push_back(x->last);
  std::vector<OpP> ops;
  for (size_t i = 0; i < x->fns.size(); ++i) {
    OpP o = std::make_shared<Op>();
    o->deps.push_back(root);
    for (size_t d : x->deps[i]) o->deps.push_back(ops[d]);
    o->fn = x->fns[i];
    ops.push_back(o);
    g_pending.push_back(o);
  }
  OpP end = enqueue(s, nullptr, nullptr);
  for (OpP& o : ops) end->deps.push_back(o);
  x->last = end;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  Lock l(g_mu);
  GraphExec* x = reinterpret_cast<GraphExec*>(e);
  if (!g_execs.count(x)) die("a graph that does not exist");
  if (x->last && !x->last->done) die("a graph destroyed while a replay of it is queued");
  g_execs.erase(x);
  delete x;
  return hipSuccess;
}
}  // extern "C"

// ---- the kernel launchers, in plain loops
namespace h2 {
namespace {

// out[out_off + a, v] (=, +=) M x for one row of the streaming tables
template <class T, class Get, class Put>
void row_product(const RowDesc& R, const int32_t* colend, const int64_t* in_off, const T* M, int nv, Get get, Put put) {
  const int ncols = R.blk_end > R.blk_begin ? colend[R.blk_end - 1] : 0;
  std::vector<double> acc((size_t)R.nrows * nv, 0.0);
  int c = 0;
  for (int b = R.blk_begin; b < R.blk_end; ++b)
    for (int64_t j = 0; c < colend[b]; ++c, ++j)
      for (int a = 0; a < R.nrows; ++a) {
        const double m = (double)M[a + (int64_t)R.nrows * c];
        for (int v = 0; v < nv; ++v) acc[(size_t)a * nv + v] += m * get(in_off[b] + j, v);
      }
  (void)ncols;
  for (int a = 0; a < R.nrows; ++a)
    for (int v = 0; v < nv; ++v) put(a, v, acc[(size_t)a * nv + v]);
}

// row-major rows (the multi-vector path)
template <class T>
hipError_t rm_rows(const char* name, const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                   const T* data, const double* in, double* out, int nvp, int mode, int max_rows, hipStream_t s,
                   const T* fl = nullptr) {
  if (nrows == 0) return hipSuccess;
  (void)fl;
  return launch(s, name, [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const RowDesc R = rows[i];
      if (R.nrows > max_rows) die("a row longer than the launch says");
      row_product(R, colend, in_off, data + R.data_off, nvp, [&](int64_t r, int v) { return in[r * nvp + v]; },
                  [&](int a, int v, double x) {
                    double* o = out + (R.out_off + a) * nvp + v;
                    *o = mode == MODE_STORE ? x : *o + x;
                  });
    }
  });
}

template <class T>
void cols_product(const RowDesc& R, const int64_t* bdata, const int32_t* bmr, const int64_t* bin, const T* data, int nv,
                  const std::function<double(int64_t, int)>& get, const std::function<void(int, int, double)>& put) {
  std::vector<double> acc((size_t)R.nrows * nv, 0.0);
  for (int b = R.blk_begin; b < R.blk_end; ++b)
    for (int c = 0; c < R.nrows; ++c)
      for (int a = 0; a < bmr[b]; ++a)
        for (int v = 0; v < nv; ++v)
          acc[(size_t)c * nv + v] += (double)data[bdata[b] + a + (int64_t)bmr[b] * c] * get(bin[b] + a, v);
  for (int c = 0; c < R.nrows; ++c)
    for (int v = 0; v < nv; ++v) put(c, v, acc[(size_t)c * nv + v]);
}

template <class T>
hipError_t cm_cols(const char* name, const RowDesc* rows, int64_t nrows, const int64_t* bdata, const int32_t* bmr,
                   const int64_t* bin, const T* data, const double* in, double* out, int nv, hipStream_t s) {
  if (nrows == 0) return hipSuccess;
  return launch(s, name, [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const RowDesc R = rows[i];
      cols_product<T>(R, bdata, bmr, bin, data, nv, [&](int64_t r, int v) { return in[r + R.in_ld * v]; },
                      [&](int c, int v, double x) { out[R.out_off + c + R.out_ld * v] = x; });
    }
  });
}

}  // namespace

hipError_t launch_permute_in(const double* X, int64_t ldx, const int32_t* perm, double* xt, int64_t n, int nv,
                             hipStream_t s) {
  return launch(s, "permute_in", [=] {
    for (int v = 0; v < nv; ++v)
      for (int64_t i = 0; i < n; ++i) xt[i + n * v] = X[perm[i] + ldx * v];
  });
}
hipError_t launch_scale(double* Y, int64_t ldy, int64_t n, int64_t nv, double beta, hipStream_t s) {
  return launch(s, "scale", [=] {
    for (int64_t v = 0; v < nv; ++v)
      for (int64_t i = 0; i < n; ++i) Y[i + ldy * v] = beta == 0.0 ? 0.0 : beta * Y[i + ldy * v];
  });
}
template <typename T>
hipError_t launch_rows(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                       const T* data, const double* in, double* out, int nv, int mode, const Epilogue& ep,
                       hipStream_t s, int64_t) {
  if (nrows == 0) return hipSuccess;
  return launch(s, "rows", [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const RowDesc R = rows[i];
      row_product(R, colend, in_off, data + R.data_off, nv, [&](int64_t r, int v) { return in[r + R.in_ld * v]; },
                  [&](int a, int v, double x) {
                    if (mode == MODE_FINAL) {
                      const int64_t i_ = R.out_off + a;
                      double* y = ep.Y + ep.perm[i_] + ep.ldy * v;
                      *y = ep.alpha * (ep.zn[i_ + ep.n * v] + x) + (ep.beta == 0.0 ? 0.0 : ep.beta * *y);
                      return;
                    }
                    double* o = out + R.out_off + a + R.out_ld * v;
                    *o = mode == MODE_STORE ? x : *o + x;
                  });
    }
  });
}
template hipError_t launch_rows<double>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const double*,
                                        const double*, double*, int, int, const Epilogue&, hipStream_t, int64_t);
template hipError_t launch_rows<float>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const float*,
                                       const double*, double*, int, int, const Epilogue&, hipStream_t, int64_t);
hipError_t launch_rows_first(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                             const double* data, const double* X, double* out, int nv, const FirstArgs& F,
                             hipStream_t s) {
  return launch(s, "rows_first", [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const RowDesc R = rows[i];
      const bool up = i >= F.ndense;
      row_product(R, colend, in_off, (up ? F.data2 : data) + R.data_off, nv,
                  [&](int64_t r, int v) { return X[F.perm[r] + F.ldx * v]; },
                  [&](int a, int v, double x) { (up ? F.out2 : out)[R.out_off + a + R.out_ld * v] = x; });
    }
  });
}
template <typename T>
hipError_t launch_rows_mfma(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                            const T* data, const double* in, double* out, int nvp, int mode, int max_rows,
                            hipStream_t s, int, int64_t, int, const float* in32) {
  if (in32) ++g_count["reads_x32"];
  return rm_rows<T>("rows_mfma", rows, nrows, colend, in_off, data, in, out, nvp, mode, max_rows, s);
}
template hipError_t launch_rows_mfma<double>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const double*,
                                             const double*, double*, int, int, int, hipStream_t, int, int64_t, int,
                                             const float*);
template hipError_t launch_rows_mfma<float>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const float*,
                                            const double*, double*, int, int, int, hipStream_t, int, int64_t, int,
                                            const float*);
hipError_t launch_batch_permute(const BatchItem* items, const int32_t* tile_op, const int32_t* tile_j0, int64_t ntiles,
                                const int32_t* pinv, double* ws, int nvp, bool out, hipStream_t s) {
  return launch(s, "batch_permute", [=] {
    for (int64_t b = 0; b < ntiles; ++b) {
      const BatchItem it = items[tile_op[b]];
      for (int64_t j = tile_j0[b]; j < std::min<int64_t>(tile_j0[b] + kPermTile, it.n); ++j) {
        const int64_t p = pinv[it.pinv_off + j];
        for (int v = 0; v < nvp; ++v) {
          if (!out) ws[(it.xt_row + p) * nvp + v] = v < it.nv && it.alpha != 0.0 ? it.X[j + it.ldx * v] : 0.0;
          else if (v < it.nv) {
            double* y = it.Y + j + it.ldy * v;
            *y = (it.alpha == 0.0 ? 0.0 : it.alpha * ws[(it.zn_row + p) * nvp + v]) + (it.beta == 0.0 ? 0.0 : it.beta * *y);
          }
        }
      }
    }
  });
}
hipError_t launch_to_f32(const double* src, float* dst, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  return launch(s, "to_f32", [=] {
    for (int64_t i = 0; i < n; ++i) dst[i] = (float)src[i];
  });
}
hipError_t launch_transpose_tasks(const TransTask* t, int64_t n, const double* mat, double* trans, hipStream_t s) {
  return launch(s, "transpose", [=] {
    for (int64_t k = 0; k < n; ++k)
      for (int r = 0; r < t[k].rows; ++r)
        for (int c = 0; c < t[k].cols; ++c)
          trans[t[k].dst + c + (int64_t)t[k].cols * r] = mat[t[k].src + r + (int64_t)t[k].rows * c];
  });
}
int run_compose(const std::vector<const Composed*>& C, const Parsed& P, const double* mat, double* trans) {
  Lock l(g_mu);
  run(nullptr);
  for (const Composed* co : C)
    for (const ComposeStage& g : co->stages) {
      int64_t down = g.reg[0];
      std::vector<int64_t> up(g.reg);
      for (int64_t c = g.c0; c < g.c0 + g.count; ++c) {
        const int64_t top = g.s - 1, m = g.points ? P.hi[c] - P.lo[c] : g.k[g.s];
        const double* A = mat + g.stored + (g.points ? P.lo[c] * g.k[top] : (c - g.c0) * g.k[g.s] * g.k[top]);
        std::vector<double> W(A, A + m * g.k[top]);
        int64_t a = g.points ? c : P.parent[c];
        for (int64_t x = top; x >= g.lo; --x) {
          if (x < top) {  // times the transfer of the ancestor on level x + 1
            const double* T = mat + g.tr[x + 1] + (a - P.level_ptr[x + 1]) * g.k[x + 1] * g.k[x];
            std::vector<double> N((size_t)(m * g.k[x]), 0.0);
            for (int64_t j = 0; j < g.k[x]; ++j)
              for (int64_t i = 0; i < g.k[x + 1]; ++i)
                for (int64_t r = 0; r < m; ++r) N[r + m * j] += W[r + m * i] * T[i + g.k[x + 1] * j];
            W.swap(N);
            a = P.parent[a];
          }
          if (!g.up) {
            std::copy(W.begin(), W.end(), trans + down);
            down += m * g.k[x];
          } else if (x < top) {
            for (int64_t r = 0; r < m; ++r)
              for (int64_t j = 0; j < g.k[x]; ++j) trans[up[x] + j + g.k[x] * r] = W[r + m * j];
            up[x] += m * g.k[x];
          }
        }
      }
    }
  return H2_OK;
}
hipError_t launch_rows_mfma_bf16(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t*,
                                 const void* data, const void*, bool, int64_t, void* out, bool, int64_t, int,
                                 int, int, hipStream_t s, int64_t, int) {
  // the layouts only: one byte of each row's operands is touched
  return launch(s, "rows_bf16", [=] {
    volatile char sink = 0;
    for (int64_t i = 0; i < nrows; ++i)
      if (rows[i].nrows > 0 && rows[i].blk_end > rows[i].blk_begin && colend[rows[i].blk_end - 1] > 0)
        sink = sink + static_cast<const char*>(data)[2 * rows[i].data_off];
    (void)out;
  });
}
hipError_t launch_rows_to_bf16(const RowDesc* rows, int64_t nrows, const int32_t* colend, const double* src, void* dst,
                               hipStream_t s) {
  return launch(s, "to_bf16", [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const int64_t e = (int64_t)rows[i].nrows * (rows[i].blk_end > rows[i].blk_begin ? colend[rows[i].blk_end - 1] : 0);
      for (int64_t k = 0; k < e; ++k) static_cast<uint16_t*>(dst)[rows[i].data_off + k] = (uint16_t)src[rows[i].data_off + k];
    }
  });
}
hipError_t launch_permute_in_rm(const double* X, int64_t ldx, const int32_t* pinv, double* xt, int64_t n, int nv,
                                int nvp, hipStream_t s) {
  return launch(s, "permute_in_rm", [=] {
    for (int64_t j = 0; j < n; ++j)
      for (int v = 0; v < nvp; ++v) xt[(int64_t)pinv[j] * nvp + v] = v < nv ? X[j + ldx * v] : 0.0;
  });
}
hipError_t launch_permute_out_rm2(const double* Z, const double* Z2, const int32_t* pinv, double alpha, double beta,
                                  double* Y, int64_t ldy, int64_t n, int nv, int nvp, hipStream_t s) {
  return launch(s, "permute_out", [=] {
    for (int64_t j = 0; j < n; ++j)
      for (int v = 0; v < nv; ++v) {
        const int64_t p = (int64_t)pinv[j] * nvp + v;
        double* y = Y + j + ldy * v;
        *y = alpha * (Z[p] + (Z2 ? Z2[p] : 0.0)) + (beta == 0.0 ? 0.0 : beta * *y);
      }
  });
}
hipError_t launch_permute_out_rm(const double* Z, const int32_t* pinv, double alpha, double beta, double* Y,
                                 int64_t ldy, int64_t n, int nv, int nvp, hipStream_t s) {
  return launch_permute_out_rm2(Z, nullptr, pinv, alpha, beta, Y, ldy, n, nv, nvp, s);
}
RowForm auto_form(int, int64_t, int max_rows) { return {max_rows > 64 ? 64 : kWaveRows, 0}; }
template <typename T>
hipError_t launch_wave_rows(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                            const T* data, const double* in, double* out, int nvp, int mode, int min_rows,
                            int max_rows, hipStream_t s, int64_t, bool, int, const T* fl, int) {
  if (max_rows > 64) return hipErrorInvalidValue;
  (void)min_rows;
  return rm_rows<T>("wave_rows", rows, nrows, colend, in_off, data, in, out, nvp, mode, max_rows, s, fl);
}
template hipError_t launch_wave_rows<double>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const double*,
                                             const double*, double*, int, int, int, int, hipStream_t, int64_t, bool,
                                             int, const double*, int);
template hipError_t launch_wave_rows<float>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const float*,
                                            const double*, double*, int, int, int, int, hipStream_t, int64_t, bool,
                                            int, const float*, int);
hipError_t launch_split_rows(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                             const double* data, const double* in, double* out, int nvp, int mode, int, int max_rows,
                             hipStream_t s, bool all, int64_t, int) {
  if (max_rows > 64) return hipErrorInvalidValue;
  return rm_rows<double>(all ? "split_dense" : "split_rows", rows, nrows, colend, in_off, data, in, out, nvp, mode,
                         max_rows, s);
}
hipError_t launch_wave_cols(const RowDesc* rows, int64_t nrows, const int64_t* bdata, const int32_t* bmr,
                            const int64_t* bin, const double* data, const double* in, double* out, int nvp, int,
                            hipStream_t s) {
  if (nrows == 0) return hipSuccess;
  return launch(s, "wave_cols", [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const RowDesc R = rows[i];
      cols_product<double>(R, bdata, bmr, bin, data, nvp, [&](int64_t r, int v) { return in[r * nvp + v]; },
                           [&](int c, int v, double x) { out[(R.out_off + c) * nvp + v] = x; });
    }
  });
}
template <typename T>
hipError_t launch_rows_to_fl(const RowDesc* rows, int64_t nrows, const int32_t* colend, const T* src, T* dst,
                             hipStream_t s) {
  return launch(s, "to_fl", [=] {
    for (int64_t i = 0; i < nrows; ++i) {
      const int64_t c = rows[i].blk_end > rows[i].blk_begin ? colend[rows[i].blk_end - 1] : 0, m = rows[i].nrows;
      for (int64_t e = 0; e < m * ((c + 7) / 8 * 8); ++e) dst[rows[i].fl_off + e] = e < m * c ? src[rows[i].data_off + e] : (T)0;
    }
  });
}
template hipError_t launch_rows_to_fl<double>(const RowDesc*, int64_t, const int32_t*, const double*, double*,
                                              hipStream_t);
template hipError_t launch_rows_to_fl<float>(const RowDesc*, int64_t, const int32_t*, const float*, float*,
                                             hipStream_t);
template <typename T>
hipError_t launch_tree(const int2* ranges, int64_t nwg, const TreeLevels& L0, const RowDesc* rows,
                       const int32_t* colend, const int64_t* in_off, const T* data, double* const bufs0[4], int nvp,
                       int, hipStream_t s) {
  const TreeLevels L = L0;
  std::vector<double*> bufs(bufs0, bufs0 + 4);
  return launch(s, "tree", [=] {
    for (int64_t w = 0; w < nwg; ++w)
      for (int lev = 0; lev < L.nlev; ++lev) {
        const int2 r = ranges[w * L.nlev + lev];
        for (int i = r.x; i < r.y; ++i) {
          const RowDesc R = rows[i];
          const double* in = bufs[L.in[lev]];
          double* out = bufs[L.out[lev]];
          row_product(R, colend, in_off, data + R.data_off, nvp, [&](int64_t q, int v) { return in[q * nvp + v]; },
                      [&](int a, int v, double x) {
                        double* o = out + (R.out_off + a) * nvp + v;
                        *o = L.mode[lev] == MODE_STORE ? x : *o + x;
                      });
        }
      }
  });
}
template hipError_t launch_tree<float>(const int2*, int64_t, const TreeLevels&, const RowDesc*, const int32_t*,
                                       const int64_t*, const float*, double* const[4], int, int, hipStream_t);
hipError_t launch_rows_wide(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                            const double* data, const double* in, double* out, int nv, hipStream_t s) {
  return launch_rows<double>(rows, nrows, colend, in_off, data, in, out, nv, MODE_STORE, Epilogue{}, s, 0);
}
int cols_slots(int max_rows, int max_mr) { return max_rows * max_mr <= 4096 ? 1 : 0; }
hipError_t launch_cols(const RowDesc* rows, int64_t nrows, const int64_t* bdata, const int32_t* bmr,
                       const int64_t* bin, const double* data, const double* in, double* out, int nv, int,
                       hipStream_t s, int64_t) {
  return cm_cols<double>("cols", rows, nrows, bdata, bmr, bin, data, in, out, nv, s);
}
template <typename T>
hipError_t launch_gather(const RowDesc* rows, int64_t nrows, const int64_t* bdata, const int32_t* bmr,
                         const int64_t* bin, const T* data, const double* in, double* out, int nv, hipStream_t s) {
  return cm_cols<T>("gather", rows, nrows, bdata, bmr, bin, data, in, out, nv, s);
}
template hipError_t launch_gather<double>(const RowDesc*, int64_t, const int64_t*, const int32_t*, const int64_t*,
                                          const double*, const double*, double*, int, hipStream_t);
template hipError_t launch_gather<float>(const RowDesc*, int64_t, const int64_t*, const int32_t*, const int64_t*,
                                         const float*, const double*, double*, int, hipStream_t);

// ---- recompression: the task lists and every operand's first and last
// element are read, counts keep half of each rank; no arithmetic
namespace {
volatile double g_sink;
void touch(const double* p, int64_t rows, int64_t cols, int64_t ld) {
  if (rows > 0 && cols > 0) g_sink = p[0] + p[rows - 1 + (cols - 1) * ld];
}
void fill(double* p, int64_t rows, int64_t cols, int64_t ld) {
  for (int64_t j = 0; j < cols; ++j)
    for (int64_t i = 0; i < rows; ++i) p[i + ld * j] = 1.0;
}
}  // namespace
hipError_t launch_qr(const QrTask* t, int64_t n, hipStream_t s, int me) {
  return launch(s, "qr", [=] {
    for (int64_t i = 0; i < n; ++i) {
      if (t[i].rows * t[i].cols > me) die("a QR operand larger than the launch says");
      touch(t[i].A, t[i].rows, t[i].cols, t[i].lda);
      fill(t[i].Q, t[i].rows, t[i].cols, t[i].ldq);
      fill(t[i].R, t[i].cols, t[i].cols, t[i].ldr);
    }
  });
}
hipError_t launch_gemm(const GemmTask* t, int64_t n, const GemmPair* p, hipStream_t s, int) {
  return launch(s, "gemm", [=] {
    for (int64_t i = 0; i < n; ++i) {
      for (int k = t[i].pbeg; k < t[i].pend; ++k) {
        touch(p[k].A, p[k].flags & 1 ? p[k].k : t[i].m, p[k].flags & 1 ? t[i].m : p[k].k, p[k].lda);
        touch(p[k].B, p[k].flags & 2 ? t[i].n : p[k].k, p[k].flags & 2 ? p[k].k : t[i].n, p[k].ldb);
      }
      fill(t[i].C, t[i].m, t[i].n, t[i].ldc);
    }
  });
}
hipError_t launch_triple(const TripleTask* t, int64_t n, hipStream_t s, int) {
  return launch(s, "triple", [=] {
    for (int64_t i = 0; i < n; ++i) {
      touch(t[i].M, t[i].k1, t[i].k2, t[i].ldm);
      touch(t[i].R, t[i].b, t[i].k2, t[i].ldr);
      fill(t[i].C, t[i].a, t[i].b, t[i].ldc);
    }
  });
}
hipError_t launch_eig(const EigTask* t, int64_t n, int nmax, hipStream_t s) {
  return launch(s, "eig", [=] {
    for (int64_t i = 0; i < n; ++i) {
      if (t[i].n > nmax) die("an eigenproblem larger than the launch says");
      touch(t[i].G, t[i].n, t[i].n, t[i].ldg);
      fill(t[i].Z, t[i].n, t[i].n, t[i].ldz);
      for (int k = 0; k < t[i].n; ++k) t[i].lam[k] = k < (t[i].n + 1) / 2 ? 1.0 : 0.0;
    }
  });
}
hipError_t launch_mask_gram(const MaskTask* t, int64_t n, hipStream_t s) {
  return launch(s, "mask", [=] {
    for (int64_t i = 0; i < n; ++i) fill(t[i].out, t[i].k, t[i].k, t[i].k);
  });
}
hipError_t launch_count(const CountTask* t, int64_t n, double, int32_t* counts, hipStream_t s) {
  return launch(s, "count", [=] {
    for (int64_t i = 0; i < n; ++i) counts[t[i].node] = (t[i].n + 1) / 2;
  });
}
hipError_t launch_max_lead(const CountTask*, int64_t n, double* out, hipStream_t s) {
  return launch(s, "max", [=] { *out = n > 0 ? 1.0 : 0.0; });
}
hipError_t launch_scale_cols(const ScaleTask* t, int64_t n, const int32_t* counts, int, hipStream_t s) {
  return launch(s, "scale_cols", [=] {
    for (int64_t i = 0; i < n; ++i) g_sink = t[i].Z[0] + counts[t[i].node];
  });
}
hipError_t launch_sqrt_factor(const EigTask* t, int64_t n, double* const* outs, const int64_t* ldo, hipStream_t s) {
  return launch(s, "sqrt", [=] {
    for (int64_t i = 0; i < n; ++i) fill(outs[i], t[i].n, t[i].n, ldo[i]);
  });
}
hipError_t launch_copy(const CopyTask* t, int64_t n, hipStream_t s) {
  return launch(s, "copy", [=] {
    for (int64_t i = 0; i < n; ++i)
      for (int c = 0; c < t[i].cols; ++c)
        for (int r = 0; r < t[i].rows; ++r)
          t[i].dst[r + t[i].ldd * c] = t[i].trans ? t[i].src[c + t[i].lds * r] : t[i].src[r + t[i].lds * c];
  });
}
}  // namespace h2
