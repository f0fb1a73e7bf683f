// The library's host sources against the stand-ins of hip_standin.cpp: whole
// calls through the C entry points, results compared with the CPU oracle.
// Compiled with the sanitizers and run by tests/test_host_standin.py:
//   standin_check CASE FILE...
// "device" buffers of the caller are heap vectors of exactly their length.
// Prints "<case> ok" or a line starting with FAIL and exit status 1.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "h2_internal.h"

extern "C" {
void h2_standin_seed(uint64_t);
void h2_standin_limit(int64_t);
void h2_standin_hide_free(int);
int64_t h2_standin_peak();
int64_t h2_standin_count(const char*);
int64_t h2_standin_live();
// the oracle (oracle/h2_oracle.c)
int h2o_open(const uint8_t*, int64_t, void**);
void h2o_close(void*);
int h2o_gemv(const void*, char, double, const double*, int64_t, int64_t, double, double*, int64_t, int);
}

namespace {

using Vec = std::vector<double>;
using Bytes = std::vector<uint64_t>;

[[noreturn]] void fail(const std::string& what) {
  std::printf("FAIL %s\n", what.c_str());
  std::exit(1);
}
#define OK(call)                                                             \
  do {                                                                       \
    const int rc_ = (call);                                                  \
    if (rc_ != H2_OK) fail(std::string(#call) + ": " + h2_last_error());     \
  } while (0)

struct File {
  Bytes mem;
  int64_t len = 0;
};
File read_file(const char* path) {
  File f;
  FILE* p = std::fopen(path, "rb");
  if (!p) fail(path);
  std::fseek(p, 0, SEEK_END);
  f.len = std::ftell(p);
  std::fseek(p, 0, SEEK_SET);
  f.mem.resize((size_t)(f.len + 7) / 8);
  if (std::fread(f.mem.data(), 1, (size_t)f.len, p) != (size_t)f.len) fail(path);
  std::fclose(p);
  return f;
}

// One operator with its oracle; products are checked elementwise against
// tol * (the oracle's product in absolute values).
struct Pair {
  h2_handle h = nullptr;
  void* ref = nullptr;
  int64_t n = 0;
  explicit Pair(const File& f) {
    OK(h2_load_mem(f.mem.data(), (size_t)f.len, 0, &h));
    if (h2o_open(reinterpret_cast<const uint8_t*>(f.mem.data()), f.len, &ref) != 0) fail("oracle");
    n = h2_n(h);
  }
  ~Pair() {
    OK(h2_free(h));
    h2o_close(ref);
  }
  void check(const Vec& X, const Vec& Y0, const Vec& Y, char op, int64_t nv, double alpha, double beta, double tol,
             const std::string& what) const {
    Vec want = Y0, B = Y0;
    h2o_gemv(ref, op, alpha, X.data(), n, nv, beta, want.data(), n, 0);
    h2o_gemv(ref, op, alpha, X.data(), n, nv, beta, B.data(), n, 1);
    for (size_t i = 0; i < Y.size(); ++i)
      if (!(std::fabs(Y[i] - want[i]) <= tol * B[i])) fail(what + ": entry " + std::to_string(i));
  }
};

uint64_t g_state = 1;
double next() {
  uint64_t z = (g_state += 0x9e3779b97f4a7c15ull);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return (double)(int64_t)((z ^ (z >> 31)) >> 12) / (double)(int64_t(1) << 51) - 1.0;
}
Vec random_vec(int64_t n) {
  Vec v((size_t)n);
  for (double& x : v) x = next();
  return v;
}

const double kTol[2] = {1e-12, 2e-5};  // FP64, FP32

void product(const Pair& p, char op, int64_t nv, int prec, hipStream_t s, const std::string& what) {
  const Vec X = random_vec(p.n * nv), Y0 = random_vec(p.n * nv);
  Vec Y = Y0;
  OK(h2_gemv_ex(p.h, op, 1.5, X.data(), p.n, nv, -0.5, Y.data(), p.n, prec, s));
  (void)hipDeviceSynchronize();
  p.check(X, Y0, Y, op, nv, 1.5, -0.5, kTol[prec], what);
}

std::string name_of(const char* what, int64_t a, int64_t b, int64_t c, char op) {
  return std::string(what) + " " + op + " " + std::to_string(a) + " " + std::to_string(b) + " " + std::to_string(c);
}

bool plan_has(h2_handle h, const char* prefix) {
  size_t need = 0;
  OK(h2_plan_info(h, nullptr, 0, &need));
  std::vector<char> buf(need);
  OK(h2_plan_info(h, buf.data(), need, &need));
  return std::string("\n").append(buf.data()).find(std::string("\n") + prefix) != std::string::npos;
}

// Products of both ops, every pass width, schedule and sweep form, in several
// orders of execution that the waits between the streams allow.
void products(const std::vector<File>& files, hipStream_t s) {
  bool down = false;
  for (size_t fi = 0; fi < files.size(); ++fi) {
    Pair p(files[fi]);
    OK(h2_prepare(p.h, H2_PREC_FP32));
    down = down || plan_has(p.h, "down ");
    for (int64_t nv : {1, 3, 20, 64, 70})
      for (char op : {'N', 'T'})
        for (int prec : {0, 1}) product(p, op, nv, prec, s, name_of("product", (int64_t)fi, nv, prec, op));
    for (int sched = 0; sched < 4; ++sched)
      for (int prec : {0, 1}) {
        OK(h2_set_schedule(p.h, prec, sched));
        for (int64_t nv : {2, 17, 64})
          for (int seed = 0; seed < 3; ++seed) {
            h2_standin_seed((uint64_t)(100 * sched + seed));
            product(p, 'N', nv, prec, s, name_of("schedule", sched, nv, prec, 'N'));
          }
        Vec X = random_vec(p.n * 5), Y((size_t)p.n * 5);
        OK(h2_gemv_noalloc(p.h, 'T', 1.0, X.data(), p.n, 5, 0.0, Y.data(), p.n, s));
        (void)hipDeviceSynchronize();
        p.check(X, Y, Y, 'T', 5, 1.0, 0.0, kTol[0], "no allocation");
      }
    if (h2_set_sweeps(p.h, H2_PREC_FP32, 1) == H2_OK) product(p, 'N', 40, 1, s, "fused sweeps");
    OK(h2_profile(p.h, 1));
    for (int64_t nv : {1, 9})
      for (char op : {'N', 'T'}) product(p, op, nv, 0, s, "profiled");
    h2_profile_t prof;
    OK(h2_profile_read(p.h, &prof));
    if (prof.calls != 4) fail("profiled calls");
  }
  if (!down) fail("no operator with a composed downsweep stage");
}

// Captured products replayed on refilled inputs: both ops, both paths, with
// the third stream (schedule 3) where the operator has a downsweep stage.
void graphs(const std::vector<File>& files, hipStream_t s) {
  for (const File& f : files) {
    Pair p(f);
    for (int sched : {0, 3})
      for (char op : {'N', 'T'})
        for (int64_t nv : {1, 20}) {
          OK(h2_set_schedule(p.h, H2_PREC_FP64, sched));
          OK(h2_graph(p.h, 1));
          Vec X((size_t)(p.n * nv)), Y((size_t)(p.n * nv));
          const int64_t before = h2_standin_count("graph");
          for (int rep = 0; rep < 4; ++rep) {
            X = random_vec(p.n * nv);
            const Vec Y0 = Y = random_vec(p.n * nv);
            OK(h2_gemv(p.h, op, 1.5, X.data(), p.n, nv, -0.5, Y.data(), p.n, s));
            (void)hipDeviceSynchronize();
            p.check(X, Y0, Y, op, nv, 1.5, -0.5, kTol[0], name_of("replay", rep, nv, sched, op));
          }
          if (h2_standin_count("graph") != before + 4) fail("replays");
        }
  }
}

// A workspace that grows while captured graphs of the smaller one are kept.
void growth(const std::vector<File>& files, hipStream_t s) {
  for (const File& f : files) {
    Pair p(f);
    OK(h2_graph(p.h, 1));
    Vec X = random_vec(p.n), Y((size_t)p.n);
    for (int rep = 0; rep < 2; ++rep) {
      OK(h2_gemv(p.h, 'N', 1.0, X.data(), p.n, 1, 0.0, Y.data(), p.n, s));
      (void)hipDeviceSynchronize();
      p.check(X, Y, Y, 'N', 1, 1.0, 0.0, kTol[0], "one vector");
      product(p, 'N', 20, 0, s, "growing");
    }
  }
}

// Graphs captured on a stream that the caller has destroyed since.
void streams(const std::vector<File>& files, hipStream_t s) {
  Pair p(files[0]);
  OK(h2_graph(p.h, 1));
  hipStream_t t = nullptr;
  (void)hipStreamCreateWithFlags(&t, hipStreamNonBlocking);
  product(p, 'N', 1, 0, t, "a stream of its own");
  (void)hipStreamDestroy(t);
  const Vec X = random_vec(p.n);
  std::vector<Vec> Y(12, Vec((size_t)p.n));
  for (Vec& y : Y) OK(h2_gemv(p.h, 'N', 1.0, X.data(), p.n, 1, 0.0, y.data(), p.n, s));
  (void)hipDeviceSynchronize();
  for (const Vec& y : Y) p.check(X, y, y, 'N', 1, 1.0, 0.0, kTol[0], "after the stream");
}

// A batch tuned while a replay of its graph is queued.
void batch(const std::vector<File>& files, hipStream_t s) {
  std::vector<const void*> bufs;
  std::vector<size_t> lens;
  std::vector<int64_t> nv;
  for (size_t i = 0; i < files.size(); ++i) {
    bufs.push_back(files[i].mem.data());
    lens.push_back((size_t)files[i].len);
    nv.push_back(i % 2 ? 3 : 33);
  }
  h2_batch b = nullptr;
  OK(h2_batch_load_ex(bufs.data(), lens.data(), (int64_t)bufs.size(), nv.data(), 0, &b));
  std::vector<Pair*> ops;
  std::vector<Vec> X, Y;
  std::vector<h2_batch_item> it;
  for (size_t i = 0; i < files.size(); ++i) {
    ops.push_back(new Pair(files[i]));
    X.push_back(random_vec(ops[i]->n * nv[i]));
    Y.emplace_back((size_t)(ops[i]->n * nv[i]));
    it.push_back({X[i].data(), ops[i]->n, Y[i].data(), ops[i]->n, nv[i], 1.0, 0.0});
  }
  OK(h2_batch_graph(b, 1));
  for (int round = 0; round < 2; ++round) {
    for (int rep = 0; rep < 3; ++rep) OK(h2_batch_gemv(b, it.data(), s));
    if (round == 0) OK(h2_batch_tune(b, it.data(), s));
  }
  (void)hipDeviceSynchronize();
  for (size_t i = 0; i < files.size(); ++i) {
    ops[i]->check(X[i], Y[i], Y[i], 'N', nv[i], 1.0, 0.0, kTol[0], "batch");
    delete ops[i];
  }
  OK(h2_batch_free(b));
}

// The least free memory with which an operator loads is that of the sweeps
// level by level, not of the composed ones.
void memory(const std::vector<File>& files, hipStream_t s) {
  for (const File& f : files) {
    h2_stats_t full{}, st{};
    {
      Pair p(f);
      OK(h2_stats(p.h, &full));
    }
    int64_t least[3] = {0, 0, 0};
    for (int hide : {0, 2}) {  // the free memory is known, or an allocation fails although it seems to be there
      int64_t lo = 0, hi = 2 * full.device_bytes + (int64_t(1) << 20);  // refused, accepted
      h2_standin_hide_free(hide);
      while (hi - lo > 64) {
        const int64_t mid = (lo + hi) / 2;
        h2_handle h = nullptr;
        h2_standin_limit(mid);
        const int rc = h2_load_mem(f.mem.data(), (size_t)f.len, 0, &h);
        if (rc == H2_OK) OK(h2_free(h));
        else if (rc != H2_ENOMEM) fail("load without memory");
        (rc == H2_OK ? hi : lo) = mid;
      }
      least[hide] = hi;
      h2_standin_limit(hi);
      Pair p(f);
      h2_standin_limit(-1);
      h2_standin_hide_free(0);
      OK(h2_stats(p.h, &st));
      for (char op : {'N', 'T'})
        for (int64_t nv : {1, 20}) product(p, op, nv, 0, s, "least memory");
      if (st.device_bytes >= full.device_bytes) fail("the composed sweeps are kept where memory is short");
    }
    if (least[2] > least[0] + 64) fail("a failed allocation needs more memory than a known shortage");
  }
}

// Recompression needs no more memory than its arrays one by one.
void compress_memory(const std::vector<File>& files, hipStream_t s) {
  for (const File& f : files) {
    h2_handle h = nullptr, c = nullptr;
    OK(h2_load_mem(f.mem.data(), (size_t)f.len, 0, &h));
    (void)h2_standin_peak();
    h2_standin_hide_free(1);
    OK(h2_compress(h, 1e-3, &c, nullptr, s));
    h2_standin_hide_free(0);
    OK(h2_free(c));
    const int64_t peak = h2_standin_peak();
    h2_standin_limit(peak);
    OK(h2_compress(h, 1e-3, &c, nullptr, s));
    h2_standin_limit(-1);
    OK(h2_free(c));
    OK(h2_free(h));
  }
}

// FP32 passes of 64 vectors convert x^ only for launches that read the copy.
void fp32(const std::vector<File>& files, hipStream_t s) {
  bool split = false;
  for (const File& f : files) {
    Pair p(f);
    OK(h2_prepare(p.h, H2_PREC_FP32));
    auto run = [&](const char* what, int64_t* conv, int64_t* reads) {
      const int64_t c = h2_standin_count("to_f32"), r = h2_standin_count("reads_x32"), w = h2_standin_count("wave_rows");
      product(p, 'N', 64, 1, s, what);
      *conv = h2_standin_count("to_f32") - c;
      *reads = h2_standin_count("reads_x32") - r;
      return h2_standin_count("wave_rows") - w;
    };
    int64_t conv, reads;
    for (int sched : {0, 2, 3}) {
      OK(h2_set_schedule(p.h, H2_PREC_FP32, sched));
      const int64_t waves = run("untuned", &conv, &reads);
      if ((conv > 0) != (reads > 0)) fail("a conversion of x^ that nothing reads");
      if (sched == 3) {
        OK(h2_set_schedule(p.h, H2_PREC_FP32, 2));
        split = split || run("schedule 2", &conv, &reads) < waves;
      }
    }
    OK(h2_tune_set(p.h, H2_PREC_FP32, 64, 0, 0, 0));
    run("staged", &conv, &reads);
    if (conv != 1 || reads == 0) fail("the staged kernel without the copy of x^");
  }
  if (!split) fail("schedule 3 taken as 2 everywhere");
}

// Profiled products run the launches that unprofiled ones run.
void profile(const std::vector<File>& files, hipStream_t s) {
  const char* names[] = {"rows_first", "rows", "cols", "wave_rows", "split_rows", "split_dense", "wave_cols", "permute_in"};
  bool first = false;
  for (const File& f : files) {
    Pair p(f);
    first = first || plan_has(p.h, "input ");
    for (char op : {'N', 'T'})
      for (int64_t nv : {1, 4, 20}) {
        std::vector<int64_t> n[2];
        for (int on : {0, 1}) {
          OK(h2_profile(p.h, on));
          for (const char* k : names) n[on].push_back(-h2_standin_count(k));
          product(p, op, nv, 0, s, "profiled");
          for (size_t k = 0; k < n[on].size(); ++k) n[on][k] += h2_standin_count(names[k]);
        }
        if (n[0] != n[1]) fail(name_of("profiled launches", nv, 0, 0, op));
        h2_profile_t t;
        OK(h2_profile_read(p.h, &t));
        if (t.calls != 1) fail("profiled calls");
      }
    OK(h2_profile(p.h, 0));
  }
  if (!first) fail("no operator of three launches");
}

// Stages of several levels with more rows than one launch of four workgroups a
// row can hold are taken level by level.
void split_rows(const std::vector<File>&, hipStream_t) {
  for (bool split : {false, true})
    for (size_t rows : {size_t(1) << 20, (size_t(1) << 22) - 1, size_t(1) << 22})
      for (int where = 0; where < 3; ++where) {
        h2::Composed c;
        std::vector<h2::RowSpec> v(rows);
        if (where == 0) c.up.push_back(std::move(v)), c.up_split.push_back(split);
        if (where == 1) c.down.push_back(std::move(v)), c.down_split.push_back(split);
        if (where == 2) c.out = std::move(v), c.out_split = split;
        const bool fits = !split || 4 * rows * 256 < size_t(1) << 32;
        if (h2::composed_fits(c) != fits) fail(name_of("rows", (int64_t)rows, split, where, ' '));
      }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  const std::string name = argv[1];
  std::vector<File> files;
  for (int i = 2; i < argc; ++i) files.push_back(read_file(argv[i]));
  hipStream_t s = nullptr;
  (void)hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  const int64_t live = h2_standin_live();
  if (name == "products") products(files, s);
  else if (name == "graphs") graphs(files, s);
  else if (name == "growth") growth(files, s);
  else if (name == "streams") streams(files, s);
  else if (name == "batch") batch(files, s);
  else if (name == "memory") memory(files, s);
  else if (name == "compress_memory") compress_memory(files, s);
  else if (name == "fp32") fp32(files, s);
  else if (name == "profile") profile(files, s);
  else if (name == "split_rows") split_rows(files, s);
  else return 2;
  if (h2_standin_live() != live) fail("streams, events, graphs or memory left behind");
  (void)hipStreamDestroy(s);
  std::printf("%s ok\n", name.c_str());
  return 0;
}
