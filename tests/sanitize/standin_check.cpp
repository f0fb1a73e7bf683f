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

#include "h2.h"

extern "C" {
void h2_standin_seed(uint64_t);
void h2_standin_limit(int64_t);
int64_t h2_standin_used();
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
  else return 2;
  if (h2_standin_live() != live) fail("streams, events, graphs or memory left behind");
  (void)hipStreamDestroy(s);
  std::printf("%s ok\n", name.c_str());
  return 0;
}
