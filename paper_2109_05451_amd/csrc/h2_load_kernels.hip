// Kernels run once when an operator is loaded.
#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "h2_internal.h"

namespace h2 {
namespace {

// The transposed copies of the leaf bases and transfer matrices (used by the
// upsweep products): task b's column-major rows x cols block at mat + src
// becomes its transpose (cols x rows, column-major) at trans + dst.  One
// workgroup per task, grid-stride; reads are contiguous.
__global__ __launch_bounds__(256) void k_transpose_tasks(const TransTask* __restrict__ tasks, int64_t ntasks,
                                                          const double* __restrict__ mat,
                                                          double* __restrict__ trans) {
  for (int64_t b = blockIdx.x; b < ntasks; b += gridDim.x) {
    const TransTask T = tasks[b];
    const int64_t total = (int64_t)T.rows * T.cols;
    for (int64_t e = threadIdx.x; e < total; e += blockDim.x) {
      const int64_t r = e % T.rows, c = e / T.rows;
      trans[T.dst + c + (int64_t)T.cols * r] = mat[T.src + e];
    }
  }
}

}  // namespace

hipError_t launch_transpose_tasks(const TransTask* tasks, int64_t ntasks, const double* mat, double* trans,
                                  hipStream_t s) {
  if (ntasks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_transpose_tasks, dim3((unsigned)std::min<int64_t>(ntasks, 65536)), dim3(256), 0, s, tasks,
                     ntasks, mat, trans);
  return hipGetLastError();
}

namespace {
// One stage of run_compose, a workgroup per node: its matrices one level after
// the other, each read back from where it was written (a few KB, in L1/L2).
// tab: per level ranks, transfer offsets, first nodes, outputs (nl each).
// Run once at load: well under a millisecond for 2^16 points.
__global__ __launch_bounds__(256) void k_compose(const int64_t* __restrict__ tab, int nl,
                                                 const int32_t* __restrict__ parent, const int32_t* __restrict__ lo_of,
                                                 int64_t leaf0, int s, int lo, int points, int up, int64_t c0,
                                                 int64_t stored, const double* __restrict__ mat, double* trans) {
  const int64_t *k = tab, *tr = tab + nl, *lp = tab + 2 * nl, *reg = tab + 3 * nl;
  const int64_t c = c0 + blockIdx.x;
  const int top = s - 1, q = nl - 1;
  const int64_t p0 = points ? lo_of[c - leaf0] : 0;
  const int m = points ? lo_of[c - leaf0 + 1] - (int)p0 : (int)k[s];
  const int64_t before = points ? p0 : blockIdx.x * (int64_t)k[s];  // rows of the nodes before this one
  const double* A = mat + stored + (points ? p0 * k[q] : blockIdx.x * (int64_t)(k[s] * k[top]));
  bool trA = false;  // A holds the transpose
  int64_t sum = 0;
  for (int l = lo; l <= top; ++l) sum += k[l];
  double* D = trans + reg[0] + before * sum;  // downsweep: this node's matrices
  int64_t a = points ? c : parent[c];         // ancestor on level l + 1
  if (!up) {
    for (int e = threadIdx.x; e < m * (int)k[top]; e += 256) D[e] = A[e];
    A = D;
    D += m * k[top];
    __syncthreads();
  }
  for (int l = top - 1; l >= lo; --l) {
    const int kk = (int)k[l + 1], kn = (int)k[l];
    const double* T = mat + tr[l + 1] + (a - lp[l + 1]) * (int64_t)(kk * kn);
    double* C = up ? trans + reg[l] + before * kn : D;
    for (int e = threadIdx.x; e < m * kn; e += 256) {
      const int r = up ? e / kn : e % m, j = up ? e % kn : e / m;
      double sum_ = 0.0;
      for (int i = 0; i < kk; ++i) sum_ += (trA ? A[i + (int64_t)kk * r] : A[r + (int64_t)m * i]) * T[i + (int64_t)kk * j];
      C[e] = sum_;
    }
    __syncthreads();  // this level's matrix is the next one's operand
    A = C;
    trA = up;
    D += (int64_t)m * kn;
    a = parent[a];
  }
}
}  // namespace

int run_compose(const std::vector<const Composed*>& C, const Parsed& P, const double* mat, double* trans) {
  // one device buffer: per stage the level tables, then the tree
  const int nl = (int)P.q + 1;
  size_t nst = 0;
  for (const Composed* c : C) nst += c->stages.size();
  if (nst == 0) return H2_OK;
  const size_t tabs = sizeof(int64_t) * 4 * nl * nst, pb = sizeof(int32_t) * P.nnodes;
  std::vector<char> host(tabs + pb + sizeof(int32_t) * (P.nleaves + 1));
  int64_t* t = reinterpret_cast<int64_t*>(host.data());
  for (const Composed* c : C)
    for (const ComposeStage& g : c->stages) {
      for (int l = 0; l < nl; ++l) {
        t[l] = g.k[l];
        t[nl + l] = g.tr[l];
        t[2 * nl + l] = P.level_ptr[l];
        t[3 * nl + l] = g.reg[l];
      }
      t += 4 * nl;
    }
  int32_t* par = reinterpret_cast<int32_t*>(host.data() + tabs);
  for (int64_t c = 0; c < P.nnodes; ++c) par[c] = (int32_t)P.parent[c];
  int32_t* lo = par + P.nnodes;
  for (int64_t i = 0; i < P.nleaves; ++i) lo[i] = (int32_t)P.lo[P.leaf0 + i];
  lo[P.nleaves] = (int32_t)P.n;
  char* d = nullptr;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&d), host.size());
  if (e == hipSuccess) e = hipMemcpy(d, host.data(), host.size(), hipMemcpyHostToDevice);
  size_t at = 0;
  for (const Composed* c : C)
    for (const ComposeStage& g : c->stages) {
      if (e == hipSuccess && g.count > 0) {
        hipLaunchKernelGGL(k_compose, dim3((unsigned)g.count), dim3(256), 0, nullptr,
                           reinterpret_cast<const int64_t*>(d) + 4 * nl * at, nl,
                           reinterpret_cast<const int32_t*>(d + tabs),
                           reinterpret_cast<const int32_t*>(d + tabs) + P.nnodes, P.leaf0, g.s, g.lo, g.points, g.up,
                           g.c0, g.stored, mat, trans);
        e = hipGetLastError();
      }
      ++at;
    }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (d) (void)hipFree(d);
  if (e == hipSuccess) return H2_OK;
  set_error(std::string("composed transfers: ") + hipGetErrorString(e));
  return e == hipErrorOutOfMemory ? H2_ENOMEM : H2_EHIP;
}

}  // namespace h2
