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
// One workgroup per task; the operands are a few KB and stay in L1/L2 (a load-
// time kernel: a few ms for the largest operators).
__global__ __launch_bounds__(256) void k_compose_tasks(const ComposeTask* __restrict__ tasks, const double* mat,
                                                       double* trans, double* scratch) {
  const ComposeTask t = tasks[blockIdx.x];
  const int w = t.where & 3;
  const double* A = (w == 0 ? mat : w == 1 ? trans : scratch) + t.a;
  const double* B = mat + t.b;
  double* C = (t.where & 4 ? scratch : trans) + t.dst;
  for (int e = threadIdx.x; e < t.m * t.n; e += 256) {
    const int r = e % t.m, c = e / t.m;
    double s = 0.0;
    if (t.k == 0) s = A[e];
    for (int i = 0; i < t.k; ++i) s += A[r + (int64_t)t.m * i] * B[i + (int64_t)t.k * c];
    C[e] = s;
  }
}
}  // namespace

hipError_t launch_compose_tasks(const ComposeTask* tasks, int64_t ntasks, const double* mat, double* trans,
                                double* scratch, hipStream_t s) {
  if (ntasks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_compose_tasks, dim3((unsigned)ntasks), dim3(256), 0, s, tasks, mat, trans, scratch);
  return hipGetLastError();
}

int run_compose(const Composed& C, const double* mat, double* trans) {
  // one device buffer: the tasks of every step, the transpositions, scratch
  size_t ntask = 0;
  for (const auto& v : C.steps) ntask += v.size();
  if (ntask == 0) return H2_OK;
  const size_t tb = sizeof(ComposeTask) * ntask, sb = sizeof(TransTask) * C.trans.size();
  std::vector<char> host(tb + sb);
  size_t at = 0;
  for (const auto& v : C.steps) {
    if (!v.empty()) std::memcpy(host.data() + at, v.data(), sizeof(ComposeTask) * v.size());
    at += sizeof(ComposeTask) * v.size();
  }
  if (sb) std::memcpy(host.data() + tb, C.trans.data(), sb);
  const size_t scratch_at = (tb + sb + 255) / 256 * 256;
  char* d = nullptr;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&d), scratch_at + sizeof(double) * (size_t)C.nscratch + 256);
  if (e == hipSuccess) e = hipMemcpy(d, host.data(), tb + sb, hipMemcpyHostToDevice);
  double* scratch = reinterpret_cast<double*>(d + scratch_at);
  at = 0;
  for (const auto& v : C.steps) {  // in stream order: a step reads what the one before it wrote
    if (e == hipSuccess)
      e = launch_compose_tasks(reinterpret_cast<const ComposeTask*>(d) + at, (int64_t)v.size(), mat, trans, scratch,
                               nullptr);
    at += v.size();
  }
  if (e == hipSuccess && sb)
    e = launch_transpose_tasks(reinterpret_cast<const TransTask*>(d + tb), (int64_t)C.trans.size(), scratch, trans,
                               nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (d) (void)hipFree(d);
  if (e == hipSuccess) return H2_OK;
  set_error(std::string("composed transfers: ") + hipGetErrorString(e));
  return e == hipErrorOutOfMemory ? H2_ENOMEM : H2_EHIP;
}

}  // namespace h2
