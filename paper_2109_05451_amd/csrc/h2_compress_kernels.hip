// Kernels of the algebraic recompression (Section 5 of the paper), FP64.
//
// Every operation works on small dense matrices (at most 64 columns; the
// QR operands at most 8192 elements), one workgroup per matrix (or per
// output block), with the operands staged in LDS:
//   k_qr       Householder QR with the thin Q formed in place (reflectors
//              applied backwards), R written separately
//   k_gemm     C = beta C + alpha sum_p op(A_p) op(B_p) over a list of pairs
//              (segmented sums such as the Gram matrix of a block row)
//   k_triple   C = beta C + L M R^T (coupling transforms, projections, the
//              Gram downsweep)
//   k_eig      symmetric eigendecomposition by parallel cyclic Jacobi
//              (eigenvalues in descending order, eigenvectors as columns)
// plus small elementwise helpers.  All index bounds come from descriptors
// that the host checks against the allocations before any launch.
#include <hip/hip_runtime.h>

#include "h2_compress.h"

namespace h2 {
namespace {

constexpr int kCT = 256;  // threads per workgroup
constexpr int kTile = 64; // largest output rows / columns of one GEMM task

// v + (the lane at the given row rotation's v): the sums of a row of 16 lanes
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return v + __hiloint2double(hi, lo);
}

// Sum over the wave in every lane, halves first: lanes 32, 16 apart by the
// lane swaps (both operands the same register: one result holds the lower
// half's value in both, the other the upper's), then 8, 4, 2, 1 by row
// rotations.  No LDS: a __shfl_xor of a double is two LDS permutes.
__device__ __forceinline__ double wave_sum(double v) {
  const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  v = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  const unsigned lo2 = (unsigned)__double2loint(v), hi2 = (unsigned)__double2hiint(v);
  const auto l2 = __builtin_amdgcn_permlane16_swap(lo2, lo2, false, false);
  const auto h2 = __builtin_amdgcn_permlane16_swap(hi2, hi2, false, false);
  v = __hiloint2double((int)h2[0], (int)l2[0]) + __hiloint2double((int)h2[1], (int)l2[1]);
  v = dpp_add<0x128>(v);  // row_ror:8
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}

// ---------------------------------------------------------------------------
// Householder QR of an r x c column-major matrix (r * c <= ELEMS).
// Reflector j (j < nr = min(r, c)) is H_j = I - tau_j v_j v_j^T with
// v_j[j] = 1, zeros above j, scal_j times the stored column below it;
// beta_j = R[j][j].
// Q (r x c): the first nr columns of H_0 ... H_{nr-1}, zero columns after.
// R (c x c): upper triangle of the factored matrix in rows < nr, zero rows
// after (so that A = Q R also when r < c).
//
// Bound by the chain of reflectors.  Every wave takes the norm itself and the
// scale stays beside the column, so a reflector is one barrier; a wave applies
// it to four columns at a time, whose dot products then overlap; the LDS is
// sized by the launch's largest operand, so the leaf level is resident at
// once.  512 stacks of 72 x 36: 231 -> 102 us, 1024 leaf bases of 64 x 36 240 -> 214.

// H_j on columns first + wave, first + wave + 4, ... below last.  Four at a
// time: past the last column the last one again, whose equal results are
// stored again, so that no load stands behind a branch.  Rows j + lane and
// j + lane + 64 stay in registers, further ones (operands of more than 128
// rows) are read twice.
__device__ __forceinline__ void reflect(double* sA, int r, int j, double tau, double scal, int first, int last,
                                        int wave, int lane) {
  const double* col = sA + j * r;
  const int i0 = min(j + lane, r - 1), i1 = min(j + lane + 64, r - 1);
  const bool in0 = j + lane < r, in1 = j + lane + 64 < r;
  const double v0 = !in0 ? 0.0 : lane == 0 ? 1.0 : col[i0] * scal, v1 = in1 ? col[i1] * scal : 0.0;
  for (int c0 = first + wave; c0 < last; c0 += 16) {
    double* a[4];
    double w[4], x0[4], x1[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = sA + min(c0 + 4 * u, c0 + (last - 1 - c0) / 4 * 4) * r;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x0[u] = a[u][i0];
      x1[u] = a[u][i1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = v0 * x0[u] + v1 * x1[u];
    for (int i = j + lane + 128; i < r; i += 64) {
      const double v = col[i] * scal;
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] += v * a[u][i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = wave_sum(w[u]) * tau;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (in0) a[u][i0] = x0[u] - w[u] * v0;
      if (in1) a[u][i1] = x1[u] - w[u] * v1;
    }
    for (int i = j + lane + 128; i < r; i += 64) {
      const double v = col[i] * scal;
      double x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = a[u][i];
#pragma unroll
      for (int u = 0; u < 4; ++u) a[u][i] = x[u] - w[u] * v;
    }
  }
}

template <int ELEMS>
__global__ __launch_bounds__(kCT) void k_qr(const QrTask* __restrict__ tasks) {
  __shared__ double sA[ELEMS];
  __shared__ double s_tau[kMaxCompressRank], s_scal[kMaxCompressRank], s_beta[kMaxCompressRank];
  const QrTask T = tasks[blockIdx.x];
  const int r = T.rows, c = T.cols, nr = min(r, c);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int j = wave; j < c; j += kCT / 64)
    for (int i = lane; i < r; i += 64) sA[i + j * r] = T.A[i + (int64_t)j * T.lda];
  __syncthreads();
  for (int j = 0; j < nr; ++j) {
    const double* col = sA + j * r;
    double x2 = 0.0;
    for (int i = j + 1 + lane; i < r; i += 64) x2 += col[i] * col[i];
    x2 = wave_sum(x2);
    const double alpha = col[j];
    double tau = 0.0, scal = 0.0, beta = alpha;
    if (x2 > 0.0) {
      const double nrm = sqrt(alpha * alpha + x2);
      beta = alpha >= 0.0 ? -nrm : nrm;
      tau = (beta - alpha) / beta;
      scal = 1.0 / (alpha - beta);
    }
    if (tid == 0) {
      s_tau[j] = tau;
      s_scal[j] = scal;
      s_beta[j] = beta;
    }
    if (tau != 0.0) reflect(sA, r, j, tau, scal, j + 1, c, wave, lane);
    __syncthreads();
  }
  // R
  for (int j = wave; j < c; j += kCT / 64)
    for (int i = lane; i < c; i += 64)
      T.R[i + (int64_t)j * T.ldr] = i >= nr || i > j ? 0.0 : i == j ? s_beta[j] : sA[i + j * r];
  __syncthreads();
  // thin Q in place, reflectors taken backwards
  for (int j = nr - 1; j >= 0; --j) {
    double* col = sA + j * r;
    const double tau = s_tau[j], scal = s_scal[j];
    // H_j on columns j+1 .. nr-1 (their rows above j are zero, so only rows >= j change)
    if (tau != 0.0) reflect(sA, r, j, tau, scal, j + 1, nr, wave, lane);
    __syncthreads();
    for (int i = tid; i < r; i += kCT) col[i] = i < j ? 0.0 : i == j ? 1.0 - tau : col[i] * scal * -tau;
    __syncthreads();
  }
  for (int j = wave; j < c; j += kCT / 64)
    for (int i = lane; i < r; i += 64) T.Q[i + (int64_t)j * T.ldq] = j < nr ? sA[i + j * r] : 0.0;
}

// ---------------------------------------------------------------------------
// GEMM tiles: thread (ty, tx) = (tid / 16, tid % 16) owns rows ty + 16 i and
// columns tx + 16 j (i, j < MI) of a 16 MI x 16 MI output (MI = 1..4, picked
// per launch from its largest task, so 36 x 36 blocks take 48 x 48 tiles);
// K in chunks of 32 staged in LDS as sA[k][row], sB[k][col] (odd stride
// against bank conflicts).  Every output sums over k in the same order
// whatever MI.
constexpr int kKc = 32;

template <int MI>
struct GemmAcc {
  double v[MI][MI];
};

__device__ inline double opA(const double* A, int64_t lda, bool t, int i, int k) {
  return t ? A[k + (int64_t)i * lda] : A[i + (int64_t)k * lda];
}

// acc += op(A) (a x K) * op(B) (K x b), operands in global memory
template <int MI>
__device__ void gemm_acc(GemmAcc<MI>& acc, const double* A, int64_t lda, bool ta, const double* B, int64_t ldb,
                         bool tb, int a, int b, int K, double* sA, double* sB) {
  constexpr int TILE = 16 * MI, LD = TILE + 1;
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  for (int k0 = 0; k0 < K; k0 += kKc) {
    const int kc = min(kKc, K - k0);
    __syncthreads();
    for (int e = tid; e < kKc * TILE; e += kCT) {
      // transposed operands: consecutive threads walk k (contiguous), else rows
      int kk, i;
      if (ta) { i = e / kKc; kk = e - i * kKc; } else { kk = e / TILE; i = e - kk * TILE; }
      sA[kk * LD + i] = (kk < kc && i < a) ? opA(A, lda, ta, i, k0 + kk) : 0.0;
    }
    for (int e = tid; e < kKc * TILE; e += kCT) {
      int kk, j;
      if (tb) { kk = e / TILE; j = e - kk * TILE; } else { j = e / kKc; kk = e - j * kKc; }
      // op(B)[k][j] = tb ? B[j][k] : B[k][j]
      sB[kk * LD + j] = (kk < kc && j < b) ? (tb ? B[j + (int64_t)(k0 + kk) * ldb] : B[(k0 + kk) + (int64_t)j * ldb])
                                          : 0.0;
    }
    __syncthreads();
    for (int kk = 0; kk < kc; ++kk) {
      double ar[MI], br[MI];
#pragma unroll
      for (int i = 0; i < MI; ++i) ar[i] = sA[kk * LD + ty + 16 * i];
#pragma unroll
      for (int j = 0; j < MI; ++j) br[j] = sB[kk * LD + tx + 16 * j];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc.v[i][j] = fma(ar[i], br[j], acc.v[i][j]);
    }
  }
}

template <int MI>
__device__ void gemm_store(const GemmAcc<MI>& acc, double* C, int64_t ldc, int a, int b, double alpha,
                           double beta) {
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j) {
      const int row = ty + 16 * i, col = tx + 16 * j;
      if (row < a && col < b) {
        double* o = C + row + (int64_t)col * ldc;
        *o = beta == 0.0 ? alpha * acc.v[i][j] : fma(alpha, acc.v[i][j], beta * *o);
      }
    }
}

template <int MI>
__global__ __launch_bounds__(kCT) void k_gemm(const GemmTask* __restrict__ tasks, const GemmPair* __restrict__ pairs) {
  constexpr int LD = 16 * MI + 1;
  __shared__ double sA[kKc * LD];
  __shared__ double sB[kKc * LD];
  const GemmTask T = tasks[blockIdx.x];
  GemmAcc<MI> acc;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j) acc.v[i][j] = 0.0;
  for (int p = T.pbeg; p < T.pend; ++p) {
    const GemmPair P = pairs[p];
    gemm_acc<MI>(acc, P.A, P.lda, P.flags & 1, P.B, P.ldb, P.flags & 2, T.m, T.n, P.k, sA, sB);
  }
  gemm_store<MI>(acc, T.C, T.ldc, T.m, T.n, T.alpha, T.beta);
}

// C = beta C + op(L) M R^T: L M (a x k2) into LDS, then times R^T; the tile
// covers a, b and k2
template <int MI>
__global__ __launch_bounds__(kCT) void k_triple(const TripleTask* __restrict__ tasks) {
  constexpr int TILE = 16 * MI, LD = TILE + 1;
  __shared__ double sA[kKc * LD];
  __shared__ double sB[kKc * LD];
  __shared__ double sT[TILE * LD];  // L M, column-major with stride LD
  const TripleTask T = tasks[blockIdx.x];
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  GemmAcc<MI> acc;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j) acc.v[i][j] = 0.0;
  gemm_acc<MI>(acc, T.L, T.ldl, T.flags & 1, T.M, T.ldm, false, T.a, T.k2, T.k1, sA, sB);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j) sT[(ty + 16 * i) + (tx + 16 * j) * LD] = acc.v[i][j];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j) acc.v[i][j] = 0.0;
  __syncthreads();
  // (L M) from LDS times R^T
  for (int k0 = 0; k0 < T.k2; k0 += kKc) {
    const int kc = min(kKc, T.k2 - k0);
    __syncthreads();
    for (int e = tid; e < kKc * TILE; e += kCT) {
      const int kk = e / TILE, j = e - kk * TILE;
      sB[kk * LD + j] = (kk < kc && j < T.b) ? T.R[j + (int64_t)(k0 + kk) * T.ldr] : 0.0;
    }
    __syncthreads();
    for (int kk = 0; kk < kc; ++kk) {
      double ar[MI], br[MI];
#pragma unroll
      for (int i = 0; i < MI; ++i) ar[i] = sT[(ty + 16 * i) + (k0 + kk) * LD];
#pragma unroll
      for (int j = 0; j < MI; ++j) br[j] = sB[kk * LD + tx + 16 * j];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc.v[i][j] = fma(ar[i], br[j], acc.v[i][j]);
    }
  }
  gemm_store<MI>(acc, T.C, T.ldc, T.a, T.b, 1.0, T.beta);
}

// ---------------------------------------------------------------------------
// Parallel cyclic Jacobi for a symmetric n x n matrix (n <= N), one
// workgroup per matrix, matrix and eigenvectors in LDS (sized by N, so small
// orders leave room for more workgroups per CU): rounds of n'/2 disjoint
// rotations (n' = n rounded up to even; the padding index only meets
// identity rotations), tournament ordering, n' - 1 rounds per sweep, until a
// sweep rotates nothing.  Rotation (c, s) from the 2 x 2 symmetric Schur
// decomposition zeroes A[p][q] in J^T A J, J = [[c, s], [-s, c]].
//
// Bound by the chain of rounds.  A round is two barriers: every thread takes
// 2 x 2 blocks of A (a row pair and a column pair, both rotations at once);
// then the first wave finds the next round's rotations while the others apply
// this round's to the eigenvectors.  1024 matrices of order 36: 1350 -> 990
// us, a level of orders up to 32 200 -> 135.
constexpr int kET = 512;
template <int N>
__global__ __launch_bounds__(kET) void k_eig(const EigTask* __restrict__ tasks) {
  constexpr int LD = N + 1;
  __shared__ double sA[N * LD];
  __shared__ double sV[N * LD];
  __shared__ double2 s_cs[2][N / 2];  // rotations, of this round and the next
  __shared__ int2 s_pq[2][N / 2];
  __shared__ int s_rot[2];  // a rotation in this sweep, and in the next
  __shared__ double s_lam[N];
  __shared__ double s_red[kET];
  const EigTask T = tasks[blockIdx.x];
  const int n = T.n, tid = threadIdx.x;
  const int np = (n + 1) & ~1, half = np / 2;
  double sq = 0.0;
  for (int e = tid; e < np * np; e += kET) {
    const int j = e / np, i = e - j * np;
    // symmetrize (the inputs are symmetric up to rounding)
    const double a = i < n && j < n ? 0.5 * (T.G[i + (int64_t)j * T.ldg] + T.G[j + (int64_t)i * T.ldg]) : 0.0;
    sA[i * LD + j] = a;
    sV[i * LD + j] = i == j ? 1.0 : 0.0;
    sq += a * a;
  }
  s_red[tid] = sq;
  __syncthreads();
  for (int w = kET / 2; w > 0; w >>= 1) {
    if (tid < w) s_red[tid] += s_red[tid + w];
    __syncthreads();
  }
  // off-diagonal entries below 1e-16 of the Frobenius norm are not rotated:
  // besides the relative test, this stops the sweeps once only rounding
  // noise among the (many) negligible eigenvalues is left, at an absolute
  // accuracy far below any threshold the truncation applies
  const double floor_abs = 1e-16 * sqrt(s_red[0]);
  if (tid < 2) s_rot[tid] = 0;
  __syncthreads();
  // rotations of a round from A into buffer b; sweeps alternate s_rot
  auto rotations = [&](int round, int b, int sweep) {
    if (tid >= half) return;
    int p, q;
    if (tid == 0) { p = round; q = np - 1; }
    else { p = (round + tid) % (np - 1); q = (round - tid + (np - 1)) % (np - 1); }
    if (p > q) { const int t = p; p = q; q = t; }
    double c = 1.0, s = 0.0;
    if (q < n) {
      const double app = sA[p * LD + p], aqq = sA[q * LD + q], apq = sA[p * LD + q];
      if (fabs(apq) > 1e-300 && fabs(apq) > floor_abs && fabs(apq) > 1e-15 * sqrt(fabs(app) * fabs(aqq))) {
        const double tau = (aqq - app) / (2.0 * apq);
        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
        c = 1.0 / sqrt(1.0 + t * t);
        s = t * c;
        s_rot[sweep & 1] = 1;
      }
    }
    s_pq[b][tid] = int2{p, q};
    s_cs[b][tid] = double2{c, s};
  };
  // quotients by half of numbers below 2^11 (half <= 32)
  const unsigned inv = half > 0 ? 65536u / (unsigned)half + 1u : 0u;
  if (np > 1) rotations(0, 0, 0);
  __syncthreads();
  for (int sweep = 0, b = 0; sweep < 40 && np > 1; ++sweep) {
    if (tid == 0) s_rot[(sweep + 1) & 1] = 0;
    for (int round = 0; round < np - 1; ++round, b ^= 1) {
      // rows p' = c p - s q, q' = s p + c q, then columns likewise
      for (int e = tid; e < half * half; e += kET) {
        const int k = (int)((unsigned)e * inv >> 16), l = e - k * half;
        const double2 rk = s_cs[b][k], rl = s_cs[b][l];
        if (rk.y == 0.0 && rl.y == 0.0) continue;
        const int2 ik = s_pq[b][k], il = s_pq[b][l];
        double *pp = sA + ik.x * LD + il.x, *pq = sA + ik.x * LD + il.y;
        double *qp = sA + ik.y * LD + il.x, *qq = sA + ik.y * LD + il.y;
        const double a = *pp, bb = *pq, c = *qp, d = *qq;
        const double a1 = rk.x * a - rk.y * c, c1 = rk.y * a + rk.x * c;
        const double b1 = rk.x * bb - rk.y * d, d1 = rk.y * bb + rk.x * d;
        *pp = rl.x * a1 - rl.y * b1;
        *pq = rl.y * a1 + rl.x * b1;
        *qp = rl.x * c1 - rl.y * d1;
        *qq = rl.y * c1 + rl.x * d1;
      }
      __syncthreads();
      const bool last = round + 1 == np - 1;
      if (tid < 64) rotations(last ? 0 : round + 1, b ^ 1, last ? sweep + 1 : sweep);
      else
        for (int e = tid - 64; e < half * n; e += kET - 64) {
          const int i = (int)((unsigned)e * inv >> 16), k = e - i * half;
          const double2 r = s_cs[b][k];
          if (r.y == 0.0) continue;
          const int2 ix = s_pq[b][k];
          double *vp = sV + i * LD + ix.x, *vq = sV + i * LD + ix.y;
          const double x = *vp, y = *vq;
          *vp = r.x * x - r.y * y;
          *vq = r.y * x + r.x * y;
        }
      __syncthreads();
    }
    if (s_rot[sweep & 1] == 0) break;
    __syncthreads();  // read by all before the next sweep clears it
  }
  // descending order (ties by index)
  for (int i = tid; i < n; i += kET) s_lam[i] = sA[i * LD + i];
  __syncthreads();
  for (int i = tid; i < n; i += kET) {
    const double li = s_lam[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) rank += (s_lam[j] > li) || (s_lam[j] == li && j < i);
    T.lam[rank] = li;
    for (int row = 0; row < n; ++row) T.Z[row + (int64_t)rank * T.ldz] = sV[row * LD + i];
  }
}

// ---------------------------------------------------------------------------
// Elementwise helpers (one workgroup per node)

// masked Gram: out = P G P, P = diag(1 if column j of the leaf basis is nonzero)
__global__ __launch_bounds__(kCT) void k_mask_gram(const MaskTask* __restrict__ tasks) {
  __shared__ int nz[kMaxCompressRank];
  const MaskTask T = tasks[blockIdx.x];
  const int k = T.k, m = T.m, tid = threadIdx.x;
  for (int j = tid; j < k; j += kCT) {
    int any = 0;
    for (int i = 0; i < m; ++i) any |= T.U[i + (int64_t)j * T.ldu] != 0.0;
    nz[j] = any;
  }
  __syncthreads();
  for (int e = tid; e < k * k; e += kCT) {
    const int j = e / k, i = e - j * k;
    T.out[i + (int64_t)j * k] = (nz[i] && nz[j]) ? T.G[i + (int64_t)j * T.ldg] : 0.0;
  }
}

// per node: count of lam > thr2 (first `n` entries), into counts[node]
__global__ void k_count(const CountTask* __restrict__ tasks, int64_t ntasks, double thr2, int32_t* counts) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= ntasks) return;
  const CountTask T = tasks[t];
  int c = 0;
  for (int i = 0; i < T.n; ++i) c += T.lam[i] > thr2;
  counts[T.node] = c;
}

// largest first eigenvalue over the tasks (one workgroup, fixed order)
__global__ __launch_bounds__(kCT) void k_max_lead(const CountTask* __restrict__ tasks, int64_t ntasks,
                                                   double* out) {
  __shared__ double red[kCT];
  double m = 0.0;
  for (int64_t t = threadIdx.x; t < ntasks; t += kCT) {
    const CountTask T = tasks[t];
    if (T.n > 0) m = fmax(m, T.lam[0]);
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int o = kCT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// column scaling of eigenvector matrices: Z[:, j] *= (j < keep ? f(lam_j) : 0)
// for j < cols, with f = 1 (mode 0) or 1/sqrt(lam) (mode 1); the kept count
// is counts[node]
__global__ __launch_bounds__(kCT) void k_scale_cols(const ScaleTask* __restrict__ tasks, const int32_t* counts,
                                                     int mode) {
  const ScaleTask T = tasks[blockIdx.x];
  const int keep = counts[T.node];
  for (int e = threadIdx.x; e < T.rows * T.cols; e += kCT) {
    const int j = e / T.rows, i = e - j * T.rows;
    double f = 0.0;
    if (j < keep) f = mode == 0 ? 1.0 : 1.0 / sqrt(T.lam[j]);
    T.Z[i + (int64_t)j * T.ldz] *= f;
  }
}

// square-root factor R = diag(sqrt(max(lam, 0))) Z^T (n x n)
__global__ __launch_bounds__(kCT) void k_sqrt_factor(const EigTask* __restrict__ tasks, double* const* outs,
                                                      const int64_t* ldo) {
  const EigTask T = tasks[blockIdx.x];
  double* R = outs[blockIdx.x];
  const int64_t ld = ldo[blockIdx.x];
  for (int e = threadIdx.x; e < T.n * T.n; e += kCT) {
    const int j = e / T.n, i = e - j * T.n;
    R[i + (int64_t)j * ld] = sqrt(fmax(T.lam[i], 0.0)) * T.Z[j + (int64_t)i * T.ldz];
  }
}

// dst (rows x cols, ldd) = src (rows x cols, lds), optionally transposed (dst = src^T)
__global__ __launch_bounds__(kCT) void k_copy(const CopyTask* __restrict__ tasks) {
  const CopyTask T = tasks[blockIdx.x];
  for (int e = threadIdx.x; e < T.rows * T.cols; e += kCT) {
    const int j = e / T.rows, i = e - j * T.rows;
    T.dst[i + (int64_t)j * T.ldd] = T.trans ? T.src[j + (int64_t)i * T.lds] : T.src[i + (int64_t)j * T.lds];
  }
}

inline dim3 grid_of(int64_t n) { return dim3((unsigned)n); }

}  // namespace

hipError_t launch_qr(const QrTask* t, int64_t n, hipStream_t s, int max_elems) {
  if (n == 0) return hipSuccess;
  if (max_elems <= 2560) hipLaunchKernelGGL((k_qr<2560>), grid_of(n), dim3(kCT), 0, s, t);
  else if (max_elems <= 4608) hipLaunchKernelGGL((k_qr<4608>), grid_of(n), dim3(kCT), 0, s, t);
  else if (max_elems <= kQrMaxElems) hipLaunchKernelGGL((k_qr<kQrMaxElems>), grid_of(n), dim3(kCT), 0, s, t);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
hipError_t launch_gemm(const GemmTask* t, int64_t n, const GemmPair* p, hipStream_t s, int maxdim) {
  if (n == 0) return hipSuccess;
  if (maxdim <= 16) hipLaunchKernelGGL((k_gemm<1>), grid_of(n), dim3(kCT), 0, s, t, p);
  else if (maxdim <= 32) hipLaunchKernelGGL((k_gemm<2>), grid_of(n), dim3(kCT), 0, s, t, p);
  else if (maxdim <= 48) hipLaunchKernelGGL((k_gemm<3>), grid_of(n), dim3(kCT), 0, s, t, p);
  else if (maxdim <= kTile) hipLaunchKernelGGL((k_gemm<4>), grid_of(n), dim3(kCT), 0, s, t, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
hipError_t launch_triple(const TripleTask* t, int64_t n, hipStream_t s, int maxdim) {
  if (n == 0) return hipSuccess;
  if (maxdim <= 16) hipLaunchKernelGGL((k_triple<1>), grid_of(n), dim3(kCT), 0, s, t);
  else if (maxdim <= 32) hipLaunchKernelGGL((k_triple<2>), grid_of(n), dim3(kCT), 0, s, t);
  else if (maxdim <= 48) hipLaunchKernelGGL((k_triple<3>), grid_of(n), dim3(kCT), 0, s, t);
  else if (maxdim <= kTile) hipLaunchKernelGGL((k_triple<4>), grid_of(n), dim3(kCT), 0, s, t);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
hipError_t launch_eig(const EigTask* t, int64_t n, int nmax, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (nmax <= 32) hipLaunchKernelGGL((k_eig<32>), grid_of(n), dim3(kET), 0, s, t);
  else if (nmax <= 48) hipLaunchKernelGGL((k_eig<48>), grid_of(n), dim3(kET), 0, s, t);
  else if (nmax <= kMaxCompressRank) hipLaunchKernelGGL((k_eig<64>), grid_of(n), dim3(kET), 0, s, t);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
hipError_t launch_mask_gram(const MaskTask* t, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_mask_gram, grid_of(n), dim3(kCT), 0, s, t);
  return hipGetLastError();
}
hipError_t launch_count(const CountTask* t, int64_t n, double thr2, int32_t* counts, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_count, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, t, n, thr2, counts);
  return hipGetLastError();
}
hipError_t launch_max_lead(const CountTask* t, int64_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_max_lead, dim3(1), dim3(kCT), 0, s, t, n, out);
  return hipGetLastError();
}
hipError_t launch_scale_cols(const ScaleTask* t, int64_t n, const int32_t* counts, int mode, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scale_cols, grid_of(n), dim3(kCT), 0, s, t, counts, mode);
  return hipGetLastError();
}
hipError_t launch_sqrt_factor(const EigTask* t, int64_t n, double* const* outs, const int64_t* ldo, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_sqrt_factor, grid_of(n), dim3(kCT), 0, s, t, outs, ldo);
  return hipGetLastError();
}
hipError_t launch_copy(const CopyTask* t, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy, grid_of(n), dim3(kCT), 0, s, t);
  return hipGetLastError();
}

}  // namespace h2
