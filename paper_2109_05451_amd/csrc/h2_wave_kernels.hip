// Wave-per-row kernel of the multi-vector path (FP64 and FP32 MFMA): a row
// list's products out (m x 16NT, row-major) = M (m x ncols, column-major) * B
// (ncols x 16NT, gathered block by block), each row on one wave or split by
// vector tiles over two or four, with no workgroup barriers.
#include <algorithm>
#include <type_traits>

#include "h2_internal.h"

namespace h2 {
namespace {

constexpr int kT = 256;  // threads per workgroup (4 wave64)
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
template <typename T> struct Mfma;
template <> struct Mfma<double> {
  typedef d4 acc;
  static __device__ __forceinline__ d4 op(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // accumulator element r of lane l: tile row 4r + l/16, column l%16
  static __device__ __forceinline__ int row(int r, int akk) { return 4 * r + akk; }
};
template <> struct Mfma<float> {
  typedef f4 acc;
  static __device__ __forceinline__ f4 op(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // accumulator element r of lane l: tile row 4(l/16) + r, column l%16
  static __device__ __forceinline__ int row(int r, int akk) { return 4 * akk + r; }
};

constexpr int kChunk = 1024;  // columns of one source-row table (4 KB of LDS per wave)

// One form: NTW vector tiles per wave; NF full 16-row tiles and, FP64 only,
// TQ four-row tails (one v_mfma_f64_4x4x4_4b each) of the row; U four-column
// steps per load group; W waves per SIMD that the register budget must allow.
//
// What bounds it: at 16 vectors the bytes (the matrix streams once, each
// block's input segment is gathered again), at 64 the FP64 matrix cores.
// So: every load of group g + 1 is issued before the MFMAs of group g (the
// kernel before this one drained its loads first, half the time with nothing
// in flight); the matrix is read at a scalar base plus per-row constant lane
// offsets and a step's input row comes from a table in LDS, so that a step
// costs one address computation and no block search; and the accumulators
// stay in VGPRs (W >= 2: with the whole register file the compiler puts them
// in AGPRs and moves all eight registers of a tile around every MFMA).
//
// A rows: lane l's pair of tiles (2i, 2i + 1) are rows 32i + 2 (l%16) + {0, 1}
// of M, one 16-byte load per step (32 rows of a column are 256 contiguous
// bytes); a last single tile is rows 16t + l%16.  B columns: lane l's tiles j
// are vectors NTW (l%16) + j of its wave's range (NTW 2 or 4: 16-byte loads).
// Which tile holds a row or a vector does not change any output's sum:
// four-column steps in column order, as in every other row kernel, so the
// results are bitwise theirs.
// Measured on the 2D operator of 2^20 points (rank 36, 517 772 coupling
// blocks), against the best kernel before: coupling launch 1.13 -> 1.08 ms at
// 16 vectors, 2.62 -> 1.83 ms (47 TF) at 64; half of the dense rows 1.19 ->
// 0.87 ms (52 TF) at 64; whole products 2.96 -> 2.85 and 6.94 -> 5.36 ms (2.80
// and 5.12 with the composed sweeps and the later output permutation).
// Lanes of rows past m and of columns past ncols read whatever follows (the
// arrays end in kRowSlack bytes of slack): the former's outputs are not
// stored, the latter's operands are zeroed.
// FL: M read from the row's fragment-ordered copy (see k_rows_to_fl): tile t
// is rows 16t + l%16, two steps per 16-byte load.
// WHOLE: every row of the launch has matrix rows in every tile, and every group
// issues the same number of loads, so that the waits before a group's MFMAs
// count past the next group's loads.  In launches of mixed rows the loads of a
// row's empty tiles are skipped (cheaper than loading them, though the waits
// then count the fewer).
// KS: a workgroup per row and vector range, the row's columns in four equal
// pieces, one per wave, the partial sums added through LDS in wave order, one
// vector tile at a time (32 KB at most, over the source-row tables): the
// composed sweep rows and the dense rows of operators of few leaves, where one
// wave's chain of loads is what the launch waits for.  Dense rows of a 3D
// operator of 131 072 points at 64 vectors: 0.73 -> 0.60 ms per half.
template <typename T, int NT, int NTW, int NF, int TQ, int U, int W, bool FL, bool WHOLE, bool KS = false>
__global__ __launch_bounds__(kT, W) void k_wave_rows(const RowDesc* __restrict__ rows, int64_t nrows,
                                                     const int32_t* __restrict__ colend,
                                                     const int64_t* __restrict__ in_off,
                                                     const T* __restrict__ data, const double* in, double* out,
                                                     int mode, int remap) {
  typedef typename Mfma<T>::acc CT;
  typedef T t2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));  // any element offset
  typedef double v2 __attribute__((ext_vector_type(2)));
  constexpr int NVP = 16 * NT, WPR = NT / NTW, RPW = KS ? 1 : 4 / WPR;
  constexpr int G = 4 * U;           // columns per load group
  constexpr int NA = NF + TQ;        // A values per step
  constexpr bool BV = NTW % 2 == 0;  // tiles j: vectors NTW * arow + j, else 16 j + arow
  constexpr int ES = sizeof(T);
  typedef const __attribute__((address_space(1))) char* gptr;
  static_assert((U == 2 || U % 4 == 0) && kChunk % G == 0, "load groups");
  // source rows of a chunk's columns; a lane's U steps of a group adjacent,
  // and two groups of padding for the reads ahead.  KS: afterwards the four
  // waves' partial sums of one vector tile
  constexpr int SRC = kChunk + 2 * G, PART = KS ? 4 * (16 * NF + 4 * TQ) * 16 * 2 : 0;
  __shared__ __align__(16) uint32_t s_mem[4 * SRC > PART ? 4 * SRC : PART];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = KS ? 0 : wave / WPR, vt0 = KS ? (int)(blockIdx.x % WPR) * NTW : (wave % WPR) * NTW;
  const int arow = lane & 15, akk = lane >> 4;
  const int vcol = 16 * vt0 + (BV ? NTW * arow : arow);  // first vector of the lane
  uint32_t* src = s_mem + wave * SRC;
  const double* inl = in + vcol;
  // rows by workgroup: grid-stride, or (remap; a grid of a multiple of 8)
  // each XCD (workgroups b with the same b % 8) takes one contiguous eighth
  // of the rows, so that rows in flight together on an XCD are neighbours in
  // the row order and their shared input segments meet in that XCD's L2
  const int64_t per = remap ? (nrows + 7) / 8 : nrows;
  const int64_t base = remap ? (int64_t)(blockIdx.x % 8) * per : 0;
  // (KS: the vector ranges of a row in neighbouring workgroups; remap only with one range)
  const int64_t wg = remap ? blockIdx.x / 8 : KS ? blockIdx.x / WPR : blockIdx.x;
  const int64_t nwg = remap ? gridDim.x / 8 : KS ? gridDim.x / WPR : gridDim.x;
  for (int64_t jr = wg * RPW + slot; jr < per; jr += nwg * RPW) {
    const int64_t ri = base + jr;
    if (ri >= nrows) break;
    const RowDesc R = rows[ri];
    const int m = R.nrows;
    if (m <= 0) continue;
    const int allcols = R.blk_end > R.blk_begin ? colend[R.blk_end - 1] : 0;
    const int piece = KS ? ((allcols + 3) / 4 + G - 1) / G * G : 0;  // columns per wave
    const int cbeg = KS ? min(wave * piece, allcols) : 0;
    const int ncols = KS ? min(cbeg + piece, allcols) : allcols;
    CT acc[NF][NTW];
    T acc4[TQ > 0 ? TQ : 1][NTW];
#pragma unroll
    for (int t = 0; t < NF; ++t)
#pragma unroll
      for (int j = 0; j < NTW; ++j) acc[t][j] = CT{0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < (TQ > 0 ? TQ : 1); ++t)
#pragma unroll
      for (int j = 0; j < NTW; ++j) acc4[t][j] = (T)0;
    const int nt = min(FL ? (m + 15) >> 4 : (m + 31) / 32 * 2, NF);  // tiles that hold rows of this row's matrix
    const bool tq = TQ > 0 && m > 16 * NF;
    // the lane's byte offset of each A value from the step's (FL: the pair of
    // steps') first element
    uint32_t voff[NA];
    if constexpr (FL) {
      const int nfullt = m >> 4, rem = m & 15;
#pragma unroll
      for (int t = 0; t < NF; ++t)
        voff[t] = (t < nfullt ? 128 * t + 2 * lane : 128 * nfullt + 2 * (akk * rem + arow)) * ES;
#pragma unroll
      for (int t = 0; t < TQ; ++t) voff[NF + t] = (128 * NF + 2 * (akk * rem + 4 * t + (arow & 3))) * ES;
    } else {
#pragma unroll
      for (int t = 0; t < NF; ++t)
        voff[t] = (akk * m + (t == NF - 1 && NF % 2 == 1 ? 16 * t + arow : 32 * (t / 2) + 2 * arow + (t & 1))) * ES;
#pragma unroll
      for (int t = 0; t < TQ; ++t) voff[NF + t] = (akk * m + 16 * NF + (TQ == 1 ? arow & 3 : 2 * (arow & 3) + t)) * ES;
    }
    gptr sbase = (gptr)(data + (FL ? R.fl_off : R.data_off) + (int64_t)m * cbeg);
    const int64_t sstep = (int64_t)4 * m * ES;  // bytes of one step

    T a[U][NA], a2[U][NA];
    double b[U][NTW], b2[U][NTW];
    uint32_t idx[U];
    auto index = [&](int g) __attribute__((always_inline)) {  // source rows of group g
      if constexpr (U % 4 == 0) {
#pragma unroll
        for (int u = 0; u < U; u += 4) {
          const uint4 v = *reinterpret_cast<const uint4*>(src + G * g + U * akk + u);
          idx[u] = v.x, idx[u + 1] = v.y, idx[u + 2] = v.z, idx[u + 3] = v.w;
        }
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(src + G * g + 2 * akk);
        idx[0] = v.x, idx[1] = v.y;
      }
    };
    // the next group's operands: the matrix at sbase, which moves on, the
    // inputs at the source rows of `idx`
    auto load = [&](T(&x)[U][NA], double(&y)[U][NTW]) __attribute__((always_inline)) {
      asm volatile("" : "+s"(sbase));  // keeps the base scalar: lane offsets stay 32-bit constants of the row
#pragma unroll
      for (int t = 0; t < NA; ++t) {
        if (!WHOLE && (t < NF ? (t > 0 && t >= nt) : !tq)) continue;  // wave-uniform
        if constexpr (FL) {
#pragma unroll
          for (int u = 0; u < U; u += 2) {
            const t2 v = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) t2*>(sbase + u * sstep + voff[t]));
            x[u][t] = v[0];
            x[u + 1][t] = v[1];
          }
        } else {
          // adjacent rows in tiles t, t + 1: one load for both
          const bool paired = t < NF ? t < NF / 2 * 2 : TQ == 2;
          const bool second = paired && ((t < NF ? t : t - NF) & 1);
          if (second) continue;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const gptr p = sbase + u * sstep + voff[t];
            if (paired) {
              const t2 v = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) t2*>(p));
              x[u][t] = v[0];
              x[u][t + 1 < NA ? t + 1 : t] = v[1];
            } else {
              x[u][t] = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) T*>(p));
            }
          }
        }
      }
      sbase += U * sstep;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const double* s = inl + (uint64_t)idx[u] * NVP;
        if constexpr (BV) {
#pragma unroll
          for (int j = 0; j < NTW; j += 2) {
            const v2 v = *reinterpret_cast<const v2*>(s + j);
            y[u][j] = v[0];
            y[u][j + 1] = v[1];
          }
        } else {
#pragma unroll
          for (int j = 0; j < NTW; ++j) y[u][j] = s[16 * j];
        }
      }
    };
    auto compute = [&](T(&x)[U][NA], double(&y)[U][NTW], int steps) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < NF; ++t) {
        if (!WHOLE && t > 0 && t >= nt) continue;  // wave-uniform
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (u < steps)
#pragma unroll
            for (int j = 0; j < NTW; ++j) acc[t][j] = Mfma<T>::op(x[u][t], (T)y[u][j], acc[t][j]);
      }
      if constexpr (TQ > 0) {
        if (WHOLE || tq)
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u < steps)
#pragma unroll
              for (int t = 0; t < TQ; ++t)
#pragma unroll
                for (int j = 0; j < NTW; ++j)
                  acc4[t][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(x[u][NF + t], y[u][j], acc4[t][j], 0, 0, 0);
      }
    };

    int bcur = R.blk_begin, bstart = 0;  // block of the chunk's first column and its first column
    for (int c0 = cbeg; c0 < ncols; c0 += kChunk) {
      const int cn = min(kChunk, ncols - c0);
      // source row of each column of the chunk: 64 blocks' table entries
      // loaded by the lanes, then one block at a time written by the wave
      auto put_src = [&](int c, uint32_t v) __attribute__((always_inline)) {
        src[c / G * G + (c & 3) * U + (c % G >> 2)] = v;
      };
      __builtin_amdgcn_wave_barrier();  // the previous chunk's table fully read
      uint32_t last = 0;
      for (bool more = true; more;) {
        const int bl = bcur + lane;
        const int e = bl < R.blk_end ? colend[bl] : 0;
        const uint32_t o = bl < R.blk_end ? (uint32_t)in_off[bl] : 0u;
        const int nbat = min(64, R.blk_end - bcur);
        int i = 0;
        for (; i < nbat; ++i) {
          const int ei = __builtin_amdgcn_readlane(e, i);
          const uint32_t oi = (uint32_t)__builtin_amdgcn_readlane((int)o, i);
          const int ce = min(ei, c0 + cn);
          for (int c = max(bstart, c0) + lane; c < ce; c += 64) put_src(c - c0, oi + (uint32_t)(c - bstart));
          if (ce > bstart) last = oi + (uint32_t)(ce - 1 - bstart);
          if (ei >= c0 + cn) {  // the chunk is covered; a block that reaches past it starts the next
            if (ei == c0 + cn) {
              ++i;
              bstart = ei;
            }
            more = false;
            break;
          }
          bstart = ei;
        }
        bcur += i;
        if (bcur >= R.blk_end) more = false;
      }
      // columns past the chunk: its last source row, up to two whole groups on
      for (int c = cn + lane; c < (cn + G - 1) / G * G + 2 * G; c += 64) put_src(c, last);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

      const int lastg = (cn - 1) / G;
      index(0);
      load(a, b);
      index(1);
      int g = 0;
      for (; g + 1 < lastg; g += 2) {
        load(a2, b2);
        index(g + 2);
        __builtin_amdgcn_sched_barrier(0);
        compute(a, b, U);
        __builtin_amdgcn_sched_barrier(0);
        load(a, b);
        index(g + 3);
        __builtin_amdgcn_sched_barrier(0);
        compute(a2, b2, U);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (g < lastg) {
        load(a2, b2);
        __builtin_amdgcn_sched_barrier(0);
        compute(a, b, U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
          for (int t = 0; t < NA; ++t) a[u][t] = a2[u][t];
#pragma unroll
          for (int j = 0; j < NTW; ++j) b[u][j] = b2[u][j];
        }
      }
      // the last group: operands past the row's last column zeroed
      const int tail = cn - lastg * G;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (4 * u + akk >= tail) {
#pragma unroll
          for (int t = 0; t < NA; ++t) a[u][t] = (T)0;
#pragma unroll
          for (int j = 0; j < NTW; ++j) b[u][j] = 0.0;
        }
      compute(a, b, (tail + 3) >> 2);
      // the next chunk's matrix starts after this one's columns
      sbase = (gptr)(data + (FL ? R.fl_off : R.data_off)) + (int64_t)m * ES * (c0 + kChunk);
    }

    // matrix row of accumulator element r of tile t, and of tail t
    auto row_of = [&](int t, int r) __attribute__((always_inline)) {
      const int i = Mfma<T>::row(r, akk);
      return FL || (t == NF - 1 && NF % 2 == 1) ? 16 * t + i : 32 * (t / 2) + 2 * i + (t & 1);
    };
    auto row_of_tail = [&](int t) __attribute__((always_inline)) {
      return 16 * NF + (FL || TQ == 1 ? 4 * t + akk : 2 * akk + t);
    };
    if constexpr (KS) {
      // one vector tile after the other through LDS
      double* part = reinterpret_cast<double*>(s_mem);
#pragma unroll
      for (int j = 0; j < NTW; ++j) {
        __syncthreads();  // the source rows, or the tile before this one, are read
#pragma unroll
        for (int t = 0; t < NF; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = row_of(t, r);
            if (row < m) part[(wave * m + row) * 16 + arow] = acc[t][j][r];
          }
        if constexpr (TQ > 0) {
#pragma unroll
          for (int t = 0; t < TQ; ++t) {
            const int row = row_of_tail(t);
            if (row < m) part[(wave * m + row) * 16 + arow] = acc4[t][j];
          }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 16 * m; e += kT) {
          double sum = part[e];
#pragma unroll
          for (int w = 1; w < 4; ++w) sum += part[16 * w * m + e];
          const int v = e & 15;
          double* o = out + (R.out_off + (e >> 4)) * NVP + 16 * vt0 + (BV ? NTW * v + j : 16 * j + v);
          *o = mode == MODE_STORE ? sum : *o + sum;
        }
      }
      __syncthreads();
      continue;
    }
    // stores: vectors vcol + j (NTW even) or vcol + 16 j of the tile's rows
    auto put = [&](int row, auto val) __attribute__((always_inline)) {
      if (row >= m) return;
      double* o = out + (R.out_off + row) * NVP + vcol;
      if constexpr (BV) {
#pragma unroll
        for (int j = 0; j < NTW; j += 2) {
          v2 v = {val(j), val(j + 1)};
          v2* p = reinterpret_cast<v2*>(o + j);
          if (mode != MODE_STORE) v += *p;
          *p = v;
        }
      } else {
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
          if (mode == MODE_STORE) o[16 * j] = val(j);
          else o[16 * j] += val(j);
        }
      }
    };
#pragma unroll
    for (int t = 0; t < NF; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) put(row_of(t, r), [&](int j) { return (double)acc[t][j][r]; });
    if constexpr (TQ > 0) {
#pragma unroll
      for (int t = 0; t < TQ; ++t) put(row_of_tail(t), [&](int j) { return acc4[t][j]; });
    }
  }
}

// Transposed row list (op 'T', FP64): out (ms x 16NT) = sum over the blocks of
// a block column of M_b^T (ms x mr_b) x_b, M_b stored column-major mr_b x ms.
// The same wave-per-row product as k_wave_rows with A[i][k] = M_b[k, i]: a
// load group is 4U rows of one block, lane l holding rows U (l/16) .. + U - 1
// of output column l%16 (16-byte loads, 32U contiguous bytes of a column), in
// a block's last group the operands past its rows zeroed.  Every group issues
// the same number of loads, so that the waits before a group's MFMAs count
// past the next group's loads.  Input rows of a block are consecutive, so no
// source-row table is needed.
// Bound by the bytes, as the streaming of the same blocks untransposed: one
// pass over the matrix for up to 64 vectors, where passes of four vectors
// through LDS read it once per four.  Measured on the 2D operator of 100 003
// points (leaf 50, rank 25) at 24 vectors: product 3.80 -> 0.53-0.57 ms.  At 32
// to 64 vectors a group is eight rows, 64 bytes of a column: half of each line
// is fetched again (3.5 GB counted for 0.85).
// KS: a workgroup per row and vector range, its blocks dealt to the four waves
// in turn and their partial sums added through LDS in wave order: for launches
// of too few rows to give every SIMD four waves, where a row's chain of loads
// is what the launch waits for.
template <int NT, int NTW, int NF, int TQ, int U, int W, bool KS>
__global__ __launch_bounds__(kT, W) void k_wave_cols(const RowDesc* __restrict__ rows, int64_t nrows,
                                                     const int64_t* __restrict__ bdata,
                                                     const int32_t* __restrict__ bmr,
                                                     const int64_t* __restrict__ bin,
                                                     const double* __restrict__ data, const double* in,
                                                     double* out) {
  typedef double t2 __attribute__((ext_vector_type(2), aligned(8)));
  typedef double v2 __attribute__((ext_vector_type(2)));
  typedef const __attribute__((address_space(1))) char* gptr;
  constexpr int NVP = 16 * NT, WPR = NT / NTW, RPW = 4 / WPR, G = 4 * U, NA = NF + TQ;
  constexpr bool BV = NTW % 2 == 0;
  constexpr int LDP = 16 * NTW;  // LDS row of the partial sums
  __shared__ __align__(16) double part[KS ? 4 * (16 * NF + 4 * TQ) * LDP : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = wave / WPR, vt0 = KS ? (int)(blockIdx.x % WPR) * NTW : (wave % WPR) * NTW;
  const int arow = lane & 15, akk = lane >> 4;
  const int vcol = 16 * vt0 + (BV ? NTW * arow : arow);
  const double* inl = in + vcol;
  const int64_t ri = KS ? blockIdx.x / WPR : (int64_t)blockIdx.x * RPW + slot;
  if (ri >= nrows) return;
  const RowDesc R = rows[ri];
  constexpr int STEP = KS ? 4 : 1;  // blocks from one of this wave's to the next
  const int ms = R.nrows;
  if (ms <= 0) return;
  d4 acc[NF][NTW];
  double acc4[TQ > 0 ? TQ : 1][NTW];
#pragma unroll
  for (int t = 0; t < NF; ++t)
#pragma unroll
    for (int j = 0; j < NTW; ++j) acc[t][j] = d4{0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < (TQ > 0 ? TQ : 1); ++t)
#pragma unroll
    for (int j = 0; j < NTW; ++j) acc4[t][j] = 0.0;
  // output column of each A value (past ms: the last one; not stored)
  int col[NA];
#pragma unroll
  for (int t = 0; t < NA; ++t) col[t] = min(t < NF ? 16 * t + arow : 16 * NF + 4 * (t - NF) + (arow & 3), ms - 1);
  const int nt = min((ms + 15) >> 4, NF);
  const bool tq = TQ > 0 && ms > 16 * NF;

  double a[U][NA], a2[U][NA], b[U][NTW], b2[U][NTW];
  int rem = 0, rem2 = 0;  // rows of the block in each buffer's group (G: a whole group)
  // the block that the next load reads, and the table entries of the one after it
  int blk = R.blk_begin + (KS ? wave : 0), k0 = 0;
  int mr = 0, mrn = 0;
  int64_t bd = 0, bi = 0, bdn = 0, bin_n = 0;
  auto peek = [&](int i) __attribute__((always_inline)) {
    if (i < R.blk_end) {
      mrn = bmr[i];
      bdn = bdata[i];
      bin_n = bin[i];
    }
  };
  auto advance = [&]() __attribute__((always_inline)) {  // to the next block with rows
    for (;;) {
      mr = mrn;
      bd = bdn;
      bi = bin_n;
      k0 = 0;
      peek(blk + STEP);
      if (blk >= R.blk_end || mr > 0) break;
      blk += STEP;
    }
  };
  auto load = [&](double(&x)[U][NA], double(&y)[U][NTW], int& left) __attribute__((always_inline)) -> bool {
    if (blk >= R.blk_end) return false;
    left = min(mr - k0, G);
    const gptr base = (gptr)(data + bd + k0);
    const double* src = inl + (bi + k0) * NVP;
    const int kl = min(U * akk, left - 1);  // the lane's first row, or the last one left
#pragma unroll
    for (int t = 0; t < NA; ++t) {
      const uint32_t off = (uint32_t)(kl + mr * col[t]) * 8u;
#pragma unroll
      for (int u = 0; u < U; u += 2) {
        const t2 v = __builtin_nontemporal_load(
            reinterpret_cast<const __attribute__((address_space(1))) t2*>(base + off + 8 * u));
        x[u][t] = v[0];
        x[u + 1][t] = v[1];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double* sv = src + min(kl + u, left - 1) * NVP;
      if constexpr (BV) {
#pragma unroll
        for (int j = 0; j < NTW; j += 2) {
          const v2 v = *reinterpret_cast<const v2*>(sv + j);
          y[u][j] = v[0];
          y[u][j + 1] = v[1];
        }
      } else {
#pragma unroll
        for (int j = 0; j < NTW; ++j) y[u][j] = sv[16 * j];
      }
    }
    k0 += G;
    if (k0 >= mr) {
      blk += STEP;
      advance();
    }
    return true;
  };
  auto compute = [&](double(&x)[U][NA], double(&y)[U][NTW], int left) __attribute__((always_inline)) {
    if (left < G) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (U * akk + u >= left) {
#pragma unroll
          for (int t = 0; t < NA; ++t) x[u][t] = 0.0;
#pragma unroll
          for (int j = 0; j < NTW; ++j) y[u][j] = 0.0;
        }
    }
#pragma unroll
    for (int t = 0; t < NF; ++t) {
      if (t > 0 && t >= nt) continue;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u < left)
#pragma unroll
          for (int j = 0; j < NTW; ++j) acc[t][j] = Mfma<double>::op(x[u][t], y[u][j], acc[t][j]);
    }
    if constexpr (TQ > 0) {
      if (tq)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (u < left)
#pragma unroll
            for (int t = 0; t < TQ; ++t)
#pragma unroll
              for (int j = 0; j < NTW; ++j)
                acc4[t][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(x[u][NF + t], y[u][j], acc4[t][j], 0, 0, 0);
    }
  };
  peek(blk);
  advance();
  bool has = load(a, b, rem);
  while (has) {
    const bool has2 = load(a2, b2, rem2);
    __builtin_amdgcn_sched_barrier(0);
    compute(a, b, rem);
    __builtin_amdgcn_sched_barrier(0);
    if (!has2) break;
    has = load(a, b, rem);
    __builtin_amdgcn_sched_barrier(0);
    compute(a2, b2, rem2);
    __builtin_amdgcn_sched_barrier(0);
  }
  auto put = [&](int row, auto val) __attribute__((always_inline)) {
    if (row >= ms) return;
    double* o = KS ? part + (wave * ms + row) * LDP + vcol - 16 * vt0 : out + (R.out_off + row) * NVP + vcol;
    if constexpr (BV) {
#pragma unroll
      for (int j = 0; j < NTW; j += 2) *reinterpret_cast<v2*>(o + j) = v2{val(j), val(j + 1)};
    } else {
#pragma unroll
      for (int j = 0; j < NTW; ++j) o[16 * j] = val(j);
    }
  };
#pragma unroll
  for (int t = 0; t < NF; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) put(16 * t + 4 * r + akk, [&](int j) { return acc[t][j][r]; });
  if constexpr (TQ > 0) {
#pragma unroll
    for (int t = 0; t < TQ; ++t) put(16 * NF + 4 * t + akk, [&](int j) { return acc4[t][j]; });
  }
  if constexpr (KS) {
    __syncthreads();
    for (int e = threadIdx.x; e < ms * 16 * NTW; e += kT) {
      const int row = e / (16 * NTW), v = e % (16 * NTW);
      double sum = part[row * LDP + v];
#pragma unroll
      for (int w = 1; w < 4; ++w) sum += part[(w * ms + row) * LDP + v];
      out[(R.out_off + row) * NVP + 16 * vt0 + v] = sum;
    }
  }
}

// Registers of a form (32-bit), and from them the waves per SIMD it is
// compiled for: 512 / W registers each, W >= 2 so that the accumulators stay
// in VGPRs.
constexpr int form_regs(int tb, int ntw, int nf, int tq, int u) {
  return (nf * 4 + tq) * ntw * tb / 4 + 2 * u * ((nf + tq) * tb / 4 + 2 * ntw) + u + 30;
}
constexpr int form_waves(int r) { return r <= 96 ? 5 : r <= 128 ? 4 : r <= 168 ? 3 : 2; }

// Workgroups of a wave-row launch of rpw rows per workgroup pass: enough
// for every row at once, or `grid`; with the XCD remap a multiple of 8
// covering eight equal row ranges.
inline int64_t wave_grid(int64_t nrows, int rpw, int64_t grid, int remap) {
  if (!remap) {
    const int64_t need = (nrows + rpw - 1) / rpw;
    return grid > 0 && grid < need ? grid : need;
  }
  const int64_t per = (nrows + 7) / 8, needx = (per + rpw - 1) / rpw;
  return grid > 0 ? std::min<int64_t>((grid + 7) / 8 * 8, 8 * needx) : 8 * needx;
}

template <typename T>
struct Args {
  const RowDesc* rows;
  int64_t nrows;
  const int32_t* colend;
  const int64_t* in_off;
  const T *data, *fl;
  const double* in;
  double* out;
  int mode, remap, min_rows;
  int64_t grid;
  hipStream_t s;
};

template <typename T, int NT, int NTW, int NF, int TQ, int U>
void launch_form(const Args<T>& A) {
  constexpr int W = form_waves(form_regs((int)sizeof(T), NTW, NF, TQ, U));
  const dim3 g((unsigned)wave_grid(A.nrows, 4 * NTW / NT, A.grid, A.remap)), b(kT);
  // the shortest row fills every tile (pairs of tiles hold interleaved rows)
  const bool whole = std::min((A.min_rows + 31) / 32 * 2, NF) == NF && (TQ == 0 || A.min_rows > 16 * NF);
  if (A.fl && whole && A.min_rows > 16 * (NF - 1))
    hipLaunchKernelGGL((k_wave_rows<T, NT, NTW, NF, TQ, U, W, true, true>), g, b, 0, A.s, A.rows, A.nrows, A.colend,
                       A.in_off, A.fl, A.in, A.out, A.mode, A.remap);
  else if (whole)
    hipLaunchKernelGGL((k_wave_rows<T, NT, NTW, NF, TQ, U, W, false, true>), g, b, 0, A.s, A.rows, A.nrows, A.colend,
                       A.in_off, A.data, A.in, A.out, A.mode, A.remap);
  else
    hipLaunchKernelGGL((k_wave_rows<T, NT, NTW, NF, TQ, U, W, false, false>), g, b, 0, A.s, A.rows, A.nrows,
                       A.colend, A.in_off, A.data, A.in, A.out, A.mode, A.remap);
}

// Row tiles by the longest row of the launch: full 16-row tiles, and for
// FP64 one or two four-row tails where at most eight rows are left over (two
// cost 36 cycles a step, a 16-row tile 64).
template <typename T, int NT, int NTW, int U>
void launch_rows_of(const Args<T>& A, int max_rows) {
  const int nf = max_rows >> 4, rem = max_rows & 15;
  if constexpr (sizeof(T) == 8) {
    if (nf >= 1 && nf <= 3 && rem >= 1 && rem <= 8) {
      if (nf == 1) return rem <= 4 ? launch_form<T, NT, NTW, 1, 1, U>(A) : launch_form<T, NT, NTW, 1, 2, U>(A);
      if (nf == 2) return rem <= 4 ? launch_form<T, NT, NTW, 2, 1, U>(A) : launch_form<T, NT, NTW, 2, 2, U>(A);
      return rem <= 4 ? launch_form<T, NT, NTW, 3, 1, U>(A) : launch_form<T, NT, NTW, 3, 2, U>(A);
    }
  }
  switch (nf + (rem > 0 ? 1 : 0)) {
    case 0:
    case 1: return launch_form<T, NT, NTW, 1, 0, U>(A);
    case 2: return launch_form<T, NT, NTW, 2, 0, U>(A);
    case 3: return launch_form<T, NT, NTW, 3, 0, U>(A);
    default: return launch_form<T, NT, NTW, 4, 0, U>(A);
  }
}

// Waves (rows times vector ranges) below which a block column is split over
// the four waves of a workgroup.
constexpr int64_t kColsSplit = 8192;

struct SplitArgs {
  const RowDesc* rows;
  int64_t nrows;
  const int32_t* colend;
  const int64_t* in_off;
  const double *data, *in;
  double* out;
  int mode, min_rows, remap;
  int64_t grid;
  hipStream_t s;
};

template <int NT, int NTW, int NF, int TQ, int U>
void launch_split_form(const SplitArgs& A) {
  constexpr int W = form_waves(form_regs(8, NTW, NF, TQ, U));
  const dim3 g((unsigned)(wave_grid(A.nrows, 1, A.grid, A.remap) * (NT / NTW))), b(kT);
  const bool whole = std::min((A.min_rows + 31) / 32 * 2, NF) == NF && (TQ == 0 || A.min_rows > 16 * NF);
  if (whole)
    hipLaunchKernelGGL((k_wave_rows<double, NT, NTW, NF, TQ, U, W, false, true, true>), g, b, 0, A.s, A.rows, A.nrows,
                       A.colend, A.in_off, A.data, A.in, A.out, A.mode, A.remap);
  else
    hipLaunchKernelGGL((k_wave_rows<double, NT, NTW, NF, TQ, U, W, false, false, true>), g, b, 0, A.s, A.rows,
                       A.nrows, A.colend, A.in_off, A.data, A.in, A.out, A.mode, A.remap);
}

template <int NT, int NTW, int U>
void launch_split_of(const SplitArgs& A, int max_rows) {
  const int nf = max_rows >> 4, rem = max_rows & 15;
  if (nf == 2 && rem >= 1 && rem <= 4) return launch_split_form<NT, NTW, 2, 1, U>(A);
  if (nf == 3 && rem >= 1 && rem <= 4) return launch_split_form<NT, NTW, 3, 1, U>(A);
  switch (nf + (rem > 0 ? 1 : 0)) {
    case 0:
    case 1: return launch_split_form<NT, NTW, 1, 0, U>(A);
    case 2: return launch_split_form<NT, NTW, 2, 0, U>(A);
    case 3: return launch_split_form<NT, NTW, 3, 0, U>(A);
    default: return launch_split_form<NT, NTW, 4, 0, U>(A);
  }
}

struct ColArgs {
  const RowDesc* rows;
  int64_t nrows;
  const int64_t* bdata;
  const int32_t* bmr;
  const int64_t* bin;
  const double *data, *in;
  double* out;
  hipStream_t s;
};

template <int NT, int NTW, int NF, int TQ, int U>
void launch_cols_form(const ColArgs& A) {
  constexpr int W = form_waves(form_regs(8, NTW, NF, TQ, U) + 10);
  constexpr int RPW = 4 * NTW / NT;
  if (A.nrows * (NT / NTW) < kColsSplit)
    hipLaunchKernelGGL((k_wave_cols<NT, NTW, NF, TQ, U, W, true>), dim3((unsigned)(A.nrows * (NT / NTW))), dim3(kT),
                       0, A.s, A.rows, A.nrows, A.bdata, A.bmr, A.bin, A.data, A.in, A.out);
  else
    hipLaunchKernelGGL((k_wave_cols<NT, NTW, NF, TQ, U, W, false>), dim3((unsigned)((A.nrows + RPW - 1) / RPW)),
                       dim3(kT), 0, A.s, A.rows, A.nrows, A.bdata, A.bmr, A.bin, A.data, A.in, A.out);
}

template <int NT, int NTW, int U>
void launch_cols_of(const ColArgs& A, int max_rows) {
  const int nf = max_rows >> 4, rem = max_rows & 15;
  if (nf >= 1 && nf <= 3 && rem >= 1 && rem <= 8) {
    if (nf == 1) return rem <= 4 ? launch_cols_form<NT, NTW, 1, 1, U>(A) : launch_cols_form<NT, NTW, 1, 2, U>(A);
    if (nf == 2) return rem <= 4 ? launch_cols_form<NT, NTW, 2, 1, U>(A) : launch_cols_form<NT, NTW, 2, 2, U>(A);
    return rem <= 4 ? launch_cols_form<NT, NTW, 3, 1, U>(A) : launch_cols_form<NT, NTW, 3, 2, U>(A);
  }
  switch (nf + (rem > 0 ? 1 : 0)) {
    case 0:
    case 1: return launch_cols_form<NT, NTW, 1, 0, U>(A);
    case 2: return launch_cols_form<NT, NTW, 2, 0, U>(A);
    case 3: return launch_cols_form<NT, NTW, 3, 0, U>(A);
    default: return launch_cols_form<NT, NTW, 4, 0, U>(A);
  }
}

}  // namespace

// Two waves per row at 64 vectors: block columns are fewer and longer than
// four waves per SIMD need, and half the accumulators leave room for them.
hipError_t launch_wave_cols(const RowDesc* rows, int64_t nrows, const int64_t* bdata, const int32_t* bmr,
                            const int64_t* bin, const double* data, const double* in, double* out, int nvp,
                            int max_rows, hipStream_t s) {
  if (nrows == 0) return hipSuccess;
  if (max_rows > 64) return hipErrorInvalidValue;
  const ColArgs A{rows, nrows, bdata, bmr, bin, data, in, out, s};
  switch (nvp) {
    case 16: launch_cols_of<1, 1, 4>(A, max_rows); break;
    case 32: launch_cols_of<2, 2, 2>(A, max_rows); break;
    case 48: launch_cols_of<3, 3, 2>(A, max_rows); break;
    case 64: launch_cols_of<4, 2, 2>(A, max_rows); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_split_rows(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                             const double* data, const double* in, double* out, int nvp, int mode, int min_rows,
                             int max_rows, hipStream_t s, bool all, int64_t grid, int remap) {
  if (nrows == 0) return hipSuccess;
  if (max_rows > 64) return hipErrorInvalidValue;
  const SplitArgs A{rows, nrows, colend, in_off, data, in, out, mode, min_rows, all || nvp == 16 ? remap : 0, grid, s};
  // all: one workgroup for a row's whole vector range (the matrix read once),
  // else one per 16 vectors
  switch (nvp) {
    case 16: launch_split_of<1, 1, 4>(A, max_rows); break;
    case 32: all ? launch_split_of<2, 2, 4>(A, max_rows) : launch_split_of<2, 1, 4>(A, max_rows); break;
    case 48: all ? launch_split_of<3, 3, 2>(A, max_rows) : launch_split_of<3, 1, 4>(A, max_rows); break;
    case 64: all ? launch_split_of<4, 4, 2>(A, max_rows) : launch_split_of<4, 1, 4>(A, max_rows); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

RowForm auto_form(int nvp, int64_t rows, int max_rows) {
  if (max_rows > 64) return {64, 0};
  if (nvp == 16) return {kWaveRows, rows >= 8192 ? 5 : 0};
  if (nvp == 48) return {kWaveRows, 0};
  if (rows < 400) return {kWaveTiles, 0};
  return {kWaveRows, nvp == 64 && rows < 1200 ? 5 : 0};
}

template <typename T>
hipError_t launch_wave_rows(const RowDesc* rows, int64_t nrows, const int32_t* colend, const int64_t* in_off,
                            const T* data, const double* in, double* out, int nvp, int mode, int min_rows,
                            int max_rows, hipStream_t s, int64_t grid, bool narrow, int remap, const T* fl, int occ) {
  if (nrows == 0) return hipSuccess;
  if (max_rows > 64) return hipErrorInvalidValue;
  const Args<T> A{rows, nrows, colend, in_off, data, fl, in, out, mode, remap, min_rows, grid, s};
  // narrow: a wave per 16-vector tile.  Otherwise a wave per row, or (occ) two
  // waves per row at 64 vectors and half the columns per load group at 16 and
  // 32: fewer registers, more waves.
  switch (nvp) {
    case 16: occ && !narrow ? launch_rows_of<T, 1, 1, 2>(A, max_rows) : launch_rows_of<T, 1, 1, 4>(A, max_rows); break;
    case 32:
      if (narrow) launch_rows_of<T, 2, 1, 4>(A, max_rows);
      else occ ? launch_rows_of<T, 2, 2, 2>(A, max_rows) : launch_rows_of<T, 2, 2, 4>(A, max_rows);
      break;
    case 48: launch_rows_of<T, 3, 3, 2>(A, max_rows); break;
    case 64:
      if (narrow) launch_rows_of<T, 4, 1, 4>(A, max_rows);
      else occ ? launch_rows_of<T, 4, 2, 2>(A, max_rows) : launch_rows_of<T, 4, 4, 2>(A, max_rows);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template hipError_t launch_wave_rows<double>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const double*,
                                             const double*, double*, int, int, int, int, hipStream_t, int64_t, bool,
                                             int, const double*, int);
template hipError_t launch_wave_rows<float>(const RowDesc*, int64_t, const int32_t*, const int64_t*, const float*,
                                            const double*, double*, int, int, int, int, hipStream_t, int64_t, bool,
                                            int, const float*, int);

}  // namespace h2
