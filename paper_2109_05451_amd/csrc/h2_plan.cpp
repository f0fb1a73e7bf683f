// Launch-plan construction shared by the single-operator handle and the
// multi-operator batch: the per-operator layout (vector-tree offsets,
// section offsets, transposed basis copies) and the rows of every op-'N'
// phase, each row a block row whose stored blocks are contiguous.
//
// The paper marshals, per call and per level, pointer arrays for batched
// kernels (Algorithm 3, Section 3.1).  The structure is static, so here the
// same information is produced once, at load time, as row lists.
#include <algorithm>
#include <vector>

#include "h2_internal.h"

namespace h2 {

int make_layout(const Parsed& P, OpLayout* L) {
  const int64_t q = P.q, n = P.n;
  const int64_t* lp = P.level_ptr;
  L->P = &P;
  L->shared = !(P.flags & 1u);
  L->kmax.assign(q + 1, 0);
  for (int64_t l = 0; l <= q; ++l) L->kmax[l] = std::max(P.krow[l], P.kcol[l]);
  const int64_t mat0 = P.off_U;
  L->oU = 0;
  L->oE = (P.off_E - mat0) / 8;
  L->oV = L->shared ? L->oU : (P.off_V - mat0) / 8;
  L->oF = L->shared ? L->oE : (P.off_F - mat0) / 8;
  L->oS = (P.off_S - mat0) / 8;
  L->oD = (P.off_D - mat0) / 8;
  L->nmat = (P.off_end - mat0) / 8;
  auto up32 = [](int64_t x) { return (x + 31) / 32 * 32; };
  const int64_t nU = n * P.krow[q], nE = P.ebase[q + 1], nV = n * P.kcol[q], nF = P.fbase[q + 1];
  L->tUT = 0;
  L->tET = up32(nU);
  L->tVT = L->shared ? L->tUT : up32(L->tET + nE);
  L->tFT = L->shared ? L->tET : up32(L->tVT + nV);
  L->ntrans = L->shared ? up32(L->tET + nE) : up32(L->tFT + nF);
  L->hoff.assign(P.nnodes, 0);
  int64_t H = 0;
  for (int64_t l = 0; l <= q; ++l)
    for (int64_t c = lp[l]; c < lp[l + 1]; ++c) {
      L->hoff[c] = H;
      H += L->kmax[l];
    }
  L->H = H;
  L->cbeg.assign(P.nnodes + 1, P.nnodes);
  int64_t next = 1;
  for (int64_t p = 0; p < P.nnodes; ++p) {
    L->cbeg[p] = next;
    while (next < P.nnodes && P.parent[next] == p) ++next;
    if (next - L->cbeg[p] > kMaxChildren) {
      set_error("h2 representation: node with more than 512 children");
      return H2_EUNSUPPORTED;
    }
  }
  L->cbeg[P.nnodes] = next;
  return H2_OK;
}

int64_t OpLayout::eoff(int64_t c, int64_t l) const {
  return P->ebase[l] + (c - P->level_ptr[l]) * P->krow[l] * P->krow[l - 1];
}
int64_t OpLayout::foff(int64_t c, int64_t l) const {
  return P->fbase[l] + (c - P->level_ptr[l]) * P->kcol[l] * P->kcol[l - 1];
}

void transpose_tasks(const OpLayout& L, std::vector<TransTask>* out) {
  const Parsed& P = *L.P;
  const int64_t q = P.q;
  out->clear();
  for (int pass = 0; pass < (L.shared ? 1 : 2); ++pass) {
    const int64_t* k = pass ? P.kcol : P.krow;
    const int64_t ob = pass ? L.oV : L.oU, ot = pass ? L.oF : L.oE;
    const int64_t tb = pass ? L.tVT : L.tUT, tt = pass ? L.tFT : L.tET;
    for (int64_t t = P.leaf0; t < P.nnodes; ++t) {  // leaf basis: m x k
      const int64_t m = P.hi[t] - P.lo[t], base = P.lo[t] * k[q];
      out->push_back({ob + base, tb + base, (int32_t)m, (int32_t)k[q]});
    }
    for (int64_t l = 1; l <= q; ++l)
      for (int64_t c = P.level_ptr[l]; c < P.level_ptr[l + 1]; ++c) {  // transfer: k[l] x k[l-1]
        const int64_t base = pass ? L.foff(c, l) : L.eoff(c, l);
        out->push_back({ot + base, tt + base, (int32_t)k[l], (int32_t)k[l - 1]});
      }
  }
}

void build_transposed(const uint8_t* buf, const OpLayout& L, double* tr) {
  std::fill(tr, tr + L.ntrans, 0.0);
  const double* M = reinterpret_cast<const double*>(buf + L.P->off_U);  // the matrix array
  std::vector<TransTask> tasks;
  transpose_tasks(L, &tasks);
  for (const TransTask& T : tasks)
    for (int64_t c = 0; c < T.cols; ++c)
      for (int64_t r = 0; r < T.rows; ++r) tr[T.dst + c + T.cols * r] = M[T.src + r + T.rows * c];
}

void emit_rows_N(const OpLayout& L, const RowBases& B, RowsN* R) {
  const Parsed& P = *L.P;
  const int64_t q = P.q;
  const int64_t* lp = P.level_ptr;
  const int64_t* kc = P.kcol;
  const int64_t* kr = P.krow;
  auto msz = [&](int64_t c) { return (int32_t)(P.hi[c] - P.lo[c]); };
  const std::vector<int64_t>& hoff = L.hoff;
  R->up.assign(q + 1, {});
  R->down.assign(q, {});
  R->couple.clear();
  R->dense.clear();
  R->out.clear();
  // leaf products x^_t = V_t^T x~_t (transposed leaf basis, contiguous rows)
  for (int64_t t = P.leaf0; t < P.nnodes; ++t)
    R->up[0].push_back({B.trans + L.tVT + P.lo[t] * kc[q], B.xh + hoff[t], B.ld_h, B.ld_x, (int32_t)kc[q],
                        {BlockRef{0, B.xt + P.lo[t], msz(t), 0}}});
  // transfer level l (h = q - l + 1 from the leaves): x^_p = [F_c1^T F_c2^T ..] [x^_c1; x^_c2; ..]
  for (int64_t l = q; l >= 1; --l) {
    std::vector<RowSpec>& rows = R->up[q - l + 1];
    for (int64_t p = lp[l - 1]; p < lp[l]; ++p) {
      RowSpec r{B.trans + L.tFT + L.foff(L.cbeg[p], l), B.xh + hoff[p], B.ld_h, B.ld_h, (int32_t)kc[l - 1], {}};
      for (int64_t c = L.cbeg[p]; c < L.cbeg[p + 1]; ++c) r.blks.push_back({0, B.xh + hoff[c], (int32_t)kc[l], 0});
      rows.push_back(std::move(r));
    }
  }
  // coupling rows of every level (Algorithm 4)
  for (int64_t l = 0; l <= q; ++l) {
    const int64_t* rp = P.s_rowptr + P.rp_base[l];
    const int64_t nl = lp[l + 1] - lp[l], bsz = P.krow[l] * P.kcol[l];
    for (int64_t t = 0; t < nl; ++t) {
      RowSpec r{B.mat + L.oS + P.sdat[l] + rp[t] * bsz, B.yh + hoff[lp[l] + t], B.ld_h, B.ld_h,
                (int32_t)P.krow[l], {}};
      for (int64_t b = rp[t]; b < rp[t + 1]; ++b)
        r.blks.push_back({0, B.xh + hoff[lp[l] + P.s_col[P.blk_base[l] + b]], (int32_t)P.kcol[l], 0});
      R->couple.push_back(std::move(r));
    }
  }
  // transfer downsweep level l: y^_c += E_c y^_parent
  for (int64_t l = 1; l <= q; ++l)
    for (int64_t c = lp[l]; c < lp[l + 1]; ++c)
      R->down[l - 1].push_back({B.mat + L.oE + L.eoff(c, l), B.yh + hoff[c], B.ld_h, B.ld_h, (int32_t)kr[l],
                                {BlockRef{0, B.yh + hoff[P.parent[c]], (int32_t)kr[l - 1], 0}}});
  // dense leaf rows: Z_t = sum_s D_ts x~_s
  for (int64_t t = 0; t < P.nleaves; ++t) {
    RowSpec r{B.mat + L.oD + P.ddat[P.d_rowptr[t]], B.zn + P.lo[P.leaf0 + t], B.ld_x, B.ld_x, msz(P.leaf0 + t), {}};
    for (int64_t b = P.d_rowptr[t]; b < P.d_rowptr[t + 1]; ++b)
      r.blks.push_back({0, B.xt + P.lo[P.leaf0 + P.d_col[b]], msz(P.leaf0 + P.d_col[b]), 0});
    R->dense.push_back(std::move(r));
  }
  // leaf expansion U_t y^_t (the caller picks the epilogue)
  for (int64_t t = P.leaf0; t < P.nnodes; ++t)
    R->out.push_back({B.mat + L.oU + P.lo[t] * kr[q], B.zn + P.lo[t], B.ld_x, B.ld_h, msz(t),
                      {BlockRef{0, B.yh + hoff[t], (int32_t)kr[q], 0}}});
}

namespace {
// One basis tree: ranks per level, offsets in the matrix array of its leaf
// bases and transfers and in the transposed array of their transposes.
struct Basis {
  const int64_t* k;
  int64_t leaf, tr, leaf_t, tr_t;
  const std::vector<int64_t>* base;  // per level: element offset of the level's first transfer
  const Parsed* P;
  // offset of the transfer of node c on level l
  int64_t at(int64_t c, int64_t l) const { return (*base)[l] + (c - P->level_ptr[l]) * k[l] * k[l - 1]; }
};

// Stages s_0 = q + 1 (the points) > s_1 > ... > s_m = lmin of one sweep:
// stage i spans the levels s_(i+1) .. s_i - 1 and level s_i.  Chosen by
// dynamic programming over the cost of a stage: a launch in a chain of
// dependent ones costs about 8 us beside the dense rows (4-5 us alone plus the
// gap), the composed matrices are read at about 4 TB/s, and a workgroup
// streams its own row at about 20 GB/s, which bounds the longest row.  For
// operators of a few thousand points one stage covers every level, for 2^20
// points only the levels of up to 2^11 nodes are grouped.
std::vector<int64_t> sweep_stages(const Parsed& P, const int64_t* k, int64_t lmin, bool up, bool group) {
  const int64_t q = P.q;
  const int64_t* lp = P.level_ptr;
  const double kLaunch = 8.0, kBytesPerUs = 4e6, kRowBytesPerUs = 2e4;
  int64_t max_leaf = 0;
  for (int64_t t = P.leaf0; t < P.nnodes; ++t) max_leaf = std::max(max_leaf, P.hi[t] - P.lo[t]);
  std::vector<double> best(q + 2, 0.0);
  std::vector<int64_t> prev(q + 2, lmin);
  if (!group) {
    std::vector<int64_t> st;
    for (int64_t s = q + 1; s >= lmin; --s) st.push_back(s);
    return st;
  }
  for (int64_t s = lmin + 1; s <= q + 1; ++s) {
    best[s] = 1e300;
    // columns of one node's composed row: points, or rows of x^ of its descendants on level s
    std::vector<int64_t> width(P.nnodes, 0);
    if (up && s <= q)
      for (int64_t c = lp[s]; c < lp[s + 1]; ++c) width[c] = k[s];
    double bytes = 0.0, longest = 0.0, sumk = 0.0;
    for (int64_t lo = s - 1; lo >= lmin; --lo) {
      bytes += 8.0 * (s <= q ? (double)(lp[s + 1] - lp[s]) * (double)k[s] : (double)P.n) * (double)k[lo];
      sumk += (double)k[lo];
      if (up) {
        for (int64_t p = lp[lo]; p < lp[lo + 1]; ++p) {
          if (s > q) width[p] = P.hi[p] - P.lo[p];
          else width[p] = 0;
        }
        if (s <= q)
          for (int64_t c = lp[lo + 1]; c < lp[lo + 2]; ++c) width[P.parent[c]] += width[c];
        for (int64_t p = lp[lo]; p < lp[lo + 1]; ++p) longest = std::max(longest, 8.0 * (double)(width[p] * k[lo]));
      } else {
        longest = 8.0 * sumk * (double)(s <= q ? k[s] : max_leaf);
      }
      const double c = best[lo] + kLaunch + std::max(bytes / kBytesPerUs, longest / kRowBytesPerUs);
      if (c < best[s]) {
        best[s] = c;
        prev[s] = lo;
      }
    }
  }
  std::vector<int64_t> st{q + 1};
  while (st.back() > lmin) st.push_back(prev[st.back()]);
  return st;
}
}  // namespace

void compose_sweeps(const OpLayout& L, const RowBases& B, bool trans_op, int64_t first, bool group, Composed* C) {
  const Parsed& P = *L.P;
  const int64_t q = P.q;
  const int64_t* lp = P.level_ptr;
  *C = Composed();
  const Basis row{P.krow, L.oU, L.oE, L.tUT, L.tET, &P.ebase, &P}, col{P.kcol, L.oV, L.oF, L.tVT, L.tFT, &P.fbase, &P};
  const Basis &bu = trans_op ? row : col, &bd = trans_op ? col : row;
  const int64_t lmin = std::min(first_coupling_level(P), q);
  int64_t ext = first;
  auto msz = [&](int64_t c) { return (int32_t)(P.hi[c] - P.lo[c]); };
  auto stage_of = [&](const Basis& b, int64_t s, int64_t lo, bool up) {
    ComposeStage g{};
    g.s = (int32_t)s;
    g.lo = (int32_t)lo;
    g.points = s > q;
    g.up = up;
    g.c0 = s > q ? lp[q] : lp[s];
    g.count = s > q ? lp[q + 1] - lp[q] : lp[s + 1] - lp[s];
    g.stored = s > q ? b.leaf : b.tr + (*b.base)[s];
    g.k.assign(b.k, b.k + q + 1);
    g.tr.assign(q + 1, 0);
    for (int64_t l = 1; l <= q; ++l) g.tr[l] = b.tr + (*b.base)[l];
    g.reg.assign(q + 1, 0);
    return g;
  };
  const std::vector<int64_t> su = sweep_stages(P, bu.k, lmin, true, group),
                             sd = sweep_stages(P, bd.k, lmin, false, group);
  // ---- upsweep, from the points towards the root
  for (size_t i = 0; i + 1 < su.size(); ++i) {
    const int64_t s = su[i], lo = su[i + 1], top = s - 1;
    C->up.emplace_back();
    C->up_split.push_back(lo < top);
    std::vector<RowSpec>& rows = C->up.back();
    const bool pts = s > q;
    const int64_t c0 = pts ? lp[q] : lp[s], c1 = pts ? lp[q + 1] : lp[s + 1];
    // rows of the level just below the source: the stored transposes
    for (int64_t p = lp[top]; p < lp[top + 1]; ++p) {
      if (pts) {
        rows.push_back({B.trans + bu.leaf_t + P.lo[p] * bu.k[q], B.xh + L.hoff[p], B.ld_h, B.ld_x, (int32_t)bu.k[q],
                        {BlockRef{0, B.xt + P.lo[p], msz(p), 0}}});
      } else {
        RowSpec r{B.trans + bu.tr_t + bu.at(L.cbeg[p], s), B.xh + L.hoff[p], B.ld_h, B.ld_h, (int32_t)bu.k[top], {}};
        for (int64_t c = L.cbeg[p]; c < L.cbeg[p + 1]; ++c)
          r.blks.push_back({0, B.xh + L.hoff[c], (int32_t)bu.k[s], 0});
        rows.push_back(std::move(r));
      }
    }
    if (lo == top) continue;
    // the levels above: transposes of the composed matrices, a node's
    // descendants side by side
    ComposeStage g = stage_of(bu, s, lo, true);
    std::vector<int64_t> anc(c1 - c0);  // ancestor on level l + 1
    for (int64_t c = c0; c < c1; ++c) anc[c - c0] = pts ? c : P.parent[c];
    for (int64_t l = top - 1; l >= lo; --l) {
      g.reg[l] = ext;
      int64_t c = c0;
      for (int64_t p = lp[l]; p < lp[l + 1]; ++p) {
        RowSpec r{B.trans + ext, B.xh + L.hoff[p], B.ld_h, pts ? B.ld_x : B.ld_h, (int32_t)bu.k[l], {}};
        if (pts) {
          r.blks.push_back({0, B.xt + P.lo[p], msz(p), 0});
          ext += (P.hi[p] - P.lo[p]) * bu.k[l];
        }
        for (; c < c1 && P.parent[anc[c - c0]] == p; ++c) {
          anc[c - c0] = p;
          if (pts) continue;
          ext += bu.k[s] * bu.k[l];
          // consecutive descendants are consecutive rows of x^ where all the level's tree rows are used
          const int64_t in = B.xh + L.hoff[c];
          if (!r.blks.empty() && r.blks.back().in_off + r.blks.back().width == in) r.blks.back().width += (int32_t)bu.k[s];
          else r.blks.push_back({0, in, (int32_t)bu.k[s], 0});
        }
        rows.push_back(std::move(r));
      }
    }
    C->stages.push_back(std::move(g));
  }
  // ---- downsweep, from the root towards the points
  for (size_t i = sd.size() - 1; i-- > 0;) {
    const int64_t s = sd[i], lo = sd[i + 1], top = s - 1;
    const bool pts = s > q, split = lo < top;
    std::vector<RowSpec> rows;
    const int64_t c0 = pts ? lp[q] : lp[s], c1 = pts ? lp[q + 1] : lp[s + 1];
    if (split) {
      C->stages.push_back(stage_of(bd, s, lo, false));
      C->stages.back().reg[0] = ext;
    }
    for (int64_t c = c0; c < c1; ++c) {
      const int32_t m = pts ? msz(c) : (int32_t)bd.k[s];
      RowSpec r{split ? B.trans + ext : B.mat + (pts ? bd.leaf + P.lo[c] * bd.k[q] : bd.tr + bd.at(c, s)),
                pts ? B.zn + P.lo[c] : B.yh + L.hoff[c], pts ? B.ld_x : B.ld_h, B.ld_h, m, {}};
      int64_t a = pts ? c : P.parent[c];  // ancestor on level l
      for (int64_t l = top; l >= lo; --l) {
        r.blks.push_back({0, B.yh + L.hoff[a], (int32_t)bd.k[l], 0});
        if (split) ext += (int64_t)m * bd.k[l];
        if (l > lo) a = P.parent[a];
      }
      rows.push_back(std::move(r));
    }
    if (pts) {
      C->out = std::move(rows);
      C->out_split = split;
    } else {
      C->down.push_back(std::move(rows));
      C->down_split.push_back(split);
    }
  }
  C->ntrans = (ext + 31) / 32 * 32;
}

bool composed_fits(const Composed& C) {
  // up to four workgroups of 256 threads a row (64 vectors), 2^32 - 1 threads a launch
  constexpr size_t kMaxSplitRows = (size_t(1) << 22) - 1;
  for (const auto* v : {&C.up, &C.down})
    for (size_t i = 0; i < v->size(); ++i) {
      const bool split = (v == &C.up ? C.up_split : C.down_split)[i] != 0;
      if (split && (*v)[i].size() > kMaxSplitRows) return false;
      for (const RowSpec& r : (*v)[i])
        if ((int64_t)r.blks.size() > kNbMax) return false;
    }
  return !C.out_split || C.out.size() <= kMaxSplitRows;
}

void append_row(RowTables& t, const RowSpec& r) {
  RowDesc R{};
  R.data_off = r.data_off;
  R.out_off = r.out_off;
  R.nrows = r.nrows;
  R.blk_begin = (int32_t)t.colend.size();
  int32_t col = 0;
  for (const BlockRef& b : r.blks) {
    col += b.width;
    t.colend.push_back(col);
    t.in_off.push_back(b.in_off);
  }
  R.blk_end = (int32_t)t.colend.size();
  R.out_ld = r.out_ld;
  R.in_ld = r.in_ld;
  t.rows.push_back(R);
}

void place_fl(RowTables& t, int64_t begin, int64_t end, int arr, FlKeys* keys, int64_t* n_fl) {
  for (int64_t i = begin; i < end; ++i) {
    RowDesc& R = t.rows[i];
    const int32_t ncols = R.blk_end > R.blk_begin ? t.colend[R.blk_end - 1] : 0;
    const int64_t size = (int64_t)R.nrows * ((ncols + 7) / 8 * 8);  // columns padded to pairs of steps
    const auto ins = keys->emplace(2 * R.data_off + arr, FlRegion{*n_fl, R.nrows, ncols});
    if (!ins.second && (ins.first->second.nrows != R.nrows || ins.first->second.ncols != ncols)) {
      R.fl_off = *n_fl;  // the same offset with another shape: a region of its own
      *n_fl += size;
      continue;
    }
    R.fl_off = ins.first->second.fl_off;
    if (ins.second) *n_fl += size;
  }
}

int64_t row_work(const RowSpec& r) {
  int64_t c = 0;
  for (const BlockRef& b : r.blks) c += b.width;
  return c * r.nrows;
}

}  // namespace h2
