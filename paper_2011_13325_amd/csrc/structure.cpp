#include "structure.hpp"

#include <algorithm>
#include <functional>
#include <map>
#include <queue>
#include <utility>

namespace eamg {

namespace {

// Row chunks of a pattern pass: contiguous ranges, a count that depends on n only, so results
// that are concatenated in chunk order do not depend on the thread count.
inline int n_chunks(int n) { return std::max(1, std::min(64, n / 1024)); }
inline int chunk_lo(int n, int nch, int64_t c) { return int(int64_t(n) * c / nch); }

}  // namespace

ProlongPlan plan_prolongation(const Pattern &A, const AuxLevel &aux, const std::vector<int> &agg_of,
                              const std::vector<char> &dmask, int cap_S, int cap_A, double tie_rtol) {
  const int n = A.n_rows;
  const int k = aux.k;
  ProlongPlan pl;
  pl.type.assign(static_cast<size_t>(n), ROW_D);
  pl.P.n_rows = n;
  pl.P.rp.assign(size_t(n) + 1, 0);
  pl.F_ptr.assign(size_t(n) + 1, 0);
  int nc = 0;
  for (int v : agg_of) nc = std::max(nc, v + 1);
  pl.P.n_cols = nc;
  // per chunk: P columns and F entries of its rows, lengths in pl.P.rp / pl.F_ptr [i + 1]
  struct Part {
    std::vector<int> col, fv, fe;
  };
  const int nch = n_chunks(n);
  std::vector<Part> parts(static_cast<size_t>(nch));
  parallel_for_dynamic(nch, [&](int64_t c) {
    Part &pt = parts[size_t(c)];
    std::vector<int> cs;
    std::vector<std::pair<int, int>> F;         // (l, e)
    for (int i = chunk_lo(n, nch, c); i < chunk_lo(n, nch, c + 1); ++i) {
      if (dmask[i]) continue;
      cs.clear();
      cs.push_back(agg_of[i]);
      for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) {
        const int j = A.col[p];
        if (!dmask[j]) cs.push_back(agg_of[j]);
      }
      std::sort(cs.begin(), cs.end());
      cs.erase(std::unique(cs.begin(), cs.end()), cs.end());
      if (int(cs.size()) <= cap_S) {
        pl.type[i] = ROW_S;
        pt.col.insert(pt.col.end(), cs.begin(), cs.end());
        pl.P.rp[i + 1] = int64_t(cs.size());
        continue;
      }
      pl.type[i] = ROW_A;
      F.clear();
      std::map<int, double> ws;
      for (int64_t p = aux.nb_ptr[i]; p < aux.nb_ptr[i + 1]; ++p) {
        const int l = aux.nb[p];
        if (dmask[l]) continue;
        const int e = aux.nb_e[p];
        double tr = 0.0;
        for (int d = 0; d < k; ++d) tr += aux.E[size_t(e) * k * k + size_t(d) * k + d];
        ws[agg_of[l]] += tr;
      }
      const int own = agg_of[i];
      std::vector<std::pair<int, double>> others;   // ascending group id
      for (const auto &g : ws)
        if (g.first != own) others.emplace_back(g.first, g.second);
      std::vector<int> keep = {own};
      while (!others.empty() && int(keep.size()) < cap_A) {
        double wmax = others[0].second;
        for (const auto &g : others) wmax = std::max(wmax, g.second);
        size_t pick = 0;
        while (!(others[pick].second >= wmax * (1.0 - tie_rtol))) ++pick;   // smallest id in band
        keep.push_back(others[pick].first);
        others.erase(others.begin() + long(pick));
      }
      std::sort(keep.begin(), keep.end());
      for (int64_t p = aux.nb_ptr[i]; p < aux.nb_ptr[i + 1]; ++p) {
        const int l = aux.nb[p];
        if (dmask[l]) continue;
        if (std::binary_search(keep.begin(), keep.end(), agg_of[l])) F.emplace_back(l, aux.nb_e[p]);
      }
      std::sort(F.begin(), F.end());
      for (const auto &le : F) {
        pt.fv.push_back(le.first);
        pt.fe.push_back(le.second);
      }
      pl.F_ptr[i + 1] = int64_t(F.size());
      pt.col.insert(pt.col.end(), keep.begin(), keep.end());
      pl.P.rp[i + 1] = int64_t(keep.size());
    }
  }, 1);
  for (int i = 0; i < n; ++i) {
    pl.P.rp[i + 1] += pl.P.rp[i];
    pl.F_ptr[i + 1] += pl.F_ptr[i];
  }
  pl.P.col.reserve(size_t(pl.P.rp[n]));
  pl.F_vtx.reserve(size_t(pl.F_ptr[n]));
  pl.F_edge.reserve(size_t(pl.F_ptr[n]));
  for (const Part &pt : parts) {
    pl.P.col.insert(pl.P.col.end(), pt.col.begin(), pt.col.end());
    pl.F_vtx.insert(pl.F_vtx.end(), pt.fv.begin(), pt.fv.end());
    pl.F_edge.insert(pl.F_edge.end(), pt.fe.begin(), pt.fe.end());
  }
  return pl;
}

Pattern spgemm_symbolic(const Pattern &A, const Pattern &B) {
  Pattern C;
  const int n = A.n_rows;
  C.n_rows = n;
  C.n_cols = B.n_cols;
  C.rp.assign(size_t(n) + 1, 0);
  const int nch = n_chunks(n);
  std::vector<std::vector<int>> parts(static_cast<size_t>(nch));
  parallel_for_dynamic(nch, [&](int64_t c) {
    std::vector<int> &out = parts[size_t(c)];
    std::vector<int> mark(size_t(B.n_cols), -1);
    std::vector<int> row;
    for (int i = chunk_lo(n, nch, c); i < chunk_lo(n, nch, c + 1); ++i) {
      row.clear();
      for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) {
        const int j = A.col[p];
        for (int64_t q = B.rp[j]; q < B.rp[j + 1]; ++q) {
          const int cc = B.col[q];
          if (mark[cc] != i) {
            mark[cc] = i;
            row.push_back(cc);
          }
        }
      }
      std::sort(row.begin(), row.end());
      out.insert(out.end(), row.begin(), row.end());
      C.rp[i + 1] = int64_t(row.size());
    }
  }, 1);
  for (int i = 0; i < n; ++i) C.rp[i + 1] += C.rp[i];
  C.col.reserve(size_t(C.rp[n]));
  for (const auto &pt : parts) C.col.insert(C.col.end(), pt.begin(), pt.end());
  return C;
}

Pattern transpose_pattern(const Pattern &P, std::vector<int64_t> &src) {
  Pattern T;
  T.n_rows = P.n_cols;
  T.n_cols = P.n_rows;
  T.rp.assign(size_t(P.n_cols) + 1, 0);
  for (int64_t q = 0; q < P.nnz(); ++q) T.rp[P.col[q] + 1]++;
  for (int c = 0; c < P.n_cols; ++c) T.rp[c + 1] += T.rp[c];
  T.col.resize(size_t(P.nnz()));
  src.resize(size_t(P.nnz()));
  std::vector<int64_t> fill(T.rp.begin(), T.rp.end() - 1);
  for (int i = 0; i < P.n_rows; ++i)
    for (int64_t q = P.rp[i]; q < P.rp[i + 1]; ++q) {
      const int64_t d = fill[P.col[q]]++;
      T.col[d] = i;
      src[d] = q;
    }
  return T;
}

std::vector<int> greedy_coloring(int n, const int64_t *rp, const int *col, int &n_colors) {
  // smallest-last order: remove a vertex of minimum remaining degree (lowest id on ties).
  // Indexed binary min-heap on the key (degree, id), one entry per vertex; a removal lowers
  // its neighbours' keys in place.
  std::vector<int64_t> key(static_cast<size_t>(n));
  for (int i = 0; i < n; ++i) {
    int64_t d = 0;
    for (int64_t p = rp[i]; p < rp[i + 1]; ++p)
      if (col[p] != i) ++d;
    key[i] = (d << 32) | int64_t(i);
  }
  std::vector<int> heap(static_cast<size_t>(n)), where(static_cast<size_t>(n));
  for (int i = 0; i < n; ++i) heap[i] = where[i] = i;
  int size = n;
  auto swap_at = [&](int a, int b) {
    std::swap(heap[a], heap[b]);
    where[heap[a]] = a;
    where[heap[b]] = b;
  };
  auto sift_up = [&](int a) {
    while (a > 0) {
      const int par = (a - 1) / 2;
      if (key[heap[par]] <= key[heap[a]]) break;
      swap_at(a, par);
      a = par;
    }
  };
  auto sift_down = [&](int a) {
    for (;;) {
      const int l = 2 * a + 1, r = l + 1;
      int m = a;
      if (l < size && key[heap[l]] < key[heap[m]]) m = l;
      if (r < size && key[heap[r]] < key[heap[m]]) m = r;
      if (m == a) break;
      swap_at(a, m);
      a = m;
    }
  };
  for (int a = n / 2 - 1; a >= 0; --a) sift_down(a);
  std::vector<char> removed(static_cast<size_t>(n), 0);
  std::vector<int> seq;
  seq.reserve(static_cast<size_t>(n));
  while (size > 0) {
    const int v = heap[0];
    swap_at(0, size - 1);
    --size;
    sift_down(0);
    removed[v] = 1;
    seq.push_back(v);
    for (int64_t p = rp[v]; p < rp[v + 1]; ++p) {
      const int u = col[p];
      if (u == v || removed[u]) continue;
      key[u] -= int64_t(1) << 32;
      sift_up(where[u]);
    }
  }
  std::vector<int> color(static_cast<size_t>(n), -1);
  std::vector<int> used;
  n_colors = 0;
  for (auto it = seq.rbegin(); it != seq.rend(); ++it) {
    const int i = *it;
    used.clear();
    for (int64_t p = rp[i]; p < rp[i + 1]; ++p) {
      const int j = col[p];
      if (j != i && color[j] >= 0) used.push_back(color[j]);
    }
    std::sort(used.begin(), used.end());
    int c = 0;
    for (int u : used) {
      if (u == c) ++c;
      else if (u > c) break;
    }
    color[i] = c;
    n_colors = std::max(n_colors, c + 1);
  }
  return color;
}

Pattern permute_pattern(const Pattern &A, const std::vector<int> &perm, const std::vector<int> &inv,
                        std::vector<int64_t> &src) {
  return permute_rect(A, perm, inv, src);
}

Pattern permute_rect(const Pattern &P, const std::vector<int> &perm_rows,
                     const std::vector<int> &inv_cols, std::vector<int64_t> &src) {
  Pattern R;
  R.n_rows = P.n_rows;
  R.n_cols = P.n_cols;
  R.rp.assign(size_t(P.n_rows) + 1, 0);
  R.col.resize(size_t(P.nnz()));
  src.resize(size_t(P.nnz()));
  for (int r = 0; r < P.n_rows; ++r) {
    const int o = perm_rows[r];
    R.rp[r + 1] = R.rp[r] + (P.rp[o + 1] - P.rp[o]);
  }
  const int n = P.n_rows, nch = n_chunks(n);
  parallel_for_dynamic(nch, [&](int64_t c) {
    std::vector<std::pair<int, int64_t>> row;
    for (int r = chunk_lo(n, nch, c); r < chunk_lo(n, nch, c + 1); ++r) {
      const int o = perm_rows[r];
      row.clear();
      for (int64_t q = P.rp[o]; q < P.rp[o + 1]; ++q) row.emplace_back(inv_cols[P.col[q]], q);
      std::sort(row.begin(), row.end());
      const int64_t base = R.rp[r];
      for (size_t t = 0; t < row.size(); ++t) {
        R.col[size_t(base) + t] = row[t].first;
        src[size_t(base) + t] = row[t].second;
      }
    }
  }, 1);
  return R;
}

// A colour launch costs kLaunch beyond its bytes (replayed graphs: launches of a few hundred
// kilobytes take 3.3 to 4.6 us), and a group's S, at most a few tens of megabytes that stay in the
// Infinity Cache, streams at kRate.  A group of g colours costs two launches and the bytes of S, g
// colours cost g launches; the couplings outside the group are read once either way.  Groups grow
// while a further colour's part of S costs less than the group's mean per colour (the mean falls until
// then), and stay if they save at least half a launch.  A block of S counts its FP64 value and column
// (both precisions share one plan) and a 32-byte sector of the scattered gather, which is most of a
// scalar block's cost.  The optimum is flat: S allowed 0.4, 1, 2 and 4 times these bytes gave 2.41,
// 2.29, 2.21, 3.07 ms per 17^3 FP64 solve, 19.8, 19.3, 18.8, 19.6 ms per 64^3 FP32 solve and 29.3,
// 29.3, 30.3, 32.6 ms in FP64.
SweepPlan plan_sweeps(const Pattern &Ap, const std::vector<int> &dg, const std::vector<int> &color_ptr,
                      int ncolors, int bs) {
  constexpr double kLaunch = 3.5e-6, kRate = 6e12;
  const double blk = bs * bs * 8.0 + 4.0 + 32.0;
  const int n = Ap.n_rows;
  SweepPlan pl;
  pl.pre = dg;
  pl.post.resize(size_t(n));
  for (int i = 0; i < n; ++i) pl.post[size_t(i)] = dg[size_t(i)] + 1;
  pl.rank.assign(size_t(n), -1);
  pl.S.n_rows = pl.S.n_cols = n;
  pl.S.rp.assign(size_t(n) + 1, 0);
  std::vector<std::vector<int>> rows;   // S rows of the groups tried
  rows.resize(size_t(color_ptr[size_t(ncolors)]));
  auto first_at = [&](int i, int r) {   // first position of row i at a column >= r
    return int(std::lower_bound(Ap.col.begin() + Ap.rp[size_t(i)], Ap.col.begin() + Ap.rp[size_t(i) + 1], r) -
               Ap.col.begin());
  };
  pl.cut.push_back(0);
  int c0 = 0;
  while (c0 < ncolors) {
    const int r0 = color_ptr[size_t(c0)];
    // a group that starts at the first colour has no earlier rows: one launch forward, two backward
    const double launches = c0 == 0 ? 1.5 : 2.0;
    double cost = launches * kLaunch, nnz = 0.0;
    int c1 = c0 + 1;
    for (int i = r0; i < color_ptr[size_t(c1)]; ++i) rows[size_t(i)].clear();
    for (; c1 < ncolors; ++c1) {
      const int a = color_ptr[size_t(c1)], b = color_ptr[size_t(c1) + 1];
      const double mean = cost / double(c1 - c0);
      // the direct couplings alone may already cost too much; a first-fit colouring gives every
      // row at least one in each lower colour
      if (double(b - a) * (c1 - c0) * blk / kRate >= mean) break;
      double direct = 0.0;
      for (int i = a; i < b; ++i) direct += double(dg[size_t(i)] - first_at(i, r0));
      if (direct * blk / kRate >= mean) break;
      // threads only where the merged rows repay starting them
      const bool many = direct * (1.0 + nnz / double(a - r0)) > 3e5;
      const int chunk = many ? 32 : b - a, nch = (b - a + chunk - 1) / std::max(1, chunk);
      parallel_for_dynamic(nch, [&](int64_t ch) {
        std::vector<uint64_t> seen(size_t(a - r0 + 63) / 64, 0);
        const auto visit = [&](int j) {   // whether j is new
          uint64_t &w = seen[size_t(j - r0) >> 6];
          const uint64_t bit = uint64_t(1) << ((j - r0) & 63);
          const bool fresh = !(w & bit);
          w |= bit;
          return fresh;
        };
        for (int i = a + int(ch) * chunk; i < std::min(b, a + int(ch + 1) * chunk); ++i) {
          std::vector<int> &R = rows[size_t(i)];
          R.clear();
          // the rows' sets are closed under their chains: those of a row already reached are in,
          // and the later colours, first here, reach the most
          for (int q = dg[size_t(i)] - 1, q0 = first_at(i, r0); q >= q0; --q) {
            const int j = Ap.col[size_t(q)];
            if (!visit(j)) continue;
            R.push_back(j);
            for (int k : rows[size_t(j)])
              if (visit(k)) R.push_back(k);
          }
          // ascending: from the marks, or sorted where there are few
          if (seen.size() < 16 * R.size()) {
            size_t m = 0;
            for (size_t w = 0; w < seen.size(); ++w)
              for (uint64_t v = std::exchange(seen[w], 0); v; v &= v - 1)
                R[m++] = r0 + int(w * 64) + __builtin_ctzll(v);
          } else {
            for (int j : R) seen[size_t(j - r0) >> 6] = 0;
            std::sort(R.begin(), R.end());
          }
        }
      }, 1);
      double add = 0.0;
      for (int i = a; i < b; ++i) add += double(rows[size_t(i)].size());
      if (add * blk / kRate >= mean) break;
      nnz += add;
      cost += add * blk / kRate;
    }
    if (cost > (double(c1 - c0) - 0.5) * kLaunch || nnz == 0.0) c1 = c0 + 1;
    if (c1 > c0 + 1) {
      const int r1 = color_ptr[size_t(c1)];
      for (int c = c0; c < c1; ++c)
        for (int i = color_ptr[size_t(c)]; i < color_ptr[size_t(c) + 1]; ++i) {
          pl.pre[size_t(i)] = first_at(i, r0);
          pl.post[size_t(i)] = first_at(i, r1);
          pl.rank[size_t(i)] = c - c0;
        }
      pl.max_rank = std::max(pl.max_rank, c1 - c0 - 1);
    }
    pl.cut.push_back(c1);
    c0 = c1;
  }
  for (int i = 0; i < n; ++i)
    pl.S.rp[size_t(i) + 1] = pl.S.rp[size_t(i)] + (pl.rank[size_t(i)] > 0 ? int64_t(rows[size_t(i)].size()) : 0);
  pl.S.col.reserve(size_t(pl.S.nnz()));
  for (int i = 0; i < n; ++i)
    if (pl.rank[size_t(i)] > 0) pl.S.col.insert(pl.S.col.end(), rows[size_t(i)].begin(), rows[size_t(i)].end());
  return pl;
}

ColourOrder colour_order(const std::vector<int> &color, int ncolors) {
  ColourOrder o;
  const size_t n = color.size();
  o.ptr.assign(size_t(ncolors) + 1, 0);
  for (int c : color) o.ptr[size_t(c) + 1]++;
  for (int c = 0; c < ncolors; ++c) o.ptr[size_t(c) + 1] += o.ptr[size_t(c)];
  o.perm.resize(n);
  o.inv.resize(n);
  std::vector<int> fill(o.ptr.begin(), o.ptr.end() - 1);
  for (size_t i = 0; i < n; ++i) o.perm[size_t(fill[size_t(color[i])]++)] = int(i);
  for (size_t r = 0; r < n; ++r) o.inv[size_t(o.perm[r])] = int(r);
  return o;
}

SweepStages prepare_sweeps(const Pattern &Ap, const std::vector<int> &dg, const std::vector<int> &color_ptr,
                           int ncolors, int bs) {
  SweepStages st;
  st.plan = plan_sweeps(Ap, dg, color_ptr, ncolors, bs);
  const SweepPlan &pl = st.plan;
  if (!pl.grouped()) return st;
  const int n = Ap.n_rows;
  st.Sb.n_rows = st.Sb.n_cols = n;
  st.Sb.rp.assign(size_t(n) + 1, 0);
  for (int c : pl.S.col) ++st.Sb.rp[size_t(c) + 1];
  for (int i = 0; i < n; ++i) st.Sb.rp[size_t(i) + 1] += st.Sb.rp[size_t(i)];
  st.Sb.col.resize(pl.S.col.size());
  std::vector<int64_t> next(st.Sb.rp.begin(), st.Sb.rp.end() - 1);
  const int *col = pl.S.col.data();
  for (int i = 0; i < n; ++i)
    for (int64_t q = pl.S.rp[size_t(i)], q1 = pl.S.rp[size_t(i) + 1]; q < q1; ++q)
      st.Sb.col[size_t(next[size_t(col[q])]++)] = i;
  st.lo_end.resize(size_t(n));
  st.right.resize(size_t(n));
  int64_t lo = 0;
  for (int i = 0; i < n; ++i) {
    st.right[size_t(i)] = dg[size_t(i)] + 1;
    st.lo_end[size_t(i)] = int(lo + (pl.pre[size_t(i)] - Ap.rp[size_t(i)]));
    lo += dg[size_t(i)] - Ap.rp[size_t(i)];
  }
  st.rank_ptr.assign(size_t(pl.max_rank) + 2, 0);
  for (int r : pl.rank)
    if (r >= 0) ++st.rank_ptr[size_t(r) + 1];
  for (int r = 0; r <= pl.max_rank; ++r) st.rank_ptr[size_t(r) + 1] += st.rank_ptr[size_t(r)];
  st.order.resize(size_t(st.rank_ptr.back()));
  std::vector<int> fill(st.rank_ptr.begin(), st.rank_ptr.end() - 1);
  for (int i = 0; i < n; ++i)
    if (pl.rank[size_t(i)] >= 0) st.order[size_t(fill[size_t(pl.rank[size_t(i)])]++)] = i;
  return st;
}

Smoothing plan_smoothing(const Pattern &A, int bs, bool sweeps) {
  Smoothing c;
  c.color = greedy_coloring(A, c.ncolors);
  c.order = colour_order(c.color, c.ncolors);
  c.Ap = permute_pattern(A, c.order.perm, c.order.inv, c.src);
  if (!sweeps) return c;
  const Pattern &P = c.Ap;
  std::vector<int> dg(size_t(P.n_rows));
  for (int i = 0; i < P.n_rows; ++i)
    dg[size_t(i)] = int(std::lower_bound(P.col.begin() + P.rp[size_t(i)], P.col.begin() + P.rp[size_t(i) + 1], i) -
                        P.col.begin());
  c.stages = prepare_sweeps(P, dg, c.order.ptr, c.ncolors, bs);
  return c;
}

}  // namespace eamg
