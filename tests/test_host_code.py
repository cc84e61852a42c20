"""Host parts of the library on their own (CPU): small C++ programs over its headers and sources."""
import os
import subprocess

import pytest

from paper_2011_13325_amd import build as B


def _run(tmp_path, source, *sources, timeout=120):
    try:
        cxx = B._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run([cxx, "-O2", "-ftrapv", "-std=c++17", "-pthread", f"-I{B.CSRC}", str(src),
                    *[os.path.join(B.CSRC, f) for f in sources], "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
    return r.stdout


POLL = r"""
#include "wait.hpp"
#include <cstdint>
#include <cstdio>
#include <stdexcept>
using namespace eamg;
struct NoRest { void operator()() const {} };
#define CHECK(c) do { if (!(c)) { std::printf("line %d: " #c "\n", __LINE__); return 1; } } while (0)
int main() {
  volatile int64_t polls = 0;
  int64_t asked = 0;
  auto poll = [&](int64_t ready_at, int64_t busy_for) {
    polls = asked = 0;
    return poll_until([&] { return (polls = polls + 1) > ready_at; },
                      [&] { return ++asked < busy_for; }, NoRest());
  };
  const int64_t never = INT64_MAX;
  CHECK(poll(0, never) && polls == 1 && asked == 0);
  CHECK(poll(kPolls - 1, never) && asked == 0);
  CHECK(poll(kPolls, never) && asked == 1);
  CHECK(poll(5 * kPolls + 3, never) && asked == 5);
  // nothing left to wait for: one last look
  CHECK(!poll(never, 3) && asked == 3 && polls == 3 * kPolls + 1);
  CHECK(poll(3 * kPolls, 3) && asked == 3);
  // a wait of more polls than an int counts is asked about as often as a short one
  const int64_t many = (int64_t(1) << 31) / kPolls + 1000;
  CHECK(!poll(never, many) && asked == many && polls == many * kPolls + 1);
  try {
    poll_until([] { return false; }, []() -> bool { throw std::runtime_error("x"); });
    CHECK(false);
  } catch (const std::runtime_error &) {
  }
  return 0;
}
"""


def test_a_wait_of_any_length_keeps_asking_whether_to_go_on(tmp_path):
    _run(tmp_path, POLL)


LOOP = r"""
#include "coarsen.hpp"
#include <new>
using namespace eamg;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: " #c "\n", __LINE__); return 1; } } while (0)
int main() {
  for (int64_t n : {int64_t(0), int64_t(1), int64_t(7), int64_t(200), int64_t(100000)})
    for (int64_t chunk : {int64_t(1), int64_t(64)}) {
      std::vector<int> seen(size_t(n), 0);
      parallel_for_dynamic(n, [&](int64_t i) { ++seen[size_t(i)]; }, chunk);
      for (int v : seen) CHECK(v == 1);
    }
  for (int64_t bad : {int64_t(0), int64_t(777), int64_t(99999)}) {
    bool caught = false;
    try {
      parallel_for_dynamic(100000, [&](int64_t i) { if (i >= bad) throw std::bad_alloc(); }, 1);
    } catch (const std::bad_alloc &) {
      caught = true;
    }
    CHECK(caught);
  }
  return 0;
}
"""


def test_a_failed_allocation_in_a_parallel_loop_reaches_the_caller(tmp_path):
    _run(tmp_path, LOOP)


RUNS = r"""
#include "coarse.hpp"
#include <cstdio>
#include <vector>
using namespace eamg;
#define CHECK(c) do { if (!(c)) { std::printf("nb %d lr %d line %d: " #c "\n", nb, lr, __LINE__); return 1; } } while (0)
int main() {
  int seen_lr[4] = {0, 0, 0, 0};
  for (int nb = 1; nb <= 128; ++nb) {   // a tail has up to 16,384 dofs
    ++seen_lr[sym_run_log2(nb)];
    for (int lr = 0; lr <= 3; ++lr) {
      const int runs = sym_first_run(nb, lr, nb);
      std::vector<int> owner(size_t(nb) * nb, -1);
      int last_i = 0;
      for (int run = 0; run < runs; ++run) {
        const SymRun r = sym_run(nb, lr, run);
        CHECK(r.i >= last_i && r.i < nb && r.j0 >= r.i && r.j1 > r.j0 && r.j1 <= nb && r.j1 - r.j0 <= 1 << lr);
        CHECK(r.i == last_i || run == sym_first_run(nb, lr, r.i));
        last_i = r.i;
        for (int j = r.j0; j < r.j1; ++j) {
          CHECK(owner[size_t(r.i) * nb + j] < 0);
          owner[size_t(r.i) * nb + j] = run;
        }
        CHECK(r.j1 - r.j0 == 1 << lr || r.j1 == nb);
      }
      for (int i = 0; i < nb; ++i)
        for (int j = 0; j < nb; ++j) CHECK((owner[size_t(i) * nb + j] >= 0) == (j >= i));
    }
  }
  const int nb = 0, lr = 0;
  CHECK(seen_lr[0] == 90 && seen_lr[1] == 37 && seen_lr[2] == 1);
  return 0;
}
"""


def test_runs_of_the_packed_panel_product_cover_every_tile_once(tmp_path):
    _run(tmp_path, RUNS)


PLAN = r"""
#include "structure.hpp"
#include <cmath>
#include <random>
#include <set>
using namespace eamg;
#define CHECK(c) do { if (!(c)) { std::printf("n %d deg %d bs %d line %d: " #c "\n", n, deg, bs, __LINE__); return 1; } } while (0)
// Random symmetric patterns near the diagonal, scalar entries; the plan's cost is that of bs x bs blocks.
int check(int n, int deg, int bs, int &groups, int &singles) {
  std::mt19937 rng(unsigned(n + 7 * deg));
  std::vector<std::set<int>> adj;
  adj.resize(size_t(n));
  for (int i = 0; i < n; ++i) {
    adj[size_t(i)].insert(i);
    for (int d = 0; d < deg / 2; ++d) {
      const int j = (i + 1 + int(rng() % unsigned(2 * deg))) % n;
      adj[size_t(i)].insert(j);
      adj[size_t(j)].insert(i);
    }
  }
  Pattern A;
  A.n_rows = A.n_cols = n;
  A.rp.push_back(0);
  for (const auto &s : adj) {
    A.col.insert(A.col.end(), s.begin(), s.end());
    A.rp.push_back(int64_t(A.col.size()));
  }
  const Smoothing c = plan_smoothing(A, bs, true);
  const Pattern &P = c.Ap;
  const SweepPlan &pl = c.stages.plan;
  const std::vector<int> &cp = c.order.ptr;
  const int ns = int(pl.cut.size()) - 1;
  CHECK(pl.cut.front() == 0 && pl.cut.back() == c.ncolors);
  // values, D^+ (every seventh row singular: zero), right-hand side
  const size_t N = size_t(n);
  std::vector<double> val(P.col.size()), D(N), b(N);
  std::vector<int> dg(N);
  for (int i = 0; i < n; ++i)
    for (int64_t q = P.rp[i]; q < P.rp[i + 1]; ++q) {
      const int j = P.col[size_t(q)];
      if (j == i) dg[size_t(i)] = int(q);
      val[size_t(q)] = j == i ? 2.0 * deg : -double((std::min(i, j) * 31 + std::max(i, j) * 17) % 101) / 101.0;
    }
  for (int i = 0; i < n; ++i) {
    D[size_t(i)] = i % 7 ? 1.0 / val[size_t(dg[size_t(i)])] : 0.0;
    b[size_t(i)] = double(rng() % 1000) / 500.0 - 1.0;
  }
  const auto row = [&](int i, int64_t q0, int64_t q1, const std::vector<double> &x) {
    double s = 0.0;
    for (int64_t q = q0; q < q1; ++q) s += val[size_t(q)] * x[size_t(P.col[size_t(q)])];
    return s;
  };
  // the group matrices by the recursion of the fill kernel, rank by rank as listed
  const auto fill = [&](const Pattern &S, bool fwd) {
    std::vector<double> v(S.col.size(), NAN);
    for (int t = 0; t <= pl.max_rank; ++t) {
      const int r = fwd ? t : pl.max_rank - t;
      for (int o = c.stages.rank_ptr[size_t(r)]; o < c.stages.rank_ptr[size_t(r) + 1]; ++o) {
        const int i = c.stages.order[size_t(o)];
        const int q0 = fwd ? pl.pre[size_t(i)] : c.stages.right[size_t(i)], q1 = fwd ? dg[size_t(i)] : pl.post[size_t(i)];
        for (int64_t e = S.rp[i]; e < S.rp[i + 1]; ++e) {
          const int k = S.col[size_t(e)];
          double a = 0.0;
          for (int q = q0; q < q1; ++q) {
            const int j = P.col[size_t(q)];
            const double p = val[size_t(q)] * D[size_t(j)];
            const auto *lo = &S.col[0] + S.rp[j], *hi = &S.col[0] + S.rp[j + 1], *at = std::lower_bound(lo, hi, k);
            if (j == k) a += p;
            else if (at != hi && *at == k) a -= p * v[size_t(at - &S.col[0])];
          }
          v[size_t(e)] = a;
        }
      }
    }
    return v;
  };
  std::vector<double> vf, vb;
  if (pl.grouped()) {
    vf = fill(pl.S, true);
    vb = fill(c.stages.Sb, false);
  }
  for (double v : vf) CHECK(std::isfinite(v));
  for (double v : vb) CHECK(std::isfinite(v));
  const auto close = [&](const std::vector<double> &x, const std::vector<double> &y) {
    double d = 0.0, m = 0.0;
    for (int i = 0; i < n; ++i) {
      d = std::max(d, std::fabs(x[size_t(i)] - y[size_t(i)]));
      m = std::max(m, std::fabs(y[size_t(i)]));
    }
    return d <= 1e-12 * m;
  };
  // forward from x = 0
  std::vector<double> x(N, 0.0), g(N, 0.0), u(N, 0.0);
  for (int i = 0; i < n; ++i) x[size_t(i)] = D[size_t(i)] * (b[size_t(i)] - row(i, P.rp[i], dg[size_t(i)], x));
  int64_t lo = 0;
  for (int k = 0; k < ns; ++k) {
    const int r0 = cp[size_t(pl.cut[size_t(k)])], r1 = cp[size_t(pl.cut[size_t(k) + 1])];
    ++(pl.cut[size_t(k) + 1] > pl.cut[size_t(k)] + 1 ? groups : singles);
    for (int i = r0; i < r1; ++i) {
      const int64_t left = dg[size_t(i)] - P.rp[i];
      if (pl.grouped()) CHECK(c.stages.lo_end[size_t(i)] - lo == pl.pre[size_t(i)] - P.rp[i]);
      lo += left;
      u[size_t(i)] = b[size_t(i)] - row(i, P.rp[i], pl.pre[size_t(i)], g);
    }
    for (int i = r0; i < r1; ++i) {
      double t = u[size_t(i)];
      for (int64_t e = pl.S.rp[i]; e < pl.S.rp[i + 1]; ++e) t -= vf[size_t(e)] * u[size_t(pl.S.col[size_t(e)])];
      g[size_t(i)] = D[size_t(i)] * t;
    }
  }
  CHECK(close(g, x));
  // backward from there
  for (int i = n - 1; i >= 0; --i) x[size_t(i)] += D[size_t(i)] * (b[size_t(i)] - row(i, P.rp[i], P.rp[i + 1], x));
  for (int k = ns - 1; k >= 0; --k) {
    const int r0 = cp[size_t(pl.cut[size_t(k)])], r1 = cp[size_t(pl.cut[size_t(k) + 1])];
    for (int i = r0; i < r1; ++i) u[size_t(i)] = b[size_t(i)] - row(i, P.rp[i], P.rp[i + 1], g);
    for (int i = r0; i < r1; ++i) {
      double t = u[size_t(i)];
      if (pl.grouped())
        for (int64_t e = c.stages.Sb.rp[i]; e < c.stages.Sb.rp[i + 1]; ++e)
          t -= vb[size_t(e)] * u[size_t(c.stages.Sb.col[size_t(e)])];
      g[size_t(i)] += D[size_t(i)] * t;
    }
  }
  CHECK(close(g, x));
  return 0;
}
int main() {
  int groups = 0, singles = 0;
  for (int n : {1, 30, 200, 1200, 5000, 40000})
    for (int deg : {4, 12, 40})
      for (int bs : {1, 3, 6})
        if (check(n, deg, bs, groups, singles)) return 1;
  std::printf("%d groups, %d single colours\n", groups, singles);
  return groups > 20 && singles > 20 ? 0 : 1;
}
"""


def test_planned_groups_are_the_colour_sweeps(tmp_path):
    """plan_smoothing on random symmetric patterns: the forward and backward sweeps by stages, the group
    matrices filled by their recursion, against the sweeps row by row (singular rows among them)."""
    _run(tmp_path, PLAN, "structure.cpp")
