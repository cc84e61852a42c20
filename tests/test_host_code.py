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
