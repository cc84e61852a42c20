// Batched block-panel PCG (eamg_solve_batch): K right-hand sides share every matrix stream of
// the V-cycle and of the CG operator, each column keeping its own CG recurrence.  The
// preconditioner is the same V-cycle as the single-vector path (same colours, same transfers,
// same coarsest inverse), applied to K columns per launch.
#include <algorithm>
#include <cmath>
#include <functional>
#include <cstdlib>
#include <memory>
#include <string>

#include "hierarchy.hpp"
#include "panel.hpp"
#include "wide.hpp"

namespace eamg {

struct BatchWork {
  int K = 0;
  DevArena arena;
  // level-0 CG panels (FP64, colour-major, interleaved)
  double *x = nullptr, *r = nullptr, *z = nullptr, *p = nullptr, *q = nullptr, *bp = nullptr;
  double *part = nullptr, *scal = nullptr;
  double *scal_h = nullptr;   // pinned
  double *dense = nullptr;    // slices of the coarsest panel product
  // V-cycle panels per precision ([0] FP64, [1] FP32) and level: x, b, r
  bool have[2] = {false, false};
  std::vector<void *> vx[2], vb[2], vr[2];
  // right-hand sides of grouped sweep stages: levels that have some, if the memory holds them (else their
  // colours run one by one)
  std::vector<void *> vu[2];
  hipStream_t cap = nullptr;
  hipGraphExec_t g[2] = {nullptr, nullptr};
  bool tried[2] = {false, false};
  ~BatchWork() {
    for (hipGraphExec_t e : g)
      if (e) (void)hipGraphExecDestroy(e);
    if (cap) (void)hipStreamDestroy(cap);
    if (scal_h) (void)hipHostFree(scal_h);
  }
};

void destroy_batch(BatchWork *w) { delete w; }

namespace {

int panel_width(int m) {
  int K = 1;
  while (K < m) K <<= 1;
  return K;
}

int64_t level_dofs(const Level &L) { return int64_t(L.n) * L.bs; }

BatchWork *ensure_work(eamg_hierarchy *h, int K, bool f32) {
  if (h->batch && h->batch->K != K) {
    hip_check(hipDeviceSynchronize(), "sync");
    destroy_batch(h->batch);
    h->batch = nullptr;
  }
  if (!h->batch) {
    auto w = std::make_unique<BatchWork>();
    w->K = K;
    const Level &L0 = h->lv[0];
    const int64_t N = level_dofs(L0) * K;
    w->x = w->arena.alloc<double>(N);
    w->r = w->arena.alloc<double>(N);
    w->z = w->arena.alloc<double>(N);
    w->p = w->arena.alloc<double>(N);
    w->q = w->arena.alloc<double>(N);
    w->bp = w->arena.alloc<double>(N);
    const int nparts = std::max(pdot_blocks(N), pspmv_blocks(L0.Am, K));
    w->part = w->arena.alloc<double>(size_t(nparts) * K);
    w->scal = w->arena.alloc<double>(size_t(PS_COUNT) * K);
    w->dense = w->arena.alloc<double>(std::max<size_t>(
        1, h->tail_level >= 0 ? sym_panel_work_doubles(h->nT, K) : dense_panel_work_doubles(h->nL, K)));
    hip_check(hipHostMalloc(reinterpret_cast<void **>(&w->scal_h), sizeof(double) * PS_COUNT * K,
                            hipHostMallocDefault),
              "hipHostMalloc");
    h->batch = w.release();
  }
  BatchWork *w = h->batch;
  const int p = f32 ? 1 : 0;
  if (!w->have[p]) {
    const size_t vsz = f32 ? sizeof(float) : sizeof(double);
    const size_t nl = h->lv.size();
    w->vx[p].assign(nl, nullptr);
    w->vb[p].assign(nl, nullptr);
    w->vr[p].assign(nl, nullptr);
    w->vu[p].assign(nl, nullptr);
    for (size_t l = 0; l < nl; ++l) {
      const size_t n = size_t(level_dofs(h->lv[l])) * K * vsz;
      const bool coarsest = l + 1 == nl;
      // FP64 level 0 uses the CG panels r (right-hand side) and z (result) directly
      if (l > 0 || f32) {
        w->vx[p][l] = w->arena.alloc<char>(n);
        w->vb[p][l] = w->arena.alloc<char>(n);
      }
      if (!coarsest) w->vr[p][l] = w->arena.alloc<char>(n);
    }
    for (size_t l = 0; l < nl; ++l) {
      if (!h->lv[l].u) continue;
      const size_t n = size_t(level_dofs(h->lv[l])) * K * vsz;
      try {
        GroupRoom().take(n);
        w->vu[p][l] = w->arena.alloc<char>(n);
      } catch (const Failure &e) {
        if (e.code != EAMG_ERR_OOM) throw;
        (void)hipGetLastError();
      }
    }
    w->have[p] = true;
  }
  return w;
}

template <class T>
T *vp(void *v) {
  return static_cast<T *>(v);
}

// Whether stage k of a panel sweep runs as a group (u: the level's vu panel).  A launch costs 4 to 7 us beyond its blocks (more
// with more columns), a block its values at 3 TB/s and its K columns of the gathered panel at 8 TB/s
// (64^3, 32 columns, FP32: 10.5 and 22.8 us for colours of 42,000 and 146,000 blocks; 37x29x33, 8 columns,
// FP64: 22 us for the 130,000 blocks of an S); the group saves its colours' launches but one or two
// and adds the blocks of S, planned for a single vector.  64^3 x 32 FP32 82.7 -> 70.1 ms.
bool panel_group(const Level &L, const void *u, int k, bool fwd, int K, double vs) {
  if (!u || !L.is_group(k)) return false;
  const double launch = 4e-6 + 5e-8 * K;
  const double block = L.bs * L.bs * vs / 3e12 + L.bs * K * vs / 8e12;
  const double colours = L.cut[size_t(k) + 1] - L.cut[size_t(k)];
  const double launches = fwd && k == 0 ? 1.0 : 2.0;
  return launches * launch + double(L.gs_blocks[size_t(k)]) * block < colours * launch;
}

// The group matrix of stage k with its row team: a workgroup per row where its sub-teams find a block
// each in an average row.
SolveMat panel_smat(const Level &L, int k, bool fwd) {
  SolveMat S = fwd ? L.Sf : L.Sb;
  S.panel_waves = double(L.gs_blocks[size_t(k)]) >= 16.0 * (L.row1(k) - L.row0(k)) ? 4 : 1;
  return S;
}

// Stage k of the panel sweeps of level L (u: the level's vu panel).
template <class T>
hipError_t pfwd_stage(const Level &L, const SolveMat &A, const T *Dinv, int k, int K, const T *b, T *x, T *r,
                      T *u, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (panel_group(L, u, k, true, K, sizeof(T))) {
    if (k > 0) {
      e = launch_pgroup_rhs<T>(A, L.lo_end, L.row0(k), L.row1(k), K, b, x, u, s);
      if (e != hipSuccess) return e;
    }
    return launch_pgroup_fwd<T>(A, panel_smat(L, k, true), Dinv, L.row0(k), L.row1(k), K, k > 0 ? u : b, x, r, s);
  }
  for (int c = L.cut[size_t(k)]; c < L.cut[size_t(k) + 1] && e == hipSuccess; ++c)
    e = launch_pgs_fwd<T>(A, Dinv, L.color_ptr[c], L.color_ptr[c + 1], K, b, x, r, s);
  return e;
}
template <class T>
hipError_t pbwd_stage(const Level &L, const SolveMat &A, const T *Dinv, int k, int K, const T *b, T *x, T *u,
                      hipStream_t s) {
  hipError_t e = hipSuccess;
  if (panel_group(L, u, k, false, K, sizeof(T))) {
    e = launch_pgroup_rhs<T>(A, nullptr, L.row0(k), L.row1(k), K, b, x, u, s);
    if (e != hipSuccess) return e;
    return launch_pgroup_bwd<T>(panel_smat(L, k, false), Dinv, L.row0(k), L.row1(k), K, u, x, s);
  }
  for (int c = L.cut[size_t(k) + 1] - 1; c >= L.cut[size_t(k)] && e == hipSuccess; --c)
    e = launch_pgs_bwd<T>(A, Dinv, L.color_ptr[c], L.color_ptr[c + 1], K, b, x, s);
  return e;
}

template <class T>
void pvcycle_t(eamg_hierarchy *h, BatchWork *w, size_t l, const T *b, T *x, hipStream_t s) {
  const int K = w->K;
  const int pi = sizeof(T) == 4 ? 1 : 0;
  const std::string ty = type_name<T>();
  const double vs = sizeof(T);
  Level &L = h->lv[l];
  if (int(l) == h->tail_level) {
    const double by = double(sym_entries(h->nT)) * 8.0 + 2.0 * 8.0 * double(sym_panel_work_doubles(h->nT, K)) +
                      2.0 * h->nT * K * vs;
    timed(h, "dense tail", lvname(h, l, "k_dense_panel_sym<" + ty + ">"), by, s,
          [&] { return launch_dense_panel_sym<T>(h->nT, K, h->tailS, b, x, w->dense, s); });
    return;
  }
  if (l + 1 == h->lv.size()) {
    const double by = double(h->nL) * h->nL * 8.0 + 2.0 * h->nL * K * vs;
    timed(h, "coarsest", lvname(h, l, "k_dense_panel_mfma<" + ty + ">"), by, s,
          [&] { return launch_dense_panel<T>(h->nL, h->ldL, K, h->Ainv, b, x, w->dense, s); });
    return;
  }
  const int bs = L.bs;
  const T *Dinv = bufs<T>(L).Dinv;
  T *R = vp<T>(w->vr[pi][l]), *U = vp<T>(w->vu[pi][l]);
  const auto run = [&](bool fwd, auto &&stage) {
    const auto grouped = [&](int k) { return panel_group(L, U, k, fwd, K, vs); };
    const auto launches = [&](int k) { return !grouped(k) ? L.cut[size_t(k) + 1] - L.cut[size_t(k)] : fwd && k == 0 ? 1 : 2; };
    sweep<T>(h, l, fwd, "k_pgs_color", K, false, grouped, launches, stage, s);
  };
  run(true, [&](int k) { return pfwd_stage<T>(L, L.Am, Dinv, k, K, b, x, R, U, s); });
  timed(h, "presid_upper", lvname(h, l, "k_presid_upper<" + ty + ", " + std::to_string(bs) + ">"),
        launch_bytes(L.sh_resid, LK_RESID, bs, bs, vs, K), s,
        [&] { return launch_presid_upper<T>(L.panel_mat(L.pw_resid), K, x, R, s); });
  T *Cb = vp<T>(w->vb[pi][l + 1]);
  T *Cx = vp<T>(w->vx[pi][l + 1]);
  timed(h, "prestrict", lvname(h, l, "k_prect<" + ty + ", " + std::to_string(L.kc) + ", " + std::to_string(bs) + ">"),
        launch_bytes(L.sh_R, LK_RECT, L.kc, bs, vs, K), s,
        [&] { return launch_prect<T>(L.Rm, K, R, Cb, false, s); });
  pvcycle_t<T>(h, w, l + 1, Cb, Cx, s);
  timed(h, "pprolong", lvname(h, l, "k_prect<" + ty + ", " + std::to_string(bs) + ", " + std::to_string(L.kc) + ">"),
        launch_bytes(L.sh_P, LK_RECT_ACC, bs, L.kc, vs, K), s,
        [&] { return launch_prect<T>(L.Pm, K, Cx, x, true, s); });
  const SolveMat Mb = L.panel_mat(L.pw_bwd);
  run(false, [&](int k) { return pbwd_stage<T>(L, Mb, Dinv, k, K, b, x, U, s); });
}

// The level-0 panels of the FP32 V-cycle: R's FP32 copy (written with R), and Z.
float *panel_r32(BatchWork *w) { return vp<float>(w->vb[1][0]); }
float *panel_z32(BatchWork *w) { return vp<float>(w->vx[1][0]); }

// Z = V(R) for the K columns of the level-0 CG panels: FP32 from panel_r32 to panel_z32, else R to Z.
void pvcycle(eamg_hierarchy *h, BatchWork *w, bool f32, hipStream_t s) {
  if (f32)
    pvcycle_t<float>(h, w, 0, panel_r32(w), panel_z32(w), s);
  else
    pvcycle_t<double>(h, w, 0, w->r, w->z, s);
}

// part <- R.Z
void pdot_rz(eamg_hierarchy *h, BatchWork *w, bool f32, hipStream_t s) {
  const int64_t N = level_dofs(h->lv[0]) * w->K;
  const int nd = pdot_blocks(N);
  timed(h, "pdot", "k_pdot", (f32 ? 12.0 : 16.0) * N + 8.0 * nd * w->K, s, [&] {
    return f32 ? launch_pdot<float>(N, w->K, w->r, panel_z32(w), w->part, s)
               : launch_pdot<double>(N, w->K, w->r, w->z, w->part, s);
  });
}

// Q = A P, alpha, X += alpha P, R -= alpha Q, R.R and the stopping tests.
void pstep(eamg_hierarchy *h, BatchWork *w, bool f32, hipStream_t s) {
  const Level &L0 = h->lv[0];
  const int K = w->K;
  const int64_t N = level_dofs(L0) * K;
  const int nd = pdot_blocks(N), ns = pspmv_blocks(L0.Am, K);
  timed(h, "pspmv", tname("k_pspmv", L0.bs), launch_bytes(L0.sh_spmv, LK_SPMV, L0.bs, L0.bs, 8.0, K) + 8.0 * ns * K, s,
        [&] { return launch_pspmv(L0.Am, K, w->p, w->q, w->part, s); });
  timed(h, "preduce", "k_preduce", 8.0 * ns * K, s,
        [&] { return launch_preduce(ns, K, w->part, w->scal, PS_PQ, PRED_ALPHA, s); });
  timed(h, "pupdate_xr", "k_pupdate_xr", (f32 ? 52.0 : 48.0) * N + 8.0 * nd * K, s, [&] {
    return launch_pupdate_xr(N, K, w->scal, w->x, w->r, w->p, w->q, w->part, f32 ? panel_r32(w) : nullptr, s);
  });
  timed(h, "preduce", "k_preduce", 8.0 * nd * K, s,
        [&] { return launch_preduce(nd, K, w->part, w->scal, PS_RR, PRED_RR, s); });
}

// One batched PCG iteration after the stopping test (the columns that are still active).
void penqueue_iteration(eamg_hierarchy *h, BatchWork *w, bool precond, bool f32, hipStream_t s) {
  const int K = w->K;
  const int64_t N = level_dofs(h->lv[0]) * K;
  const int nd = pdot_blocks(N);
  if (precond)
    pvcycle(h, w, f32, s);
  else
    hip_check(launch_copy(N, w->r, w->z, s), "copy");
  pdot_rz(h, w, f32, s);
  timed(h, "preduce", "k_preduce", 8.0 * nd * K, s,
        [&] { return launch_preduce(nd, K, w->part, w->scal, PS_RZ, PRED_BETA, s); });
  timed(h, "pupdate_p", "k_pupdate_p", (f32 ? 20.0 : 24.0) * N, s, [&] {
    return f32 ? launch_pupdate_p<float>(N, K, w->scal, panel_z32(w), w->p, s)
               : launch_pupdate_p<double>(N, K, w->scal, w->z, w->p, s);
  });
  pstep(h, w, f32, s);
  hip_check(hipMemcpyAsync(w->scal_h, w->scal, sizeof(double) * PS_COUNT * K, hipMemcpyDeviceToHost, s),
            "copy");
}

void ptry_graph(eamg_hierarchy *h, BatchWork *w, bool f32) {
  w->tried[f32] = true;
  if (const char *e = std::getenv("EAMG_GRAPH"))
    if (std::atoi(e) == 0) return;
  if (!w->cap && hipStreamCreateWithFlags(&w->cap, hipStreamNonBlocking) != hipSuccess) {
    w->cap = nullptr;
    return;
  }
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(w->cap, hipStreamCaptureModeRelaxed) != hipSuccess) return;
  bool ok = true;
  try {
    penqueue_iteration(h, w, true, f32, w->cap);
  } catch (const Failure &) {
    ok = false;
  }
  if (hipStreamEndCapture(w->cap, &g) != hipSuccess || !ok) {
    if (g) (void)hipGraphDestroy(g);
    (void)hipGetLastError();
    return;
  }
  hipGraphExec_t ex = nullptr;
  if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) == hipSuccess) w->g[f32] = ex;
  (void)hipGraphDestroy(g);
  (void)hipGetLastError();
}

void pfetch(BatchWork *w, hipStream_t s) {
  hip_check(hipMemcpyAsync(w->scal_h, w->scal, sizeof(double) * PS_COUNT * w->K, hipMemcpyDeviceToHost, s),
            "copy");
  hip_check(hipStreamSynchronize(s), "sync");
}

bool any_active(const BatchWork *w) {
  for (int k = 0; k < w->K; ++k)
    if (w->scal_h[PS_ACTIVE * w->K + k] != 0.0) return true;
  return false;
}

// Solve the m <= 64 columns of one panel; returns whether all of them converged.
bool solve_panel(eamg_hierarchy *h, int m, const double *B, int64_t ld, double *X,
                 const eamg_solve_params &sp, hipStream_t s, eamg_solve_info *infos) {
  const int K = panel_width(m);
  const bool precond = sp.precond != EAMG_PRECOND_NONE;
  const bool f32 = sp.precond == EAMG_PRECOND_VCYCLE_FP32;
  BatchWork *w = ensure_work(h, K, f32);
  const Level &L0 = h->lv[0];
  const SolveMat &A = L0.Am;
  const int64_t N = level_dofs(L0) * K;
  const int nd = pdot_blocks(N);
  struct Events {
    hipEvent_t a = nullptr, b = nullptr;
    ~Events() {
      if (a) (void)hipEventDestroy(a);
      if (b) (void)hipEventDestroy(b);
    }
  } ev;
  hip_check(hipEventCreate(&ev.a), "event");
  hip_check(hipEventCreate(&ev.b), "event");
  hipEvent_t e0 = ev.a, e1 = ev.b;
  hip_check(hipEventRecord(e0, s), "event");
  hip_check(launch_pinit_scal(K, sp.rtol, sp.max_it, w->scal, s), "pinit");
  hip_check(launch_ppack(L0.n, L0.bs, K, m, L0.perm_d, h->dir, B, ld, w->bp, s), "ppack");
  hip_check(launch_pfinite(N, K, w->bp, w->scal, s), "pfinite");
  hip_check(launch_pdot<double>(N, K, w->bp, w->bp, w->part, s), "pdot");
  hip_check(launch_preduce(nd, K, w->part, w->scal, PS_BB, PRED_INIT, s), "preduce");
  if (sp.use_x0) {
    hip_check(launch_ppack(L0.n, L0.bs, K, m, L0.perm_d, h->dir, X, ld, w->x, s), "ppack");
    hip_check(launch_pspmv(A, K, w->x, w->q, nullptr, s), "pspmv");
    hip_check(launch_sub(N, w->bp, w->q, w->r, s), "sub");
  } else {
    hip_check(launch_fill(N, 0.0, w->x, s), "fill");
    hip_check(launch_copy(N, w->bp, w->r, s), "copy");
  }
  hip_check(launch_pdot<double>(N, K, w->r, w->r, w->part, s), "pdot");
  hip_check(launch_preduce(nd, K, w->part, w->scal, PS_RR0, PRED_STORE, s), "preduce");
  if (f32) hip_check(launch_convert<double, float>(N, w->r, panel_r32(w), s), "convert");
  if (precond)
    pvcycle(h, w, f32, s);
  else
    hip_check(launch_copy(N, w->r, w->z, s), "copy");
  if (f32)
    hip_check(launch_convert<float, double>(N, panel_z32(w), w->p, s), "convert");
  else
    hip_check(launch_copy(N, w->z, w->p, s), "copy");
  pdot_rz(h, w, f32, s);
  hip_check(launch_preduce(nd, K, w->part, w->scal, PS_RHO, PRED_RHO0, s), "preduce");
  // first iteration (p = z), then one graph replay per further iteration
  pstep(h, w, f32, s);
  pfetch(w, s);
  const bool graphs = precond && !h->prof_on;
  if (graphs && !w->tried[f32]) ptry_graph(h, w, f32);
  // every active column stops by MAXIT; the bound only guards the host loop
  for (int it = 1; any_active(w) && it <= sp.max_it; ++it) {
    if (graphs && w->g[f32]) {
      hip_check(hipGraphLaunch(w->g[f32], s), "graph launch");
      hip_check(hipStreamSynchronize(s), "sync");
    } else {
      penqueue_iteration(h, w, precond, f32, s);
      hip_check(hipStreamSynchronize(s), "sync");
    }
  }
  // true residuals, x of columns that never started, unpack
  hip_check(launch_pspmv(A, K, w->x, w->q, nullptr, s), "pspmv");
  hip_check(launch_sub(N, w->bp, w->q, w->z, s), "sub");
  hip_check(launch_pdot<double>(N, K, w->z, w->z, w->part, s), "pdot");
  hip_check(launch_preduce(nd, K, w->part, w->scal, PS_RZ, PRED_STORE, s), "preduce");
  hip_check(launch_pzero_unstarted(N, K, w->scal, w->x, s), "pzero");
  hip_check(launch_punpack(L0.n, L0.bs, K, m, L0.perm_d, w->x, X, ld, s), "punpack");
  hip_check(hipEventRecord(e1, s), "event");
  pfetch(w, s);
  float fms = 0.0f;
  hip_check(hipEventElapsedTime(&fms, e0, e1), "event");
  bool all = true;
  for (int k = 0; k < m; ++k) {
    const double *S = w->scal_h;
    auto at = [&](int slot) { return S[slot * K + k]; };
    const double bn = std::sqrt(at(PS_BB));
    const bool conv = at(PS_CONV) != 0.0;
    const bool bad = at(PS_BAD) != 0.0;
    all = all && conv && !bad;
    if (infos) {
      eamg_solve_info &inf = infos[k];
      inf.iterations = int32_t(at(PS_ITS));
      inf.rel_res = (bn > 0.0 && std::isfinite(bn)) ? std::sqrt(at(PS_RR)) / bn : 0.0;
      inf.rel_res_true = (bn > 0.0 && std::isfinite(bn)) ? std::sqrt(at(PS_RZ)) / bn : 0.0;
      if (bad && at(PS_ITS) == 0.0) inf.rel_res = inf.rel_res_true = 0.0;
      inf.ms = fms;
      inf.status = bad ? EAMG_ERR_BREAKDOWN : conv ? EAMG_OK : EAMG_NOT_CONVERGED;
    }
  }
  return all;
}

// Time one launch sequence on the stream (events), median of reps.
template <class F>
double time_ms(hipStream_t s, int reps, F &&f) {
  hipEvent_t a, b;
  hip_check(hipEventCreate(&a), "event");
  hip_check(hipEventCreate(&b), "event");
  std::vector<float> t;
  for (int r = 0; r < reps; ++r) {
    hip_check(hipEventRecord(a, s), "event");
    f();
    hip_check(hipEventRecord(b, s), "event");
    hip_check(hipEventSynchronize(b), "sync");
    float ms = 0.0f;
    hip_check(hipEventElapsedTime(&ms, a, b), "event");
    t.push_back(ms);
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  std::sort(t.begin(), t.end());
  return t[t.size() / 2];
}

}  // namespace

namespace {

// Work panels of a level below the tail's first: right-hand side, solution and residual.
struct WideLevel {
  WidePanel b, x, r;
};

// x = V_l(b) for K columns on level l (b.p == nullptr: columns j0 .. j0 + K - 1 of the identity,
// and x is zero on entry).  The forward sweep of an identity right-hand side stays at or below
// the diagonal, so each colour takes only the columns that reach its rows; r is zeroed for the
// rest.  The result's columns beyond the diagonal are its rows (V is symmetric), so the backward
// sweep leaves them too: a row needs the later rows' new values, theirs reach at least as far, and
// the earlier rows' old ones, which are complete.  x ends up valid on and below the diagonal only.
void wide_vcycle(eamg_hierarchy *h, std::vector<WideLevel> &w, size_t l, WidePanel b, int j0, WidePanel x,
                 int K, hipStream_t s) {
  Level &L = h->lv[l];
  if (l + 1 == h->lv.size()) {
    hip_check(launch_wide_dense(h->nL, h->ldL, h->Ainv, K, b, x, s), "wide coarsest");
    return;
  }
  const WidePanel r = w[l].r;
  // columns of the launch that reach rows before r1
  const auto reach = [&](int r1) {
    if (b.p) return K;
    const int64_t d = int64_t(r1) * L.bs - j0;
    return int(std::max<int64_t>(0, std::min<int64_t>(K, (d + 1) / 2 * 2)));
  };
  if (!b.p) hip_check(launch_fill(level_dofs(L) * r.ld, 0.0, r.p, s), "fill");
  for (int c = 0; c < L.ncolors; ++c) {
    const int r0 = L.color_ptr[c], r1 = L.color_ptr[c + 1];
    hip_check(launch_wide_fwd(L.Am, L.Dinv, r0, r1, reach(r1), b, j0, x, r, s), "wide fwd");
  }
  hip_check(launch_wide_resid(L.Am, K, x, r, s), "wide resid");
  WideLevel &C = w[l + 1];
  hip_check(launch_wide_rect(L.Rm, K, r, C.b, false, s), "wide restrict");
  wide_vcycle(h, w, l + 1, C.b, 0, C.x, K, s);
  hip_check(launch_wide_rect(L.Pm, K, C.x, x, true, s), "wide prolong");
  for (int c = L.ncolors - 1; c >= 0; --c) {
    const int r0 = L.color_ptr[c], r1 = L.color_ptr[c + 1];
    hip_check(launch_wide_bwd(L.Am, L.Dinv, r0, r1, reach(r1), b, j0, x, s), "wide bwd");
  }
}

}  // namespace

DenseTail make_dense_tail(eamg_hierarchy *h, size_t t, DevArena &out, hipStream_t s) {
  if (t == 0 || t + 1 >= h->lv.size()) fail(EAMG_ERR_INVALID_ARG, "dense tail must start above the coarsest level, below the finest");
  const Level &Lt = h->lv[t];
  const int n = Lt.n * Lt.bs;
  if (n > kMaxCoarsestDofs) fail(EAMG_ERR_INVALID_ARG, "dense tail too large");
  // columns per pass: few, wide passes fill the chip on levels of a few dozen rows per colour;
  // kWideCols bounds the residual panel to half of the largest tail matrix.  Each pass's solution
  // panel is its columns of T itself.
  constexpr int kWideCols = 8192;
  const int ld = dense_ld(n);
  double *T = out.alloc<double>(size_t(ld) * ld);
  int K = std::min(ld, kWideCols);
  // EAMG_WIDE_COLS: the columns of a pass, as if the memory held no more (for tests)
  if (const char *e = std::getenv("EAMG_WIDE_COLS")) K = std::min(ld, std::max(2, (std::atoi(e) + 1) / 2 * 2));
  std::unique_ptr<DevArena> work;
  std::vector<WideLevel> w(h->lv.size());
  for (;; K = (K / 2 + 1) / 2 * 2) {
    // narrower passes where the panels do not fit in the free memory
    work = std::make_unique<DevArena>();
    try {
      for (size_t l = t; l < h->lv.size(); ++l) {
        auto panel = [&] { return WidePanel{work->alloc<double>(size_t(level_dofs(h->lv[l])) * K), K}; };
        if (l > t) {
          w[l].b = panel();
          w[l].x = panel();
        }
        if (l + 1 < h->lv.size()) w[l].r = panel();
      }
      break;
    } catch (const Failure &e) {
      if (e.code != EAMG_ERR_OOM || K <= 128) throw;
      (void)hipGetLastError();
    }
  }
  hip_check(launch_fill(int64_t(ld) * ld, 0.0, T, s), "fill");
  for (int j0 = 0; j0 < n; j0 += K)
    wide_vcycle(h, w, t, WidePanel{}, j0, WidePanel{T + j0, ld}, std::min(K, (n - j0 + 1) / 2 * 2), s);
  DenseTail d;
  d.T = T;
  d.n = n;
  d.ld = ld;
  hip_check(hipStreamSynchronize(s), "sync");
  return d;
}

void build_dense_tail(eamg_hierarchy *h, size_t t, hipStream_t s) {
  DevArena full;
  const DenseTail d = make_dense_tail(h, t, full, s);
  h->nT = d.n;
  h->tailS = h->arena.alloc<double>(sym_entries(d.n));
  hip_check(launch_pack_lower<double>(d.n, d.ld, d.T, h->tailS, s), "pack tail");
  if (h->prm.vcycle_fp32 && h->prm.dense_tail_fp32) {
    h->tailS32 = h->arena.alloc<float>(sym_entries(d.n));
    hip_check(launch_pack_lower<float>(d.n, d.ld, d.T, h->tailS32, s), "pack tail f32");
  }
  h->tailW = h->arena.alloc<double>(sym_work_doubles(d.n));
  hip_check(hipStreamSynchronize(s), "sync");
  h->tail_level = int(t);
}

// Panel launch shapes measured on the hierarchy's own matrices for K columns (FP64 V-cycle
// kernels): per level, the sweep + upper-residual sequence and each transfer with one or four
// wavefronts per row; the faster is kept in SolveMat::panel_waves.  Returns the summed time of the
// tuned kernels before / after (ms).
std::pair<double, double> tune_panels(eamg_hierarchy *h, int K, hipStream_t s) {
  BatchWork *w = ensure_work(h, K, false);
  const int reps = 5;
  double before = 0.0, after = 0.0;
  for (size_t l = 0; l + 1 < h->lv.size(); ++l) {
    if (h->tail_level >= 0 && int(l) >= h->tail_level) break;   // applied as the dense tail
    Level &L = h->lv[l];
    double *b = l == 0 ? w->r : vp<double>(w->vb[0][l]);
    double *x = l == 0 ? w->z : vp<double>(w->vx[0][l]);
    double *r = vp<double>(w->vr[0][l]), *u = vp<double>(w->vu[0][l]);
    double *cb = vp<double>(w->vb[0][l + 1]);
    double *cx = vp<double>(w->vx[0][l + 1]);
    const int64_t nv = level_dofs(L) * K, nc = level_dofs(h->lv[l + 1]) * K;
    for (double *v : {b, x, r}) hip_check(launch_fill(nv, 0.0, v, s), "fill");
    for (double *v : {cb, cx}) hip_check(launch_fill(nc, 0.0, v, s), "fill");
    // forward sweep, residual update and backward sweep tuned apart (each reads a different part
    // of the rows), then the transfers
    auto fwd = [&] {
      for (int k = 0; k < L.stages(); ++k)
        hip_check(pfwd_stage<double>(L, L.Am, L.Dinv, k, K, b, x, r, u, s), "pgs");
    };
    auto resid = [&] {
      hip_check(launch_presid_upper<double>(L.panel_mat(L.pw_resid), K, x, r, s), "presid");
    };
    auto bwd = [&] {
      const SolveMat Mb = L.panel_mat(L.pw_bwd);
      for (int k = L.stages() - 1; k >= 0; --k)
        hip_check(pbwd_stage<double>(L, Mb, L.Dinv, k, K, b, x, u, s), "pgs");
    };
    auto restrict_ = [&] { hip_check(launch_prect<double>(L.Rm, K, r, cb, false, s), "prect"); };
    auto prolong = [&] { hip_check(launch_prect<double>(L.Pm, K, cx, x, true, s), "prect"); };
    L.pw_resid = L.pw_bwd = 0;
    struct Item {
      int *pw;   // the choice: 0 (built-in / the forward sweep's), 1 or 4 wavefronts per row
      std::function<void()> run;
    } items[] = {{&L.Am.panel_waves, fwd}, {&L.pw_resid, resid}, {&L.pw_bwd, bwd},
                 {&L.Rm.panel_waves, restrict_}, {&L.Pm.panel_waves, prolong}};
    for (Item &it : items) {
      const int orig = *it.pw;
      int best_w = orig;
      const double t0 = time_ms(s, reps, it.run);
      before += t0;
      double best = t0;
      for (int wv : {1, 4}) {
        *it.pw = wv;
        const double t = time_ms(s, reps, it.run);
        if (t < best) {
          best = t;
          best_w = wv;
        }
      }
      *it.pw = best_w;
      after += best;
    }
  }
  // captured iteration graphs hold the old launch shapes
  for (int p = 0; p < 2; ++p) {
    if (w->g[p]) (void)hipGraphExecDestroy(w->g[p]);
    w->g[p] = nullptr;
    w->tried[p] = false;
  }
  return {before, after};
}

}  // namespace eamg

using namespace eamg;

extern "C" eamg_status eamg_solve_batch(eamg_hierarchy *h, int32_t nrhs, const double *B_dev,
                                        int64_t ld, double *X_dev, const eamg_solve_params *params,
                                        void *stream, eamg_solve_info *infos) {
  bool all = true;
  const eamg_status st = guarded([&] {
    if (!h || !B_dev || !X_dev) fail(EAMG_ERR_INVALID_ARG, "NULL argument");
    reject_fused(h);
    if (nrhs < 1) fail(EAMG_ERR_INVALID_ARG, "nrhs must be >= 1");
    const int64_t ndof = level_dofs(h->lv[0]);
    if (ld < ndof) fail(EAMG_ERR_INVALID_ARG, "ld must be >= n*dim");
    {
      const char *b0 = reinterpret_cast<const char *>(B_dev);
      const char *x0 = reinterpret_cast<const char *>(X_dev);
      const int64_t span = (int64_t(nrhs - 1) * ld + ndof) * int64_t(sizeof(double));
      if (b0 < x0 + span && x0 < b0 + span) fail(EAMG_ERR_INVALID_ARG, "B and X may not overlap");
    }
    eamg_solve_params sp;
    eamg_default_solve_params(&sp);
    if (params) sp = *params;
    if (sp.max_it < 1) fail(EAMG_ERR_INVALID_ARG, "max_it must be >= 1");
    if (!(sp.rtol >= 0.0)) fail(EAMG_ERR_INVALID_ARG, "rtol must be >= 0");
    if (sp.precond < EAMG_PRECOND_NONE || sp.precond > EAMG_PRECOND_VCYCLE_FP32)
      fail(EAMG_ERR_INVALID_ARG, "precond must be 0, 1 or 2");
    if (sp.precond == EAMG_PRECOND_VCYCLE_FP32 && !h->prm.vcycle_fp32)
      fail(EAMG_ERR_INVALID_ARG, "FP32 V-cycle needs setup with vcycle_fp32 = 1");
    hipStream_t s = static_cast<hipStream_t>(stream);
    constexpr int kMaxPanel = 64;
    for (int c0 = 0; c0 < nrhs; c0 += kMaxPanel) {
      const int m = std::min(kMaxPanel, nrhs - c0);
      all = solve_panel(h, m, B_dev + int64_t(c0) * ld, ld, X_dev + int64_t(c0) * ld, sp, s,
                        infos ? infos + c0 : nullptr) && all;
    }
  });
  if (st == EAMG_OK && !all) {
    g_last_error = "some right-hand sides did not converge";
    return EAMG_NOT_CONVERGED;
  }
  return st;
}
