// Launchers of the gfx950 kernels (kernels.hip).  All pointers are device pointers; every
// launcher enqueues on `s` and returns the launch status.
//
// Solve-phase matrices (SolveMat) are block CSR with row-major blocks stored one after another:
// value (r, c) of block q lives at val[q * BR * BC + r * BC + c], so a lane that owns a block
// reads it as a few wide loads of consecutive bytes (measured on a level-1-shaped 6 x 6 FP32
// matrix: 11 % more bandwidth than element planes, where value (r, c) of every block forms one
// array).  Rows of every level are numbered colour-major, so a colour is a contiguous row range
// and, within a row, the columns below the row index are exactly the neighbours of lower colour.
// diag[i] is the position of the diagonal block of row i.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eamg {

// ---- setup -------------------------------------------------------------------------------
// Dirichlet rows / columns of A_N -> identity / zero blocks (AoS row-major blocks).
hipError_t launch_dirichlet(int n, int bs, const int64_t *rp, const int *col, double *val,
                            const uint8_t *dir, hipStream_t s);

// Dinv[i] = pinv_tau(A_ii) for every row (AoS blocks, natural numbering).
hipError_t launch_diag_pinv(int n, int bs, const int64_t *rp, const int *col, const double *val,
                            double *Dinv, double tau, hipStream_t s);

struct PsArgs {
  int n, k, bs;
  const int *type;        // ROW_S / ROW_A / ROW_D
  const int *agg;         // coarse vertex or -1
  const double *x;        // fine positions n*3
  const double *xc;       // coarse positions nc*3
  const int64_t *Prp;     // P_s pattern
  const int *Pcol;
  const int64_t *Arp;     // A_l (AoS bs x bs)
  const int *Acol;
  const double *Aval;
  const int64_t *Fptr;    // filtered neighbours of edge-matrix rows
  const int *Fvtx, *Fedge;
  const double *E;        // edge weights m*k*k
  double omega, tau;
  double *Pval;           // out: nnz(P) * bs * k (AoS)
};
hipError_t launch_ps_numeric(const PsArgs &a, hipStream_t s);

// C = A * B on a given pattern (AoS blocks: A ra x ca, B ca x cb, C ra x cb).
// crow[q] = block row of entry q of C.
hipError_t launch_spgemm_numeric(int64_t nnzC, int ra, int ca, int cb, const int *crow,
                                 const int *Ccol, const int64_t *Arp, const int *Acol,
                                 const double *Aval, const int64_t *Brp, const int *Bcol,
                                 const double *Bval, double *Cval, hipStream_t s);

// out[q] = transpose(in[src[q]]) for r x c input blocks (AoS).
hipError_t launch_transpose_blocks(int64_t nnz, int r, int c, const int64_t *src, const double *in,
                                   double *out, hipStream_t s);

// Block gather: out[q * bsz + e] = in[src[q] * bsz + e].
hipError_t launch_gather_blocks(int64_t nnz, int bsz, const int64_t *src, const double *in, double *out,
                                hipStream_t s);

// AoS -> AoS row gather: out[r * bsz + e] = in[perm[r] * bsz + e].
hipError_t launch_gather_rows(int n, int bsz, const int *perm, const double *in, double *out,
                              hipStream_t s);

// ---- solve -------------------------------------------------------------------------------
constexpr int kBlock = 256;          // threads per workgroup of the solve kernels
constexpr double kWideRowBlocks = 96; // square matrices with longer average rows: group = kBlock

struct SolveMat {
  // group: lanes per row (a power of two <= 64), or 128 / kBlock for two wavefronts / a whole
  // workgroup per row (square matrices with diag only)
  int n_rows = 0, n_cols = 0, br = 0, bc = 0, group = 16;
  // lanes per row of the backward sweep (whole rows), or 0 for `group` (forward sweep and the
  // residual update read about half of each row)
  int group_bwd = 0;
  // panel kernels: wavefronts per row (1 or 4), or 0 for the built-in choice
  int panel_waves = 0;
  int64_t nnz = 0;
  const int *rp = nullptr;   // int32 row offsets (nnz < 2^31 for one level)
  const int *col = nullptr;
  const double *val = nullptr;
  const float *val32 = nullptr;  // FP32 copy of val (FP32 V-cycle), or nullptr
  const int *diag = nullptr; // square matrices only
  // Square colour-major level matrices also hold the blocks left of the diagonal, the blocks
  // right of it and the diagonal blocks each in storage of their own (row offsets, columns,
  // blocks; the diagonal block of row i is block i of dg_val), so that the forward sweep and
  // the residual update, which read one side of every row, stream contiguous memory instead of
  // touching partly used cache lines at both ends of every row segment.
  const int *lo_rp = nullptr, *lo_col = nullptr;
  const double *lo_val = nullptr;
  const float *lo_val32 = nullptr;
  int64_t lo_nnz = 0;
  const int *up_rp = nullptr, *up_col = nullptr;
  const double *up_val = nullptr;
  const float *up_val32 = nullptr;
  int64_t up_nnz = 0;
  const double *dg_val = nullptr;   // nnz = n_rows
  const float *dg_val32 = nullptr;
};

// y = A x ; if part != nullptr also writes per-workgroup partial sums of x.y (spmv_blocks(A)
// entries)
hipError_t launch_spmv(const SolveMat &A, const double *x, double *y, double *part, hipStream_t s);
int spmv_blocks(const SolveMat &A);
// The V-cycle kernels are instantiated for T = double (values SolveMat::val) and T = float
// (values SolveMat::val32); they accumulate in T.
// Forward colour sweep with x = 0 initially on rows [r0, r1):
//   t = b_i - sum_{j < i} A_ij x_j ; x_i = Dinv_i t ; r_i = t - A_ii x_i
template <class T>
hipError_t launch_gs_fwd(const SolveMat &A, const T *Dinv, int r0, int r1, const T *b, T *x, T *r,
                         hipStream_t s);
// r_i -= sum_{j > i} A_ij x_j on rows [r0, r1) (completes r = b - A x after the forward sweep).
template <class T>
hipError_t launch_resid_upper(const SolveMat &A, int r0, int r1, const T *x, T *r, hipStream_t s);
// Backward colour sweep on rows [r0, r1): x_i += Dinv_i (b_i - sum_j A_ij x_j).
template <class T>
hipError_t launch_gs_bwd(const SolveMat &A, const T *Dinv, int r0, int r1, const T *b, T *x,
                         hipStream_t s);
// Grouped sweep stages (SweepPlan, structure.hpp) on rows [r0, r1):
//   launch_group_rhs: u_i = b_i - sum over the row's couplings outside the group of A_ij x_j; forward:
//     the blocks left of the diagonal up to lo_end[i] (those inside the group are left out, and
//     the later rows' x is zero); backward (lo_end null): the whole row, so that u = b - A x.
//   launch_group_fwd: t_i = u_i - sum_j S_ij u_j; x_i = Dinv_i t_i; r_i = t_i - A_ii x_i.
//   launch_group_bwd: t_i = u_i - sum_j S_ij u_j; x_i += Dinv_i t_i.
template <class T>
hipError_t launch_group_rhs(const SolveMat &A, const int *lo_end, int r0, int r1, const T *b, const T *x,
                            T *u, hipStream_t s);
template <class T>
hipError_t launch_group_fwd(const SolveMat &A, const SolveMat &S, const T *Dinv, int r0, int r1,
                            const T *u, T *x, T *r, hipStream_t s);
template <class T>
hipError_t launch_group_bwd(const SolveMat &S, const T *Dinv, int r0, int r1, const T *u, T *x,
                            hipStream_t s, const double *cg_r = nullptr, double *rz = nullptr);
// Workgroups of a group's launch over rows [r0, r1), and with rz (launch_group_bwd) its partials of
// the CG's r.z there: cg_r times the new x.
int group_blocks(const SolveMat &S, int r0, int r1);
// One rank of a group matrix, rows[0 .. nrows): row i's couplings inside the group are the positions
// [q0[i], q1[i]) of A (col, val, FP64 blocks in the solve numbering), and
//   S_ik = sum over those q, j = col[q], of A_q Dinv_j ([j == k] I - S_jk)
// for the row's columns k in S (rp, col of `longest` entries at most; val is written).
struct GroupRank {
  const int *rows;
  int nrows;
  const int *q0, *q1;
  const int *rp, *col;
  double *val;
};
// A rank of the forward and one of the backward matrix.
hipError_t launch_group_fill(const GroupRank &fwd, const GroupRank &bwd, int longest, int bs, const int *col,
                             const double *val, const double *Dinv, hipStream_t s);
// y = M x (rectangular, overwrite) or y += M x (accumulate = true).
template <class T>
hipError_t launch_rect(const SolveMat &M, const T *x, T *y, bool accumulate, hipStream_t s);
// out[i] = D(in[i])
template <class S, class D>
hipError_t launch_convert(int64_t n, const S *in, D *out, hipStream_t s);
// Block gather to FP32: out[q * bsz + e] = float(in[src[q] * bsz + e]).
hipError_t launch_gather_blocks_f32(int64_t nnz, int bsz, const int64_t *src, const double *in,
                                    float *out, hipStream_t s);

// Vector operations with deterministic reductions; grid size fixed by the length.
int dot_blocks(int64_t n);
// part <- partials of a.b (b in double, or in float: the FP32 V-cycle's output, each value
// converted exactly)
hipError_t launch_dot(int64_t n, const double *a, const double *b, double *part, hipStream_t s);
hipError_t launch_dot(int64_t n, const double *a, const float *b, double *part, hipStream_t s);
// Sum of the partials into scal[slot].
hipError_t launch_reduce(int nparts, const double *part, double *scal, int slot, hipStream_t s);
// p = z + beta p (z in double or float), beta = r.z / scal[SC_RHO], r.z summed from the partials in
// `part` by every workgroup alike; also stores SC_RZ and SC_BETA.
hipError_t launch_update_p(int64_t n, double *scal, const double *z, double *p, int nparts,
                           const double *part, hipStream_t s);
hipError_t launch_update_p(int64_t n, double *scal, const float *z, double *p, int nparts,
                           const double *part, hipStream_t s);
// x += alpha p ; r -= alpha q ; part <- partials of r.r, alpha = scal[SC_RZ] / p.q, p.q summed from the
// npq partials in `pq` (npq = 0: scal[SC_PQ]); also stores SC_PQ, SC_ALPHA and SC_RHO = SC_RZ.  With
// r32, also r32 = float(r) (the next FP32 V-cycle's right-hand side).  Once scal[SC_DONE] is set, x and
// r stay as they are.  With pold, pold = p (launch_spmv_dir's direction).  With ring, one workgroup
// does all of it and publishes (launch_publish), without partials: up to kOneBlock entries, from where
// the launch that publishes is cheaper than one workgroup's longer loop (elasticity cubes: 375 dofs
// 102.2 -> 97.6 us a solve, 1,029 dofs 530 -> 518, 3,993 dofs 854, not 865).
constexpr int64_t kOneBlock = 1536;
hipError_t launch_update_xr(int64_t n, double *scal, double *x, double *r, const double *p,
                            const double *q, double *part, int npq, const double *pq, hipStream_t s,
                            float *r32 = nullptr, double *pold = nullptr, double *ring = nullptr);
// p' = z + beta p in pn and q = A p', beta as in launch_update_p (from the nparts partials in rz);
// part <- partials of p'.q.  For up to kDirEntries entries, where the p update's launch costs more than
// the rows' second gather (solves of elasticity cubes of 1,029 dofs 530 -> 523 us, 3,993 dofs 854 ->
// 811, 14,739 dofs 2,039 -> 2,021, 41,472 dofs 4,505 -> 4,487; scalar 262,000 dofs 7.66 ms, not 7.87).
constexpr int64_t kDirEntries = 1 << 16;
template <class TZ>
hipError_t launch_spmv_dir(const SolveMat &A, double *scal, const TZ *z, const double *p, double *pn, double *q,
                           int nparts, const double *rz, double *part, hipStream_t s);
// Partial counts up to this many are summed by the kernel that uses the sum.
constexpr int kInlineParts = 1024;
// End of an iteration: SC_RR from the partials, SC_ITER + 1, SC_DONE if sqrt(r.r) <= SC_RTOL sqrt(SC_BB),
// then the scalars published in ring entry SC_ITER mod kRing (host memory; kRecord doubles, the last
// one, the iteration's number, stored after the others).
constexpr int kRing = 4, kRecord = 16;
hipError_t launch_publish(int nparts, const double *part, double *scal, double *ring, hipStream_t s);
// Start of a solve: bp = the right-hand side b in solve order (as launch_perm_in); with x also x = 0,
// r = bp and (r32) its FP32 copy; scal := 0 but SC_RTOL, SC_BB = bp.bp and SC_NONFINITE = whether an
// entry of bp is not finite.  part, bad: dot_blocks(n) entries each.
hipError_t launch_start(int64_t n, int bs, const int *perm, const uint8_t *mask, const double *b, double *bp,
                        double *x, double *r, float *r32, double rtol, double *part, double *bad, double *scal,
                        hipStream_t s);
// p = z; part <- partials of r.z
template <class TZ>
hipError_t launch_start_p(int64_t n, const TZ *z, const double *r, double *p, double *part, hipStream_t s);
// End of a solve: out = x in natural order; part <- partials of |b - q|^2
hipError_t launch_finish(int64_t n, int bs, const int *perm, const double *x, const double *b, const double *q,
                         double *out, double *part, hipStream_t s);
// y = a - b
hipError_t launch_sub(int64_t n, const double *a, const double *b, double *y, hipStream_t s);
hipError_t launch_copy(int64_t n, const double *a, double *y, hipStream_t s);
// out[r*bs+c] = mask[perm[r]] ? 0 : in[perm[r]*bs+c]   (natural -> colour-major, Dirichlet zeroed)
hipError_t launch_perm_in(int n, int bs, const int *perm, const uint8_t *mask, const double *in,
                          double *out, hipStream_t s);
// out[perm[r]*bs+c] = in[r*bs+c]   (colour-major -> natural)
hipError_t launch_perm_out(int n, int bs, const int *perm, const double *in, double *out,
                           hipStream_t s);
hipError_t launch_fill(int64_t n, double v, double *a, hipStream_t s);

// Scalar slots on the device.
enum Scalar : int {
  SC_RHO = 0, SC_PQ = 1, SC_RR = 2, SC_ALPHA = 3, SC_BETA = 4, SC_RZ = 5, SC_BB = 6,
  SC_BAD = 7, SC_NONFINITE = 8, SC_DONE = 9, SC_RTOL = 10, SC_ITER = 11, SC_COUNT = 15
};

}  // namespace eamg
