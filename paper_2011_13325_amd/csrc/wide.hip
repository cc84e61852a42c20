// Wide-panel V-cycle kernels for gfx950 (layouts in wide.hpp).
//
// A workgroup owns one block row and 128 columns (two per lane); its four wavefronts share the row's
// blocks and their sums meet in LDS.  A block is the same for all lanes, so the compiler reads it through
// scalar loads and every FMA takes its matrix value from a scalar register; the panel rows come as
// 16-byte loads, 1 KB per wavefront.  Bound: the chain of a wavefront through its blocks (72 scalar
// registers each, so one at a time: column index, panel rows and scalar block, then FMAs), with the
// panel rows from L2 and the Infinity Cache behind it.  Against 64-column panels (a row team summing
// lane parts, one panel after another: 9 to 13 us for each of 2 x colours x n / 64 launches) the tail of
// a 21^3 cube with inclusions (15,200 dofs on its first level) took 49 ms instead of 475 ms with a
// wavefront per row and 512 columns a workgroup; the backward sweep on the columns up to the diagonal
// 43, each XCD on neighbouring workgroups 38, the rows shared by four wavefronts 29.  Fewer columns a
// pass only repeat the chain: another tail of that mesh, of 15,444 dofs, takes 49 ms in passes of 8192
// columns, 57 of 4096, 81 of 2048.
#include "wide.hpp"

namespace eamg {
namespace {

constexpr int kWB = 256;              // threads per workgroup
constexpr int kWaveCols = 128;        // columns per wavefront
constexpr int kWaves = kWB / 64;

inline unsigned wide_slices(int K, int cols) { return unsigned((K + cols - 1) / cols); }

// Row and first column of this lane, rows x slices workgroups: workgroup b runs on XCD b mod 8, which
// takes one contiguous run of them, rows first, so that the panel rows that neighbours share come
// through one L2.
struct Place {
  int row, c0;
};
template <int COLS>   // columns of a workgroup, two per lane
__device__ inline Place place(int rows) {
  const int nb = int(gridDim.x), b = int(blockIdx.x);
  const int x = b & 7, q = nb >> 3, rem = nb & 7;
  const int l = x * q + min(x, rem) + (b >> 3);
  return {l % rows, l / rows * COLS + int(threadIdx.x) * 2 % COLS};
}

__device__ inline double2 ld2(const double *p) { return *reinterpret_cast<const double2 *>(p); }

// acc += sum over blocks p in [p0, p1) of M_p X_col(p), this lane's two columns of X at `x`.
template <int BR, int BC>
__device__ inline void wide_accumulate(int p0, int p1, const int *__restrict__ col,
                                       const double *__restrict__ val, const double *__restrict__ x,
                                       int64_t ldx, double2 (&acc)[BR]) {
#pragma unroll 2
  for (int p = p0; p < p1; ++p) {
    const double *xr = x + int64_t(col[p]) * BC * ldx;
    const double *a = val + int64_t(p) * (BR * BC);
    double2 xv[BC];
#pragma unroll
    for (int c = 0; c < BC; ++c) xv[c] = ld2(xr + c * ldx);
#pragma unroll
    for (int r = 0; r < BR; ++r)
#pragma unroll
      for (int c = 0; c < BC; ++c) {
        acc[r].x = fma(a[r * BC + c], xv[c].x, acc[r].x);
        acc[r].y = fma(a[r * BC + c], xv[c].y, acc[r].y);
      }
  }
}

// The row's sums: each wavefront takes a contiguous share of its blocks, the shares meet in LDS in
// wavefront order.  True on wavefront 0, which holds the sums; the others are done.
template <int BR, int BC>
__device__ inline bool wide_row(int p0, int p1, const int *__restrict__ col, const double *__restrict__ val,
                                const double *__restrict__ x, int64_t ldx, double2 (&acc)[BR]) {
  __shared__ double2 sh[kWaves - 1][BR][64];
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = int(threadIdx.x) & 63;
  const int share = (p1 - p0 + kWaves - 1) / kWaves;
#pragma unroll
  for (int q = 0; q < BR; ++q) acc[q] = make_double2(0.0, 0.0);
  wide_accumulate<BR, BC>(min(p1, p0 + w * share), min(p1, p0 + (w + 1) * share), col, val, x, ldx, acc);
  if (w > 0)
#pragma unroll
    for (int q = 0; q < BR; ++q) sh[w - 1][q][lane] = acc[q];
  __syncthreads();
  if (w > 0) return false;
#pragma unroll
  for (int k = 0; k < kWaves - 1; ++k)
#pragma unroll
    for (int q = 0; q < BR; ++q) {
      const double2 v = sh[k][q][lane];
      acc[q].x += v.x;
      acc[q].y += v.y;
    }
  return true;
}

// Right-hand side of dof `d` in this lane's columns: a panel row, or the identity's columns from j0.
__device__ inline double2 rhs_pair(const double *b, int64_t ldb, int64_t d, int c0, int j0) {
  if (b) return ld2(b + d * ldb + c0);
  return make_double2(d == j0 + c0 ? 1.0 : 0.0, d == j0 + c0 + 1 ? 1.0 : 0.0);
}

// One colour row of the block Gauss-Seidel sweeps (see launch_wide_fwd / launch_wide_bwd).
template <int B, bool FWD>
__global__ __launch_bounds__(kWB) void k_wide_gs(int r0, int rows, int K, const int *__restrict__ rp,
                                                 const int *__restrict__ col,
                                                 const double *__restrict__ val,
                                                 const double *__restrict__ dval,
                                                 const double *__restrict__ Dinv,
                                                 const double *b, int64_t ldb, int j0, double *x,
                                                 int64_t ldx, double *r, int64_t ldr) {
  const Place at = place<kWaveCols>(rows);
  const int i = r0 + at.row, c0 = min(at.c0, K - 2);   // lanes past K repeat the last columns' work
  double2 acc[B];
  if (!wide_row<B, B>(rp[i], rp[i + 1], col, val, x + c0, ldx, acc) || at.c0 >= K) return;
  const int64_t d0 = int64_t(i) * B;
  const double *Di = Dinv + d0 * B;
  double2 t[B], z[B];
#pragma unroll
  for (int q = 0; q < B; ++q) {
    const double2 bq = rhs_pair(b, ldb, d0 + q, c0, j0);
    t[q] = make_double2(bq.x - acc[q].x, bq.y - acc[q].y);
  }
#pragma unroll
  for (int q = 0; q < B; ++q) {
    z[q] = make_double2(0.0, 0.0);
#pragma unroll
    for (int c = 0; c < B; ++c) {
      z[q].x = fma(Di[q * B + c], t[c].x, z[q].x);
      z[q].y = fma(Di[q * B + c], t[c].y, z[q].y);
    }
  }
#pragma unroll
  for (int q = 0; q < B; ++q) {
    double2 *xq = reinterpret_cast<double2 *>(x + (d0 + q) * ldx + c0);
    if (FWD) {
      *xq = z[q];
    } else {
      const double2 o = *xq;
      *xq = make_double2(o.x + z[q].x, o.y + z[q].y);
    }
  }
  if (FWD) {
    const double *Ai = dval + d0 * B;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      double2 v = t[q];
#pragma unroll
      for (int c = 0; c < B; ++c) {
        v.x = fma(-Ai[q * B + c], z[c].x, v.x);
        v.y = fma(-Ai[q * B + c], z[c].y, v.y);
      }
      *reinterpret_cast<double2 *>(r + (d0 + q) * ldr + c0) = v;
    }
  }
}

// y_i (+ or -)= (M x)_i: mode 0 y = M x, 1 y += M x, 2 y -= M x.
template <int BR, int BC>
__global__ __launch_bounds__(kWB) void k_wide_rect(int rows, int K, const int *__restrict__ rp,
                                                   const int *__restrict__ col,
                                                   const double *__restrict__ val,
                                                   const double *__restrict__ x, int64_t ldx,
                                                   double *__restrict__ y, int64_t ldy, int mode) {
  const Place at = place<kWaveCols>(rows);
  const int i = at.row, c0 = min(at.c0, K - 2);
  double2 acc[BR];
  if (!wide_row<BR, BC>(rp[i], rp[i + 1], col, val, x + c0, ldx, acc) || at.c0 >= K) return;
#pragma unroll
  for (int q = 0; q < BR; ++q) {
    double2 *yq = reinterpret_cast<double2 *>(y + (int64_t(i) * BR + q) * ldy + c0);
    double2 v = acc[q];
    if (mode) {
      const double2 o = *yq;
      v = mode == 1 ? make_double2(o.x + v.x, o.y + v.y) : make_double2(o.x - v.x, o.y - v.y);
    }
    *yq = v;
  }
}

// y = D x, four rows of D per wavefront.
constexpr int kDR = 4;
__global__ __launch_bounds__(kWB) void k_wide_dense(int n, int ldD, const double *__restrict__ D, int K,
                                                    const double *__restrict__ x, int64_t ldx,
                                                    double *__restrict__ y, int64_t ldy) {
  const Place at = place<kWaveCols * kWaves>((n + kDR - 1) / kDR);
  const int i0 = at.row * kDR, c0 = at.c0;
  if (c0 >= K) return;
  const double *Dr[kDR];
  double2 acc[kDR];
#pragma unroll
  for (int q = 0; q < kDR; ++q) {
    Dr[q] = D + int64_t(i0 + q < n ? i0 + q : n - 1) * ldD;
    acc[q] = make_double2(0.0, 0.0);
  }
#pragma unroll 4
  for (int j = 0; j < n; ++j) {
    const double2 xv = ld2(x + j * ldx + c0);
#pragma unroll
    for (int q = 0; q < kDR; ++q) {
      acc[q].x = fma(Dr[q][j], xv.x, acc[q].x);
      acc[q].y = fma(Dr[q][j], xv.y, acc[q].y);
    }
  }
#pragma unroll
  for (int q = 0; q < kDR; ++q)
    if (i0 + q < n) *reinterpret_cast<double2 *>(y + int64_t(i0 + q) * ldy + c0) = acc[q];
}

bool panel_ok(const WidePanel &v, int K) {
  return v.p && v.ld >= K && v.ld % 2 == 0 && reinterpret_cast<uintptr_t>(v.p) % 16 == 0;
}

}  // namespace

hipError_t launch_wide_fwd(const SolveMat &A, const double *Dinv, int r0, int r1, int K, WidePanel b,
                           int j0, WidePanel x, WidePanel r, hipStream_t s) {
  if (r1 <= r0 || K == 0) return hipSuccess;
  if (K % 2 || (b.p && !panel_ok(b, K)) || !panel_ok(x, K) || !panel_ok(r, K) || !A.lo_val || !A.dg_val ||
      r0 < 0 || r1 > A.n_rows)
    return hipErrorInvalidValue;
  const int rows = r1 - r0;
  const dim3 grid(unsigned(rows) * wide_slices(K, kWaveCols));
  if (A.br == 1)
    hipLaunchKernelGGL((k_wide_gs<1, true>), grid, dim3(kWB), 0, s, r0, rows, K, A.lo_rp, A.lo_col, A.lo_val,
                       A.dg_val, Dinv, b.p, b.ld, j0, x.p, x.ld, r.p, r.ld);
  else if (A.br == 6)
    hipLaunchKernelGGL((k_wide_gs<6, true>), grid, dim3(kWB), 0, s, r0, rows, K, A.lo_rp, A.lo_col, A.lo_val,
                       A.dg_val, Dinv, b.p, b.ld, j0, x.p, x.ld, r.p, r.ld);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_wide_bwd(const SolveMat &A, const double *Dinv, int r0, int r1, int K, WidePanel b,
                           int j0, WidePanel x, hipStream_t s) {
  if (r1 <= r0 || K == 0) return hipSuccess;
  if (K % 2 || (b.p && !panel_ok(b, K)) || !panel_ok(x, K) || r0 < 0 || r1 > A.n_rows)
    return hipErrorInvalidValue;
  const int rows = r1 - r0;
  const dim3 grid(unsigned(rows) * wide_slices(K, kWaveCols));
  double *none = nullptr;
  const double *none_c = nullptr;
  if (A.br == 1)
    hipLaunchKernelGGL((k_wide_gs<1, false>), grid, dim3(kWB), 0, s, r0, rows, K, A.rp, A.col, A.val, none_c,
                       Dinv, b.p, b.ld, j0, x.p, x.ld, none, int64_t(0));
  else if (A.br == 6)
    hipLaunchKernelGGL((k_wide_gs<6, false>), grid, dim3(kWB), 0, s, r0, rows, K, A.rp, A.col, A.val, none_c,
                       Dinv, b.p, b.ld, j0, x.p, x.ld, none, int64_t(0));
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

namespace {
template <int BR, int BC>
void rect_go(int rows, int K, const int *rp, const int *col, const double *val, WidePanel x, WidePanel y,
             int mode, hipStream_t s) {
  hipLaunchKernelGGL((k_wide_rect<BR, BC>), dim3(unsigned(rows) * wide_slices(K, kWaveCols)), dim3(kWB), 0, s, rows, K, rp,
                     col, val, x.p, x.ld, y.p, y.ld, mode);
}
}  // namespace

hipError_t launch_wide_resid(const SolveMat &A, int K, WidePanel x, WidePanel r, hipStream_t s) {
  if (A.n_rows == 0 || K == 0) return hipSuccess;
  if (K % 2 || !panel_ok(x, K) || !panel_ok(r, K) || !A.up_val) return hipErrorInvalidValue;
  if (A.br == 1)
    rect_go<1, 1>(A.n_rows, K, A.up_rp, A.up_col, A.up_val, x, r, 2, s);
  else if (A.br == 6)
    rect_go<6, 6>(A.n_rows, K, A.up_rp, A.up_col, A.up_val, x, r, 2, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_wide_rect(const SolveMat &M, int K, WidePanel x, WidePanel y, bool accumulate,
                            hipStream_t s) {
  if (M.n_rows == 0 || K == 0) return hipSuccess;
  if (K % 2 || !panel_ok(x, K) || !panel_ok(y, K)) return hipErrorInvalidValue;
  const int mode = accumulate ? 1 : 0;
  if (M.br == 1 && M.bc == 1)
    rect_go<1, 1>(M.n_rows, K, M.rp, M.col, M.val, x, y, mode, s);
  else if (M.br == 6 && M.bc == 6)
    rect_go<6, 6>(M.n_rows, K, M.rp, M.col, M.val, x, y, mode, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_wide_dense(int n, int ldD, const double *D, int K, WidePanel x, WidePanel y,
                             hipStream_t s) {
  if (n == 0 || K == 0) return hipSuccess;
  if (K % 2 || ldD < n || !panel_ok(x, K) || !panel_ok(y, K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_wide_dense, dim3(unsigned((n + kDR - 1) / kDR) * wide_slices(K, kWaveCols * kWaves)), dim3(kWB), 0, s, n,
                     ldD, D, K, x.p, x.ld, y.p, y.ld);
  return hipGetLastError();
}

}  // namespace eamg
