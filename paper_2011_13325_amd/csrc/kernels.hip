// gfx950 kernels of the edge-matrix AMG-PCG library.  See kernels.hpp for the data layouts.
//
// Every floating point reduction has a fixed order (per-lane strided sums, then a fixed
// butterfly / tree), so results are bitwise reproducible run to run; no floating point
// atomics are used anywhere.
#include "kernels.hpp"

#include <cmath>
#include <cstdlib>
#include <type_traits>

namespace eamg {

namespace {


inline int cdiv64(int64_t a, int64_t b) { return int((a + b - 1) / b); }

// Workgroups are dispatched round-robin over the eight XCDs (workgroup b to XCD b mod 8), each
// XCD with its own L2.  The colour sweeps use this logical workgroup index instead of
// blockIdx.x: XCD x gets one contiguous run of logical workgroups (the first nb mod 8 XCDs one
// more), so the rows of a colour that one XCD updates are neighbours in the numbering and share
// their gathered x blocks in that XCD's L2 (sweeps 3 % faster at 64^3).  A bijection on
// [0, gridDim.x), so results do not change.  Not used where row lengths drift along the
// numbering: the residual update over all colour-major rows (upper blocks only, long rows first)
// would load one XCD with the longest rows (+33 % measured).
__device__ inline int xcd_block() {
  const int nb = int(gridDim.x), b = int(blockIdx.x);
  const int x = b & 7, q = nb >> 3, rem = nb & 7;
  return x * q + min(x, rem) + (b >> 3);
}

// ---- small dense helpers (one thread; every size a constant, so that the arrays are registers) ---

// X := X Q(t), Q(t) = [I Skew(t); 0 I] (K = 6; Skew(t) r = t x r) or 1 (K = 1); X is R x K.
template <int R, int K>
__device__ __forceinline__ void mul_q(double (&X)[R * K], const double (&t)[3]) {
  if constexpr (K == 6) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double a = X[r * 6], b = X[r * 6 + 1], c = X[r * 6 + 2];
      X[r * 6 + 3] += b * t[2] - c * t[1];
      X[r * 6 + 4] += c * t[0] - a * t[2];
      X[r * 6 + 5] += a * t[1] - b * t[0];
    }
  }
}
// X := Q(t)^T X
template <int K>
__device__ __forceinline__ void tmul_q(double (&X)[K * K], const double (&t)[3]) {
  if constexpr (K == 6) {
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const double a = X[j], b = X[6 + j], c = X[12 + j];
      X[18 + j] += b * t[2] - c * t[1];
      X[24 + j] += c * t[0] - a * t[2];
      X[30 + j] += a * t[1] - b * t[0];
    }
  }
}
// out (R x P) = A (R x N, the first R rows of a matrix with rows of N) B (N x P)
template <int R, int N, int P>
__device__ __forceinline__ void mul_rows(const double *A, const double (&B)[N * P], double (&out)[R * P]) {
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < P; ++j) {
      double v = 0.0;
#pragma unroll
      for (int l = 0; l < N; ++l) v += A[i * N + l] * B[l * P + j];
      out[i * P + j] = v;
    }
}

// Symmetric pseudo-inverse by cyclic Jacobi; eigenvalues <= tau * max(lambda_max, 0) dropped.
template <int N>
__device__ __forceinline__ void dev_pinv(const double (&X)[N * N], double (&P)[N * N], double tau) {
  double A[N * N], V[N * N];
  double fro2 = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      A[i * N + j] = 0.5 * (X[i * N + j] + X[j * N + i]);
      V[i * N + j] = i == j ? 1.0 : 0.0;
      fro2 += A[i * N + j] * A[i * N + j];
    }
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0;
#pragma unroll
    for (int p = 0; p < N; ++p)
#pragma unroll
      for (int q = p + 1; q < N; ++q) off += A[p * N + q] * A[p * N + q];
    if (off <= 1e-40 * fro2 || off == 0.0) break;
#pragma unroll
    for (int p = 0; p < N; ++p)
#pragma unroll
      for (int q = p + 1; q < N; ++q) {
        const double apq = A[p * N + q];
        if (apq == 0.0) continue;
        const double theta = (A[q * N + q] - A[p * N + p]) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        const double cs = 1.0 / sqrt(t * t + 1.0), sn = t * cs;
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const double akp = A[k * N + p], akq = A[k * N + q];
          A[k * N + p] = cs * akp - sn * akq;
          A[k * N + q] = sn * akp + cs * akq;
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const double apk = A[p * N + k], aqk = A[q * N + k];
          A[p * N + k] = cs * apk - sn * aqk;
          A[q * N + k] = sn * apk + cs * aqk;
        }
        A[p * N + q] = 0.0;
        A[q * N + p] = 0.0;
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const double vkp = V[k * N + p], vkq = V[k * N + q];
          V[k * N + p] = cs * vkp - sn * vkq;
          V[k * N + q] = sn * vkp + cs * vkq;
        }
      }
  }
  double lmax = A[0];
#pragma unroll
  for (int i = 0; i < N; ++i) lmax = A[i * N + i] > lmax ? A[i * N + i] : lmax;
#pragma unroll
  for (int i = 0; i < N * N; ++i) P[i] = 0.0;
  if (!(lmax > 0.0)) return;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double wk = A[k * N + k];
    if (!(wk > tau * lmax)) continue;
    const double inv = 1.0 / wk;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) P[i * N + j] += V[i * N + k] * inv * V[j * N + k];
  }
}

template <int N>
__device__ __forceinline__ void load_block(const double *src, double (&dst)[N]) {
#pragma unroll
  for (int e = 0; e < N; ++e) dst[e] = src[e];
}

// Block (i, i) of a matrix in rows [rp[i], rp[i + 1]), zero if it has none.
template <int B>
__device__ __forceinline__ void diagonal_block(int i, const int64_t *rp, const int *col, const double *val,
                                               double (&out)[B * B]) {
#pragma unroll
  for (int e = 0; e < B * B; ++e) out[e] = 0.0;
  for (int64_t p = rp[i]; p < rp[i + 1]; ++p)
    if (col[p] == i) {
      load_block<B * B>(val + p * (B * B), out);
      break;
    }
}

// ---- setup kernels --------------------------------------------------------------------------

__global__ void k_dirichlet(int n, int bs, const int64_t *rp, const int *col, double *val,
                            const uint8_t *dir) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int bsz = bs * bs;
  for (int64_t p = rp[i]; p < rp[i + 1]; ++p) {
    const int j = col[p];
    if (!(dir[i] || dir[j])) continue;
    for (int e = 0; e < bsz; ++e)
      val[p * bsz + e] = (i == j && dir[i] && (e / bs == e % bs)) ? 1.0 : 0.0;
  }
}

template <int B>
__global__ __launch_bounds__(64) void k_diag_pinv(int n, const int64_t *rp, const int *col, const double *val,
                                                 double *Dinv, double tau) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double blk[B * B], P[B * B];
  diagonal_block<B>(i, rp, col, val, blk);
  dev_pinv<B>(blk, P, tau);
#pragma unroll
  for (int e = 0; e < B * B; ++e) Dinv[int64_t(i) * (B * B) + e] = P[e];
}

// One fine row of the auxiliary smoothed prolongation (Def. def:aux_sp), one thread.  Bound: the chain
// of a row (its pseudo-inverse, then a congruence per neighbour); the blocks' sizes are constants and
// the transformations Q are applied as the cross products they are, so that a row's blocks stay in
// registers: 0.40 ms for the 9,261 rows of a cube with inclusions and its three coarse levels, 13.0 ms
// with arrays in scratch memory.
template <int K, int BS>
__global__ __launch_bounds__(64) void k_ps_numeric(PsArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const int type = a.type[i];
  if (type == 2) return;  // dropped row: no entries
  const int Ji = a.agg[i];
  const double *xi = a.x + 3 * int64_t(i);
  if (type == 0) {
    // real-matrix row: P_i - omega pinv(A_ii) sum_j A_ij P_j, P_j the first BS rows of Q^{J->j}
    double Dp[BS * BS];
    {
      double Aii[BS * BS];
      diagonal_block<BS>(i, a.Arp, a.Acol, a.Aval, Aii);
      dev_pinv<BS>(Aii, Dp, a.tau);
    }
    for (int64_t q = a.Prp[i]; q < a.Prp[i + 1]; ++q) {
      const int J = a.Pcol[q];
      const double *xJ = a.xc + 3 * int64_t(J);
      double acc[BS * K], X[BS * K];
#pragma unroll
      for (int e = 0; e < BS * K; ++e) acc[e] = 0.0;
      for (int64_t p = a.Arp[i]; p < a.Arp[i + 1]; ++p) {
        const int j = a.Acol[p];
        if (a.agg[j] != J) continue;
        const double *xj = a.x + 3 * int64_t(j);
        const double t[3] = {xj[0] - xJ[0], xj[1] - xJ[1], xj[2] - xJ[2]};
#pragma unroll
        for (int r = 0; r < BS; ++r)
#pragma unroll
          for (int c = 0; c < K; ++c) X[r * K + c] = c < BS ? a.Aval[p * (BS * BS) + r * BS + c] : 0.0;
        mul_q<BS, K>(X, t);
#pragma unroll
        for (int e = 0; e < BS * K; ++e) acc[e] += X[e];
      }
      mul_rows<BS, BS, K>(Dp, acc, X);
      double *out = a.Pval + q * (BS * K);
      double T[BS * K];
#pragma unroll
      for (int e = 0; e < BS * K; ++e) T[e] = J == Ji && e / K == e % K ? 1.0 : 0.0;
      const double t[3] = {xi[0] - xJ[0], xi[1] - xJ[1], xi[2] - xJ[2]};
      mul_q<BS, K>(T, t);
#pragma unroll
      for (int e = 0; e < BS * K; ++e) out[e] = T[e] - a.omega * X[e];
    }
    return;
  }
  // edge-matrix row: P_i - omega pinv(Dhat0_ii) (Dhat0_ii P_i + sum_{l in F} Ahat0_il P_l)
  constexpr int KK = K * K;
  double Dh[KK], Dp[KK], X[KK];
#pragma unroll
  for (int e = 0; e < KK; ++e) Dh[e] = 0.0;
  for (int64_t f = a.Fptr[i]; f < a.Fptr[i + 1]; ++f) {
    const double *xl = a.x + 3 * int64_t(a.Fvtx[f]);
    const double th[3] = {0.5 * (xl[0] - xi[0]), 0.5 * (xl[1] - xi[1]), 0.5 * (xl[2] - xi[2])};
    load_block<KK>(a.E + int64_t(a.Fedge[f]) * KK, X);
    tmul_q<K>(X, th);
    mul_q<K, K>(X, th);   // Q^{il,T} E Q^{il}
#pragma unroll
    for (int e = 0; e < KK; ++e) Dh[e] += X[e];
  }
  dev_pinv<K>(Dh, Dp, a.tau);
  for (int64_t q = a.Prp[i]; q < a.Prp[i + 1]; ++q) {
    const int J = a.Pcol[q];
    const double *xJ = a.xc + 3 * int64_t(J);
    const double ti[3] = {xi[0] - xJ[0], xi[1] - xJ[1], xi[2] - xJ[2]};
    double acc[KK];
#pragma unroll
    for (int e = 0; e < KK; ++e) acc[e] = J == Ji ? Dh[e] : 0.0;
    mul_q<K, K>(acc, ti);   // Dhat0_ii Q^{J->i}
    for (int64_t f = a.Fptr[i]; f < a.Fptr[i + 1]; ++f) {
      const int l = a.Fvtx[f];
      if (a.agg[l] != J) continue;
      const double *xl = a.x + 3 * int64_t(l);
      const double th[3] = {0.5 * (xl[0] - xi[0]), 0.5 * (xl[1] - xi[1]), 0.5 * (xl[2] - xi[2])};
      const double mh[3] = {-th[0], -th[1], -th[2]};
      const double t[3] = {xl[0] - xJ[0], xl[1] - xJ[1], xl[2] - xJ[2]};
      load_block<KK>(a.E + int64_t(a.Fedge[f]) * KK, X);
      tmul_q<K>(X, th);
      mul_q<K, K>(X, mh);   // Q^{il,T} E Q^{li}
      mul_q<K, K>(X, t);    // ... Q^{J->l}
#pragma unroll
      for (int e = 0; e < KK; ++e) acc[e] -= X[e];
    }
    double R[BS * K], T[BS * K];
    mul_rows<BS, K, K>(Dp, acc, R);
#pragma unroll
    for (int e = 0; e < BS * K; ++e) T[e] = J == Ji && e / K == e % K ? 1.0 : 0.0;
    mul_q<BS, K>(T, ti);
    double *out = a.Pval + q * (BS * K);
#pragma unroll
    for (int e = 0; e < BS * K; ++e) out[e] = T[e] - a.omega * R[e];
  }
}

__global__ void k_spgemm_numeric(int64_t nnzC, int ra, int ca, int cb, const int *crow,
                                 const int *Ccol, const int64_t *Arp, const int *Acol,
                                 const double *Aval, const int64_t *Brp, const int *Bcol,
                                 const double *Bval, double *Cval) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= nnzC * ra) return;
  const int64_t q = gid / ra;
  const int r = int(gid % ra);
  const int i = crow[q], J = Ccol[q];
  double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t p = Arp[i]; p < Arp[i + 1]; ++p) {
    const int kk = Acol[p];
    int64_t lo = Brp[kk], hi = Brp[kk + 1];
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (Bcol[mid] < J)
        lo = mid + 1;
      else
        hi = mid;
    }
    if (lo == Brp[kk + 1] || Bcol[lo] != J) continue;
    const double *Ab = Aval + p * ra * ca + r * ca;
    const double *Bb = Bval + lo * ca * cb;
    for (int c = 0; c < cb; ++c) {
      double s = 0.0;
      for (int t = 0; t < ca; ++t) s += Ab[t] * Bb[t * cb + c];
      acc[c] += s;
    }
  }
  for (int c = 0; c < cb; ++c) Cval[q * ra * cb + r * cb + c] = acc[c];
}

__global__ void k_transpose_blocks(int64_t nnz, int r, int c, const int64_t *src, const double *in,
                                   double *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int bsz = r * c;
  if (gid >= nnz * bsz) return;
  const int64_t q = gid / bsz;
  const int e = int(gid % bsz);
  const int oi = e / r, oj = e % r;   // out block is c x r: (oi, oj) = in (oj, oi)
  out[q * bsz + e] = in[src[q] * bsz + oj * c + oi];
}

// Block q of out := block src[q] of in (blocks of bsz values).
__global__ void k_gather_blocks(int64_t nnz, int bsz, const int64_t *src, const double *in, double *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= nnz * bsz) return;
  const int64_t q = gid / bsz;
  const int e = int(gid % bsz);
  out[gid] = in[src[q] * bsz + e];
}

__global__ void k_gather_rows(int n, int bsz, const int *perm, const double *in, double *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= int64_t(n) * bsz) return;
  const int64_t r = gid / bsz;
  const int e = int(gid % bsz);
  out[gid] = in[int64_t(perm[r]) * bsz + e];
}

// ---- solve kernels ---------------------------------------------------------------------------

__device__ inline double block_sum(double v, double *sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  return sh[0];
}

// The solve-phase kernels below are templated on the value type T of the matrices and vectors
// they stream (double, or float for the FP32 V-cycle); they accumulate in T.

template <class T, int BR>
__device__ inline void group_reduce(T (&acc)[BR], int G) {
  for (int off = G >> 1; off > 0; off >>= 1)
#pragma unroll
    for (int r = 0; r < BR; ++r) acc[r] += __shfl_xor(acc[r], off, G);
}

// A row team of W wavefronts (64 W lanes, "wide"; kBlock / (64 W) rows per workgroup):
// butterfly within each wavefront, then the W wavefront sums of the row added in wavefront order
// through LDS; every lane of the row gets the total.  sh: kBlock / 64 * BR values.
template <class T, int BR, int W>
__device__ inline void wide_reduce(T (&acc)[BR], T *sh) {
  group_reduce<T, BR>(acc, 64);
  const int wv = threadIdx.x / 64;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int r = 0; r < BR; ++r) sh[wv * BR + r] = acc[r];
  __syncthreads();
  const int w0 = wv - wv % W;   // first wavefront of this row
#pragma unroll
  for (int r = 0; r < BR; ++r) {
    T v = sh[w0 * BR + r];
    for (int w = 1; w < W; ++w) v += sh[(w0 + w) * BR + r];
    acc[r] = v;
  }
}

// xv = the BC entries of block column c of x.  Six-entry blocks start at a multiple of 24 (FP32)
// or 48 (FP64) bytes, so they are gathered as three 8- or 16-byte pairs: half the load
// instructions of a scattered gather (every lane of it touches its own cache line).
template <class T, int BC>
__device__ inline void gather_block(const T *x, int64_t c, T (&xv)[BC]) {
  if constexpr (BC % 2 == 0) {
    using T2 = typename std::conditional<sizeof(T) == 4, float2, double2>::type;
    const T2 *x2 = reinterpret_cast<const T2 *>(x + c * BC);
#pragma unroll
    for (int h = 0; h < BC / 2; ++h) {
      const T2 v = x2[h];
      xv[2 * h] = v.x;
      xv[2 * h + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int cc = 0; cc < BC; ++cc) xv[cc] = x[c * BC + cc];
  }
}

// acc[r] += sum over blocks p in [p0, p1) (strided by G) of A_p x_col(p), x_c read by load(c, out)
template <class T, int BR, int BC, class F>
__device__ inline void row_accumulate_of(int p0, int p1, int lane, int G, const int *__restrict__ col,
                                         const T *__restrict__ val, T (&acc)[BR], F &&load) {
  for (int p = p0 + lane; p < p1; p += G) {
    const int64_t c = col[p];
    T v[BR * BC];
#pragma unroll
    for (int e = 0; e < BR * BC; ++e) v[e] = val[int64_t(p) * (BR * BC) + e];
    // every value load is issued before the gathers of x, which wait for the column index
    __builtin_amdgcn_sched_barrier(0);
    T xv[BC];
    load(c, xv);
#pragma unroll
    for (int r = 0; r < BR; ++r)
#pragma unroll
      for (int cc = 0; cc < BC; ++cc) acc[r] = fma(v[r * BC + cc], xv[cc], acc[r]);
  }
}
template <class T, int BR, int BC>
__device__ inline void row_accumulate(int p0, int p1, int lane, int G, const int *__restrict__ col,
                                      const T *__restrict__ val, int64_t nnz, const T *x,
                                      T (&acc)[BR]) {
  row_accumulate_of<T, BR, BC>(p0, p1, lane, G, col, val, acc,
                               [x](int64_t c, T (&xv)[BC]) { gather_block<T, BC>(x, c, xv); });
}

template <int BR, int BC>
__global__ __launch_bounds__(kBlock) void k_spmv(int n_rows, int G, const int *__restrict__ rp,
                                                const int *__restrict__ col,
                                                const double *__restrict__ val, int64_t nnz,
                                                const double *__restrict__ x, double *__restrict__ y,
                                                double *part) {
  __shared__ double sh[kBlock];
  const int lane = threadIdx.x & (G - 1);
  const int wg = xcd_block();
  const int row = wg * (kBlock / G) + threadIdx.x / G;
  double acc[BR];
#pragma unroll
  for (int r = 0; r < BR; ++r) acc[r] = 0.0;
  if (row < n_rows) row_accumulate<double, BR, BC>(rp[row], rp[row + 1], lane, G, col, val, nnz, x, acc);
  group_reduce<double, BR>(acc, G);
  double d = 0.0;
  if (row < n_rows && lane == 0) {
#pragma unroll
    for (int r = 0; r < BR; ++r) {
      y[int64_t(row) * BR + r] = acc[r];
      d += x[int64_t(row) * BR + r] * acc[r];
    }
  }
  if (part) {
    const double s = block_sum(d, sh);
    if (threadIdx.x == 0) part[wg] = s;
  }
}

template <class T, int B>
__device__ inline T pick(const T (&v)[B], int i) {
  T out = T(0);
#pragma unroll
  for (int q = 0; q < B; ++q) out = (q == i) ? v[q] : out;
  return out;
}

// One row of a multicolour block Gauss-Seidel sweep, computed by the G lanes of a row group.
// FWD: x = 0 before the sweep, so only the blocks left of the diagonal (lower colours) are read
// (rp, col, val: the lower part) and A_ii is block `row` of dval;
// also writes r_i = t - A_ii x_i.  BWD: x_i += Dinv_i (b_i - sum_j A_ij x_j) over the whole row
// (rp, col, val: the full matrix).
// Lane q < B owns component q: it prefetches b_i[q], row q of Dinv_i and (FWD) row q of A_ii,
// (BWD) x_i[q], together with the row's blocks, so a row costs one round of row loads plus the
// x gathers; a butterfly all-reduce leaves the row sum on every lane.  No other row of the
// colour writes x_i, so the prefetched x_i[q] is the value the gathers see.
// y: the vector the blocks multiply, x itself for a colour.  For a group of colours b and
// y are both its right-hand side u and (rp, col, val) the group's matrix S (SweepPlan).
// Returns the lane's component of the new x_i (lanes < B of a valid row).
template <class T, int B, bool FWD, int W>
__device__ inline T gs_row(int row, bool valid, int lane, int G, const int *__restrict__ rp,
                              const int *__restrict__ col, const T *__restrict__ val, int64_t nnz,
                              const T *__restrict__ dval, int64_t nd, const T *__restrict__ Dinv,
                              const T *__restrict__ b, const T *y, T *x, T *r, T *sh) {
  const bool own = valid && lane < B;
  int p0 = 0, p1 = 0;
  if (valid) {
    p0 = rp[row];
    p1 = rp[row + 1];
  }
  T bq = T(0), xo = T(0), Dq[B], Aq[B];
#pragma unroll
  for (int c = 0; c < B; ++c) {
    Dq[c] = T(0);
    Aq[c] = T(0);
  }
  if (own) {
    bq = b[int64_t(row) * B + lane];
    if (!FWD) xo = x[int64_t(row) * B + lane];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      Dq[c] = Dinv[int64_t(row) * B * B + lane * B + c];
      if (FWD) Aq[c] = dval[int64_t(row) * (B * B) + lane * B + c];
    }
  }
  T acc[B];
#pragma unroll
  for (int q = 0; q < B; ++q) acc[q] = T(0);
  if (valid) row_accumulate<T, B, B>(p0, p1, lane, G, col, val, nnz, y, acc);
  if (W > 1)
    wide_reduce<T, B, W>(acc, sh);
  else
    group_reduce<T, B>(acc, G);
  // wide teams: the owning lanes (< B) are in the row's first wavefront; shuffles stay within
  // wavefronts
  const int GS = W > 1 ? 64 : G;
  const T tq = bq - pick<T, B>(acc, lane);   // t component of this lane (lanes < B)
  T t[B];
#pragma unroll
  for (int c = 0; c < B; ++c) t[c] = __shfl(tq, c, GS);
  T xq = T(0);
#pragma unroll
  for (int c = 0; c < B; ++c) xq = fma(Dq[c], t[c], xq);
  if (FWD) {
    T xi[B];
#pragma unroll
    for (int c = 0; c < B; ++c) xi[c] = __shfl(xq, c, GS);
    T rq = tq;
#pragma unroll
    for (int c = 0; c < B; ++c) rq = fma(-Aq[c], xi[c], rq);
    if (own) {
      x[int64_t(row) * B + lane] = xq;
      r[int64_t(row) * B + lane] = rq;
    }
  } else {
    xq = xo + xq;
    if (own) x[int64_t(row) * B + lane] = xq;
  }
  return xq;
}

// r_i = b_i - sum over the blocks [rp[i], re[i]) of A_ij x_j for one row (b may be r).
template <class T, int B, int W>
__device__ inline void resid_row(int row, bool valid, int lane, int G, const int *__restrict__ rp,
                                 const int *__restrict__ re, const int *__restrict__ col,
                                 const T *__restrict__ val, int64_t nnz, const T *x, const T *b, T *r,
                                 T *sh) {
  T rq = T(0);
  int p0 = 0, p1 = 0;
  if (valid) {
    p0 = rp[row];
    p1 = re[row];
    if (lane < B) rq = b[int64_t(row) * B + lane];
  }
  T acc[B];
#pragma unroll
  for (int a = 0; a < B; ++a) acc[a] = T(0);
  if (valid) row_accumulate<T, B, B>(p0, p1, lane, G, col, val, nnz, x, acc);
  if (W > 1)
    wide_reduce<T, B, W>(acc, sh);
  else
    group_reduce<T, B>(acc, G);
  if (valid && lane < B) r[int64_t(row) * B + lane] = rq - pick<T, B>(acc, lane);
}

// One colour (rows [r0, r1)) per launch, kBlock / G rows per workgroup.  G = 64 W lanes per
// row with W = 2 or 4 wavefronts ("wide", W = 4: one row per workgroup) for levels whose rows
// are long; else G <= 64 (W = 1).
template <class T, int B, bool FWD, int W>
__global__ __launch_bounds__(kBlock) void k_gs_color(int r0, int r1, int G, const int *__restrict__ rp,
                                                    const int *__restrict__ col,
                                                    const T *__restrict__ val, int64_t nnz,
                                                    const T *__restrict__ dval, int64_t nd,
                                                    const T *__restrict__ Dinv,
                                                    const T *__restrict__ b, T *x, T *r) {
  __shared__ T sh[W > 1 ? (kBlock / 64) * B : 1];
  const int lane = threadIdx.x & (G - 1);
  const int row = r0 + xcd_block() * (kBlock / G) + threadIdx.x / G;
  gs_row<T, B, FWD, W>(row, row < r1, lane, G, rp, col, val, nnz, dval, nd, Dinv, b, x, x, r, sh);
}

// Groups of colours.  On the levels of a few hundred rows per colour a colour launch is a chain of
// dependent steps (dispatch, row offsets, blocks, gathers, reduction, store) of 3.3 to 5 us that its
// bytes hardly add to, and a sweep is 20 to 70 such launches.  A group runs any number of colours
// in two: u = b - (couplings outside the group) x over all its rows, then its colours' recursion
// multiplied out, t = u - S u.  Solves with groups against one launch per colour, without a dense tail:
// 17^3 FP64 9.22 -> 2.25 ms (1536 colour launches -> 132 group launches), Poisson 65x57x71 15.1 -> 7.9
// ms; with the tail 64^3 FP32 25.9 -> 19.6 ms, FP64 35.9 -> 29.3 ms, 128^3 FP32 155 -> 143 ms.
template <class T, int B, int W>
__global__ __launch_bounds__(kBlock) void k_group_rhs(int r0, int r1, int G, const int *__restrict__ rp,
                                                     const int *__restrict__ re,
                                                     const int *__restrict__ col,
                                                     const T *__restrict__ val, int64_t nnz,
                                                     const T *__restrict__ b, const T *__restrict__ x,
                                                     T *__restrict__ u) {
  __shared__ T sh[W > 1 ? (kBlock / 64) * B : 1];
  const int lane = threadIdx.x & (G - 1);
  const int row = r0 + xcd_block() * (kBlock / G) + int(threadIdx.x) / G;
  resid_row<T, B, W>(row, row < r1, lane, G, rp, re, col, val, nnz, x, b, u, sh);
}

// The second launch: t = u - S u, x and (forward) r; u = launch_group_rhs's, or b for the first group.
// rz (backward): the workgroup's part of the CG's r.z over its rows, z the new x, in rz[workgroup]
// (the sweep's last launch, of a level that is one group).
template <class T, int B, bool FWD, int W, bool RZ>
__global__ __launch_bounds__(kBlock) void k_gs_group(int r0, int r1, int G, const int *__restrict__ rp,
                                                    const int *__restrict__ col,
                                                    const T *__restrict__ val, int64_t nnz,
                                                    const T *__restrict__ dval, int64_t nd,
                                                    const T *__restrict__ Dinv,
                                                    const T *__restrict__ u, T *__restrict__ x,
                                                    T *__restrict__ r, const double *__restrict__ cg_r,
                                                    double *__restrict__ rz) {
  __shared__ T sh[W > 1 ? (kBlock / 64) * B : 1];
  const int lane = threadIdx.x & (G - 1);
  const int row = r0 + xcd_block() * (kBlock / G) + threadIdx.x / G;
  const bool own = RZ && row < r1 && lane < B;
  const double rq = own ? cg_r[int64_t(row) * B + lane] : 0.0;
  const T z = gs_row<T, B, FWD, W>(row, row < r1, lane, G, rp, col, val, nnz, dval, nd, Dinv, u, u, x, r, sh);
  if (RZ) {
    __shared__ double shd[kBlock];
    const double t = block_sum(own ? rq * double(z) : 0.0, shd);
    if (threadIdx.x == 0) rz[blockIdx.x] = t;
  }
}

// 256 entries of a row of S per workgroup (launch_group_fill), one per thread.  The products A_q Dinv_j of
// FillSize::chunk couplings at a time sit in LDS.  Setup only.  Bound: the chain of ranks, each waiting for the
// one before, and in it the searches of S_jk's position in row j, dependent loads through L2; FillSize::ahead
// couplings are searched for at once, the forward and the backward matrix fill beside each other, and a
// row's entries are shared out over workgroups.  A scalar level of 895 rows in one group of 59 colours
// (S of 361,684 entries) took 38 ms with one workgroup a row, one search after the other and the
// matrices in turn, 6 ms now (the level's stages with uploads and allocations).
template <int B>
struct FillSize {
  static constexpr int chunk = B == 1 ? 256 : B == 3 ? 64 : 32, ahead = B == 6 ? 4 : 8;
};
template <int B>
__global__ __launch_bounds__(kBlock) void k_group_fill(GroupRank fwd, GroupRank bwd, const int *__restrict__ col,
                                                      const double *__restrict__ val,
                                                      const double *__restrict__ Dinv) {
  constexpr int BB = B * B, kChunk = FillSize<B>::chunk, kAhead = FillSize<B>::ahead;
  static_assert(kChunk % kAhead == 0, "a batch stays inside a chunk");
  __shared__ double P[kChunk * BB];
  __shared__ int J[kChunk], J0[kChunk], J1[kChunk];
  const GroupRank g = blockIdx.z ? bwd : fwd;
  if (int(blockIdx.x) >= g.nrows) return;
  const int i = g.rows[blockIdx.x];
  const int s0 = g.rp[i] + int(blockIdx.y) * kBlock, s1 = g.rp[i + 1];
  if (s0 >= s1) return;
  const int a = g.q0[i], b = g.q1[i];
  const int e = s0 + int(threadIdx.x);
  const int k = e < s1 ? g.col[e] : -1;
  double acc[BB];
#pragma unroll
  for (int v = 0; v < BB; ++v) acc[v] = 0.0;
  for (int qa = a; qa < b; qa += kChunk) {
    const int m = min(kChunk, b - qa);
    __syncthreads();
    for (int t = threadIdx.x; t < m * BB; t += kBlock) {
      const int q = t / BB, r = (t % BB) / B, c = t % B;
      const int j = col[qa + q];
      double v = 0.0;
#pragma unroll
      for (int l = 0; l < B; ++l) v = fma(val[int64_t(qa + q) * BB + r * B + l], Dinv[int64_t(j) * BB + l * B + c], v);
      P[t] = v;
      if (r == 0 && c == 0) {
        J[q] = j;
        J0[q] = g.rp[j];
        J1[q] = g.rp[j + 1];
      }
    }
    __syncthreads();
    for (int qb = 0; qb < m; qb += kAhead) {
      // lo[u]: the first entry of row j at a column >= k
      int lo[kAhead], hi[kAhead], longest = 0;
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int q = min(qb + u, m - 1);
        lo[u] = J0[q];
        hi[u] = J1[q];
        longest = max(longest, hi[u] - lo[u]);
      }
      for (; longest > 0; longest >>= 1)
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int mid = (lo[u] + hi[u]) >> 1;
          const bool in = lo[u] < hi[u];
          const bool less = g.col[in ? mid : s0] < k;
          hi[u] = in && !less ? mid : hi[u];
          lo[u] = in && less ? mid + 1 : lo[u];
        }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int q = min(qb + u, m - 1), at = lo[u];
        hi[u] = at < J1[q] && g.col[at < J1[q] ? at : s0] == k ? at : -1;
      }
      if (k < 0) continue;
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (qb + u >= m) break;
        const double *Pq = P + (qb + u) * BB;
        if (J[qb + u] == k) {
#pragma unroll
          for (int v = 0; v < BB; ++v) acc[v] += Pq[v];
          continue;
        }
        if (hi[u] < 0) continue;
        const double *Sj = g.val + int64_t(hi[u]) * BB;
#pragma unroll
        for (int l = 0; l < B; ++l) {
          double sj[B];
#pragma unroll
          for (int c = 0; c < B; ++c) sj[c] = Sj[l * B + c];
#pragma unroll
          for (int r = 0; r < B; ++r)
#pragma unroll
            for (int c = 0; c < B; ++c) acc[r * B + c] = fma(-Pq[r * B + l], sj[c], acc[r * B + c]);
        }
      }
    }
  }
  if (k >= 0)
#pragma unroll
    for (int v = 0; v < BB; ++v) g.val[int64_t(e) * BB + v] = acc[v];
}

template <class T, int B, int W>
__global__ __launch_bounds__(kBlock) void k_resid_upper(int r0, int r1, int G, const int *__restrict__ rp,
                                                       const int *__restrict__ col,
                                                       const T *__restrict__ val, int64_t nnz,
                                                       const T *x, T *r) {
  __shared__ T sh[W > 1 ? (kBlock / 64) * B : 1];
  const int lane = threadIdx.x & (G - 1);
  const int row = r0 + int(blockIdx.x) * (kBlock / G) + int(threadIdx.x) / G;
  resid_row<T, B, W>(row, row < r1, lane, G, rp, rp + 1, col, val, nnz, x, r, r, sh);
}

template <class T, int BR, int BC>
__global__ __launch_bounds__(kBlock) void k_rect(int n_rows, int G, const int *__restrict__ rp,
                                                const int *__restrict__ col,
                                                const T *__restrict__ val, int64_t nnz,
                                                const T *__restrict__ x, T *__restrict__ y,
                                                int accumulate) {
  const int lane = threadIdx.x & (G - 1);
  const int row = xcd_block() * (kBlock / G) + threadIdx.x / G;
  // the old y_i is read with the row's first loads, not after the reduction
  T acc[BR], yo[BR];
#pragma unroll
  for (int r = 0; r < BR; ++r) {
    acc[r] = T(0);
    yo[r] = T(0);
  }
  if (accumulate && row < n_rows && lane == 0)
#pragma unroll
    for (int r = 0; r < BR; ++r) yo[r] = y[int64_t(row) * BR + r];
  if (row < n_rows) row_accumulate<T, BR, BC>(rp[row], rp[row + 1], lane, G, col, val, nnz, x, acc);
  group_reduce<T, BR>(acc, G);
  if (row < n_rows && lane == 0) {
#pragma unroll
    for (int r = 0; r < BR; ++r) y[int64_t(row) * BR + r] = accumulate ? yo[r] + acc[r] : acc[r];
  }
}

template <class S, class D>
__global__ void k_convert(int64_t n, const S *__restrict__ in, D *__restrict__ out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] = D(in[i]);
}

__global__ void k_gather_blocks_f32(int64_t nnz, int bsz, const int64_t *src, const double *in, float *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= nnz * bsz) return;
  const int64_t q = gid / bsz;
  const int e = int(gid % bsz);
  out[gid] = float(in[src[q] * bsz + e]);
}

// b in double, or the FP32 V-cycle's output read as it is (each value converted exactly)
template <class TB>
__global__ __launch_bounds__(kBlock) void k_dot(int64_t n, const double *__restrict__ a,
                                               const TB *__restrict__ b, double *part) {
  __shared__ double sh[kBlock];
  double s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
    s = fma(a[i], double(b[i]), s);
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// The sum of the partials, on every thread: the same strided sums and tree wherever it is taken.
__device__ inline double sum_parts(int nparts, const double *__restrict__ part, double *sh) {
  double s = 0.0;
  // unrolled so that the loads are in flight together (the CG SpMV leaves one partial per
  // workgroup: hundreds of thousands on a large level); the sum keeps its order
#pragma unroll 16
  for (int i = threadIdx.x; i < nparts; i += kBlock) s += part[i];
  const double t = block_sum(s, sh);
  __syncthreads();
  return t;
}

__global__ __launch_bounds__(kBlock) void k_reduce(int nparts, const double *__restrict__ part,
                                                  double *scal, int slot) {
  __shared__ double sh[kBlock];
  const double t = sum_parts(nparts, part, sh);
  if (threadIdx.x == 0) scal[slot] = t;
}

// End of an iteration, one thread: t = r.r (see launch_publish).
__device__ inline void publish(double t, double *scal, double *ring) {
  const double it = scal[SC_ITER] + 1.0;
  scal[SC_RR] = t;
  scal[SC_ITER] = it;
  if (sqrt(t) <= scal[SC_RTOL] * sqrt(scal[SC_BB])) scal[SC_DONE] = 1.0;
  double *rec = ring + (int(it) & (kRing - 1)) * kRecord;
  for (int i = 0; i < SC_COUNT; ++i) rec[i] = scal[i];
  __threadfence_system();
  __hip_atomic_store(rec + kRecord - 1, it, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The scalars of an iteration are formed by the kernels that use them: a kernel that only sums a
// thousand partials costs 2.5 to 4.7 us in the chain of an iteration, the sum inside the next kernel
// about one.  Every workgroup takes the same sum; workgroup 0 stores the scalars, in slots that no
// workgroup of the same launch reads.
__global__ __launch_bounds__(kBlock) void k_update_xr(int64_t n, double *scal, double *__restrict__ x,
                                                     double *__restrict__ r, const double *__restrict__ p,
                                                     const double *__restrict__ q,
                                                     double *__restrict__ part, int npq,
                                                     const double *__restrict__ pq,
                                                     float *__restrict__ r32, double *__restrict__ pold,
                                                     double *ring) {
  __shared__ double sh[kBlock];
  const double rz = scal[SC_RZ];
  const bool done = scal[SC_DONE] != 0.0;
  const double t = npq > 0 ? sum_parts(npq, pq, sh) : scal[SC_PQ];
  const double alpha = rz / t;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (!(t > 0.0) || !isfinite(t)) scal[SC_BAD] = 1.0;
    if (npq > 0) scal[SC_PQ] = t;
    scal[SC_ALPHA] = alpha;
    scal[SC_RHO] = rz;
  }
  double s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    double ri = r[i];
    const double pi = p[i];
    if (pold) pold[i] = pi;
    if (!done) {
      x[i] = fma(alpha, pi, x[i]);
      ri = fma(-alpha, q[i], ri);
      r[i] = ri;
      if (r32) r32[i] = float(ri);
    }
    s = fma(ri, ri, s);
  }
  const double rr = block_sum(s, sh);
  if (threadIdx.x != 0) return;
  if (ring)
    publish(rr, scal, ring);
  else
    part[blockIdx.x] = rr;
}

template <class TZ>
__global__ __launch_bounds__(kBlock) void k_update_p(int64_t n, double *scal, const TZ *__restrict__ z,
                                                    double *__restrict__ p, int nparts,
                                                    const double *__restrict__ part) {
  __shared__ double sh[kBlock];
  const double rho = scal[SC_RHO];
  const double t = sum_parts(nparts, part, sh);
  const double beta = t / rho;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (!(t > 0.0) || !isfinite(t)) scal[SC_BAD] = 1.0;
    scal[SC_RZ] = t;
    scal[SC_BETA] = beta;
  }
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
    p[i] = fma(beta, p[i], double(z[i]));
}

__global__ __launch_bounds__(kBlock) void k_publish(int nparts, const double *__restrict__ part,
                                                   double *scal, double *ring) {
  __shared__ double sh[kBlock];
  const double t = sum_parts(nparts, part, sh);
  if (threadIdx.x == 0) publish(t, scal, ring);
}

// p' = z + beta p, formed where the rows gather it, and q = A p': the p update's launch and its pass
// over the vectors, for a second gather per block.  p' goes to pn (other rows still gather p), and
// the x and r update copies it back.
template <int B, class TZ>
__global__ __launch_bounds__(kBlock) void k_spmv_dir(int n_rows, int G, const int *__restrict__ rp,
                                                    const int *__restrict__ col,
                                                    const double *__restrict__ val,
                                                    const TZ *__restrict__ z, const double *__restrict__ p,
                                                    double *__restrict__ pn, double *__restrict__ q,
                                                    double *scal, int nparts,
                                                    const double *__restrict__ rz, double *__restrict__ part) {
  __shared__ double sh[kBlock];
  const int lane = threadIdx.x & (G - 1);
  const int wg = xcd_block();
  const int row = wg * (kBlock / G) + threadIdx.x / G;
  int p0 = 0, p1 = 0;
  if (row < n_rows) {
    p0 = rp[row];
    p1 = rp[row + 1];
  }
  const double rho = scal[SC_RHO];
  const double t = sum_parts(nparts, rz, sh);
  const double beta = t / rho;
  if (wg == 0 && threadIdx.x == 0) {
    if (!(t > 0.0) || !isfinite(t)) scal[SC_BAD] = 1.0;
    scal[SC_RZ] = t;
    scal[SC_BETA] = beta;
  }
  const auto load = [&](int64_t c, double (&xv)[B]) {
    TZ zv[B];
    double pv[B];
    gather_block<TZ, B>(z, c, zv);
    gather_block<double, B>(p, c, pv);
#pragma unroll
    for (int e = 0; e < B; ++e) xv[e] = fma(beta, pv[e], double(zv[e]));
  };
  double acc[B];
#pragma unroll
  for (int r = 0; r < B; ++r) acc[r] = 0.0;
  row_accumulate_of<double, B, B>(p0, p1, lane, G, col, val, acc, load);
  group_reduce<double, B>(acc, G);
  double d = 0.0;
  if (row < n_rows && lane == 0) {
    double pi[B];
    load(row, pi);
#pragma unroll
    for (int r = 0; r < B; ++r) {
      const int64_t i = int64_t(row) * B + r;
      q[i] = acc[r];
      pn[i] = pi[r];
      d += pi[r] * acc[r];
    }
  }
  const double s = block_sum(d, sh);
  if (threadIdx.x == 0) part[wg] = s;
}

// Start of a solve, one pass over the vectors: bp = the right-hand side in solve order (Dirichlet
// zeroed), with x also x = 0, r = bp and (r32) its FP32 copy; part <- partials of bp.bp, bad <-
// whether a workgroup's entries are not all finite.  Launches bound the small solves: with the end's
// k_finish and r.z taken by the last sweep launch, a solve of 1,029 dofs takes 530 us instead of 561
// (ten passes of their own before and after the iterations), one of 14,739 dofs 2.04 ms instead of 2.08.
__global__ __launch_bounds__(kBlock) void k_start(int64_t n, int bs, const int *__restrict__ perm,
                                                 const uint8_t *__restrict__ mask,
                                                 const double *__restrict__ b, double *__restrict__ bp,
                                                 double *__restrict__ x, double *__restrict__ r,
                                                 float *__restrict__ r32, double *__restrict__ part,
                                                 double *__restrict__ bad) {
  __shared__ double sh[kBlock];
  double s = 0.0;
  int wrong = 0;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const int64_t row = i / bs;
    const int o = perm[row];
    const double v = (mask && mask[o]) ? 0.0 : b[int64_t(o) * bs + (i - row * bs)];
    bp[i] = v;
    if (x) {
      x[i] = 0.0;
      r[i] = v;
      if (r32) r32[i] = float(v);
    }
    s = fma(v, v, s);
    wrong |= !isfinite(v);
  }
  wrong = __syncthreads_or(wrong);
  const double t = block_sum(s, sh);
  if (threadIdx.x != 0) return;
  part[blockIdx.x] = t;
  bad[blockIdx.x] = wrong ? 1.0 : 0.0;
}

// The scalars of a new solve: SC_RTOL, SC_BB and SC_NONFINITE from the start's partials, else 0.
__global__ __launch_bounds__(kBlock) void k_start_scal(int nparts, const double *__restrict__ part,
                                                      const double *__restrict__ bad, double rtol,
                                                      double *__restrict__ scal) {
  __shared__ double sh[kBlock];
  int wrong = 0;
  for (int i = threadIdx.x; i < nparts; i += kBlock) wrong |= bad[i] != 0.0;
  wrong = __syncthreads_or(wrong);
  const double t = sum_parts(nparts, part, sh);
  if (threadIdx.x < SC_COUNT)
    scal[threadIdx.x] = threadIdx.x == SC_RTOL ? rtol
                        : threadIdx.x == SC_BB ? t
                        : threadIdx.x == SC_NONFINITE ? (wrong ? 1.0 : 0.0)
                                                      : 0.0;
}

// p = z, part <- partials of r.z
template <class TZ>
__global__ __launch_bounds__(kBlock) void k_start_p(int64_t n, const TZ *__restrict__ z,
                                                   const double *__restrict__ r, double *__restrict__ p,
                                                   double *__restrict__ part) {
  __shared__ double sh[kBlock];
  double s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const double zi = double(z[i]);
    p[i] = zi;
    s = fma(r[i], zi, s);
  }
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// End of a solve: out = x in natural order, part <- partials of |b - q|^2 (q = A x)
__global__ __launch_bounds__(kBlock) void k_finish(int64_t n, int bs, const int *__restrict__ perm,
                                                  const double *__restrict__ x, const double *__restrict__ b,
                                                  const double *__restrict__ q, double *__restrict__ out,
                                                  double *__restrict__ part) {
  __shared__ double sh[kBlock];
  double s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const int64_t row = i / bs;
    out[int64_t(perm[row]) * bs + (i - row * bs)] = x[i];
    const double d = b[i] - q[i];
    s = fma(d, d, s);
  }
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ void k_sub(int64_t n, const double *a, const double *b, double *y) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a[i] - b[i];
}

__global__ void k_copy(int64_t n, const double *a, double *y) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a[i];
}

__global__ void k_fill(int64_t n, double v, double *a) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

__global__ void k_perm_in(int n, int bs, const int *perm, const uint8_t *mask, const double *in,
                          double *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= int64_t(n) * bs) return;
  const int64_t r = gid / bs;
  const int c = int(gid % bs);
  const int o = perm[r];
  out[gid] = (mask && mask[o]) ? 0.0 : in[int64_t(o) * bs + c];
}

__global__ void k_perm_out(int n, int bs, const int *perm, const double *in, double *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= int64_t(n) * bs) return;
  const int64_t r = gid / bs;
  const int c = int(gid % bs);
  out[int64_t(perm[r]) * bs + c] = in[gid];
}

int groups_for(int G) { return kBlock / G; }

}  // namespace

// ---- launchers ---------------------------------------------------------------------------------

#define EAMG_LAUNCH_CHECK() return hipGetLastError()

hipError_t launch_dirichlet(int n, int bs, const int64_t *rp, const int *col, double *val,
                            const uint8_t *dir, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_dirichlet, dim3(cdiv64(n, 128)), dim3(128), 0, s, n, bs, rp, col, val, dir);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_diag_pinv(int n, int bs, const int64_t *rp, const int *col, const double *val,
                            double *Dinv, double tau, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const dim3 grid(cdiv64(n, 64));
  switch (bs) {
    case 1: hipLaunchKernelGGL(k_diag_pinv<1>, grid, dim3(64), 0, s, n, rp, col, val, Dinv, tau); break;
    case 3: hipLaunchKernelGGL(k_diag_pinv<3>, grid, dim3(64), 0, s, n, rp, col, val, Dinv, tau); break;
    case 6: hipLaunchKernelGGL(k_diag_pinv<6>, grid, dim3(64), 0, s, n, rp, col, val, Dinv, tau); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_ps_numeric(const PsArgs &a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const dim3 grid(cdiv64(a.n, 64));
  if (a.k == 6 && a.bs == 3)
    hipLaunchKernelGGL((k_ps_numeric<6, 3>), grid, dim3(64), 0, s, a);
  else if (a.k == 6 && a.bs == 6)
    hipLaunchKernelGGL((k_ps_numeric<6, 6>), grid, dim3(64), 0, s, a);
  else if (a.k == 1 && a.bs == 1)
    hipLaunchKernelGGL((k_ps_numeric<1, 1>), grid, dim3(64), 0, s, a);
  else
    return hipErrorInvalidValue;
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_spgemm_numeric(int64_t nnzC, int ra, int ca, int cb, const int *crow,
                                 const int *Ccol, const int64_t *Arp, const int *Acol,
                                 const double *Aval, const int64_t *Brp, const int *Bcol,
                                 const double *Bval, double *Cval, hipStream_t s) {
  if (nnzC == 0) return hipSuccess;
  hipLaunchKernelGGL(k_spgemm_numeric, dim3(cdiv64(nnzC * ra, 256)), dim3(256), 0, s, nnzC, ra, ca,
                     cb, crow, Ccol, Arp, Acol, Aval, Brp, Bcol, Bval, Cval);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_transpose_blocks(int64_t nnz, int r, int c, const int64_t *src, const double *in,
                                   double *out, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_transpose_blocks, dim3(cdiv64(nnz * r * c, 256)), dim3(256), 0, s, nnz, r, c,
                     src, in, out);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_gather_blocks(int64_t nnz, int bsz, const int64_t *src, const double *in, double *out,
                             hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_blocks, dim3(cdiv64(nnz * bsz, 256)), dim3(256), 0, s, nnz, bsz, src, in,
                     out);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_gather_rows(int n, int bsz, const int *perm, const double *in, double *out,
                              hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rows, dim3(cdiv64(int64_t(n) * bsz, 256)), dim3(256), 0, s, n, bsz,
                     perm, in, out);
  EAMG_LAUNCH_CHECK();
}

#define EAMG_DISPATCH_SQ(B, KERNEL, ...)                                                        \
  switch (B) {                                                                                  \
    case 1: hipLaunchKernelGGL(KERNEL<1>, __VA_ARGS__); break;                                  \
    case 3: hipLaunchKernelGGL(KERNEL<3>, __VA_ARGS__); break;                                  \
    case 6: hipLaunchKernelGGL(KERNEL<6>, __VA_ARGS__); break;                                  \
    default: return hipErrorInvalidValue;                                                       \
  }

// k_spmv reduces within wavefronts: a matrix with one row per workgroup runs it with 64 lanes
// per row.
inline int spmv_group(const SolveMat &A) { return A.group > 64 ? 64 : A.group; }

int spmv_blocks(const SolveMat &A) { return int(cdiv64(A.n_rows, groups_for(spmv_group(A)))); }

hipError_t launch_spmv(const SolveMat &A, const double *x, double *y, double *part, hipStream_t s) {
  if (A.n_rows == 0) return hipSuccess;
  const int G = spmv_group(A);
  const dim3 grid(spmv_blocks(A));
  if (A.br != A.bc) return hipErrorInvalidValue;
  switch (A.br) {
    case 1: hipLaunchKernelGGL((k_spmv<1, 1>), grid, dim3(kBlock), 0, s, A.n_rows, G, A.rp, A.col, A.val, A.nnz, x, y, part); break;
    case 3: hipLaunchKernelGGL((k_spmv<3, 3>), grid, dim3(kBlock), 0, s, A.n_rows, G, A.rp, A.col, A.val, A.nnz, x, y, part); break;
    case 6: hipLaunchKernelGGL((k_spmv<6, 6>), grid, dim3(kBlock), 0, s, A.n_rows, G, A.rp, A.col, A.val, A.nnz, x, y, part); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

template <class T>
const T *solve_vals(const SolveMat &M);
template <>
const double *solve_vals<double>(const SolveMat &M) {
  return M.val;
}
template <>
const float *solve_vals<float>(const SolveMat &M) {
  return M.val32;
}

// Wavefronts per row team for G lanes per row: 4 (kBlock), 2 (128) or 1 (<= 64).
#define EAMG_GS_W(W_, ...)                                                                       \
  if (G == kBlock) { constexpr int W_ = 4; __VA_ARGS__; }                                       \
  else if (G == 128) { constexpr int W_ = 2; __VA_ARGS__; }                                     \
  else { constexpr int W_ = 1; __VA_ARGS__; }

template <class T>
hipError_t launch_gs_fwd(const SolveMat &A, const T *Dinv, int r0, int r1, const T *b, T *x, T *r,
                         hipStream_t s) {
  if (r1 <= r0) return hipSuccess;
  const T *lo = sizeof(T) == 4 ? reinterpret_cast<const T *>(A.lo_val32) : reinterpret_cast<const T *>(A.lo_val);
  const T *dg = sizeof(T) == 4 ? reinterpret_cast<const T *>(A.dg_val32) : reinterpret_cast<const T *>(A.dg_val);
  if (!lo || !dg || !A.lo_rp || r0 < 0 || r1 > A.n_rows) return hipErrorInvalidValue;
  const int G = A.group;
  const dim3 grid(cdiv64(r1 - r0, groups_for(G)));
  const int64_t nd = A.n_rows;
  switch (A.br) {
    case 1: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_color<T, 1, true, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.lo_rp, A.lo_col, lo, A.lo_nnz, dg, nd, Dinv, b, x, r)); break;
    case 3: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_color<T, 3, true, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.lo_rp, A.lo_col, lo, A.lo_nnz, dg, nd, Dinv, b, x, r)); break;
    case 6: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_color<T, 6, true, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.lo_rp, A.lo_col, lo, A.lo_nnz, dg, nd, Dinv, b, x, r)); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

template <class T>
hipError_t launch_gs_bwd(const SolveMat &A, const T *Dinv, int r0, int r1, const T *b, T *x,
                         hipStream_t s) {
  if (r1 <= r0) return hipSuccess;
  const T *val = solve_vals<T>(A);
  if (!val) return hipErrorInvalidValue;
  const int G = A.group_bwd ? A.group_bwd : A.group;
  const dim3 grid(cdiv64(r1 - r0, groups_for(G)));
  T *none = nullptr;
  const T *none_c = nullptr;
  switch (A.br) {
    case 1: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_color<T, 1, false, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.rp, A.col, val, A.nnz, none_c, int64_t(0), Dinv, b, x, none)); break;
    case 3: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_color<T, 3, false, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.rp, A.col, val, A.nnz, none_c, int64_t(0), Dinv, b, x, none)); break;
    case 6: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_color<T, 6, false, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.rp, A.col, val, A.nnz, none_c, int64_t(0), Dinv, b, x, none)); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

template <class T>
hipError_t launch_resid_upper(const SolveMat &A, int r0, int r1, const T *x, T *r, hipStream_t s) {
  if (r0 < 0 || r1 > A.n_rows) return hipErrorInvalidValue;
  if (r1 <= r0) return hipSuccess;
  const T *up = sizeof(T) == 4 ? reinterpret_cast<const T *>(A.up_val32) : reinterpret_cast<const T *>(A.up_val);
  if (!up || !A.up_rp) return hipErrorInvalidValue;
  const int G = A.group;
  const dim3 grid(cdiv64(r1 - r0, groups_for(G)));
  switch (A.br) {
    case 1: EAMG_GS_W(W_, hipLaunchKernelGGL((k_resid_upper<T, 1, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.up_rp, A.up_col, up, A.up_nnz, x, r)); break;
    case 3: EAMG_GS_W(W_, hipLaunchKernelGGL((k_resid_upper<T, 3, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.up_rp, A.up_col, up, A.up_nnz, x, r)); break;
    case 6: EAMG_GS_W(W_, hipLaunchKernelGGL((k_resid_upper<T, 6, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, A.up_rp, A.up_col, up, A.up_nnz, x, r)); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

template <class T>
hipError_t launch_group_rhs(const SolveMat &A, const int *lo_end, int r0, int r1, const T *b, const T *x,
                            T *u, hipStream_t s) {
  if (r0 < 0 || r1 > A.n_rows) return hipErrorInvalidValue;
  if (r1 <= r0) return hipSuccess;
  const bool f32 = sizeof(T) == 4;
  const T *val = lo_end ? reinterpret_cast<const T *>(f32 ? (const void *)A.lo_val32 : (const void *)A.lo_val)
                        : solve_vals<T>(A);
  const int *rp = lo_end ? A.lo_rp : A.rp, *re = lo_end ? lo_end : A.rp + 1;
  const int *col = lo_end ? A.lo_col : A.col;
  const int64_t nnz = lo_end ? A.lo_nnz : A.nnz;
  if (!val || !rp) return hipErrorInvalidValue;
  const int G = !lo_end && A.group_bwd ? A.group_bwd : A.group;
  const dim3 grid(cdiv64(r1 - r0, groups_for(G)));
  switch (A.br) {
    case 1: EAMG_GS_W(W_, hipLaunchKernelGGL((k_group_rhs<T, 1, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, rp, re, col, val, nnz, b, x, u)); break;
    case 3: EAMG_GS_W(W_, hipLaunchKernelGGL((k_group_rhs<T, 3, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, rp, re, col, val, nnz, b, x, u)); break;
    case 6: EAMG_GS_W(W_, hipLaunchKernelGGL((k_group_rhs<T, 6, W_>), grid, dim3(kBlock), 0, s, r0, r1, G, rp, re, col, val, nnz, b, x, u)); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

int group_blocks(const SolveMat &S, int r0, int r1) { return int(cdiv64(r1 - r0, groups_for(S.group))); }

namespace {
template <class T, bool FWD, bool RZ>
hipError_t launch_group(const SolveMat &S, const T *dg, const T *Dinv, int r0, int r1, const T *u, T *x,
                        T *r, const double *cg_r, double *rz, hipStream_t s) {
  if (r0 < 0 || r1 > S.n_rows) return hipErrorInvalidValue;
  if (r1 <= r0) return hipSuccess;
  const T *val = solve_vals<T>(S);
  if (!val || !S.rp || (FWD && !dg)) return hipErrorInvalidValue;
  const int G = S.group;
  const dim3 grid(group_blocks(S, r0, r1));
  const int64_t nd = S.n_rows;
  switch (S.br) {
    case 1: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_group<T, 1, FWD, W_, RZ>), grid, dim3(kBlock), 0, s, r0, r1, G, S.rp, S.col, val, S.nnz, dg, nd, Dinv, u, x, r, cg_r, rz)); break;
    case 3: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_group<T, 3, FWD, W_, RZ>), grid, dim3(kBlock), 0, s, r0, r1, G, S.rp, S.col, val, S.nnz, dg, nd, Dinv, u, x, r, cg_r, rz)); break;
    case 6: EAMG_GS_W(W_, hipLaunchKernelGGL((k_gs_group<T, 6, FWD, W_, RZ>), grid, dim3(kBlock), 0, s, r0, r1, G, S.rp, S.col, val, S.nnz, dg, nd, Dinv, u, x, r, cg_r, rz)); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}
}  // namespace

template <class T>
hipError_t launch_group_fwd(const SolveMat &A, const SolveMat &S, const T *Dinv, int r0, int r1,
                            const T *u, T *x, T *r, hipStream_t s) {
  const T *dg = sizeof(T) == 4 ? reinterpret_cast<const T *>(A.dg_val32) : reinterpret_cast<const T *>(A.dg_val);
  return launch_group<T, true, false>(S, dg, Dinv, r0, r1, u, x, r, nullptr, nullptr, s);
}

template <class T>
hipError_t launch_group_bwd(const SolveMat &S, const T *Dinv, int r0, int r1, const T *u, T *x,
                            hipStream_t s, const double *cg_r, double *rz) {
  if (rz) return launch_group<T, false, true>(S, nullptr, Dinv, r0, r1, u, x, nullptr, cg_r, rz, s);
  return launch_group<T, false, false>(S, nullptr, Dinv, r0, r1, u, x, nullptr, nullptr, nullptr, s);
}

hipError_t launch_group_fill(const GroupRank &fwd, const GroupRank &bwd, int longest, int bs, const int *col,
                             const double *val, const double *Dinv, hipStream_t s) {
  const int nrows = fwd.nrows > bwd.nrows ? fwd.nrows : bwd.nrows;
  if (nrows == 0 || longest == 0) return hipSuccess;
  for (const GroupRank *g : {&fwd, &bwd})
    if (!g->rows || !g->q0 || !g->q1 || !g->rp || !g->col || !g->val) return hipErrorInvalidValue;
  if (!col || !val || !Dinv) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(nrows), static_cast<unsigned>(cdiv64(longest, kBlock)), 2);
  switch (bs) {
    case 1: hipLaunchKernelGGL(k_group_fill<1>, grid, dim3(kBlock), 0, s, fwd, bwd, col, val, Dinv); break;
    case 3: hipLaunchKernelGGL(k_group_fill<3>, grid, dim3(kBlock), 0, s, fwd, bwd, col, val, Dinv); break;
    case 6: hipLaunchKernelGGL(k_group_fill<6>, grid, dim3(kBlock), 0, s, fwd, bwd, col, val, Dinv); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}

template <class T>
hipError_t launch_rect(const SolveMat &M, const T *x, T *y, bool accumulate, hipStream_t s) {
  if (M.n_rows == 0) return hipSuccess;
  const T *val = solve_vals<T>(M);
  if (!val) return hipErrorInvalidValue;
  const dim3 grid(cdiv64(M.n_rows, groups_for(M.group)));
  const int accf = accumulate ? 1 : 0;
#define EAMG_RECT(BR_, BC_)                                                                          \
  hipLaunchKernelGGL((k_rect<T, BR_, BC_>), grid, dim3(kBlock), 0, s, M.n_rows, M.group, M.rp, M.col, \
                     val, M.nnz, x, y, accf)
  if (M.br == 1 && M.bc == 1) EAMG_RECT(1, 1);
  else if (M.br == 3 && M.bc == 6) EAMG_RECT(3, 6);
  else if (M.br == 6 && M.bc == 3) EAMG_RECT(6, 3);
  else if (M.br == 6 && M.bc == 6) EAMG_RECT(6, 6);
  else return hipErrorInvalidValue;
#undef EAMG_RECT
  EAMG_LAUNCH_CHECK();
}

template <class S, class D>
hipError_t launch_convert(int64_t n, const S *in, D *out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((k_convert<S, D>), dim3(cdiv64(n, 256)), dim3(256), 0, s, n, in, out);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_gather_blocks_f32(int64_t nnz, int bsz, const int64_t *src, const double *in,
                                 float *out, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_blocks_f32, dim3(cdiv64(nnz * bsz, 256)), dim3(256), 0, s, nnz, bsz, src,
                     in, out);
  EAMG_LAUNCH_CHECK();
}

template hipError_t launch_gs_fwd<double>(const SolveMat &, const double *, int, int, const double *, double *, double *, hipStream_t);
template hipError_t launch_gs_fwd<float>(const SolveMat &, const float *, int, int, const float *, float *, float *, hipStream_t);
template hipError_t launch_gs_bwd<double>(const SolveMat &, const double *, int, int, const double *, double *, hipStream_t);
template hipError_t launch_gs_bwd<float>(const SolveMat &, const float *, int, int, const float *, float *, hipStream_t);
template hipError_t launch_resid_upper<double>(const SolveMat &, int, int, const double *, double *, hipStream_t);
template hipError_t launch_resid_upper<float>(const SolveMat &, int, int, const float *, float *, hipStream_t);
template hipError_t launch_group_rhs<double>(const SolveMat &, const int *, int, int, const double *, const double *, double *, hipStream_t);
template hipError_t launch_group_rhs<float>(const SolveMat &, const int *, int, int, const float *, const float *, float *, hipStream_t);
template hipError_t launch_group_fwd<double>(const SolveMat &, const SolveMat &, const double *, int, int, const double *, double *, double *, hipStream_t);
template hipError_t launch_group_fwd<float>(const SolveMat &, const SolveMat &, const float *, int, int, const float *, float *, float *, hipStream_t);
template hipError_t launch_group_bwd<double>(const SolveMat &, const double *, int, int, const double *, double *, hipStream_t, const double *, double *);
template hipError_t launch_group_bwd<float>(const SolveMat &, const float *, int, int, const float *, float *, hipStream_t, const double *, double *);
template hipError_t launch_rect<double>(const SolveMat &, const double *, double *, bool, hipStream_t);
template hipError_t launch_rect<float>(const SolveMat &, const float *, float *, bool, hipStream_t);
template hipError_t launch_convert<double, float>(int64_t, const double *, float *, hipStream_t);
template hipError_t launch_convert<float, double>(int64_t, const float *, double *, hipStream_t);

int dot_blocks(int64_t n) {
  const int64_t b = (n + kBlock - 1) / kBlock;
  return int(b < 1 ? 1 : (b > 1024 ? 1024 : b));
}

hipError_t launch_dot(int64_t n, const double *a, const double *b, double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_dot<double>, dim3(dot_blocks(n)), dim3(kBlock), 0, s, n, a, b, part);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_dot(int64_t n, const double *a, const float *b, double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_dot<float>, dim3(dot_blocks(n)), dim3(kBlock), 0, s, n, a, b, part);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_reduce(int nparts, const double *part, double *scal, int slot, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(kBlock), 0, s, nparts, part, scal, slot);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_update_xr(int64_t n, double *scal, double *x, double *r, const double *p,
                            const double *q, double *part, int npq, const double *pq, hipStream_t s,
                            float *r32, double *pold, double *ring) {
  if (npq < 0 || npq > kInlineParts || (npq && (!pq || pq == part))) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_update_xr, dim3(ring ? 1 : dot_blocks(n)), dim3(kBlock), 0, s, n, scal, x, r, p, q, part,
                     npq, pq, r32, pold, ring);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_update_p(int64_t n, double *scal, const double *z, double *p, int nparts,
                           const double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_update_p<double>, dim3(dot_blocks(n)), dim3(kBlock), 0, s, n, scal, z, p, nparts, part);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_update_p(int64_t n, double *scal, const float *z, double *p, int nparts,
                           const double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_update_p<float>, dim3(dot_blocks(n)), dim3(kBlock), 0, s, n, scal, z, p, nparts, part);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_publish(int nparts, const double *part, double *scal, double *ring, hipStream_t s) {
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(kBlock), 0, s, nparts, part, scal, ring);
  EAMG_LAUNCH_CHECK();
}

template <class TZ>
hipError_t launch_spmv_dir(const SolveMat &A, double *scal, const TZ *z, const double *p, double *pn, double *q,
                           int nparts, const double *rz, double *part, hipStream_t s) {
  if (A.n_rows == 0) return hipSuccess;
  if (A.br != A.bc || !pn || pn == p || rz == part || nparts < 1 || nparts > kInlineParts) return hipErrorInvalidValue;
  const int G = spmv_group(A);
  const dim3 grid(spmv_blocks(A));
  switch (A.br) {
    case 1: hipLaunchKernelGGL((k_spmv_dir<1, TZ>), grid, dim3(kBlock), 0, s, A.n_rows, G, A.rp, A.col, A.val, z, p, pn, q, scal, nparts, rz, part); break;
    case 3: hipLaunchKernelGGL((k_spmv_dir<3, TZ>), grid, dim3(kBlock), 0, s, A.n_rows, G, A.rp, A.col, A.val, z, p, pn, q, scal, nparts, rz, part); break;
    case 6: hipLaunchKernelGGL((k_spmv_dir<6, TZ>), grid, dim3(kBlock), 0, s, A.n_rows, G, A.rp, A.col, A.val, z, p, pn, q, scal, nparts, rz, part); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_LAUNCH_CHECK();
}
template hipError_t launch_spmv_dir<double>(const SolveMat &, double *, const double *, const double *, double *, double *, int, const double *, double *, hipStream_t);
template hipError_t launch_spmv_dir<float>(const SolveMat &, double *, const float *, const double *, double *, double *, int, const double *, double *, hipStream_t);

hipError_t launch_start(int64_t n, int bs, const int *perm, const uint8_t *mask, const double *b, double *bp,
                        double *x, double *r, float *r32, double rtol, double *part, double *bad, double *scal,
                        hipStream_t s) {
  const int nd = dot_blocks(n);
  hipLaunchKernelGGL(k_start, dim3(nd), dim3(kBlock), 0, s, n, bs, perm, mask, b, bp, x, r, r32, part, bad);
  hipLaunchKernelGGL(k_start_scal, dim3(1), dim3(kBlock), 0, s, nd, part, bad, rtol, scal);
  EAMG_LAUNCH_CHECK();
}

template <class TZ>
hipError_t launch_start_p(int64_t n, const TZ *z, const double *r, double *p, double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_start_p<TZ>, dim3(dot_blocks(n)), dim3(kBlock), 0, s, n, z, r, p, part);
  EAMG_LAUNCH_CHECK();
}
template hipError_t launch_start_p<double>(int64_t, const double *, const double *, double *, double *, hipStream_t);
template hipError_t launch_start_p<float>(int64_t, const float *, const double *, double *, double *, hipStream_t);

hipError_t launch_finish(int64_t n, int bs, const int *perm, const double *x, const double *b, const double *q,
                         double *out, double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_finish, dim3(dot_blocks(n)), dim3(kBlock), 0, s, n, bs, perm, x, b, q, out, part);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_sub(int64_t n, const double *a, const double *b, double *y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_sub, dim3(cdiv64(n, 256)), dim3(256), 0, s, n, a, b, y);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_copy(int64_t n, const double *a, double *y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy, dim3(cdiv64(n, 256)), dim3(256), 0, s, n, a, y);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_fill(int64_t n, double v, double *a, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, dim3(cdiv64(n, 256)), dim3(256), 0, s, n, v, a);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_perm_in(int n, int bs, const int *perm, const uint8_t *mask, const double *in,
                          double *out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_perm_in, dim3(cdiv64(int64_t(n) * bs, 256)), dim3(256), 0, s, n, bs, perm,
                     mask, in, out);
  EAMG_LAUNCH_CHECK();
}

hipError_t launch_perm_out(int n, int bs, const int *perm, const double *in, double *out,
                           hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_perm_out, dim3(cdiv64(int64_t(n) * bs, 256)), dim3(256), 0, s, n, bs, perm,
                     in, out);
  EAMG_LAUNCH_CHECK();
}

}  // namespace eamg
