// Batched exact coarsening criteria on the device (Lemma thm:mu2, Thm thm:mu1).
//
// The kernels perform the arithmetic of crit_core.hpp in FP64, compiled with -ffp-contract=off
// like the host, so every value equals the host's bit for bit.  This is latency-bound work on
// small matrices (k x k blocks, k 1 or 6, and union matrices up to 24 x 24), not a dense
// contraction: neither HBM nor MFMA bounds it, the chain of dependent operations per pair does.
//
//  * mu_b: one thread per pair, its blocks in registers.  A pair's chain is short; batches of
//    thousands of pairs fill the chip.
//  * mu_g: one wavefront per union.  The chain of a union (two cyclic Jacobi solves of order up
//    to 24, about 2000 rotations each) is far too long for one thread, so the wavefront spreads
//    the independent entries of every step over its lanes with the matrices in LDS, and the
//    pseudo-inverses of the outside neighbours over its lanes, one each.  Each entry
//    still sees the host's operations in the host's order: block products accumulate in the same
//    index order with the same zero skips, a rotation updates column and row entries with the
//    same formulas, sums of squares run sequentially in the same order on every lane, and the
//    eigenvalue sort applies the host's stable insertion sort as a permutation.
#include "criteria.hpp"
#include "hierarchy.hpp"

#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

namespace eamg {
namespace {

constexpr int kCritBlock = 64;

// ---- mu_g, one wavefront (one 64-lane workgroup) per union ---------------------------------

// leading dimension of the union matrices: odd, so that the lanes of a column access hit different banks
constexpr int kWLd = crit::kMaxUnionDim + 1;
constexpr int kWMat = crit::kMaxUnionDim * kWLd;
constexpr int kWInv = 32;                  // outside neighbours whose pseudo-inverses are held at a time
static_assert(kWInv * 36 <= 2 * kWMat, "they share the space of U and G");
constexpr int kWOut = 192;                 // outside-neighbour entries held (NaN beyond)
constexpr int kMaxGWaves = 256 * 8;        // mu_g grid (grid-stride over the unions)

// small k x k matrices (row-major, leading dimension k) in LDS
enum {
  S_Y = 0,            // Y[a] = D_a Q^{H->a}, kMaxUnion slots
  S_Z = 4, S_ZP, S_YZ, S_S, S_T1, S_Q1, S_Q2, S_EE, S_X,
  S_KCC,              // kMaxUnion slots
  S_KCW = S_KCC + 4,  // kMaxUnion slots
  S_KW = S_KCW + 4,
  S_COUNT
};

struct WShared {
  double L[kWMat], R[kWMat];
  double UG[2 * kWMat];   // U and G of the pencil; before it, kWInv pseudo-inverses
  double w[crit::kMaxUnionDim];
  double sm[S_COUNT][36];
  int ol[kWOut], oa[kWOut], oe[kWOut];   // outside entries in encounter order
  int sl[kWOut], sa[kWOut], se[kWOut];   // the same, sorted by neighbour (stable)
  int perm[crit::kMaxUnionDim];
};

__device__ __forceinline__ void wsync() { __syncthreads(); }

// the value every lane holds, as a wave-uniform value (all lanes hold the same)
__device__ __forceinline__ double uni(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane(int(b & 0xffffffffLL));
  const int hi = __builtin_amdgcn_readfirstlane(int(b >> 32));
  return __longlong_as_double(static_cast<long long>(static_cast<unsigned>(lo)) |
                              (static_cast<long long>(hi) << 32));
}

// The k x k helpers have K as a constant: an entry's operands are then read together instead of one
// LDS round trip per term.

// C = A B, C = A^T B, C = A B^T (crit::mul with tr() operands): entry (i, j) accumulates over l
// ascending from 0.0, skipping zero entries of the left factor.
template <int K, int SA, int TA, int SB, int TB>
__device__ __forceinline__ void w_product(double *C, const double *A, const double *B) {
  const int t = threadIdx.x;
  if (t < K * K) {
    const int i = t / K, j = t - i * K;
    double av[K], bv[K];
#pragma unroll
    for (int l = 0; l < K; ++l) {
      av[l] = A[i * SA + l * TA];
      bv[l] = B[l * SB + j * TB];
    }
    double c = 0.0;
#pragma unroll
    for (int l = 0; l < K; ++l) c = av[l] == 0.0 ? c : c + av[l] * bv[l];
    C[t] = c;
  }
  wsync();
}
template <int K>
__device__ void w_mul(double *C, const double *A, const double *B) {
  w_product<K, K, 1, K, 1>(C, A, B);
}
template <int K>
__device__ void w_mul_tA(double *C, const double *A, const double *B) {
  w_product<K, 1, K, K, 1>(C, A, B);
}
template <int K>
__device__ void w_mul_tB(double *C, const double *A, const double *B) {
  w_product<K, K, 1, 1, K>(C, A, B);
}
// out = A^T B C (crit::t3), tmp a scratch slot
template <int K>
__device__ void w_t3(double *out, const double *A, const double *B, const double *C, double *tmp) {
  w_mul_tA<K>(tmp, A, B);
  w_mul<K>(out, tmp, C);
}
// Q(t) of crit::q
template <int K>
__device__ void w_q(double *Q, const double *tv) {
  const int t = threadIdx.x;
  if (t < K * K) {
    const int i = t / K, j = t - i * K;
    double v = i == j ? 1.0 : 0.0;
    if (K == 6) {
      if (i == 0 && j == 4) v = -tv[2];
      if (i == 0 && j == 5) v = tv[1];
      if (i == 1 && j == 3) v = tv[2];
      if (i == 1 && j == 5) v = -tv[0];
      if (i == 2 && j == 3) v = -tv[1];
      if (i == 2 && j == 4) v = tv[0];
    }
    Q[t] = v;
  }
  wsync();
}
template <int K>
__device__ void w_qtrans(double *Q, const double *xa, const double *xb) {
  const double tv[3] = {xb[0] - xa[0], xb[1] - xa[1], xb[2] - xa[2]};
  w_q<K>(Q, tv);
}
template <int K>
__device__ void w_qhalf(double *Q, const double *xa, const double *xb) {
  const double tv[3] = {0.5 * (xb[0] - xa[0]), 0.5 * (xb[1] - xa[1]), 0.5 * (xb[2] - xa[2])};
  w_q<K>(Q, tv);
}
template <int K>
__device__ void w_load(double *S, const double *src) {
  if (threadIdx.x < K * K) S[threadIdx.x] = src[threadIdx.x];
  wsync();
}
template <int K>
__device__ void w_zero(double *S) {
  if (threadIdx.x < K * K) S[threadIdx.x] = 0.0;
  wsync();
}
// Y += s X (crit::axpy)
template <int K>
__device__ void w_axpy(double *Y, double s, const double *X) {
  if (threadIdx.x < K * K) Y[threadIdx.x] += s * X[threadIdx.x];
  wsync();
}
template <int K>
__device__ void w_neg(double *Y) {
  if (threadIdx.x < K * K) Y[threadIdx.x] = -Y[threadIdx.x];
  wsync();
}
// block (a, b) of X (leading dimension ld) += s S, or s S^T (crit::put)
template <int K>
__device__ void w_put(double *X, int a, int b, const double *S, double s, bool trans) {
  const int t = threadIdx.x;
  if (t < K * K) {
    const int u = t / K, v = t - u * K;
    X[(a * K + u) * kWLd + b * K + v] += s * (trans ? S[v * K + u] : S[t]);
  }
  wsync();
}

// The LDS accesses of this wavefront before the call precede those after it (they are performed in
// program order; nothing is waited for).
__device__ __forceinline__ void worder() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// lane's v, on every lane (lane the same on all)
__device__ __forceinline__ double from_lane(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(int(b & 0xffffffffLL), lane);
  const int hi = __builtin_amdgcn_readlane(int(b >> 32), lane);
  return __longlong_as_double(static_cast<long long>(static_cast<unsigned>(lo)) |
                              (static_cast<long long>(hi) << 32));
}

// crit::jacobi on the n x n matrix A (leading dimension ld) in LDS; A must be symmetric bit for bit (it
// stays so: both entries of a pair see the same operations).  A rotation is one step: lane t < n holds
// A(p, t) in a register over all rotations of row p, lane 32 + t the same of V^T (kept in tmp), and
// row q + 1 is read while rotation (p, q) computes its angle; the two entries of it that this
// rotation changes, and the next rotation's a_pq, come from lane q + 1.  What is left is the chain of
// the angle, two square roots and three divisions.  A batch of unions up to 24 x 24 takes 2.21 ms instead
// of 3.05 (columns, rows and the zeroed pair in three steps through LDS; the outside neighbours'
// pseudo-inverses one after the other).
__device__ __forceinline__ void w_jacobi(double *A, int n, int ld, double *w, double *V, double *tmp, int *perm) {
  const int t = threadIdx.x;
  if (V)
    for (int idx = t; idx < n * n; idx += kCritBlock) {
      const int i = idx / n, j = idx - i * n;
      tmp[i * ld + j] = i == j ? 1.0 : 0.0;
    }
  wsync();
  double fro2 = 0.0;
  for (int i = 0; i < n; ++i)
#pragma unroll 8
    for (int j = 0; j < n; ++j) fro2 += A[i * ld + j] * A[i * ld + j];
  fro2 = uni(fro2);
  const bool la = t < n, act = la || (V && t >= 32 && t < 32 + n);
  // this lane's entry of row r: mine[r * ld] (if act); A and tmp are parts of one WShared
  double *const mine = A + (la || !V ? t : int(tmp - A) + t - 32);
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0;
    for (int p = 0; p < n; ++p)
#pragma unroll 8
      for (int q = p + 1; q < n; ++q) off += A[p * ld + q] * A[p * ld + q];
    off = uni(off);
    if (off <= 1e-40 * fro2 || off == 0.0) break;
    for (int p = 0; p + 1 < n; ++p) {
      double x = act ? mine[p * ld] : 0.0, y = act ? mine[(p + 1) * ld] : 0.0;
      double app = uni(A[p * ld + p]), apq = uni(A[p * ld + p + 1]), aqq = uni(A[(p + 1) * ld + p + 1]);
      for (int q = p + 1; q < n; ++q) {
        const int r = q + 1 < n ? q + 1 : q;   // the next row
        double yn = act ? mine[r * ld] : 0.0;
        const double arr = A[r * ld + r];
        double nx = x, ny = y;
        if (apq != 0.0) {
          const double theta = (aqq - app) / (2.0 * apq);
          const double tt = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
          const double cs = 1.0 / sqrt(tt * tt + 1.0), sn = tt * cs;
          nx = cs * x - sn * y;
          ny = sn * x + cs * y;
          // the 2 x 2 block: columns, then rows, then the pair zeroed
          const double cpp = cs * app - sn * apq, cpq = sn * app + cs * apq;
          const double cqp = cs * apq - sn * aqq, cqq = sn * apq + cs * aqq;
          app = cs * cpp - sn * cqp;
          if (t == p) {
            nx = app;
            ny = 0.0;
          } else if (t == q) {
            nx = 0.0;
            ny = sn * cpq + cs * cqq;
          }
          if (act) mine[q * ld] = ny;
          if (la) A[t * ld + q] = ny;
          worder();
        }
        apq = from_lane(nx, r);
        const double b = from_lane(ny, r);
        if (t == p) yn = apq;
        if (t == q) yn = b;
        x = nx;
        y = yn;
        aqq = uni(arr);
      }
      if (act) mine[p * ld] = x;
      if (la) A[t * ld + p] = x;
      wsync();
    }
  }
  // eigenvalues ascending by the host's stable insertion sort, applied to V as a permutation
  if (t == 0) {
    for (int i = 0; i < n; ++i) {
      w[i] = A[i * ld + i];
      perm[i] = i;
    }
    for (int i = 1; i < n; ++i)
      for (int j = i; j > 0 && w[j] < w[j - 1]; --j) {
        const double x = w[j];
        w[j] = w[j - 1];
        w[j - 1] = x;
        const int pj = perm[j];
        perm[j] = perm[j - 1];
        perm[j - 1] = pj;
      }
  }
  wsync();
  if (V) {
    for (int idx = t; idx < n * n; idx += kCritBlock) {
      const int r = idx / n, c = idx - r * n;
      V[r * ld + c] = tmp[perm[c] * ld + r];
    }
    wsync();
  }
}

// P = pinv(X, tau) of crit::pinv, one thread, on registers: any number of lanes take one matrix each in
// the time of one (a whole wavefront per matrix takes as long, its chain of rotations being the same).
template <int K>
__device__ __forceinline__ void t_pinv(double (&P)[K * K], const double (&X)[K * K], double tau) {
  double A[K * K], V[K * K], w[K];
#pragma unroll
  for (int i = 0; i < K; ++i)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      A[i * K + j] = 0.5 * (X[i * K + j] + X[j * K + i]);
      V[i * K + j] = i == j ? 1.0 : 0.0;
    }
  double fro2 = 0.0;
#pragma unroll
  for (int e = 0; e < K * K; ++e) fro2 += A[e] * A[e];
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0;
#pragma unroll
    for (int p = 0; p < K; ++p)
#pragma unroll
      for (int q = p + 1; q < K; ++q) off += A[p * K + q] * A[p * K + q];
    if (off <= 1e-40 * fro2 || off == 0.0) break;
#pragma unroll
    for (int p = 0; p < K; ++p)
#pragma unroll
      for (int q = p + 1; q < K; ++q) {
        const double apq = A[p * K + q];
        if (apq == 0.0) continue;
        const double theta = (A[q * K + q] - A[p * K + p]) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        const double cs = 1.0 / sqrt(t * t + 1.0), sn = t * cs;
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const double x = A[i * K + p], y = A[i * K + q];
          A[i * K + p] = cs * x - sn * y;
          A[i * K + q] = sn * x + cs * y;
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const double x = A[p * K + i], y = A[q * K + i];
          A[p * K + i] = cs * x - sn * y;
          A[q * K + i] = sn * x + cs * y;
        }
        A[p * K + q] = 0.0;
        A[q * K + p] = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const double x = V[i * K + p], y = V[i * K + q];
          V[i * K + p] = cs * x - sn * y;
          V[i * K + q] = sn * x + cs * y;
        }
      }
  }
  // the host's stable insertion sort
#pragma unroll
  for (int i = 0; i < K; ++i) w[i] = A[i * K + i];
#pragma unroll
  for (int i = 1; i < K; ++i) {
    bool go = true;
#pragma unroll
    for (int j = i; j > 0; --j) {
      go = go && w[j] < w[j - 1];
      const double lo = go ? w[j] : w[j - 1], hi = go ? w[j - 1] : w[j];
      w[j - 1] = lo;
      w[j] = hi;
#pragma unroll
      for (int r = 0; r < K; ++r) {
        const double a = V[r * K + j - 1], b = V[r * K + j];
        V[r * K + j - 1] = go ? b : a;
        V[r * K + j] = go ? a : b;
      }
    }
  }
  const double lmax = w[K - 1];
#pragma unroll
  for (int e = 0; e < K * K; ++e) P[e] = 0.0;
  if (lmax <= 0.0) return;
#pragma unroll
  for (int m = 0; m < K; ++m) {
    if (!(w[m] > tau * lmax)) continue;
    const double inv = 1.0 / w[m];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const double vi = V[i * K + m] * inv;
#pragma unroll
      for (int j = 0; j < K; ++j) P[i * K + j] += vi * V[j * K + m];
    }
  }
}

// crit::genmax_n on L, R (n x n, leading dimension kWLd); U, G and R's storage are scratch.
__device__ double w_genmax(int n, double tau, WShared &sh) {
  const int t = threadIdx.x, ld = kWLd;
  double *L = sh.L, *R = sh.R, *U = sh.UG, *G = sh.UG + kWMat;
  for (int idx = t; idx < n * n; idx += kCritBlock) {
    const int i = idx / n, j = idx - i * n;
    if (i < j) {
      const double l = 0.5 * (L[i * ld + j] + L[j * ld + i]);
      L[i * ld + j] = L[j * ld + i] = l;
      const double r = 0.5 * (R[i * ld + j] + R[j * ld + i]);
      R[i * ld + j] = R[j * ld + i] = r;
    }
  }
  wsync();
  double nL = 0.0;
  for (int i = 0; i < n; ++i)
#pragma unroll 8
    for (int j = 0; j < n; ++j) nL += L[i * ld + j] * L[i * ld + j];
  nL = uni(sqrt(nL));
  if (nL == 0.0) return 0.0;
  w_jacobi(R, n, ld, sh.w, U, G, sh.perm);
  const double lmax = sh.w[n - 1];
  int nk = 0, nd = 0;
  for (int m = 0; m < n; ++m) {
    if (lmax > 0.0 && sh.w[m] > tau * lmax)
      ++nk;
    else
      ++nd;
  }
  // T(i, b) = sum_j L(i, j) U(j, c0 + b) into R's storage (the host's inner sums, computed once
  // per (i, b) instead of once per (a, i, b): the same values)
  auto tcols = [&](int c0, int nc) {
    for (int idx = t; idx < n * nc; idx += kCritBlock) {
      const int i = idx / nc, b = idx - i * nc;
      double li = 0.0;
#pragma unroll 8
      for (int j = 0; j < n; ++j) li += L[i * ld + j] * U[j * ld + c0 + b];
      R[i * ld + b] = li;
    }
    wsync();
  };
  if (nd) {
    tcols(0, nd);
    for (int idx = t; idx < nd * nd; idx += kCritBlock) {
      const int a = idx / nd, b = idx - a * nd;
      double v = 0.0;
#pragma unroll 8
      for (int i = 0; i < n; ++i) v += U[i * ld + a] * R[i * ld + b];
      G[a * ld + b] = v;
    }
    wsync();
    double s = 0.0;
    for (int a = 0; a < nd; ++a)
      for (int b = 0; b < nd; ++b) s += G[a * ld + b] * G[a * ld + b];
    if (uni(sqrt(s)) > tau * nL) return crit::inf();
    wsync();
  }
  if (!nk) return 0.0;
  tcols(nd, nk);
  for (int idx = t; idx < nk * nk; idx += kCritBlock) {
    const int a = idx / nk, b = idx - a * nk;
    double v = 0.0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) v += U[i * ld + nd + a] * R[i * ld + b];
    G[a * ld + b] = v / (sqrt(sh.w[nd + a]) * sqrt(sh.w[nd + b]));
  }
  wsync();
  for (int idx = t; idx < nk * nk; idx += kCritBlock) {
    const int a = idx / nk, b = idx - a * nk;
    if (a < b) {
      const double g = 0.5 * (G[a * ld + b] + G[b * ld + a]);
      G[a * ld + b] = G[b * ld + a] = g;
    }
  }
  wsync();
  w_jacobi(G, nk, ld, sh.w, nullptr, nullptr, sh.perm);
  return uni(sh.w[nk - 1]);
}

template <int K>
__device__ __forceinline__ void load_sq(const double *src, double (&X)[K * K]) {
#pragma unroll
  for (int e = 0; e < K * K; ++e) X[e] = src[e];
}
// Y += Q^T X Q, Q = crit::q(t): crit::axpy(Y, 1.0, crit::t3(Q, X, Q)); X is overwritten
template <int K>
__device__ __forceinline__ void add_t3(double (&Y)[K * K], double (&X)[K * K], const double (&t)[3]) {
  if constexpr (K == 6) {
    // rows 3..5 of Q^T X
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const double a = X[j], b = X[6 + j], c = X[12 + j];
      X[18 + j] = 0.0 + t[2] * b + -t[1] * c + X[18 + j];
      X[24 + j] = 0.0 + -t[2] * a + t[0] * c + X[24 + j];
      X[30 + j] = 0.0 + t[1] * a + -t[0] * b + X[30 + j];
    }
    // columns 3..5 of the product by Q
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const double a = X[6 * r], b = X[6 * r + 1], c = X[6 * r + 2];
      X[6 * r + 3] = 0.0 + b * t[2] + c * -t[1] + X[6 * r + 3];
      X[6 * r + 4] = 0.0 + a * -t[2] + c * t[0] + X[6 * r + 4];
      X[6 * r + 5] = 0.0 + a * t[1] + b * -t[0] + X[6 * r + 5];
    }
  }
#pragma unroll
  for (int e = 0; e < K * K; ++e) Y[e] += X[e];
}
// The vectors of crit::qtrans and crit::qhalf
struct Vec3 {
  double v[3];
};
__device__ __forceinline__ Vec3 vtrans(const double *xa, const double *xb) {
  return {{xb[0] - xa[0], xb[1] - xa[1], xb[2] - xa[2]}};
}
__device__ __forceinline__ Vec3 vhalf(const double *xa, const double *xb) {
  return {{0.5 * (xb[0] - xa[0]), 0.5 * (xb[1] - xa[1]), 0.5 * (xb[2] - xa[2])}};
}
// The vector of crit::mul(q(a), q(b)): the skew block of a product is the sum, the right factor's first
__device__ __forceinline__ Vec3 vprod(const Vec3 &a, const Vec3 &b) {
  return {{b.v[0] + a.v[0], b.v[1] + a.v[1], b.v[2] + a.v[2]}};
}

// ---- mu_b, one thread per pair ----------------------------------------------------------------

// C = A B (crit::mul), one thread
template <int K>
__device__ __forceinline__ void t_mul(double (&C)[K * K], const double (&A)[K * K], const double (&B)[K * K]) {
#pragma unroll
  for (int i = 0; i < K; ++i)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      double c = 0.0;
#pragma unroll
      for (int l = 0; l < K; ++l) c = A[i * K + l] == 0.0 ? c : c + A[i * K + l] * B[l * K + j];
      C[i * K + j] = c;
    }
}
// H = crit::harmonic(A, B, tau)
template <int K>
__device__ __forceinline__ void t_harmonic(double (&H)[K * K], const double (&A)[K * K], const double (&B)[K * K],
                                           double tau) {
  double S[K * K], P[K * K];
#pragma unroll
  for (int e = 0; e < K * K; ++e) S[e] = A[e] + B[e];
  t_pinv<K>(P, S, tau);
  t_mul<K>(S, A, P);
  t_mul<K>(P, S, B);
#pragma unroll
  for (int i = 0; i < K; ++i)
#pragma unroll
    for (int j = 0; j < K; ++j) H[i * K + j] = 0.5 * (P[i * K + j] + P[j * K + i]);
}
// X = Q^T src Q, Q = crit::q(t)
template <int K>
__device__ __forceinline__ void t_t3(double (&X)[K * K], const double *src, const Vec3 &t) {
  double S[K * K];
  load_sq<K>(src, S);
#pragma unroll
  for (int e = 0; e < K * K; ++e) X[e] = 0.0;
  add_t3<K>(X, S, t.v);
}

// crit::mu_b on registers up to the final pencil: a pair's chain is one pseudo-inverse per common
// neighbour.  The first pass's pairs of 9,261 vertices take 0.56 ms instead of 6.0 with the matrices in
// scratch memory.
template <int K>
__global__ __launch_bounds__(kCritBlock) void k_mu_b(LevelView w, const Sq *D, int np,
                                                     const int *pairs, double tau, double *out) {
  constexpr int KK = K * K;
  const int stride = gridDim.x * kCritBlock;
  for (int u = blockIdx.x * kCritBlock + threadIdx.x; u < np; u += stride) {
    const int i = pairs[2 * u], j = pairs[2 * u + 1];
    const double *xi = w.xp(i), *xj = w.xp(j);
    const Vec3 vji = vhalf(xj, xi);
    Sq L(K), R(K);
    {
      double A[KK], B[KK], H[KK];
      t_t3<K>(A, D[i].a, vji);
      t_t3<K>(B, D[j].a, vhalf(xi, xj));
      t_harmonic<K>(H, A, B, tau);
#pragma unroll
      for (int e = 0; e < KK; ++e) L.a[e] = H[e];
    }
    double Rr[KK];
    load_sq<K>(w.E + int64_t(w.edge_id(i, j)) * KK, Rr);
    for (int64_t p = w.nb_ptr[i]; p < w.nb_ptr[i + 1]; ++p) {
      const int l = w.nb[p];
      if (l == j) continue;
      const int ejl = w.edge_id(j, l);
      if (ejl < 0) continue;
      const double *xl = w.xp(l);
      double A[KK], B[KK], H[KK];
      t_t3<K>(A, w.E + int64_t(w.nb_e[p]) * KK, vhalf(xl, xi));
      t_t3<K>(B, w.E + int64_t(ejl) * KK, vhalf(xl, xj));
      t_harmonic<K>(H, A, B, tau);
#pragma unroll
      for (int e = 0; e < KK; ++e) A[e] = 0.0;
      add_t3<K>(A, H, vprod(vtrans(xi, xl), vji).v);
#pragma unroll
      for (int e = 0; e < KK; ++e) Rr[e] += 0.5 * A[e];
    }
#pragma unroll
    for (int e = 0; e < KK; ++e) R.a[e] = Rr[e];
    out[u] = crit::genmax(L, R, tau);
  }
}

// crit::mu_g of the union mem[0..nC) (ascending) with the whole wavefront
template <int K>
__device__ __forceinline__ double w_mu_g(const LevelView &lev, const Sq *D, const int *mem, int nC, double tau,
                         WShared &sh) {
  constexpr int KK = K * K;
  const int t = threadIdx.x, n = nC * K, ld = kWLd;
  double xH[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < nC; ++a)
    for (int d = 0; d < 3; ++d) xH[d] = xH[d] + lev.x[int64_t(3) * mem[a] + d];
  for (int d = 0; d < 3; ++d) xH[d] = xH[d] / double(nC);
  double *Z = sh.sm[S_Z], *Zp = sh.sm[S_ZP], *YZ = sh.sm[S_YZ], *S = sh.sm[S_S];
  double *T1 = sh.sm[S_T1], *Q1 = sh.sm[S_Q1], *Q2 = sh.sm[S_Q2], *Ee = sh.sm[S_EE];
  double *X = sh.sm[S_X];
  // L = D_C - D_C P_C pinv(P_C^T D_C P_C) P_C^T D_C
  w_zero<K>(Z);
  for (int a = 0; a < nC; ++a) {
    w_qtrans<K>(Q1, xH, lev.xp(mem[a]));
    w_mul<K>(sh.sm[S_Y + a], D[mem[a]].a, Q1);
    w_mul_tA<K>(X, Q1, sh.sm[S_Y + a]);
    w_axpy<K>(Z, 1.0, X);
  }
  if (t == 0) {
    double z[KK], zp[KK];
    load_sq<K>(Z, z);
    t_pinv<K>(zp, z, tau);
#pragma unroll
    for (int e = 0; e < KK; ++e) Zp[e] = zp[e];
  }
  for (int idx = t; idx < n * n; idx += kCritBlock) {
    const int i = idx / n, j = idx - i * n;
    sh.L[i * ld + j] = 0.0;
    sh.R[i * ld + j] = 0.0;
  }
  wsync();
  for (int a = 0; a < nC; ++a) {
    w_mul<K>(YZ, sh.sm[S_Y + a], Zp);
    for (int b = 0; b < nC; ++b) {
      w_mul_tB<K>(S, YZ, sh.sm[S_Y + b]);
      w_put<K>(sh.L, a, b, S, -1.0, false);
    }
    w_put<K>(sh.L, a, a, D[mem[a]].a, 1.0, false);
    w_put<K>(sh.R, a, a, lev.M + int64_t(mem[a]) * KK, 1.0, false);
  }
  // edges inside C and, in encounter order, the edges to outside neighbours
  int no = 0;
  for (int a = 0; a < nC; ++a) {
    const int i = mem[a];
    for (int64_t p = lev.nb_ptr[i]; p < lev.nb_ptr[i + 1]; ++p) {
      const int l = lev.nb[p], e = lev.nb_e[p];
      int b = -1;
      for (int c = 0; c < nC; ++c)
        if (mem[c] == l) b = c;
      if (b >= 0) {
        if (i < l) {
          w_qhalf<K>(Q1, lev.xp(i), lev.xp(l));
          w_qhalf<K>(Q2, lev.xp(l), lev.xp(i));
          w_load<K>(Ee, lev.E + int64_t(e) * KK);
          w_t3<K>(X, Q1, Ee, Q1, T1);
          w_put<K>(sh.R, a, a, X, 1.0, false);
          w_t3<K>(X, Q2, Ee, Q2, T1);
          w_put<K>(sh.R, b, b, X, 1.0, false);
          w_t3<K>(X, Q1, Ee, Q2, T1);
          w_put<K>(sh.R, a, b, X, -1.0, false);
          w_t3<K>(X, Q2, Ee, Q1, T1);
          w_put<K>(sh.R, b, a, X, -1.0, false);
        }
      } else {
        if (no == kWOut) return __builtin_nan("");
        if (t == 0) {
          sh.ol[no] = l;
          sh.oa[no] = a;
          sh.oe[no] = e;
        }
        ++no;
      }
    }
  }
  wsync();
  // group by outside neighbour, ascending, keeping encounter order within a neighbour: the
  // host's stable insertion sort, as ranks
  for (int s0 = t; s0 < no; s0 += kCritBlock) {
    const int l = sh.ol[s0];
    int r = 0;
    for (int q = 0; q < no; ++q) r += (sh.ol[q] < l || (sh.ol[q] == l && q < s0)) ? 1 : 0;
    sh.sl[r] = l;
    sh.sa[r] = sh.oa[s0];
    sh.se[r] = sh.oe[s0];
  }
  wsync();
  // outside neighbours that meet at least two members: their first entry, in order
  int ng = 0;
  for (int s0 = 0; s0 < no;) {
    int s1 = s0 + 1;
    while (s1 < no && sh.sl[s1] == sh.sl[s0]) ++s1;
    if (s1 - s0 > crit::kMaxUnion) return __builtin_nan("");
    if (s1 - s0 >= 2) {
      if (t == 0) {
        sh.ol[ng] = s0;
        sh.oa[ng] = s1 - s0;
      }
      ++ng;
    }
    s0 = s1;
  }
  wsync();
  // kWInv of them at a time: the pseudo-inverses of their vertex blocks K_ww, one per lane, then the
  // Schur complements on v_C in order
  double *W = sh.UG;
  for (int g0 = 0; g0 < ng; g0 += kWInv) {
    if (t < kWInv && g0 + t < ng) {
      const int s0 = sh.ol[g0 + t], cnt = sh.oa[g0 + t], l = sh.sl[s0];
      double kww[KK], x[KK];
#pragma unroll
      for (int e = 0; e < KK; ++e) kww[e] = 0.0;
      for (int c = 0; c < cnt; ++c) {
        load_sq<K>(lev.E + int64_t(sh.se[s0 + c]) * KK, x);
        add_t3<K>(kww, x, vhalf(lev.xp(l), lev.xp(mem[sh.sa[s0 + c]])).v);
      }
      t_pinv<K>(x, kww, tau);
#pragma unroll
      for (int e = 0; e < KK; ++e) W[t * KK + e] = x[e];
    }
    wsync();
    for (int g = g0; g < ng && g < g0 + kWInv; ++g) {
      const int s0 = sh.ol[g], cnt = sh.oa[g], l = sh.sl[s0];
      int am[crit::kMaxUnion];
      for (int x = 0; x < cnt; ++x) {
        const int a = sh.sa[s0 + x], e = sh.se[s0 + x], i = mem[a];
        w_qhalf<K>(Q1, lev.xp(i), lev.xp(l));
        w_qhalf<K>(Q2, lev.xp(l), lev.xp(i));
        w_load<K>(Ee, lev.E + int64_t(e) * KK);
        am[x] = a;
        w_mul_tA<K>(T1, Q1, Ee);
        w_mul<K>(sh.sm[S_KCC + x], T1, Q1);
        w_mul<K>(sh.sm[S_KCW + x], T1, Q2);
        w_neg<K>(sh.sm[S_KCW + x]);
      }
      double *KW = sh.sm[S_KW];
      for (int x = 0; x < cnt; ++x) {
        w_mul<K>(KW, sh.sm[S_KCW + x], W + (g - g0) * KK);
        for (int y = 0; y < cnt; ++y) {
          w_mul_tB<K>(S, KW, sh.sm[S_KCW + y]);
          w_neg<K>(S);
          if (x == y) w_axpy<K>(S, 1.0, sh.sm[S_KCC + x]);
          w_put<K>(sh.R, am[x], am[y], S, 0.25, false);
          w_put<K>(sh.R, am[y], am[x], S, 0.25, true);
        }
      }
    }
  }
  return w_genmax(n, tau, sh);
}

template <int K>
__global__ __launch_bounds__(kCritBlock) void k_mu_g_wave(LevelView lev, const Sq *D, int nu,
                                                          const int *unions, double tau,
                                                          double *out) {
  __shared__ WShared sh;
  for (int u = blockIdx.x; u < nu; u += gridDim.x) {
    int mem[crit::kMaxUnion];
    int nC = 0;
    for (int a = 0; a < crit::kMaxUnion; ++a) mem[a] = unions[crit::kMaxUnion * u + a];
    while (nC < crit::kMaxUnion && mem[nC] >= 0) ++nC;
    const double v = w_mu_g<K>(lev, D, mem, nC, tau, sh);
    if (threadIdx.x == 0) out[u] = v;
    wsync();
  }
}

// ---- coarse level weights (Thm thm:cemats), one thread per aggregate / coarse edge ------------
//
// A thread's chain over its edges bounds them.  K is a constant and Q, the identity with the skew
// block of a vector, is applied as the sums that its entries leave of crit::t3, in their order (the
// zeros' terms change nothing), so that a congruence is 72 multiplications on registers instead of
// two general products in scratch memory: 47 us a level's vertex weights and 12 us its edge weights
// (cube of 9,261 vertices with inclusions, mean of its levels) instead of 1.57 and 0.72 ms.

// M^I = sum over members i (ascending) of Q^T W_i Q, Q = Q^{I->i}, W_i = M^i + the edges from i
// to dropped vertices pulled to i
template <int K>
__global__ __launch_bounds__(kCritBlock) void k_coarse_M(LevelView f, int nc, const int *mptr,
                                                         const int *mem,
                                                         const unsigned char *dmask,
                                                         const double *cc, double *Mout) {
  constexpr int KK = K * K;
  const int stride = gridDim.x * kCritBlock;
  for (int I = blockIdx.x * kCritBlock + threadIdx.x; I < nc; I += stride) {
    double acc[KK];
#pragma unroll
    for (int e = 0; e < KK; ++e) acc[e] = 0.0;
    for (int a = mptr[I]; a < mptr[I + 1]; ++a) {
      const int i = mem[a];
      double W[KK], X[KK];
      load_sq<K>(f.M + int64_t(i) * KK, W);
      for (int64_t p = f.nb_ptr[i]; p < f.nb_ptr[i + 1]; ++p)
        if (dmask[f.nb[p]]) {
          load_sq<K>(f.E + int64_t(f.nb_e[p]) * KK, X);
          add_t3<K>(W, X, vhalf(f.xp(i), f.xp(f.nb[p])).v);
        }
      add_t3<K>(acc, W, vtrans(cc + int64_t(3) * I, f.xp(i)).v);
    }
#pragma unroll
    for (int e = 0; e < KK; ++e) Mout[int64_t(I) * KK + e] = acc[e];
  }
}

// E^{IJ} = sum over the fine edges (i, j) of the group, in order, of T^T E^{ij} T with
// T = Q^{ij} Q^{I->i} Q^{JI}
template <int K>
__global__ __launch_bounds__(kCritBlock) void k_coarse_E(LevelView f, const int *e0, const int *e1,
                                                         const int *agg_of, const double *cc,
                                                         int64_t ne, const int64_t *start,
                                                         const int64_t *order, double *Eout) {
  constexpr int KK = K * K;
  const int64_t stride = int64_t(gridDim.x) * kCritBlock;
  for (int64_t g = int64_t(blockIdx.x) * kCritBlock + threadIdx.x; g < ne; g += stride) {
    double acc[KK], X[KK];
#pragma unroll
    for (int e = 0; e < KK; ++e) acc[e] = 0.0;
    for (int64_t q = start[g]; q < start[g + 1]; ++q) {
      const int64_t e = order[q];
      const int i = e0[e], j = e1[e];
      const int I = agg_of[i], J = agg_of[j];
      const double *cI = cc + int64_t(3) * I, *cJ = cc + int64_t(3) * J;
      const Vec3 T = vprod(vprod(vhalf(f.xp(i), f.xp(j)), vtrans(cI, f.xp(i))), vhalf(cJ, cI));
      load_sq<K>(f.E + e * KK, X);
      add_t3<K>(acc, X, T.v);
    }
#pragma unroll
    for (int e = 0; e < KK; ++e) Eout[g * KK + e] = acc[e];
  }
}

// Device buffer that only grows.
struct DBuf {
  void *p = nullptr;
  size_t cap = 0;
  DBuf() = default;
  DBuf(const DBuf &) = delete;
  DBuf &operator=(const DBuf &) = delete;
  ~DBuf() {
    if (p) (void)hipFree(p);
  }
  void *reserve(size_t bytes) {
    if (bytes == 0) bytes = 1;
    if (bytes > cap) {
      if (p) hip_check(hipFree(p), "hipFree");
      p = nullptr;
      cap = 0;
      hip_check(hipMalloc(&p, bytes), "hipMalloc");
      cap = bytes;
    }
    return p;
  }
  template <class T>
  T *put(const T *h, size_t count, hipStream_t s) {
    T *d = static_cast<T *>(reserve(count * sizeof(T)));
    hip_check(copy_h2d_sync(d, h, count * sizeof(T), s), "upload");
    return d;
  }
};

// Device copy of one auxiliary level and its D-hat blocks.
struct DevLevel {
  DBuf x, E, M, nb_ptr, nb, nb_e, D, e0b, e1b;
  LevelView v;
  const Sq *d = nullptr;
  const int *e0 = nullptr, *e1 = nullptr;
  int64_t m = 0;
  void upload(const AuxLevel &l, const std::vector<Sq> &Dh, hipStream_t s) {
    if (l.n > 0 && Dh.size() != size_t(l.n)) fail(EAMG_ERR_INVALID_ARG, "criteria: D-hat size");
    v.n = l.n;
    v.k = l.k;
    v.x = x.put(l.x.data(), l.x.size(), s);
    v.E = E.put(l.E.data(), l.E.size(), s);
    v.M = M.put(l.M.data(), l.M.size(), s);
    v.nb_ptr = nb_ptr.put(l.nb_ptr.data(), l.nb_ptr.size(), s);
    v.nb = nb.put(l.nb.data(), l.nb.size(), s);
    v.nb_e = nb_e.put(l.nb_e.data(), l.nb_e.size(), s);
    d = D.put(Dh.data(), Dh.size(), s);
    e0 = e0b.put(l.e0.data(), l.e0.size(), s);
    e1 = e1b.put(l.e1.data(), l.e1.size(), s);
    m = l.m();
    // the sources may change once this returns
    hip_check(hipStreamSynchronize(s), "sync");
  }
};

class DeviceCriteria final : public CritBatch {
 public:
  explicit DeviceCriteria(hipStream_t s) : s_(s) {}

  void level(const AuxLevel &lev, const std::vector<Sq> &D) override {
    lev_.upload(lev, D, s_);
    lev_src_ = &lev;
    work_ = &lev_;
    wrk_src_ = nullptr;
  }
  void work(const AuxLevel &w, const std::vector<Sq> &D) override {
    if (&w == lev_src_) {
      work_ = &lev_;
      return;
    }
    wrk_.upload(w, D, s_);
    work_ = &wrk_;
    wrk_src_ = &w;
  }
  bool coarse_weights(const AuxLevel &fine, const std::vector<std::vector<int>> &aggs,
                      const std::vector<int> &agg_of, const std::vector<char> &dmask,
                      const std::vector<double> &cc, const std::vector<int64_t> &order,
                      const std::vector<int64_t> &start, WeightVec &M,
                      WeightVec &E) override {
    const DevLevel *dl = nullptr;
    if (&fine == lev_src_)
      dl = &lev_;
    else if (&fine == wrk_src_ && work_ == &wrk_)
      dl = &wrk_;
    if (!dl || dl->v.n != fine.n || dl->m != fine.m() || dl->v.k != fine.k || (fine.k != 1 && fine.k != 6))
      return false;
    const auto t0 = std::chrono::steady_clock::now();
    const int k = fine.k, kk = k * k, nc = int(aggs.size());
    const int64_t ne = int64_t(start.size()) - 1;
    // host checks of everything the kernels index with
    if (int64_t(agg_of.size()) != fine.n || int64_t(dmask.size()) != fine.n ||
        int64_t(cc.size()) != int64_t(3) * nc || ne < 0 || start.front() != 0 ||
        start.back() != int64_t(order.size()))
      fail(EAMG_ERR_INVALID_ARG, "coarse weights: sizes");
    std::vector<int> mptr(size_t(nc) + 1, 0), mem;
    for (int I = 0; I < nc; ++I) {
      for (int i : aggs[I]) {
        if (i < 0 || i >= fine.n || agg_of[i] != I) fail(EAMG_ERR_INVALID_ARG, "coarse weights: member");
        mem.push_back(i);
      }
      mptr[I + 1] = int(mem.size());
    }
    for (int64_t e : order)
      if (e < 0 || e >= fine.m() || agg_of[fine.e0[e]] < 0 || agg_of[fine.e1[e]] < 0)
        fail(EAMG_ERR_INVALID_ARG, "coarse weights: edge");
    for (int64_t g = 0; g < ne; ++g)
      if (start[g] > start[g + 1]) fail(EAMG_ERR_INVALID_ARG, "coarse weights: groups");
    std::vector<unsigned char> dm(dmask.begin(), dmask.end());
    const int *d_mptr = cw_mptr_.put(mptr.data(), mptr.size(), s_);
    const int *d_mem = cw_mem_.put(mem.data(), mem.size(), s_);
    const unsigned char *d_dm = cw_dm_.put(dm.data(), dm.size(), s_);
    const double *d_cc = cw_cc_.put(cc.data(), cc.size(), s_);
    const int *d_agg = cw_agg_.put(agg_of.data(), agg_of.size(), s_);
    const int64_t *d_start = cw_start_.put(start.data(), start.size(), s_);
    const int64_t *d_order = cw_order_.put(order.data(), order.size(), s_);
    double *d_M = static_cast<double *>(cw_M_.reserve(size_t(nc) * kk * sizeof(double)));
    double *d_E = static_cast<double *>(cw_E_.reserve(size_t(ne) * kk * sizeof(double)));
    if (nc > 0) {
      const int grid = std::min((nc + kCritBlock - 1) / kCritBlock, 8192);
      if (k == 6)
        hipLaunchKernelGGL(k_coarse_M<6>, dim3(grid), dim3(kCritBlock), 0, s_, dl->v, nc, d_mptr, d_mem, d_dm, d_cc,
                           d_M);
      else
        hipLaunchKernelGGL(k_coarse_M<1>, dim3(grid), dim3(kCritBlock), 0, s_, dl->v, nc, d_mptr, d_mem, d_dm, d_cc,
                           d_M);
      hip_check(hipGetLastError(), "k_coarse_M");
    }
    if (ne > 0) {
      const int grid = int(std::min<int64_t>((ne + kCritBlock - 1) / kCritBlock, 16384));
      if (k == 6)
        hipLaunchKernelGGL(k_coarse_E<6>, dim3(grid), dim3(kCritBlock), 0, s_, dl->v, dl->e0, dl->e1, d_agg, d_cc, ne,
                           d_start, d_order, d_E);
      else
        hipLaunchKernelGGL(k_coarse_E<1>, dim3(grid), dim3(kCritBlock), 0, s_, dl->v, dl->e0, dl->e1, d_agg, d_cc, ne,
                           d_start, d_order, d_E);
      hip_check(hipGetLastError(), "k_coarse_E");
    }
    M.resize(size_t(nc) * kk);   // every entry is downloaded below
    E.resize(size_t(ne) * kk);
    hip_check(copy_d2h_sync(M.data(), d_M, M.size() * sizeof(double), s_), "download");
    hip_check(copy_d2h_sync(E.data(), d_E, E.size() * sizeof(double), s_), "download");
    note("coarse weights", int(ne), t0);
    return true;
  }
  void mu_b(const std::vector<int32_t> &pairs, double tau, std::vector<double> &out) override {
    const int np = int(pairs.size() / 2);
    out.assign(size_t(np), 0.0);
    if (np == 0) return;
    if (!work_) fail(EAMG_ERR_INVALID_ARG, "criteria: no working level");
    // every pair must be an edge of the working level (the kernel reads its edge matrix)
    const AuxLevel *hw = work_ == &lev_ ? lev_src_ : wrk_src_;
    for (int u = 0; u < np; ++u) {
      const int i = pairs[2 * size_t(u)], j = pairs[2 * size_t(u) + 1];
      if (i < 0 || i >= work_->v.n || j < 0 || j >= work_->v.n || !hw || hw->edge_id(i, j) < 0)
        fail(EAMG_ERR_INVALID_ARG, "criteria: pair is not an edge of the working level");
    }
    const auto t0 = std::chrono::steady_clock::now();
    const int *dp = idx_.put(pairs.data(), pairs.size(), s_);
    double *dout = static_cast<double *>(res_.reserve(size_t(np) * sizeof(double)));
    const int grid = std::min((np + kCritBlock - 1) / kCritBlock, 4096);
    if (work_->v.k == 6)
      hipLaunchKernelGGL(k_mu_b<6>, dim3(grid), dim3(kCritBlock), 0, s_, work_->v, work_->d, np, dp, tau, dout);
    else if (work_->v.k == 1)
      hipLaunchKernelGGL(k_mu_b<1>, dim3(grid), dim3(kCritBlock), 0, s_, work_->v, work_->d, np, dp, tau, dout);
    else
      fail(EAMG_ERR_INVALID_ARG, "criteria: k must be 1 or 6");
    hip_check(hipGetLastError(), "k_mu_b");
    hip_check(copy_d2h_sync(out.data(), dout, size_t(np) * sizeof(double), s_), "download");
    note("mu_b", np, t0);
  }
  void mu_g(const std::vector<int32_t> &unions, double tau, std::vector<double> &out) override {
    const int nu = int(unions.size() / crit::kMaxUnion);
    out.assign(size_t(nu), 0.0);
    if (nu == 0) return;
    if (!lev_src_) fail(EAMG_ERR_INVALID_ARG, "criteria: no level");
    if (lev_.v.k != 1 && lev_.v.k != 6) fail(EAMG_ERR_INVALID_ARG, "criteria: k must be 1 or 6");
    for (int u = 0; u < nu; ++u) {
      // members ascending and distinct, at least one, padding only at the end
      const int32_t *m = &unions[size_t(u) * crit::kMaxUnion];
      if (m[0] < 0) fail(EAMG_ERR_INVALID_ARG, "criteria: empty union");
      for (int a = 0; a < crit::kMaxUnion; ++a) {
        if (m[a] >= lev_.v.n) fail(EAMG_ERR_INVALID_ARG, "criteria: union member out of range");
        if (a > 0 && m[a] >= 0 && !(m[a - 1] >= 0 && m[a - 1] < m[a]))
          fail(EAMG_ERR_INVALID_ARG, "criteria: union not ascending");
      }
    }
    const auto t0 = std::chrono::steady_clock::now();
    const int *du = idx_.put(unions.data(), unions.size(), s_);
    double *dout = static_cast<double *>(res_.reserve(size_t(nu) * sizeof(double)));
    const int grid = std::min(nu, kMaxGWaves);
    if (lev_.v.k == 6)
      hipLaunchKernelGGL(k_mu_g_wave<6>, dim3(grid), dim3(kCritBlock), 0, s_, lev_.v, lev_.d, nu, du, tau, dout);
    else
      hipLaunchKernelGGL(k_mu_g_wave<1>, dim3(grid), dim3(kCritBlock), 0, s_, lev_.v, lev_.d, nu, du, tau, dout);
    hip_check(hipGetLastError(), "k_mu_g");
    hip_check(copy_d2h_sync(out.data(), dout, size_t(nu) * sizeof(double), s_), "download");
    if (verbose_) {
      int nan = 0;
      for (double v : out) nan += std::isnan(v) ? 1 : 0;
      if (nan) std::fprintf(stderr, "[eamg]     device mu_g: %d unions beyond the device capacity\n", nan);
    }
    note("mu_g", nu, t0);
  }

 private:
  void note(const char *what, int count, std::chrono::steady_clock::time_point t0) const {
    if (!verbose_) return;
    const double dt = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    std::fprintf(stderr, "[eamg]     device %s: %d in %.4f s\n", what, count, dt);
  }
  const bool verbose_ = std::getenv("EAMG_VERBOSE") != nullptr;
  hipStream_t s_;
  DevLevel lev_, wrk_;
  const AuxLevel *lev_src_ = nullptr, *wrk_src_ = nullptr;
  const DevLevel *work_ = nullptr;
  DBuf idx_, res_;
  DBuf cw_mptr_, cw_mem_, cw_dm_, cw_cc_, cw_agg_, cw_start_, cw_order_, cw_M_, cw_E_;
};

}  // namespace

std::unique_ptr<CritBatch> make_device_criteria(hipStream_t s) {
  return std::unique_ptr<CritBatch>(new DeviceCriteria(s));
}

}  // namespace eamg
