// Block-panel kernels for gfx950: K right-hand sides per launch (layout and lane mapping in
// panel.hpp).  The V-cycle kernels are templated on the value type T of matrices and vectors
// (double, or float for the FP32 V-cycle) and accumulate in T; the CG kernels are FP64.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "panel.hpp"

namespace eamg {
namespace {

constexpr int kPB = 256;   // threads per workgroup; a multiple of every panel width K

inline unsigned pgrid(int64_t items, int per_block) {
  return unsigned((items + per_block - 1) / per_block);
}

// Logical workgroup index of the colour sweeps: workgroup b runs on XCD b mod 8 (round-robin
// dispatch, one L2 per XCD); XCD x takes one contiguous run of logical workgroups so that the
// rows it updates are neighbours and share their gathered x panel blocks in its L2.  A
// bijection on [0, gridDim.x): results do not change.
__device__ inline int xcd_block() {
  const int nb = int(gridDim.x), b = int(blockIdx.x);
  const int x = b & 7, q = nb >> 3, rem = nb & 7;
  return x * q + min(x, rem) + (b >> 3);
}

template <class T>
const T *pvals(const SolveMat &M);
template <>
const double *pvals<double>(const SolveMat &M) {
  return M.val;
}
template <>
const float *pvals<float>(const SolveMat &M) {
  return M.val32;
}

// Logical workgroup of the launches over all rows of a level, whose row lengths may drift along the
// numbering (upper halves): chunks of kChunkWg consecutive workgroups go to the XCDs in turn, so each
// XCD's L2 still sees neighbouring rows together and no XCD gets all the long ones.  The grid is
// rounded up to whole rounds of chunks; workgroups past the rows do nothing.
constexpr int kChunkWg = 32;
__device__ inline int chunk_block(int b) {
  const int x = b & 7, i = b >> 3;
  return (i / kChunkWg * 8 + x) * kChunkWg + i % kChunkWg;
}
inline unsigned chunk_grid(unsigned wgs) { return (wgs + 8 * kChunkWg - 1) / (8 * kChunkWg) * (8 * kChunkWg); }

// A block row belongs to a team of 64 W lanes (W = 1: one wavefront per row, four rows per
// workgroup; W = 4: the whole workgroup on one row, for levels of few long rows).  A lane owns C
// consecutive columns (register blocking: every matrix value it loads serves C columns, and the
// C values of one dof are one vector load); the K / C lanes covering a panel form a sub-team,
// and the S = 64 W C / K sub-teams of the team take the row's blocks in turn: sub-team s reads
// blocks p0 + s, p0 + s + S, ...  At every step the S sub-teams read S consecutive blocks (one
// contiguous run of memory), and the column index of a sub-team's next block is
// fetched one step ahead, so a step waits for one round of gathers only.
//
// The lanes of a sub-team need the same block.  Q neighbours among them (all blocks of 6x6, 3x6 and 6x3
// entries; Q = 2 or 4, see share_log2) load 1/Q of it each and hand the values round by DPP: the loads
// of a block's entries, 9 of the 15 vector loads of a 6x6 block in FP32, drop to 3, and their registers
// with them.  64^3 x 32 FP32 69.9 -> 65.3 ms, 37x29x33 x 7 FP64 13.6 -> 12.8 ms.  Bound then: the x
// panels from L2 (level 1's backward colours gather 14 TB/s); more wavefronts per SIMD (five for four)
// change nothing.
//
// The row's BR K sums then spread over the lanes: halving exchanges across the sub-teams of a
// wavefront (each lane ends with its share of the values, 21 shuffles for 6 x 4 values over eight
// sub-teams where a butterfly takes 72), the wavefronts' shares meeting in LDS in wavefront order.
// Output o of a row is entry (dof o / K, column o mod K), at o past the row's first entry of every
// panel, so lane t of the team finishes outputs t, t + 64 W, ...: every lane works on the row's end,
// its loads of b, x and y are coalesced and are issued with the row's first loads, and D^+ costs one
// register per lane.  (Before, the K / C lanes of sub-team 0 finished the row, each loading all of
// D^+ and, after the sums, its old x or A_ii: FP64 sweeps in 304 registers, 13.4 and 11.7 us per colour
// of 400 rows and 8 columns; now 5.8 and 6.0 us.)
constexpr int kWave = 64;
constexpr int kMaxK = 64;

template <class T, int C>
struct PVec {
  T v[C];
};

// X entries of one dof for columns g C .. g C + C - 1 (C-aligned, contiguous).
template <class T, int C>
__device__ inline PVec<T, C> pload(const T *p) {
  PVec<T, C> out;
  if constexpr (C == 1) {
    out.v[0] = p[0];
  } else {
    typedef T vec_t __attribute__((ext_vector_type(C)));
    const vec_t w = *reinterpret_cast<const vec_t *>(p);
#pragma unroll
    for (int i = 0; i < C; ++i) out.v[i] = w[i];
  }
  return out;
}

// Columns per lane C, and how many consecutive lanes Q share a block's values (pteam_sums):
// CQ = C + kQuad log2(Q).
constexpr int kQuad = 16;

// Where a thread sits in a row team of 64 W lanes for K columns, C per lane.
template <int CQ, int W>
struct PTeam {
  static constexpr int C = CQ % kQuad;

  int row_in_wg;   // which of the kPB / (64 W) rows of the workgroup
  int t;           // lane within the row team
  int lg;          // log2(K / C)
  int g;           // column group (columns g C .. g C + C - 1)
  int s;           // sub-team
  int S;           // sub-teams per row
  __device__ PTeam(int K) {
    row_in_wg = threadIdx.x / (kWave * W);
    t = threadIdx.x % (kWave * W);
    lg = __builtin_ctz(K / C);
    g = t & ((K / C) - 1);
    s = t >> lg;
    S = (kWave * W) >> lg;
  }
};

// LDS values written by the team's lanes become visible to all of them: a workgroup barrier, or
// for a team of one wavefront (whose LDS operations are in order) a compiler fence.
template <int W>
__device__ inline void pteam_sync() {
  if constexpr (W > 1) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// One halving exchange: the lanes of a pair (lane bit `off`) each keep half of the first 2 H values,
// summed with the partner's.
template <int H, class T, int N>
__device__ __forceinline__ void phalve(T (&v)[N], int off) {
  const bool up = (threadIdx.x & off) != 0;
#pragma unroll
  for (int k = 0; k < H; ++k) {
    const T send = up ? v[k] : v[k + H];
    const T keep = up ? v[k + H] : v[k];
    v[k] = keep + __shfl_xor(send, off, kWave);
  }
}

template <int N, class T, int M>
__device__ __forceinline__ void pbutterfly(T (&v)[M], int off) {
  for (; off < kWave; off <<= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += __shfl_xor(v[k], off, kWave);
}

// The value that lane q of this lane's group of Q (2 or 4) consecutive lanes holds in v.
template <int Q, int q>
__device__ __forceinline__ int shared_bits(int v) {
  constexpr int perm = Q == 4 ? q * 0x55 : (q ? 0xf5 : 0xa0);   // quad_perm: q q q q, or q q q+2 q+2
  return __builtin_amdgcn_mov_dpp(v, perm, 0xf, 0xf, true);
}
template <int Q>
__device__ __forceinline__ int shared_bits(int v, int q) {
  if constexpr (Q == 2) return q == 0 ? shared_bits<2, 0>(v) : shared_bits<2, 1>(v);
  return q == 0 ? shared_bits<4, 0>(v) : q == 1 ? shared_bits<4, 1>(v) : q == 2 ? shared_bits<4, 2>(v) : shared_bits<4, 3>(v);
}
template <int Q>
__device__ __forceinline__ float shared_value(float v, int q) {
  return __int_as_float(shared_bits<Q>(__float_as_int(v), q));
}
template <int Q>
__device__ __forceinline__ double shared_value(double v, int q) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(shared_bits<Q>(int(b & 0xffffffffLL), q));
  const int hi = shared_bits<Q>(int(b >> 32), q);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | lo);
}

// The row's sums over blocks p in [p0, p1) of M_p X_col(p), by wavefront: entry (r, column k) of
// wavefront w's share at red[(w BR + r) K + k], visible to the team on return.
template <class T, int BR, int BC, int CQ, int W>
__device__ inline void pteam_sums(int p0, int p1, int K, const PTeam<CQ, W> &tm,
                                  const int *__restrict__ col, const T *__restrict__ val,
                                  const T *__restrict__ x, T *red) {
  constexpr int C = CQ % kQuad;
  constexpr int Q = 1 << (CQ / kQuad), per = BR * BC / Q;   // lanes that share a block, values each loads
  constexpr int NV = BR * C;
  T acc[NV];
#pragma unroll
  for (int e = 0; e < NV; ++e) acc[e] = T(0);
  int p = p0 + tm.s;
  int cn = p < p1 ? col[p] : 0;
  for (; p < p1; p += tm.S) {
    const int64_t c = cn;
    const int pn = p + tm.S;
    cn = pn < p1 ? col[pn] : 0;
    T a[per];
    const T *mine = val + int64_t(p) * (BR * BC) + (Q > 1 ? (tm.g & (Q - 1)) * per : 0);
#pragma unroll
    for (int e = 0; e < per; ++e) a[e] = mine[e];
    PVec<T, C> xv[BC];
#pragma unroll
    for (int cc = 0; cc < BC; ++cc) xv[cc] = pload<T, C>(x + (c * BC + cc) * K + tm.g * C);
    // the whole block and its gathers in flight together (64^3 x 32 FP32 86.1 -> 84.6 ms, 37x29x33 x 7
    // FP64 17.8 -> 17.0 ms); a further block ahead only costs registers (68.0 ms, not 65.3)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < BR; ++r)
#pragma unroll
      for (int cc = 0; cc < BC; ++cc)
#pragma unroll
        for (int i = 0; i < C; ++i) {
          const int e = r * BC + cc;
          T m;
          if constexpr (Q > 1)
            m = shared_value<Q>(a[e % per], e / per);
          else
            m = a[e];
          acc[r * C + i] = fma(m, xv[cc].v[i], acc[r * C + i]);
        }
  }
  // K <= 64: a wavefront has at least four sub-teams
  constexpr int H1 = NV % 2 == 0 ? NV / 2 : 0, H2 = NV % 4 == 0 ? NV / 4 : 0, H3 = NV % 8 == 0 ? NV / 8 : 0;
  T *rw = red + size_t(tm.t / kWave) * BR * K;
  const int ln = tm.t % kWave;
  int off = K / C, base = 0;
  if constexpr (H1 > 0) {
    phalve<H1>(acc, off);
    base += (ln & off) ? H1 : 0;
    off <<= 1;
  }
  if constexpr (H2 > 0) {
    phalve<H2>(acc, off);
    base += (ln & off) ? H2 : 0;
    off <<= 1;
  }
  auto put = [&](auto count) {
    constexpr int n = decltype(count)::value;
    pbutterfly<n>(acc, off);
    if (ln < off)   // the remaining lane bits hold copies
#pragma unroll
      for (int k = 0; k < n; ++k) {
        const int e = base + k;
        rw[(e / C) * K + tm.g * C + e % C] = acc[k];
      }
  };
  constexpr int N2 = H2 > 0 ? H2 : (H1 > 0 ? H1 : NV);
  if constexpr (H3 > 0) {
    if (off < kWave) {
      phalve<H3>(acc, off);
      base += (ln & off) ? H3 : 0;
      off <<= 1;
      put(std::integral_constant<int, H3>{});
    } else {
      put(std::integral_constant<int, N2>{});
    }
  } else {
    put(std::integral_constant<int, N2>{});
  }
  pteam_sync<W>();
}

// Output o of the row: the wavefronts' shares in wavefront order.
template <class T, int BR, int W>
__device__ inline T pout(const T *red, int K, int o) {
  T v = red[o];
#pragma unroll
  for (int w = 1; w < W; ++w) v += red[size_t(w) * BR * K + o];
  return v;
}

// Outputs per lane at the widest panel, and LDS values of a workgroup's shares.
template <int B, int W>
struct PSize {
  static constexpr int outs = (B * kMaxK + kWave * W - 1) / (kWave * W);
  static constexpr int red = (kPB / kWave) * B * kMaxK;
  static constexpr int rows = kPB / (kWave * W);
};

// One colour of the symmetric block Gauss-Seidel sweep for K columns (see launch_pgs_fwd /
// launch_pgs_bwd).  FWD: rp, col, val hold the blocks left of the diagonal and dval the diagonal
// blocks (block i for row i); BWD: rp, col, val hold whole rows.  y: the panel the blocks multiply
// (x itself, or b for a group of colours: see launch_pgs_group).
template <class T, int B, bool FWD, int C, int W>
__global__ __launch_bounds__(kPB) void k_pgs_color(int r0, int r1, int K, const int *__restrict__ rp,
                                                   const int *__restrict__ col,
                                                   const T *__restrict__ val,
                                                   const T *__restrict__ dval,
                                                   const T *__restrict__ Dinv,
                                                   const T *__restrict__ b, const T *y, T *x, T *r) {
  using Z = PSize<B, W>;
  __shared__ T red_s[Z::red], x_s[FWD ? Z::rows * B * kMaxK : 1], D_s[Z::rows][B * B],
      A_s[FWD ? Z::rows : 1][FWD ? B * B : 1];
  const PTeam<C, W> tm(K);
  const int row = r0 + xcd_block() * Z::rows + tm.row_in_wg;
  if (row >= r1) return;   // W = 4: the whole workgroup leaves together; W = 1: whole wavefronts
  const int n = B * K;
  const int64_t rb = int64_t(row) * n;
  const int p0 = rp[row], p1 = rp[row + 1];
  T bq[Z::outs], xo[Z::outs], Dv = T(0), Av = T(0);
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    bq[j] = o < n ? b[rb + o] : T(0);
    xo[j] = !FWD && o < n ? x[rb + o] : T(0);
  }
  if (tm.t < B * B) {
    Dv = Dinv[int64_t(row) * (B * B) + tm.t];
    if (FWD) Av = dval[int64_t(row) * (B * B) + tm.t];
  }
  T *red = red_s + size_t(tm.row_in_wg) * W * n;
  T *xs = x_s + (FWD ? size_t(tm.row_in_wg) * n : 0);
  T *Ds = D_s[tm.row_in_wg], *As = A_s[FWD ? tm.row_in_wg : 0];
  if (tm.t < B * B) {
    Ds[tm.t] = Dv;
    if (FWD) As[tm.t] = Av;
  }
  pteam_sums<T, B, B, C, W>(p0, p1, K, tm, col, val, y, red);
  T t[Z::outs];
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    if (o < n) {
      t[j] = bq[j] - pout<T, B, W>(red, K, o);
      red[o] = t[j];   // only this lane reads entry o of any share before the next sync
    }
  }
  pteam_sync<W>();
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    if (o < n) {
      const int q = o / K, k = o % K;
      T v = T(0);
#pragma unroll
      for (int c = 0; c < B; ++c) v = fma(Ds[q * B + c], red[c * K + k], v);
      if (FWD) {
        xs[o] = v;
        x[rb + o] = v;
      } else {
        x[rb + o] = xo[j] + v;
      }
    }
  }
  if constexpr (FWD) {
    pteam_sync<W>();
#pragma unroll
    for (int j = 0; j < Z::outs; ++j) {
      const int o = tm.t + j * kWave * W;
      if (o < n) {
        const int q = o / K, k = o % K;
        T v = t[j];
#pragma unroll
        for (int c = 0; c < B; ++c) v = fma(-As[q * B + c], xs[c * K + k], v);
        r[rb + o] = v;
      }
    }
  }
}

// r_i = b_i - sum over the blocks [rp[i], re[i]) of A_ij x_j on rows [r0, r1) (b may be r).
// CHUNK: rows of every colour (the residual update); else one group's rows.
template <class T, int B, int C, int W, bool CHUNK>
__global__ __launch_bounds__(kPB) void k_presid(int r0, int r1, int K, const int *__restrict__ rp,
                                                const int *__restrict__ re, const int *__restrict__ col,
                                                const T *__restrict__ val, const T *__restrict__ x,
                                                const T *b, T *r) {
  using Z = PSize<B, W>;
  __shared__ T red_s[Z::red];
  const PTeam<C, W> tm(K);
  const int row = r0 + (CHUNK ? chunk_block(int(blockIdx.x)) : xcd_block()) * Z::rows + tm.row_in_wg;
  if (row >= r1) return;
  const int n = B * K;
  const int64_t rb = int64_t(row) * n;
  T bq[Z::outs];
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    bq[j] = o < n ? b[rb + o] : T(0);
  }
  T *red = red_s + size_t(tm.row_in_wg) * W * n;
  pteam_sums<T, B, B, C, W>(rp[row], re[row], K, tm, col, val, x, red);
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    if (o < n) r[rb + o] = bq[j] - pout<T, B, W>(red, K, o);
  }
}

template <class T, int BR, int BC, int C, int W>
__global__ __launch_bounds__(kPB) void k_prect(int n_rows, int K, const int *__restrict__ rp,
                                               const int *__restrict__ col,
                                               const T *__restrict__ val, const T *__restrict__ x,
                                               T *__restrict__ y, int accumulate) {
  using Z = PSize<BR, W>;
  __shared__ T red_s[Z::red];
  const PTeam<C, W> tm(K);
  const int row = chunk_block(int(blockIdx.x)) * Z::rows + tm.row_in_wg;
  if (row >= n_rows) return;
  const int n = BR * K;
  const int64_t rb = int64_t(row) * n;
  T yo[Z::outs];
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    yo[j] = accumulate && o < n ? y[rb + o] : T(0);
  }
  T *red = red_s + size_t(tm.row_in_wg) * W * n;
  pteam_sums<T, BR, BC, C, W>(rp[row], rp[row + 1], K, tm, col, val, x, red);
#pragma unroll
  for (int j = 0; j < Z::outs; ++j) {
    const int o = tm.t + j * kWave * W;
    if (o < n) y[rb + o] = yo[j] + pout<T, BR, W>(red, K, o);
  }
}

// Reduce v over the threads of a workgroup that share t mod K; the sums end in threads t < K.
__device__ inline double pcol_sum(double v, int K, double *sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = kPB / 2; s >= K; s >>= 1) {
    if (int(threadIdx.x) < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  return sh[threadIdx.x];
}

// Y = A X (W = 1 teams), the workgroups striding over groups of four rows so that the
// per-column partial sums of X.Y come in at most kPSpmvMax workgroups.  A lane's outputs all belong
// to column (lane mod K).
constexpr int kPSpmvMax = 2048;

template <int B, int C>
__global__ __launch_bounds__(kPB) void k_pspmv(int n_rows, int K, const int *__restrict__ rp,
                                               const int *__restrict__ col,
                                               const double *__restrict__ val,
                                               const double *__restrict__ x, double *__restrict__ y,
                                               double *part) {
  using Z = PSize<B, 1>;
  __shared__ double red_s[Z::red], sh[kPB];
  const PTeam<C, 1> tm(K);
  const int n = B * K;
  double *red = red_s + size_t(tm.row_in_wg) * n;
  double d = 0.0;
  for (int wg = int(blockIdx.x); wg * Z::rows < n_rows + 8 * kChunkWg * Z::rows; wg += int(gridDim.x)) {
    const int row = chunk_block(wg) * Z::rows + tm.row_in_wg;
    if (row >= n_rows) continue;   // whole wavefronts; no workgroup barrier inside
    const int64_t rb = int64_t(row) * n;
    pteam_sums<double, B, B, C, 1>(rp[row], rp[row + 1], K, tm, col, val, x, red);
#pragma unroll
    for (int j = 0; j < Z::outs; ++j) {
      const int o = tm.t + j * kWave;
      if (o < n) {
        const double v = red[o];
        y[rb + o] = v;
        d = fma(x[rb + o], v, d);
      }
    }
    pteam_sync<1>();   // the next row's shares overwrite this one's
  }
  if (part) {
    const double t = pcol_sum(d, K, sh);
    if (int(threadIdx.x) < K) part[int64_t(blockIdx.x) * K + threadIdx.x] = t;
  }
}

// ---- panel CG vectors -------------------------------------------------------------------------
// Entry e of a panel vector belongs to column e mod K; grid strides are multiples of K, so a
// thread always meets the same column.

constexpr int kPDotMax = 1024;

// b in double, or the FP32 V-cycle's output read as it is
template <class TB>
__global__ __launch_bounds__(kPB) void k_pdot(int64_t n, int K, const double *__restrict__ a,
                                              const TB *__restrict__ b, double *part) {
  __shared__ double sh[kPB];
  double s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kPB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kPB)
    s = fma(a[i], double(b[i]), s);
  const double t = pcol_sum(s, K, sh);
  if (int(threadIdx.x) < K) part[int64_t(blockIdx.x) * K + threadIdx.x] = t;
}

__global__ __launch_bounds__(kPB) void k_preduce(int nparts, int K, const double *__restrict__ part,
                                                 double *scal, int slot, int op) {
  __shared__ double sh[kPB];
  const int k = threadIdx.x & (K - 1);
  double s = 0.0;
  // unrolled so that the loads are in flight together; the sum keeps its order
#pragma unroll 16
  for (int j = threadIdx.x / K; j < nparts; j += kPB / K) s += part[int64_t(j) * K + k];
  const double t = pcol_sum(s, K, sh);
  if (int(threadIdx.x) >= K) return;
  double *S = scal;
  auto at = [&](int sl) -> double & { return S[sl * K + k]; };
  at(slot) = t;
  const bool active = at(PS_ACTIVE) != 0.0;
  auto stop_bad = [&]() {
    at(PS_BAD) = 1.0;
    at(PS_ACTIVE) = 0.0;
  };
  switch (op) {
    case PRED_INIT: {
      const bool finite = at(PS_NONFINITE) == 0.0 && isfinite(t);
      at(PS_ACTIVE) = (finite && t > 0.0) ? 1.0 : 0.0;
      at(PS_CONV) = (finite && t == 0.0) ? 1.0 : 0.0;
      at(PS_BAD) = finite ? 0.0 : 1.0;
      break;
    }
    case PRED_RHO0:
      if (active && !(t > 0.0 && isfinite(t))) {
        at(PS_ACTIVE) = 0.0;
        if (at(PS_RR0) == 0.0)
          at(PS_CONV) = 1.0;
        else
          at(PS_BAD) = 1.0;
      }
      break;
    case PRED_ALPHA:
      if (active) {
        if (!(t > 0.0) || !isfinite(t)) {
          stop_bad();
          at(PS_ALPHA) = 0.0;
        } else {
          at(PS_ALPHA) = at(PS_RHO) / t;
        }
      }
      break;
    case PRED_BETA:
      if (active) {
        if (!(t > 0.0) || !isfinite(t)) {
          stop_bad();
        } else {
          at(PS_BETA) = t / at(PS_RHO);
          at(PS_RHO) = t;
        }
      }
      break;
    case PRED_RR:
      if (active) {
        at(PS_ITS) += 1.0;
        if (!isfinite(t)) {
          stop_bad();
        } else if (sqrt(t) <= at(PS_RTOL) * sqrt(at(PS_BB))) {
          at(PS_ACTIVE) = 0.0;
          at(PS_CONV) = 1.0;
        } else if (at(PS_ITS) >= at(PS_MAXIT)) {
          at(PS_ACTIVE) = 0.0;
        }
      }
      break;
    default: break;
  }
}

__global__ __launch_bounds__(kPB) void k_pupdate_xr(int64_t n, int K, const double *__restrict__ scal,
                                                    double *x, double *r, const double *__restrict__ p,
                                                    const double *__restrict__ q, double *part,
                                                    float *__restrict__ r32) {
  __shared__ double sh[kPB];
  const int k = threadIdx.x & (K - 1);
  const bool active = scal[PS_ACTIVE * K + k] != 0.0;
  const double alpha = scal[PS_ALPHA * K + k];
  double s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kPB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kPB) {
    double ri = r[i];
    if (active) {
      x[i] = fma(alpha, p[i], x[i]);
      ri = fma(-alpha, q[i], ri);
      r[i] = ri;
      if (r32) r32[i] = float(ri);
    }
    s = fma(ri, ri, s);
  }
  const double t = pcol_sum(s, K, sh);
  if (int(threadIdx.x) < K) part[int64_t(blockIdx.x) * K + threadIdx.x] = t;
}

template <class TZ>
__global__ __launch_bounds__(kPB) void k_pupdate_p(int64_t n, int K, const double *__restrict__ scal,
                                                   const TZ *__restrict__ z, double *p) {
  const int k = threadIdx.x & (K - 1);
  if (scal[PS_ACTIVE * K + k] == 0.0) return;
  const double beta = scal[PS_BETA * K + k];
  for (int64_t i = int64_t(blockIdx.x) * kPB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kPB)
    p[i] = fma(beta, p[i], double(z[i]));
}

__global__ void k_pinit_scal(int K, double rtol, double max_it, double *scal) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= PS_COUNT * K) return;
  const int slot = i / K;
  scal[i] = slot == PS_RTOL ? rtol : slot == PS_MAXIT ? max_it : 0.0;
}

__global__ void k_pfinite(int64_t n, int K, const double *a, double *scal) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n && !isfinite(a[i])) scal[PS_NONFINITE * K + int(i % K)] = 1.0;
}

__global__ void k_pzero_unstarted(int64_t n, int K, const double *scal, double *x) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k = int(i % K);
  if (scal[PS_BB * K + k] == 0.0 || scal[PS_NONFINITE * K + k] != 0.0) x[i] = 0.0;
}

__global__ void k_ppack(int n, int bs, int K, int nrhs, const int *perm, const uint8_t *mask,
                        const double *in, int64_t ld, double *out) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= int64_t(n) * bs * K) return;
  const int k = int(gid % K);
  const int64_t d = gid / K;
  const int64_t r = d / bs;
  const int c = int(d % bs);
  const int o = perm[r];
  out[gid] = (k >= nrhs || (mask && mask[o])) ? 0.0 : in[int64_t(k) * ld + int64_t(o) * bs + c];
}

__global__ void k_punpack(int n, int bs, int K, int nrhs, const int *perm, const double *in,
                          double *out, int64_t ld) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= int64_t(n) * bs * K) return;
  const int k = int(gid % K);
  if (k >= nrhs) return;
  const int64_t d = gid / K;
  const int64_t r = d / bs;
  const int c = int(d % bs);
  out[int64_t(k) * ld + int64_t(perm[r]) * bs + c] = in[gid];
}

bool valid_k(int K) { return K >= 1 && K <= 64 && (K & (K - 1)) == 0; }

}  // namespace

#define EAMG_PCHECK() return hipGetLastError()

// Columns per lane: 4 when the panel is at least 4 wide.
inline int pcols(int K) { return K >= 4 ? 4 : K; }

// Team width: a whole workgroup per row when its 64 * 4 * C / K sub-teams still find a block
// each in an average row, else one wavefront per row.
inline int pwaves(const SolveMat &M, int K) {
  if (M.panel_waves == 1 || M.panel_waves == 4) return M.panel_waves;   // tuned
  const double avg = M.n_rows ? double(M.nnz) / M.n_rows : 0.0;
  return (kWave * 4.0 * pcols(K) / K <= avg) ? 4 : 1;
}

inline unsigned pteam_grid(int rows, int W) { return pgrid(rows, kPB / (kWave * W)); }

// SHARE_: log2 of the lanes that may share a block (0: none); a sub-team has K / 4 of them
#define EAMG_PCOLS_Q(C_, SHARE_, ...)                                                          \
  switch (pcols(K)) {                                                                          \
    case 1: { constexpr int C_ = 1; __VA_ARGS__; } break;                                      \
    case 2: { constexpr int C_ = 2; __VA_ARGS__; } break;                                      \
    default:                                                                                   \
      if (K >= 16) { constexpr int C_ = 4 + kQuad * (SHARE_); __VA_ARGS__; }                   \
      else if (K >= 8) { constexpr int C_ = 4 + kQuad * ((SHARE_) ? 1 : 0); __VA_ARGS__; }     \
      else { constexpr int C_ = 4; __VA_ARGS__; }                                              \
      break;                                                                                   \
  }
#define EAMG_PCOLS(C_, ...) EAMG_PCOLS_Q(C_, 0, __VA_ARGS__)
// 9 entries a lane: 36 over four lanes, 18 over two; blocks of 1 or 9 stay whole.
constexpr int share_log2(int br, int bc) { return br * bc == 36 ? 2 : br * bc == 18 ? 1 : 0; }
#define EAMG_PTEAM(W_, M_, ...)                                 \
  if (pwaves(M_, K) == 4) { constexpr int W_ = 4; __VA_ARGS__; } \
  else { constexpr int W_ = 1; __VA_ARGS__; }

template <class T, bool FWD>
hipError_t launch_pgs(const SolveMat &A, const T *Dinv, int r0, int r1, int K, const T *b, T *x, T *r,
                      hipStream_t s) {
  if (r1 <= r0) return hipSuccess;
  const bool f32 = sizeof(T) == 4;
  const T *val = FWD ? reinterpret_cast<const T *>(f32 ? (const void *)A.lo_val32 : (const void *)A.lo_val)
                     : pvals<T>(A);
  const T *dval = FWD ? reinterpret_cast<const T *>(f32 ? (const void *)A.dg_val32 : (const void *)A.dg_val)
                      : nullptr;
  const int *rp = FWD ? A.lo_rp : A.rp;
  const int *col = FWD ? A.lo_col : A.col;
  if (!val || !rp || !valid_k(K) || (FWD && !dval) || r0 < 0 || r1 > A.n_rows) return hipErrorInvalidValue;
#define EAMG_PGS(B_)                                                                                \
  EAMG_PTEAM(W, A, EAMG_PCOLS_Q(C, share_log2(B_, B_), hipLaunchKernelGGL((k_pgs_color<T, B_, FWD, C, W>),               \
                                                    dim3(pteam_grid(r1 - r0, W)), dim3(kPB), 0, s, \
                                                    r0, r1, K, rp, col, val, dval, Dinv, b, x, x,  \
                                                    r)))
  switch (A.br) {
    case 1: EAMG_PGS(1); break;
    case 3: EAMG_PGS(3); break;
    case 6: EAMG_PGS(6); break;
    default: return hipErrorInvalidValue;
  }
#undef EAMG_PGS
  EAMG_PCHECK();
}

template <class T>
hipError_t launch_pgs_fwd(const SolveMat &A, const T *Dinv, int r0, int r1, int K, const T *b, T *x,
                          T *r, hipStream_t s) {
  return launch_pgs<T, true>(A, Dinv, r0, r1, K, b, x, r, s);
}

template <class T>
hipError_t launch_pgs_bwd(const SolveMat &A, const T *Dinv, int r0, int r1, int K, const T *b, T *x,
                          hipStream_t s) {
  return launch_pgs<T, false>(A, Dinv, r0, r1, K, b, x, nullptr, s);
}

template <class T>
hipError_t launch_pgroup_rhs(const SolveMat &A, const int *lo_end, int r0, int r1, int K, const T *b,
                             const T *x, T *u, hipStream_t s) {
  if (r0 < 0 || r1 > A.n_rows || !valid_k(K)) return hipErrorInvalidValue;
  if (r1 <= r0) return hipSuccess;
  const bool f32 = sizeof(T) == 4;
  const T *val = lo_end ? reinterpret_cast<const T *>(f32 ? (const void *)A.lo_val32 : (const void *)A.lo_val)
                        : pvals<T>(A);
  const int *rp = lo_end ? A.lo_rp : A.rp, *re = lo_end ? lo_end : A.rp + 1;
  const int *col = lo_end ? A.lo_col : A.col;
  if (!val || !rp) return hipErrorInvalidValue;
#define EAMG_PRHS(B_)                                                                             \
  EAMG_PTEAM(W, A, EAMG_PCOLS_Q(C, share_log2(B_, B_), hipLaunchKernelGGL((k_presid<T, B_, C, W, false>),              \
                                                    dim3(pteam_grid(r1 - r0, W)), dim3(kPB), 0,  \
                                                    s, r0, r1, K, rp, re, col, val, x, b, u)))
  switch (A.br) {
    case 1: EAMG_PRHS(1); break;
    case 3: EAMG_PRHS(3); break;
    case 6: EAMG_PRHS(6); break;
    default: return hipErrorInvalidValue;
  }
#undef EAMG_PRHS
  EAMG_PCHECK();
}

namespace {
template <class T, bool FWD>
hipError_t launch_pgroup(const SolveMat &S, const T *dval, const T *Dinv, int r0, int r1, int K,
                         const T *u, T *x, T *r, hipStream_t s) {
  if (r0 < 0 || r1 > S.n_rows || !valid_k(K)) return hipErrorInvalidValue;
  if (r1 <= r0) return hipSuccess;
  const T *val = pvals<T>(S);
  if (!val || !S.rp || (FWD && !dval)) return hipErrorInvalidValue;
#define EAMG_PGRP(B_)                                                                               \
  EAMG_PTEAM(W, S, EAMG_PCOLS_Q(C, share_log2(B_, B_), hipLaunchKernelGGL((k_pgs_color<T, B_, FWD, C, W>),               \
                                                    dim3(pteam_grid(r1 - r0, W)), dim3(kPB), 0, s, \
                                                    r0, r1, K, S.rp, S.col, val, dval, Dinv, u, u, \
                                                    x, r)))
  switch (S.br) {
    case 1: EAMG_PGRP(1); break;
    case 3: EAMG_PGRP(3); break;
    case 6: EAMG_PGRP(6); break;
    default: return hipErrorInvalidValue;
  }
#undef EAMG_PGRP
  EAMG_PCHECK();
}
}  // namespace

template <class T>
hipError_t launch_pgroup_fwd(const SolveMat &A, const SolveMat &S, const T *Dinv, int r0, int r1, int K,
                             const T *u, T *x, T *r, hipStream_t s) {
  const T *dval = reinterpret_cast<const T *>(sizeof(T) == 4 ? (const void *)A.dg_val32 : (const void *)A.dg_val);
  return launch_pgroup<T, true>(S, dval, Dinv, r0, r1, K, u, x, r, s);
}

template <class T>
hipError_t launch_pgroup_bwd(const SolveMat &S, const T *Dinv, int r0, int r1, int K, const T *u, T *x,
                             hipStream_t s) {
  return launch_pgroup<T, false>(S, nullptr, Dinv, r0, r1, K, u, x, nullptr, s);
}

template <class T>
hipError_t launch_presid_upper(const SolveMat &A, int K, const T *x, T *r, hipStream_t s) {
  if (A.n_rows == 0) return hipSuccess;
  const T *val = reinterpret_cast<const T *>(sizeof(T) == 4 ? (const void *)A.up_val32 : (const void *)A.up_val);
  if (!val || !A.up_rp || !valid_k(K)) return hipErrorInvalidValue;
#define EAMG_PRES(B_)                                                                             \
  EAMG_PTEAM(W, A, EAMG_PCOLS_Q(C, share_log2(B_, B_), hipLaunchKernelGGL((k_presid<T, B_, C, W, true>),               \
                                                    dim3(chunk_grid(pteam_grid(A.n_rows, W))),   \
                                                    dim3(kPB), 0, s, 0, A.n_rows, K, A.up_rp,    \
                                                    A.up_rp + 1, A.up_col, val, x, r, r)))
  switch (A.br) {
    case 1: EAMG_PRES(1); break;
    case 3: EAMG_PRES(3); break;
    case 6: EAMG_PRES(6); break;
    default: return hipErrorInvalidValue;
  }
#undef EAMG_PRES
  EAMG_PCHECK();
}

template <class T>
hipError_t launch_prect(const SolveMat &M, int K, const T *x, T *y, bool accumulate, hipStream_t s) {
  if (M.n_rows == 0) return hipSuccess;
  const T *val = pvals<T>(M);
  if (!val || !valid_k(K)) return hipErrorInvalidValue;
  const int accf = accumulate ? 1 : 0;
#define EAMG_PRECT(BR_, BC_)                                                                      \
  EAMG_PTEAM(W, M, EAMG_PCOLS_Q(C, share_log2(BR_, BC_), hipLaunchKernelGGL((k_prect<T, BR_, BC_, C, W>),                \
                                                    dim3(chunk_grid(pteam_grid(M.n_rows, W))),   \
                                                    dim3(kPB), 0, s, M.n_rows, K, M.rp, M.col,   \
                                                    val, x, y, accf)))
  if (M.br == 1 && M.bc == 1) { EAMG_PRECT(1, 1); }
  else if (M.br == 3 && M.bc == 6) { EAMG_PRECT(3, 6); }
  else if (M.br == 6 && M.bc == 3) { EAMG_PRECT(6, 3); }
  else if (M.br == 6 && M.bc == 6) { EAMG_PRECT(6, 6); }
  else return hipErrorInvalidValue;
#undef EAMG_PRECT
  EAMG_PCHECK();
}

int pspmv_blocks(const SolveMat &A, int K) {
  const int g = K > 0 ? int(pgrid(A.n_rows, kPB / kWave)) : 0;
  return g < kPSpmvMax ? (g < 1 ? 1 : g) : kPSpmvMax;
}

hipError_t launch_pspmv(const SolveMat &A, int K, const double *x, double *y, double *part,
                        hipStream_t s) {
  if (A.n_rows == 0) return hipSuccess;
  if (!valid_k(K) || A.br != A.bc) return hipErrorInvalidValue;
  const dim3 grid(pspmv_blocks(A, K));
  switch (A.br) {
    case 1: EAMG_PCOLS(C, hipLaunchKernelGGL((k_pspmv<1, C>), grid, dim3(kPB), 0, s, A.n_rows, K, A.rp, A.col, A.val, x, y, part)); break;
    case 3: EAMG_PCOLS(C, hipLaunchKernelGGL((k_pspmv<3, C>), grid, dim3(kPB), 0, s, A.n_rows, K, A.rp, A.col, A.val, x, y, part)); break;
    case 6: EAMG_PCOLS(C, hipLaunchKernelGGL((k_pspmv<6, C>), grid, dim3(kPB), 0, s, A.n_rows, K, A.rp, A.col, A.val, x, y, part)); break;
    default: return hipErrorInvalidValue;
  }
  EAMG_PCHECK();
}

int pdot_blocks(int64_t n) {
  const int64_t b = (n + kPB - 1) / kPB;
  return int(b < kPDotMax ? (b < 1 ? 1 : b) : kPDotMax);
}

template <class TB>
hipError_t launch_pdot(int64_t n, int K, const double *a, const TB *b, double *part, hipStream_t s) {
  if (!valid_k(K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pdot<TB>, dim3(pdot_blocks(n)), dim3(kPB), 0, s, n, K, a, b, part);
  EAMG_PCHECK();
}

hipError_t launch_preduce(int nparts, int K, const double *part, double *scal, int slot, int op,
                          hipStream_t s) {
  if (!valid_k(K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_preduce, dim3(1), dim3(kPB), 0, s, nparts, K, part, scal, slot, op);
  EAMG_PCHECK();
}

hipError_t launch_pupdate_xr(int64_t n, int K, const double *scal, double *x, double *r,
                             const double *p, const double *q, double *part, float *r32, hipStream_t s) {
  if (!valid_k(K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pupdate_xr, dim3(pdot_blocks(n)), dim3(kPB), 0, s, n, K, scal, x, r, p, q, part, r32);
  EAMG_PCHECK();
}

template <class TZ>
hipError_t launch_pupdate_p(int64_t n, int K, const double *scal, const TZ *z, double *p, hipStream_t s) {
  if (!valid_k(K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pupdate_p<TZ>, dim3(pdot_blocks(n)), dim3(kPB), 0, s, n, K, scal, z, p);
  EAMG_PCHECK();
}

hipError_t launch_pinit_scal(int K, double rtol, int max_it, double *scal, hipStream_t s) {
  if (!valid_k(K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pinit_scal, dim3(pgrid(PS_COUNT * K, kPB)), dim3(kPB), 0, s, K, rtol,
                     double(max_it), scal);
  EAMG_PCHECK();
}

hipError_t launch_pfinite(int64_t n, int K, const double *a, double *scal, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pfinite, dim3(pgrid(n, kPB)), dim3(kPB), 0, s, n, K, a, scal);
  EAMG_PCHECK();
}

hipError_t launch_pzero_unstarted(int64_t n, int K, const double *scal, double *x, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pzero_unstarted, dim3(pgrid(n, kPB)), dim3(kPB), 0, s, n, K, scal, x);
  EAMG_PCHECK();
}

hipError_t launch_ppack(int n, int bs, int K, int nrhs, const int *perm, const uint8_t *mask,
                        const double *in, int64_t ld, double *out, hipStream_t s) {
  const int64_t tot = int64_t(n) * bs * K;
  if (tot == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ppack, dim3(pgrid(tot, kPB)), dim3(kPB), 0, s, n, bs, K, nrhs, perm, mask,
                     in, ld, out);
  EAMG_PCHECK();
}

hipError_t launch_punpack(int n, int bs, int K, int nrhs, const int *perm, const double *in,
                          double *out, int64_t ld, hipStream_t s) {
  const int64_t tot = int64_t(n) * bs * K;
  if (tot == 0) return hipSuccess;
  hipLaunchKernelGGL(k_punpack, dim3(pgrid(tot, kPB)), dim3(kPB), 0, s, n, bs, K, nrhs, perm, in,
                     out, ld);
  EAMG_PCHECK();
}

template hipError_t launch_pgroup_rhs<double>(const SolveMat &, const int *, int, int, int, const double *, const double *, double *, hipStream_t);
template hipError_t launch_pgroup_fwd<double>(const SolveMat &, const SolveMat &, const double *, int, int, int, const double *, double *, double *, hipStream_t);
template hipError_t launch_pgroup_bwd<double>(const SolveMat &, const double *, int, int, int, const double *, double *, hipStream_t);
template hipError_t launch_pgroup_rhs<float>(const SolveMat &, const int *, int, int, int, const float *, const float *, float *, hipStream_t);
template hipError_t launch_pgroup_fwd<float>(const SolveMat &, const SolveMat &, const float *, int, int, int, const float *, float *, float *, hipStream_t);
template hipError_t launch_pgroup_bwd<float>(const SolveMat &, const float *, int, int, int, const float *, float *, hipStream_t);
template hipError_t launch_pdot<double>(int64_t, int, const double *, const double *, double *, hipStream_t);
template hipError_t launch_pdot<float>(int64_t, int, const double *, const float *, double *, hipStream_t);
template hipError_t launch_pupdate_p<double>(int64_t, int, const double *, const double *, double *, hipStream_t);
template hipError_t launch_pupdate_p<float>(int64_t, int, const double *, const float *, double *, hipStream_t);
template hipError_t launch_pgs_fwd<double>(const SolveMat &, const double *, int, int, int, const double *, double *, double *, hipStream_t);
template hipError_t launch_pgs_fwd<float>(const SolveMat &, const float *, int, int, int, const float *, float *, float *, hipStream_t);
template hipError_t launch_pgs_bwd<double>(const SolveMat &, const double *, int, int, int, const double *, double *, hipStream_t);
template hipError_t launch_pgs_bwd<float>(const SolveMat &, const float *, int, int, int, const float *, float *, hipStream_t);
template hipError_t launch_presid_upper<double>(const SolveMat &, int, const double *, double *, hipStream_t);
template hipError_t launch_presid_upper<float>(const SolveMat &, int, const float *, float *, hipStream_t);
template hipError_t launch_prect<double>(const SolveMat &, int, const double *, double *, bool, hipStream_t);
template hipError_t launch_prect<float>(const SolveMat &, int, const float *, float *, bool, hipStream_t);

}  // namespace eamg
