// Wide-panel V-cycle kernels (wide.hip): the V-cycle of a hierarchy's small levels applied to
// thousands of columns at once, the setup of the dense V-cycle tails.  FP64, blocks of 1 x 1 or
// 6 x 6 (the levels below the finest).
//
// A wide panel is row-major with a row stride of its own: entry (dof d, column k) at
// p[d * ld + k], 16-byte aligned rows, an even number of columns.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace eamg {

struct WidePanel {
  double *p = nullptr;
  int64_t ld = 0;
};

// Forward colour sweep from x = 0 on rows [r0, r1) (as launch_gs_fwd) for columns [0, K):
// t = b_i - sum_{j < i} A_ij x_j; x_i = Dinv_i t; r_i = t - A_ii x_i.  b.p == nullptr: b holds
// columns j0 .. j0 + K - 1 of the identity.
hipError_t launch_wide_fwd(const SolveMat &A, const double *Dinv, int r0, int r1, int K, WidePanel b,
                           int j0, WidePanel x, WidePanel r, hipStream_t s);
// r_i -= sum_{j > i} A_ij x_j on every row.
hipError_t launch_wide_resid(const SolveMat &A, int K, WidePanel x, WidePanel r, hipStream_t s);
// Backward colour sweep on rows [r0, r1): x_i += Dinv_i (b_i - sum_j A_ij x_j); b as above.
hipError_t launch_wide_bwd(const SolveMat &A, const double *Dinv, int r0, int r1, int K, WidePanel b,
                           int j0, WidePanel x, hipStream_t s);
// y = M x, or y += M x.
hipError_t launch_wide_rect(const SolveMat &M, int K, WidePanel x, WidePanel y, bool accumulate,
                            hipStream_t s);
// y = D x, D dense n x n row-major with leading dimension ldD.
hipError_t launch_wide_dense(int n, int ldD, const double *D, int K, WidePanel x, WidePanel y,
                             hipStream_t s);

}  // namespace eamg
