// Host-side sparse structure of the hierarchy: row split and pattern of the auxiliary smoothed
// prolongation (Def. def:aux_sp), symbolic Galerkin product, transposes, colouring.
#pragma once

#include <cstdint>
#include <vector>

#include "coarsen.hpp"

namespace eamg {

// Block sparsity pattern, column indices ascending within each row.
struct Pattern {
  int n_rows = 0, n_cols = 0;
  std::vector<int64_t> rp;
  std::vector<int> col;
  int64_t nnz() const { return rp.empty() ? 0 : rp.back(); }
};

enum RowType : int { ROW_S = 0, ROW_A = 1, ROW_D = 2 };

// Everything the device needs to assemble P_s numerically.
struct ProlongPlan {
  std::vector<int> type;          // per fine row
  Pattern P;                      // P_s pattern
  std::vector<int64_t> F_ptr;     // per fine row, into F_vtx / F_edge (A rows only)
  std::vector<int> F_vtx, F_edge; // filtered neighbour l and the aux edge {i, l}
};

// Row types and P_s pattern.  cap_S / cap_A: column caps of real-matrix / edge-matrix rows.
//  * cols_S(i) = {agg(i)} U {agg(j) : A_ij structurally nonzero, j not in D}; S row iff
//    |cols_S(i)| <= cap_S, else an edge-matrix (A) row.
//  * F^i: edge neighbours l not in D grouped by agg(l); the group agg(i) and the cap_A - 1 other
//    groups with the largest sum of tr E^il are kept, picked one at a time; sums within the
//    relative band tie_rtol of the largest tie and the smaller coarse id wins.
ProlongPlan plan_prolongation(const Pattern &A, const AuxLevel &aux, const std::vector<int> &agg_of,
                              const std::vector<char> &dmask, int cap_S, int cap_A, double tie_rtol);

// Structural pattern of A * B.
Pattern spgemm_symbolic(const Pattern &A, const Pattern &B);

// Transposed pattern; src[q] = index in P of entry q of the transpose.
Pattern transpose_pattern(const Pattern &P, std::vector<int64_t> &src);

// Greedy colouring in smallest-last order (vertices removed by minimum remaining degree, lowest
// id on ties; coloured in reverse removal order with the smallest colour unused by neighbours).
std::vector<int> greedy_coloring(int n, const int64_t *rp, const int *col, int &n_colors);
inline std::vector<int> greedy_coloring(const Pattern &A, int &n_colors) {
  return greedy_coloring(A.n_rows, A.rp.data(), A.col.data(), n_colors);
}

// Symmetric permutation of a square pattern: row/col v -> inv[v].  Columns re-sorted;
// src[q] = index in A of entry q of the result.
Pattern permute_pattern(const Pattern &A, const std::vector<int> &perm, const std::vector<int> &inv,
                        std::vector<int64_t> &src);

// Sweep stages of a colour-major level.  A stage covers the colours [cut[k], cut[k + 1]): one
// colour, or a group of consecutive colours done in two launches instead of one per colour.  With
// u_i = b_i - (couplings of row i to the rows outside the group), the forward sweep inside a group is
//   t = (I + L D^+)^{-1} u,   x_i = D_i^+ t_i,
// L the group's blocks left of the diagonal: t_i = u_i - sum_j S_ij u_j with a sparse S whose
// pattern holds, for each row, every row of the group from which a chain of couplings through
// ascending colours leads to it.  The backward sweep's matrix, of (I + L^T D^+)^{-1}, has the
// transposed pattern.
struct SweepPlan {
  std::vector<int> cut;           // stage boundaries (colours), 0 .. ncolors
  Pattern S;                      // forward matrix (rows of one-colour stages are empty)
  // positions in the level's pattern of a row's couplings inside its group: left [pre, diag),
  // right (diag, post)
  std::vector<int> pre, post;
  std::vector<int> rank;          // a row's colour counted from its group's first, -1 if none
  int max_rank = 0;
  bool grouped() const { return S.nnz() > 0; }
};
// Ap: the level's colour-major pattern, dg its diagonal positions, color_ptr the colours' first
// rows, bs the block size.
SweepPlan plan_sweeps(const Pattern &Ap, const std::vector<int> &dg, const std::vector<int> &color_ptr,
                      int ncolors, int bs);

// Colour-major numbering: colour c holds the rows [ptr[c], ptr[c + 1]), row r is natural row perm[r],
// inv its inverse; ascending natural rows within a colour.
struct ColourOrder {
  std::vector<int> ptr, perm, inv;
};
ColourOrder colour_order(const std::vector<int> &color, int ncolors);

// A plan and what its group matrices are built from on the device.
struct SweepStages {
  SweepPlan plan;
  Pattern Sb;                     // the backward matrix's pattern
  std::vector<int> lo_end;        // per row: end of [row start, plan.pre) among the blocks left of the diagonal
  std::vector<int> right;         // per row: first position right of the diagonal
  std::vector<int> order, rank_ptr;   // rows of rank r: order[rank_ptr[r]] .. order[rank_ptr[r + 1] - 1]
};
// Arguments as plan_sweeps.
SweepStages prepare_sweeps(const Pattern &Ap, const std::vector<int> &dg, const std::vector<int> &color_ptr,
                           int ncolors, int bs);

// A smoothed level's colouring and what follows from it on the host.
struct Smoothing {
  std::vector<int> color;
  int ncolors = 0;
  ColourOrder order;
  Pattern Ap;                  // colour-major pattern
  std::vector<int64_t> src;    // its positions in the natural pattern
  SweepStages stages;          // if asked for
};
// A: the level's natural pattern (structurally symmetric, with every diagonal block).
Smoothing plan_smoothing(const Pattern &A, int bs, bool sweeps);

// Rows permuted by the fine permutation, columns renumbered by the coarse one (re-sorted).
Pattern permute_rect(const Pattern &P, const std::vector<int> &perm_rows,
                     const std::vector<int> &inv_cols, std::vector<int64_t> &src);

}  // namespace eamg
