// Exact coarsening criteria of a matching pass evaluated on the device (criteria.hip).
//
// The greedy walk of Algorithm alg:pwagg stays on the host; the criteria it asks for (mu_b of
// Lemma thm:mu2 for a pair, mu_g of Thm thm:mu1 for the union of two agglomerates) are
// independent of each other and are evaluated in batches, a GPU thread per pair and a wavefront per
// union, with the arithmetic of crit_core.hpp compiled for the device without contraction so that
// every value equals the host's bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <memory>

#include "coarsen.hpp"

namespace eamg {

// Smallest batches that the device takes by default.  A batch there lasts as long as its longest chain,
// on the host as long as its share of 16 threads.  6x6 weights (9,261 vertices with inclusions; a
// level's upload not counted), host / device: unions 64 in 1.16 / 1.48 ms, 128 in 2.07 / 1.51, 512 in
// 5.5 / 1.6; pairs 512 in 0.54 / 0.65 ms, 1,024 in 0.84 / 0.66, 4,096 in 2.4 / 0.66.  Scalar weights are
// faster on the device at any size (64 pairs 0.20 / 0.08 ms).  So the line for unions lies where the
// two meet; pairs meet near 700 already, and batches up to the line still go to the host.
constexpr int kGpuCritMinPairs = 4096;
constexpr int kGpuCritMinUnions = 128;

// Batch evaluator on `s` (the device current at creation).  Device copies of the levels are kept
// until the evaluator is destroyed or another level is handed over.
std::unique_ptr<CritBatch> make_device_criteria(hipStream_t s);

}  // namespace eamg
