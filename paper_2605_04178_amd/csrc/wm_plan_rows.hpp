// wm_plan_rows.hpp -- row counters of the fusion-planning programme, apart from
// its kernels so that a host program can run them on the longest chains.
#pragma once
#include <cstdint>

namespace wm {

// Rows per batch: their costs are loaded together (one wait per batch), their
// cut lengths stay in registers, a byte each, equal on every lane of the
// group, until the next batch begins (cut bytes of all but the last batch go
// through memory).
constexpr int kPlanBatch = 16;

// A chain's L rows in batches, first row `at`.  Offsets are 32-bit, so L is at
// most 2^31 - 1 and `at` ends up to a batch beyond it; the groups of a wave
// step together, so a chain's own rows may end long before.  Unsigned, and the
// rows left are formed only where there are some: signed, `at` would pass 2^31 -
// 1 on a chain within a batch of it, and L - at on a short chain beside it.
struct PlanRows {
    uint32_t L, at;
    __host__ __device__ explicit PlanRows(int32_t rows) : L((uint32_t)rows), at(0u) {}
    __host__ __device__ bool more() const { return at < L; }
    __host__ __device__ int32_t left() const { return at < L ? (int32_t)(L - at) : 0; }   // rows from `at` on
    __host__ __device__ void next() { at += (uint32_t)kPlanBatch; }
};

// First row of the last batch of L rows, -1 with no rows.
__host__ __device__ inline int32_t last_batch(int32_t L) { return L > 0 ? (L - 1) & ~(kPlanBatch - 1) : -1; }

// The batch at w0 (0 <= w0 < L) is not the chain's last one.
__host__ __device__ inline bool batch_stored(int32_t w0, int32_t L) { return L - w0 > kPlanBatch; }

}  // namespace wm
