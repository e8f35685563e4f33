// Pieces of the LoRA projection shared between source files of the library.
#pragma once
#include <cstddef>
#include <cstdint>

#include "common.hpp"

namespace localk {

// One low-rank product of token_shrink: u[t][j] = x[t] . A[a_t][j] (float32,
// not scaled) for j < r_max and every token t with an adapter a_t; rows of
// tokens without one are not written. x [T][K], A [n_ad][r_max][K] (rows past
// an adapter's rank give values that the caller drops), K a multiple of 64.
struct ShrinkJob {
  const uint16_t* x;
  const uint16_t* A;
  float* u;  // [T][r_max]
  int64_t K;
};
constexpr int kShrinkJobs = 8;

// Up to kShrinkJobs of them in one launch; T >= 1.
local_status_t token_shrink(const ShrinkJob* jobs, int n_jobs, int64_t T, int n_ad, int r_max,
                            const int32_t* idx, hipStream_t s);

}  // namespace localk
