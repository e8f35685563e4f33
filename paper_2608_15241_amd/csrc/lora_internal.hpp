// Pieces of the LoRA projection shared between source files of the library.
#pragma once
#include <cstddef>
#include <cstdint>

#include "common.hpp"

namespace localk {

// One low-rank product of token_shrink: u[z][t][j] = the sum over K slice z of
// x[t][k] A[a_t][j][k] (float32, not scaled; rows at or past an adapter's rank
// give values that the caller drops), or with one slice us[t][j] =
// bf16(scale_t u[0][t][j]), zero at or past the rank; for j < r_max and every
// token t with an adapter a_t (rows of tokens without one are not written).
// x [T][K], A [n_ad][r_max][K], K a multiple of 64.
struct ShrinkJob {
  const uint16_t* x;
  const uint16_t* A;
  float* u;  // [ks][T][r_max], or NULL
  int64_t K;
  uint16_t* us;          // [T][r_max], where u is NULL
  const int32_t* ranks;  // with us: [n_ad], or NULL (every rank = r_max)
};
constexpr int kShrinkJobs = 8;

// Up to kShrinkJobs of them over ks K slices in one launch; T >= 1. scale: for
// us; zero16 (or NULL): 16 bytes that are set to zero.
local_status_t token_shrink(const ShrinkJob* jobs, int n_jobs, int64_t T, int n_ad, int r_max,
                            const int32_t* idx, int ks, hipStream_t s,
                            const float* scale = nullptr, uint16_t* zero16 = nullptr);

// The most K slices of a long chunk's shrink that a workspace holds.
int long_slices(int64_t T, int64_t K, int r_max, int G);

}  // namespace localk
