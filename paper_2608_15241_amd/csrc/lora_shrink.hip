// The low-rank product of long token runs, u[t][j] = x[t] . A[a_t][j] with
// token t's own adapter a_t, over the whole of K in one launch: the shrink of
// the backward (u = x A^T and dy B, float32), for several (x, A) pairs at
// once.
//
// Bound by the reads of x and A (2 r flop per byte). A workgroup takes 16
// tokens and one pair; its waves cut K between them, so that no partial sum
// leaves the compute unit. Each wave streams its K slice of the 16 token rows
// and of 16 RT adapter rows through a ring of its own in LDS (64 k a stage,
// no barrier in the loop) and runs S^T = A X^T on the matrix cores; the
// waves' tiles are added through LDS in wave order. Direct global-to-LDS
// loads, because the matrix-core lane layout (16 rows side by side) is the
// one the load path cannot merge. The six products of a q/k/v backward (2048
// tokens, 4096 x 4096, rank 16; 196 MB out of the caches): 23.4 us, 38.0 us
// with the operands loaded straight into registers, 41 us as four launches of
// the K-sliced shrink whose slices the reader summed. Tokens of other adapters
// in the tile are computed and dropped: adapters come in runs (a request's
// chunk), so a tile rarely holds more than two.
#include "common.hpp"
#include "lora_internal.hpp"

namespace localk {
namespace {

constexpr int kSkWaves = 4;
constexpr int kSkThreads = kSkWaves * kWave;
constexpr int kSkTokens = 16;

struct SkArgs {
  ShrinkJob job[kShrinkJobs];
  int64_t T;
  int n_ad, r_max;
  const int32_t* idx;
};

template <int RT>
struct SkShape {
  static constexpr int DMA = 2 + 2 * RT;       // 1 KB loads per stage
  static constexpr int STAGE = 1024 * DMA;     // x rows, then A rows, 128 bytes each
  static constexpr int S = RT == 1 ? 4 : 3;    // stages: two workgroups per unit up to RT = 2
  static constexpr int RED = RT * kSkWaves * kWave * 16;
  static constexpr int LDS = kSkWaves * S * STAGE + RED;
};

__device__ __forceinline__ void sk_load16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
}
template <int N>
__device__ __forceinline__ void sk_wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}

template <int RT>
__global__ __launch_bounds__(kSkThreads) void token_shrink_kernel(SkArgs a) {
  using SK = SkShape<RT>;
  constexpr int S = SK::S, D = SK::DMA;
  extern __shared__ __attribute__((aligned(16))) uint8_t sk_lds[];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane % 16, kgrp = lane / 16;
  uint8_t* ring = sk_lds + wave * S * SK::STAGE;
  f32x4* red = reinterpret_cast<f32x4*>(sk_lds + kSkWaves * S * SK::STAGE);  // [RT][waves][64]
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kSkTokens;
  const int64_t t = t0 + col;
  const ShrinkJob& jb = a.job[blockIdx.y];

  int my = t < a.T ? a.idx[t] : -1;
  if (my < 0 || my >= a.n_ad) my = -1;
  // the wave's 64-k steps [s_lo, s_lo + n)
  const int64_t K = jb.K;
  const int steps = static_cast<int>(K / 64);
  const int s_lo = wave * steps / kSkWaves, n = (wave + 1) * steps / kSkWaves - s_lo;
  // lane l of a load writes 16 bytes at block + 16 l: row 8 q + l / 8,
  // position l % 8, which holds chunk (l % 8) ^ (l / 8) of that row
  const int lrow = lane / 8;
  const int64_t loff = 64 * static_cast<int64_t>(s_lo) + 8 * ((lane % 8) ^ lrow);
  const uint16_t* xs[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int64_t tr = t0 + 8 * q + lrow;  // rows past T repeat row t0, never stored
    xs[q] = jb.x + (tr < a.T ? tr : t0) * K + loff;
  }
  const int rd0 = col * 128 + 16 * (kgrp ^ (col % 8));

  uint64_t pending = __ballot(my >= 0) & 0xffffull;
  bool again = false;
  while (pending) {
    const int ad = __builtin_amdgcn_readlane(my, __ffsll(static_cast<long long>(pending)) - 1);
    pending &= ~__ballot(my == ad);
    for (int j0 = 0; j0 < a.r_max; j0 += 16 * RT) {
      const uint16_t* as[2 * RT];
#pragma unroll
      for (int q = 0; q < 2 * RT; ++q) {  // rows past r_max repeat its last, never stored
        const int j = min(j0 + 8 * q + lrow, a.r_max - 1);
        as[q] = jb.A + (static_cast<int64_t>(ad) * a.r_max + j) * K + loff;
      }
      auto issue = [&](int s) {
        uint8_t* st = ring + (s % S) * SK::STAGE;
        const int64_t k = 64 * static_cast<int64_t>(s);
#pragma unroll
        for (int q = 0; q < 2; ++q) sk_load16(xs[q] + k, st + 1024 * q);
#pragma unroll
        for (int q = 0; q < 2 * RT; ++q) sk_load16(as[q] + k, st + 2048 + 1024 * q);
      };
      f32x4 acc[2][RT];  // the two halves of the steps apart: shorter sums
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[0][rt] = acc[1][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < min(S - 1, n); ++s) issue(s);
      for (int s = 0; s < n; ++s) {
        // stage s % S has landed; stage (s - 1) % S was read before the last
        // step's products, so the loads of step s + S - 1 may refill it
        if (s + S - 1 < n) {
          sk_wait_loads<D * (S - 2)>();
          issue(s + S - 1);
        } else {
          sk_wait_loads<0>();
        }
        const uint8_t* st = ring + (s % S) * SK::STAGE;
        u32x4 xf[2], af[2][RT];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          xf[m] = *reinterpret_cast<const u32x4*>(st + (rd0 ^ (64 * m)));
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            af[m][rt] = *reinterpret_cast<const u32x4*>(st + 2048 * (1 + rt) + (rd0 ^ (64 * m)));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[m][rt] = mfma16x16x32(as_bf16x8(af[m][rt]), as_bf16x8(xf[m]), acc[m][rt]);
      }
      if (again) __syncthreads();  // the previous sums have been read
      again = true;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) red[(rt * kSkWaves + wave) * kWave + lane] = acc[0][rt] + acc[1][rt];
      __syncthreads();
      for (int rt = wave; rt < RT; rt += kSkWaves) {
        f32x4 v = red[rt * kSkWaves * kWave + lane];
#pragma unroll
        for (int w = 1; w < kSkWaves; ++w) v += red[(rt * kSkWaves + w) * kWave + lane];
        const int j = j0 + 16 * rt + 4 * kgrp;
        if (my == ad && j < a.r_max) *reinterpret_cast<f32x4*>(jb.u + t * a.r_max + j) = v;
      }
    }
  }
}

template <int RT>
local_status_t launch_sk(const SkArgs& a, int n_jobs, hipStream_t s) {
  static bool done = false;
  if (!done) {  // benign race: every caller sets the same value
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(token_shrink_kernel<RT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, SkShape<RT>::LDS);
    done = true;
  }
  const dim3 grid(static_cast<unsigned>((a.T + kSkTokens - 1) / kSkTokens),
                  static_cast<unsigned>(n_jobs));
  token_shrink_kernel<RT><<<grid, kSkThreads, SkShape<RT>::LDS, s>>>(a);
  return local_check_launch("lora (token shrink)");
}

}  // namespace

local_status_t token_shrink(const ShrinkJob* jobs, int n_jobs, int64_t T, int n_ad, int r_max,
                            const int32_t* idx, hipStream_t s) {
  SkArgs a{};
  for (int q = 0; q < n_jobs; ++q) a.job[q] = jobs[q];
  a.T = T;
  a.n_ad = n_ad;
  a.r_max = r_max;
  a.idx = idx;
  if (r_max <= 16) return launch_sk<1>(a, n_jobs, s);
  if (r_max <= 32) return launch_sk<2>(a, n_jobs, s);
  return launch_sk<4>(a, n_jobs, s);
}

}  // namespace localk
