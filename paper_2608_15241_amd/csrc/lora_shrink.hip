// The low-rank product of long token runs, u[t][j] = x[t] . A[a_t][j] with
// token t's own adapter a_t: the shrink of long chunks and of the backward
// (u = x A^T and dy B), for several (x, A) pairs in one launch.
//
// Bound by the reads of x and A (2 r flop per byte). A workgroup takes 16
// tokens of one adapter and one pair; its waves cut K between them, so that no
// partial sum leaves the compute unit (with few tiles K is also cut into slices,
// each its own workgroups and output, which the reader adds in order). Each wave
// streams its K slice of the 16 token rows and of 16 RT adapter rows through a
// ring of its own in LDS (64 k a stage, no barrier in the loop) and runs
// S^T = A X^T on the matrix cores; the waves' tiles are added through LDS in wave
// order. Direct global-to-LDS loads, because the matrix-core lane layout (16 rows
// side by side) is the one the load path cannot merge. The six products of a
// q/k/v backward (2048 tokens, 4096 x 4096, rank 16; 196 MB out of the caches):
// 22 to 27 us, 38 us with the operands loaded straight into registers, 41 us as
// four launches of a K-sliced shrink whose slices the reader summed.
//
// The tiles are gathered from groups of 64 tokens, adapter by adapter in the
// order of their first tokens, four or eight workgroups a group (tile i to
// workgroup i % 4 or i % 8). Requests' chunks (runs of one adapter) make four full tiles, as 16
// tokens in order would; with an adapter per token, 16 tokens in order hold up
// to 16 adapters and stream x and A again for each: q, k and v of 2048 tokens at
// 4096 x 4096 / 1024 / 1024 over 8 adapters at random 156 -> 122 us a call. A sum
// does not depend on the tile that it is formed in.
#include "common.hpp"
#include "lora_internal.hpp"

namespace localk {
namespace {

constexpr int kSkTokens = 16;  // tokens of a tile
constexpr int kSkGroup = kWave;  // tokens that tiles are gathered from

struct SkArgs {
  ShrinkJob job[kShrinkJobs];
  int64_t T;
  int n_ad, r_max;
  const int32_t* idx;
  int ks;     // K slices (each its own workgroups and output)
  int split;  // workgroups of a group, a power of two
  const float* scale;  // for bf16 outputs
  uint16_t* zero16;    // 16 bytes or null
};

template <int RT_, int W_, int S_>
struct SkShape {
  static constexpr int RT = RT_, W = W_, S = S_;  // 16-row tiles of A, waves, stages
  static constexpr int DMA = 2 + 2 * RT;          // 1 KB loads per stage
  static constexpr int STAGE = 1024 * DMA;        // x rows, then A rows, 128 bytes each
  static constexpr int LDS = W * S * STAGE;
  static_assert(LDS <= 163840 && S >= 2, "ring");
};

__device__ __forceinline__ void sk_load16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
}
template <int N>
__device__ __forceinline__ void sk_wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}

template <class SK>
__global__ __launch_bounds__(SK::W * kWave) void token_shrink_kernel(SkArgs a) {
  constexpr int S = SK::S, D = SK::DMA, RT = SK::RT, W = SK::W;
  extern __shared__ __attribute__((aligned(16))) uint8_t sk_lds[];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane % 16, kgrp = lane / 16;
  uint8_t* ring = sk_lds + wave * S * SK::STAGE;
  // after the loop a wave's tiles take the start of its ring: [RT][64] f32x4
  auto red = [&](int w, int rt) {
    return reinterpret_cast<f32x4*>(sk_lds + w * S * SK::STAGE) + rt * kWave + lane;
  };
  const int z = static_cast<int>(blockIdx.x) % a.ks;
  const int wg = static_cast<int>(blockIdx.x) / a.ks, sub = wg & (a.split - 1);
  const int64_t t0 = static_cast<int64_t>(wg / a.split) * kSkGroup;
  const ShrinkJob& jb = a.job[blockIdx.y];

  int my = t0 + lane < a.T ? a.idx[t0 + lane] : -1;  // the adapter of the group's token `lane`
  if (my < 0 || my >= a.n_ad) my = -1;
  // the wave's 64-k steps [s_lo, s_lo + n)
  const int64_t K = jb.K;
  const int steps = static_cast<int>(K / 64);
  const int zw = z * W + wave, all = a.ks * W;
  const int s_lo = zw * steps / all, n = (zw + 1) * steps / all - s_lo;
  // lane l of a load writes 16 bytes at block + 16 l: row 8 q + l / 8,
  // position l % 8, which holds chunk (l % 8) ^ (l / 8) of that row
  const int lrow = lane / 8;
  const int64_t loff = 64 * static_cast<int64_t>(s_lo) + 8 * ((lane % 8) ^ lrow);
  const int rd0 = col * 128 + 16 * (kgrp ^ (col % 8));

  if (a.zero16 && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid < 8)
    a.zero16[tid] = 0;
  const int j0 = 16 * RT * blockIdx.z;
  bool again = false;
  int first = 0;  // the adapter's first tile of the group
  for (uint64_t pending = __ballot(my >= 0); pending;) {
    const int ad = __builtin_amdgcn_readlane(my, __ffsll(static_cast<long long>(pending)) - 1);
    const uint64_t m = __ballot(my == ad);
    pending &= ~m;
    const int cnt = __popcll(m);
    // the group's tokens in the order: this adapter's, then the others'
    const int below = __builtin_amdgcn_mbcnt_hi(
        static_cast<uint32_t>(m >> 32),
        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
    const int order =
        __builtin_amdgcn_ds_permute(4 * (my == ad ? below : cnt + lane - below), lane);
    const int tile0 = first;
    first += (cnt + kSkTokens - 1) / kSkTokens;
    for (int i = (sub - tile0) & (a.split - 1); kSkTokens * i < cnt; i += a.split) {
      if (again) __syncthreads();  // the previous tile's sums have been read
      again = true;
      // token c of the tile (past the last one: that again, never stored)
      const int left = cnt - kSkTokens * i;
      auto token = [&](int c) {
        return t0 + __shfl(order, kSkTokens * i + min(c, left - 1));
      };
      const int64_t t = token(col);
      const uint16_t* xs[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) xs[q] = jb.x + token(8 * q + lrow) * K + loff;
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
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) *red(wave, rt) = acc[0][rt] + acc[1][rt];
      __syncthreads();
      for (int rt = wave; rt < RT; rt += W) {
        f32x4 v = *red(0, rt);
#pragma unroll
        for (int w = 1; w < W; ++w) v += *red(w, rt);
        const int j = j0 + 16 * rt + 4 * kgrp;
        if (col >= left || j >= a.r_max) continue;
        if (jb.u) {
          *reinterpret_cast<f32x4*>(jb.u + (z * a.T + t) * a.r_max + j) = v;
        } else {
          const int rk = jb.ranks ? jb.ranks[ad] : a.r_max;
          const float sc = a.scale[t];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = j + q < rk ? sc * v[q] : 0.f;
          *reinterpret_cast<u32x2*>(jb.us + t * a.r_max + j) =
              u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        }
      }
    }
  }
}

template <class SK>
local_status_t launch_sk(const SkArgs& a, int n_jobs, hipStream_t s) {
  static bool done = false;
  if (!done) {  // benign race: every caller sets the same value
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(token_shrink_kernel<SK>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, SK::LDS);
    done = true;
  }
  const dim3 grid(static_cast<unsigned>((a.T + kSkGroup - 1) / kSkGroup * a.split * a.ks),
                  static_cast<unsigned>(n_jobs),
                  static_cast<unsigned>((a.r_max + 16 * SK::RT - 1) / (16 * SK::RT)));
  token_shrink_kernel<SK><<<grid, SK::W * kWave, SK::LDS, s>>>(a);
  return local_check_launch("lora (token shrink)");
}

}  // namespace

local_status_t token_shrink(const ShrinkJob* jobs, int n_jobs, int64_t T, int n_ad, int r_max,
                            const int32_t* idx, int ks, hipStream_t s, const float* scale,
                            uint16_t* zero16) {
  SkArgs a{};
  for (int q = 0; q < n_jobs; ++q) a.job[q] = jobs[q];
  a.T = T;
  a.n_ad = n_ad;
  a.r_max = r_max;
  a.idx = idx;
  a.ks = ks;
  a.scale = scale;
  a.zero16 = zero16;
  // Rank rows per workgroup: all of them (token rows read once) when the
  // tiles alone fill the chip, else half, side by side. Measured (K = 4096):
  // rank 32, 63 tiles: 10.1 us with 16 rows, 11.7 with 32; rank 64, 94 tiles:
  // 18.5, 15.4 and 17.4 with 16, 32 and 64; rank 64, 768 tiles: 72.9, 60.1
  // and 55.7.
  const bool full = (T + kSkTokens - 1) / kSkTokens * n_jobs * ks >= 256;
  // A group holds four tiles, and more where its tokens have several adapters:
  // room for eight at once where that leaves every workgroup a compute unit (1000
  // tokens in 4 slices, which would not: 46.4 us a call with four, 47.3 with eight).
  const int rows = r_max <= 16 || (r_max <= 32 && !full) ? 16 : r_max <= 32 || !full ? 32 : 64;
  const int64_t wgs = (T + kSkGroup - 1) / kSkGroup * 8 * n_jobs * ks * ((r_max + rows - 1) / rows);
  a.split = wgs <= 256 ? 8 : 4;
  if (rows == 16) return launch_sk<SkShape<1, 8, 2>>(a, n_jobs, s);
  if (rows == 32) return launch_sk<SkShape<2, 8, 3>>(a, n_jobs, s);
  return launch_sk<SkShape<4, 8, 2>>(a, n_jobs, s);
}

}  // namespace localk
