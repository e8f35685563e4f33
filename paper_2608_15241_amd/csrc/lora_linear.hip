// local_lora_linear: y = res + x W^T + s_t (x A_a^T) B_a^T with a per-token
// adapter a = adapter_idx[t] (§2.2 "LoRA adapters": one frozen base shared by
// many low-rank adapters, every request routed to its own adapter).
//
// Design, SGMV-style but on the matrix cores end to end. Every tile is
// computed transposed, Y^T = W X^T: features are MFMA rows (A operand, rows
// of W), tokens are columns (B operand, rows of x), so a lane ends with 4
// consecutive features of one token.
//
//  * Decode sizes (T <= 256), none waiting on another kernel's workgroups:
//    - base product split over K, streamed: a workgroup owns 16*FN features
//      x up to 128 tokens of one K slice; its W rows (with the shrink's
//      stacked-A rows as extra row tiles when they fit) and x rows stream
//      through an LDS ring by direct global-to-LDS loads, whole 128-byte rows
//      per load instruction; fp32 partial sums per slice. Wider feature
//      tiles for fewer tokens cut the re-reads of x.
//    - SGMV shrink, when the stacked rows are too many to ride along (more
//      than 4 extra row tiles a workgroup): workgroups per (K slice,
//      adapter, projection) gather the
//      tokens routed to that adapter and compute x_t . A[a,j,:] for j below
//      its rank over their slice of K on the matrix cores; fp32 partial sums
//      per slice.
//    - epilogue: sums the base slices, forms U_s = bf16(s_t * u) for the
//      token's own adapter and rank, adds U_s B_a^T and the residual, and
//      rounds once to bf16.
//  * Long prefill chunks (T > 256), two kernels:
//    - shrink (lora_shrink.hip): U_s[t] = bf16(s_t x_t . A[a_t]) of every
//      token with an adapter, for every projection of the call.
//    - main product: 128 x 256 down to 64 x 64 tokens x features per
//      workgroup by the size of the call, both operands brought to LDS by
//      direct global-to-LDS loads; the delta U_s Btilde^T over stacked columns
//      c = a*r_max + j (U_s zero unless a is t's adapter; Btilde[n, c] =
//      B[a, n, j]) runs as extra K-steps, only over adapters used in the tile
//      and columns below their rank.
//  Both paths sum the base K-steps in an order that does not depend on which
//  adapters are present, so a zero up-projection leaves y bit-identical.
#include <algorithm>
#include <climits>

#include "common.hpp"
#include "lora_internal.hpp"

namespace localk {

// The most K slices of a long chunk's shrink that its workspace holds: the
// fewest (a divisor of the 64-k steps) whose slices of 64 tokens and of every
// projection's rank rows fit 144 KB and give 256 workgroups, at most 8 unless
// more are needed to fit.
int long_slices(int64_t T, int64_t K, int r_max, int G) {
  const int steps = static_cast<int>(K / 64);
  const int64_t rows = 64 + static_cast<int64_t>(G) * ((r_max + 15) / 16 * 16);
  int best = steps;
  for (int ks = 1; ks <= steps; ++ks) {
    if (steps % ks || rows * (steps / ks) * 128 > 147456) continue;
    best = ks;
    if ((T + 63) / 64 * ks >= 256 || ks >= 8) break;
  }
  return best;
}

namespace {

constexpr int kMaxGroup = 4;            // projections sharing x in one grouped call
constexpr int kNumXcd = 8;

struct GemmArgs {
  const uint16_t* x;     // [T][K]
  const uint16_t* w;     // main: W [N][K]; shrink: stacked A [R][K]
  int64_t T, K, N;       // N = output width
  float* pout;           // shrink: fp32 partial sums [up_ks][T][p_stride]
  int up_ks;             // K slices of the shrink partial sums
  float* part;           // partial mode: fp32 base partial sums [ksplit][T][N]
  int xrows;             // stacked-A rows per feature-tile workgroup (0 = none)
  // Skinny kernel and epilogue: G projections that share x, taken as one
  // virtual weight whose rows [gstart[g], gstart[g+1]) are the rows of W_g
  // (N = gstart[G]); their stacked A rows are likewise concatenated, R rows
  // per projection.
  int G;
  int64_t gstart[kMaxGroup + 1];
  const uint16_t* gw[kMaxGroup];     // W_g [N_g][K]
  const uint16_t* ga[kMaxGroup];     // A_g [n_ad][r_max][K]
  const uint16_t* gb[kMaxGroup];     // B_g [n_ad][N_g][r_max]
  const int32_t* granks[kMaxGroup];  // ranks_g [n_ad] or null
  const uint16_t* gres[kMaxGroup];   // residual_g [T][N_g] or null
  uint16_t* gy[kMaxGroup];           // y_g [T][N_g]
  int p_stride;          // row length of the shrink partial sums (R or r_max)
  int p_stacked;         // 1: shrink sums indexed by stacked row a*r_max + j
  const int32_t* ranks;  // [n_ad] or null
  const int32_t* idx;    // [T] or null
  const float* scale;    // [T]
  int n_ad, r_max, R;
  const uint16_t* res;   // optional residual [T][N] (main mode)
  uint16_t* y;           // bf16 output [T][N]
  int ksplit;            // K slices of the decode base product (grid.z)
  // long chunks: the tile grid of the main product, and what the shrink wrote:
  // U_s of every projection [G][T][r_max] bf16 and 16 bytes of zeros, or (us
  // null) sums over K slices, pout [G][up_ks][T][r_max]
  int gm, gn;
  const uint16_t* us;
  const uint16_t* zero16;
};

// Entry g of a per-projection argument array. Compare-and-select over the
// array (instead of indexing it) keeps the by-value argument in registers.
template <typename T>
__device__ __forceinline__ T pick(const T (&v)[kMaxGroup], int g) {
  T r = v[0];
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i) r = g == i ? v[i] : r;
  return r;
}

// Projection of virtual row n of a grouped call.
__device__ __forceinline__ int group_of(const GemmArgs& a, int64_t n) {
  int g = 0;
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i) g += (i < a.G && n >= a.gstart[i]) ? 1 : 0;
  return g;
}

// First virtual row of projection g (g may be G: the end of the last one).
__device__ __forceinline__ int64_t gstart_of(const GemmArgs& a, int g) {
  int64_t r = a.gstart[0];
#pragma unroll
  for (int i = 1; i <= kMaxGroup; ++i) r = g == i ? a.gstart[i] : r;
  return r;
}

// Rank of adapter ad of projection g, clamped to [0, r_max] so that no rank reads
// past the adapter's own rows.
__device__ __forceinline__ int rank_g(const GemmArgs& a, int g, int ad) {
  const int32_t* r = pick(a.granks, g);
  return r ? min(max(r[ad], 0), a.r_max) : a.r_max;
}

// Adapter of token t, or -1 (past the batch, no adapter, or out of range).
__device__ __forceinline__ int token_adapter(const GemmArgs& a, int64_t t) {
  if (t >= a.T) return -1;
  const int ad = a.idx[t];
  return (ad >= 0 && ad < a.n_ad) ? ad : -1;
}

// s_waitcnt encodings (gfx9 layout): wait until at most N vector memory
// operations are outstanding / until all LDS operations are done.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void wait_lgkm0_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The first `keep` (clamped to 0..8) of 8 packed bf16 values; the rest zero.
__device__ __forceinline__ u32x4 keep_first8(u32x4 v, int keep) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e >= keep) w[e / 2] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;
  return u32x4{w[0], w[1], w[2], w[3]};
}



// Direct global-to-LDS load of 16 bytes per lane: lane l's bytes land at
// lds + 16 l (lds is the wave's common base). A plain function: the builtin
// called with template-dependent arguments fails the host compilation pass
// of a kernel template.
__device__ __forceinline__ void lds_load16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
}

// ------------------------------------------------------------------ stream
// Decode sizes (T <= 256): the base product, with the shrink's stacked-A rows
// as extra row tiles, of one K slice, streamed through LDS. Workgroup:
// features [n0, n0 + 16 FN) (+ XT tiles of stacked-A rows) x tokens
// [t0, t0 + 16 FM) over the z-th of ksplit K slices. Each 64-k step of the
// slice is one LDS stage holding the tile's W and A rows and its x rows
// (128-byte rows, chunk-swizzled as in the long-chunk product), brought in
// by direct global-to-LDS loads: every load instruction moves 8 whole rows,
// and a ring of S stages keeps S - 2 steps in flight while one is computed.
// Each wave owns whole output tiles, so there is no reduction across waves. Rows past N or T and stacked-A rows past the adapter's rank read
// clamped rows; their outputs are never stored (rows past the rank are
// masked by the epilogue). Workgroups start their slice at different steps
// (by feature tile), so that those running together read different parts
// of x; the order depends on the feature tile only, as with the K slices.
constexpr int kStThreads = 256;
constexpr int kStWaves = kStThreads / kWave;
constexpr int kStLdsMax = 147456;

template <int FN, int FM, int XT>
struct StreamShape {
  static constexpr int FT = FN + XT;                                // W and A row tiles
  static constexpr int ROWS = 16 * (FT + FM);                       // rows of a stage
  static constexpr int DMA = (ROWS / 8 + kStWaves - 1) / kStWaves;  // loads per wave and stage
  static constexpr int STAGE = 8 * DMA * kStWaves * 128;            // bytes, padded
  static constexpr int S = kStLdsMax / STAGE < 8 ? kStLdsMax / STAGE : 8;
  // Output tiles of a wave: token tiles j = wave % FM (with 8 of them wave and
  // wave + 4) x every feature tile, or every second or fourth one where there
  // are fewer token tiles than waves, so that a step reads each of the wave's
  // operands from LDS once.
  static constexpr int NX = FM > kStWaves ? FM / kStWaves : 1;
  static constexpr int IS = FM > kStWaves ? 1 : kStWaves / FM;      // stride of the feature tiles
  static constexpr int NI = (FT + IS - 1) / IS;
  static_assert(FM <= kStWaves ? kStWaves % FM == 0 : FM % kStWaves == 0, "tiles of a wave");
  static_assert(S >= 3 && DMA * (S - 2) < 64, "stream ring");
};

template <int FN, int FM, int XT>
__global__ __launch_bounds__(kStThreads) void lora_stream_kernel(GemmArgs a) {
  using SS = StreamShape<FN, FM, XT>;
  constexpr int FT = SS::FT, S = SS::S, D = SS::DMA, NX = SS::NX, NI = SS::NI, IS = SS::IS;
  extern __shared__ __attribute__((aligned(16))) uint8_t st_lds[];

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane % 16, kgrp = lane / 16;
  const int64_t n0 = static_cast<int64_t>(blockIdx.x) * 16 * FN;
  const int64_t t0 = static_cast<int64_t>(blockIdx.y) * 16 * FM;
  const int64_t x0 = static_cast<int64_t>(blockIdx.x) * a.xrows;  // first stacked-A row
  const int z = blockIdx.z;
  const int ksteps = static_cast<int>(a.K / 64);
  const int z_lo = (z * ksteps) / a.ksplit, z_hi = ((z + 1) * ksteps) / a.ksplit;
  const int nsteps = z_hi - z_lo;
  const int rot = static_cast<int>(blockIdx.x % static_cast<unsigned>(nsteps));

  // the lane's rows of its loads: stage row 8 (wave + 4q) + lane/8
  const int dchunk = (lane % 8) ^ (lane / 8);
  const uint16_t* src[D];
#pragma unroll
  for (int q = 0; q < D; ++q) {
    const int r = 8 * (wave + kStWaves * q) + lane / 8;
    const uint16_t* p;
    if (r < 16 * FN) {  // W row (a 16-row tile lies in one projection)
      const int g = group_of(a, n0 + 16 * (r / 16));
      const int64_t n = n0 + r;
      p = pick(a.gw, g) + (n < a.N ? n - gstart_of(a, g) : 0) * a.K;
    } else if (r < 16 * FT) {  // stacked-A row
      const int64_t row = x0 + (r - 16 * FN);
      const bool ok = r - 16 * FN < a.xrows && row < static_cast<int64_t>(a.G) * a.R;
      const int g = ok ? static_cast<int>(row / a.R) : 0;
      p = pick(a.ga, g) + (ok ? row % a.R : 0) * a.K;
    } else {  // x row (also the padding rows, never read)
      const int64_t t = t0 + (r < 16 * (FT + FM) ? r - 16 * FT : 0);
      p = a.x + (t < a.T ? t : t0) * a.K;
    }
    src[q] = p + 8 * dchunk;
  }
  // k offset of relative step rs (rotated, clamped into the slice)
  auto step_k = [&](int rs) {
    int as = rs < nsteps ? rs + rot : rot;
    as = z_lo + (as >= nsteps ? as - nsteps : as);
    return static_cast<int64_t>(as) * 64;
  };

  // this wave's tiles (past the last feature tile: the last again, not stored)
  const int i0 = FM >= kStWaves ? 0 : wave / FM, j0 = FM >= kStWaves ? wave : wave % FM;
  int woff[NI], xoff[NX];
#pragma unroll
  for (int i = 0; i < NI; ++i) woff[i] = 16 * min(i0 + IS * i, FT - 1) * 128;
#pragma unroll
  for (int j = 0; j < NX; ++j) xoff[j] = 16 * (FT + j0 + kStWaves * j) * 128;
  const int rd0 = col * 128 + 16 * (kgrp ^ (col % 8));  // chunk kgrp of row col
  const int rd1 = rd0 ^ 64;                              // chunk 4 + kgrp
  f32x4 acc[NI][NX];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NX; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Step rs: each wave waits for its own loads of stage rs % S (those of the
  // S - 2 later steps may stay in flight); after the barrier every wave's
  // loads of the step are visible and stage (rs - 1) % S is free for the
  // loads of step rs + S - 1.
  auto issue = [&](int rs, uint8_t* st) {
    const int64_t k = step_k(rs);
#pragma unroll
    for (int q = 0; q < D; ++q)
      lds_load16(src[q] + k, st + 8 * (wave + kStWaves * q) * 128);
  };
#pragma unroll
  for (int p = 0; p < S - 1; ++p) issue(p, st_lds + p * SS::STAGE);
  for (int rs = 0; rs < nsteps; ++rs) {
    const int cur = rs % S;
    wait_vmcnt<D * (S - 2)>();
    wait_lgkm0_barrier();
    issue(rs + S - 1, st_lds + (cur == 0 ? S - 1 : cur - 1) * SS::STAGE);
    const uint8_t* st = st_lds + cur * SS::STAGE;
    u32x4 wv[2][NI], xv[2][NX];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
      for (int j = 0; j < NX; ++j)
        xv[m][j] = *reinterpret_cast<const u32x4*>(st + xoff[j] + (m ? rd1 : rd0));
#pragma unroll
      for (int i = 0; i < NI; ++i)
        wv[m][i] = *reinterpret_cast<const u32x4*>(st + woff[i] + (m ? rd1 : rd0));
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j)
          acc[i][j] = mfma16x16x32(as_bf16x8(wv[m][i]), as_bf16x8(xv[m][j]), acc[i][j]);
  }
  wait_vmcnt<0>();

  // partial sums of the slice: lane holds rows 4 (l/16) .. +4 of tile row i,
  // token column l % 16 of tile j
#pragma unroll
  for (int ii = 0; ii < NI; ++ii)
#pragma unroll
    for (int jj = 0; jj < NX; ++jj) {
      const int i = i0 + IS * ii, j = j0 + kStWaves * jj;
      const int64_t t = t0 + 16 * j + col;
      if (i >= FT || t >= a.T) continue;
      if (i >= FN) {  // stacked-A rows: the shrink's partial sums of this slice
        const int rr = 16 * (i - FN) + 4 * kgrp;
        const int64_t rows = static_cast<int64_t>(a.G) * a.R;
        float* dst = a.pout + (static_cast<int64_t>(z) * a.T + t) * rows + x0 + rr;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (rr + q < a.xrows && x0 + rr + q < rows) dst[q] = acc[ii][jj][q];
        continue;
      }
      const int64_t n = n0 + 16 * i + 4 * kgrp;
      if (n < a.N)
        *reinterpret_cast<f32x4*>(a.part + (static_cast<int64_t>(z) * a.T + t) * a.N + n) =
            acc[ii][jj];
    }
}

// ------------------------------------------------------------- SGMV shrink
// Decode-size shrink, segmented by adapter as in SGMV. Workgroup (z, a, g)
// takes adapter a of projection g and the z-th of up_ks slices of K: the tokens routed to a are
// compacted (ascending) into groups of 16 that become the columns of
// S^T = A_a X_g^T on the matrix cores, with the adapter's rank rows as MFMA
// rows. Each of the 4 waves holds at most U steps of 32 k, so it loads its
// whole slice of A before it even knows the tokens; the waves' partial tiles
// are summed through LDS in wave order. The result, the unscaled fp32 partial
// sum of slice z, goes to P[z][t][j] for the adapter's tokens t and rows
// j < rank; the main kernel sums the slices in order, scales and rounds.
constexpr int kSgThreads = 256;
constexpr int kSgWaves = kSgThreads / kWave;
constexpr int kSgMaxTokens = 256;  // decode sizes only (one token per thread)
constexpr int kSgMaxTiles = 8;     // r_max <= 128

#ifndef LOCAL_SG_U1
#define LOCAL_SG_U1 4  // K-steps of 32 per wave when r_max <= 16
#endif

template <int RT, int U>  // RT 16-row tiles of the rank dimension (r_max <= 16*RT)
__global__ __launch_bounds__(kSgThreads) void lora_sgmv_shrink_kernel(GemmArgs a) {
  __shared__ int toks[kSgMaxTokens];
  __shared__ int wave_cnt[kSgWaves];
  __shared__ f32x4 red[kSgWaves][RT][kWave];
  const int z = blockIdx.x, ad = blockIdx.y, g = blockIdx.z;  // slice, adapter, projection
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int col = lane % 16, kgrp = lane / 16;
  const int rk = rank_g(a, g, ad);
  if (rk == 0) return;  // uniform: no row of this adapter is used
  const int tiles = (rk + 15) / 16;

  // this wave's steps: [s_lo, s_hi) of 32 k, at most U of them
  const int ksteps = static_cast<int>(a.K / 32);
  const int z_lo = (z * ksteps) / a.up_ks, z_hi = ((z + 1) * ksteps) / a.up_ks;
  const int s_lo = z_lo + (wave * (z_hi - z_lo)) / kSgWaves;
  const int s_hi = z_lo + ((wave + 1) * (z_hi - z_lo)) / kSgWaves;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  // A: rank rows 16i + col of the slice, loaded first (rows past the rank
  // read row 0 and are zeroed; steps past s_hi read a valid step and are
  // dropped below)
  const uint16_t* abase = pick(a.ga, g) + static_cast<int64_t>(ad) * a.r_max * a.K + 8 * kgrp;
  bool aok[RT];
  u32x4 av[U][RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) aok[i] = 16 * i + col < rk;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t k = static_cast<int64_t>(max(min(s_lo + u, s_hi - 1), 0)) * 32;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int64_t row = aok[i] ? 16 * i + col : 0;
      av[u][i] = i < tiles ? ld_global<u32x4>(abase + row * a.K + k) : zero4;
    }
  }

  // tokens routed to this adapter, ascending
  const bool mine = token_adapter(a, tid) == ad;
  const uint64_t m = __ballot(mine);
  if (lane == 0) wave_cnt[wave] = __popcll(m);
  __syncthreads();
  int off = 0, n_tok = 0;
  for (int w = 0; w < kSgWaves; ++w) {
    if (w < wave) off += wave_cnt[w];
    n_tok += wave_cnt[w];
  }
  if (mine) toks[off + __popcll(m & ((1ull << lane) - 1ull))] = tid;
  __syncthreads();

#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int i = 0; i < RT; ++i) av[u][i] = (aok[i] && s_lo + u < s_hi) ? av[u][i] : zero4;

  float* pz = a.pout + static_cast<int64_t>(z) * a.T * a.p_stride + g * a.r_max;
  for (int g0 = 0; g0 < n_tok; g0 += 16) {
    const bool xok = g0 + col < n_tok;
    const uint16_t* xrow = a.x + static_cast<int64_t>(toks[xok ? g0 + col : g0]) * a.K + 8 * kgrp;
    u32x4 xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      xv[u] = ld_global<u32x4>(xrow + static_cast<int64_t>(max(min(s_lo + u, s_hi - 1), 0)) * 32);
    f32x4 acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u32x4 xb = xok ? xv[u] : zero4;
#pragma unroll
      for (int i = 0; i < RT; ++i)
        if (i < tiles) acc[i] = mfma16x16x32(as_bf16x8(av[u][i]), as_bf16x8(xb), acc[i]);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) red[wave][i][lane] = acc[i];
    __syncthreads();
    for (int e = tid; e < tiles * kWave; e += kSgThreads) {
      const int i = e / kWave, l = e % kWave;
      f32x4 v = red[0][i][l];
#pragma unroll
      for (int w = 1; w < kSgWaves; ++w) v += red[w][i][l];
      const int slot = g0 + l % 16;
      const int j = 16 * i + 4 * (l / 16);  // first of 4 rank rows
      if (slot < n_tok && j < rk) {
        float* dst = pz + static_cast<int64_t>(toks[slot]) * a.p_stride + j;
        if (j + 4 <= rk) {
          *reinterpret_cast<f32x4*>(dst) = v;
        } else {
          for (int q = 0; j + q < rk; ++q) dst[q] = v[q];
        }
      }
    }
    __syncthreads();
  }
}

// Launch of the SGMV shrink: U steps per wave for the rank tiles, K cut into
// enough slices that no wave has more than U steps.
template <int RT, int U>
local_status_t launch_sgmv_shrink(GemmArgs a, hipStream_t s) {
  lora_sgmv_shrink_kernel<RT, U><<<dim3(static_cast<unsigned>(a.up_ks), static_cast<unsigned>(a.n_ad),
                                        static_cast<unsigned>(a.G)),
                                   kSgThreads, 0, s>>>(a);
  return local_check_launch("lora_linear (SGMV shrink)");
}

// Steps per wave of the SGMV shrink for a given r_max.
int sgmv_steps_per_wave(int r_max) {
  const int rt = (r_max + 15) / 16;
  return rt <= 1 ? LOCAL_SG_U1 : rt <= 2 ? 8 : rt <= 4 ? 4 : 2;
}

// K slices of the SGMV shrink.
int sgmv_slices(int64_t K, int r_max) {
  const int64_t steps = K / 32;
  const int64_t per = static_cast<int64_t>(kSgWaves) * sgmv_steps_per_wave(r_max);
  return static_cast<int>((steps + per - 1) / per);
}

local_status_t run_sgmv_shrink(const GemmArgs& a, hipStream_t s) {
  const int rt = (a.r_max + 15) / 16;
  const int u = sgmv_steps_per_wave(a.r_max);
  if (rt <= 1 && u == 4) return launch_sgmv_shrink<1, 4>(a, s);
  if (rt <= 1) return launch_sgmv_shrink<1, 8>(a, s);
  if (rt <= 2) return launch_sgmv_shrink<2, 8>(a, s);
  if (rt <= 4) return launch_sgmv_shrink<4, 4>(a, s);
  return launch_sgmv_shrink<kSgMaxTiles, 2>(a, s);
}

// --------------------------------------------------------------- epilogue
// Decode sizes, after the base partial sums and the shrink:
//   y[t, n] = bf16( sum_z part[z][t][n] + sum_j U_s[t][j] B[a_t][n][j] + res[t][n] )
// with U_s[t][j] = bf16(s_t * sum_z P[z][t][c]) for j < rank(a_t), both sums
// in slice order; c = a_t*r_max + j when the shrink ran fused with the base
// product (sums for every stacked row), c = j after the SGMV shrink. Workgroup:
// 16 tokens x 64 features; each thread finishes 4 consecutive features of one
// token (16-byte partial loads, an 8-byte store), and with few rank columns its
// share of the delta too, from its own loads of B. With more columns those are
// the bound (every load instruction touches 64 rows of B, and each token reads
// its adapter's rows again), and a wave takes 16 features on the matrix cores
// instead, reading the B rows of each adapter of the tile once, 16 rows by 64
// bytes an instruction. The tokens of other adapters select their own product,
// so a value that is not finite stays with its adapter. Measured (whole calls,
// a thread's own loads / matrix cores): rank 64, 64 tokens x 6144 features over
// 16 adapters 35.1 / 32.3 us (this kernel 14.8 / 11.8), 256 tokens x 12288 144 /
// 130; rank 32, 256 tokens x 4096 45.5 / 41.6, 3 tokens 14.6 / 14.4; rank 24, 3
// tokens x 4096 14.0 / 14.6, 12 x 6144 18.2 / 19.0, 256 x 6144 44.9 / 51.9; rank 16, 32
// tokens x 6144 19.7 / 20.5 (the list of adapters comes first).
constexpr int kEpThreads = 256;
constexpr int kEpTokens = 16;
constexpr int kEpFeatures = 64;

constexpr int kEpFewColumns = 24;
constexpr int kEpBatch = 16;      // B operands in flight per wave
constexpr int kEpUsRow = 128 + 8;  // bf16 values of an LDS row of U_s (padded: bank spread)

// r_max <= 8 STEPS, or no adapters (its registers grow with STEPS).
template <int KSB, int STEPS>
__global__ __launch_bounds__(kEpThreads) void lora_epilogue_kernel(GemmArgs a) {
  constexpr int kSteps = STEPS;
  __shared__ float us[kEpTokens][8 * STEPS + 1];
  const int tid = threadIdx.x;
  const int tt = tid / (kEpFeatures / 4), ng = tid % (kEpFeatures / 4);
  const int64_t t0 = static_cast<int64_t>(blockIdx.y) * kEpTokens;
  const int64_t nv0 = static_cast<int64_t>(blockIdx.x) * kEpFeatures;  // virtual row
  const int64_t t = t0 + tt, nv = nv0 + 4 * ng;
  const bool live = t < a.T && nv < a.N;
  const bool lora = a.n_ad > 0;  // uniform
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  // the tile's projection (a 64-row tile lies in one) and its own row index
  const int g = group_of(a, nv0);
  const int64_t Ng = gstart_of(a, g + 1) - gstart_of(a, g);
  const int64_t n = nv - gstart_of(a, g);

  // Every load that needs no other load's result is issued first: the base
  // slices, the residual, this token's adapter; then, needing only the
  // adapter, its B rows and the shrink slices.
  f32x4 pv[KSB];
#pragma unroll
  for (int z = 0; z < KSB; ++z)
    pv[z] = live ? ld_global<f32x4>(a.part + (static_cast<int64_t>(z) * a.T + t) * a.N + nv)
                 : f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* res = pick(a.gres, g);
  u32x2 rv = {0u, 0u};
  if (live && res) rv = ld_global<u32x2>(res + t * Ng + n);
  const int my_ad = (lora && live) ? token_adapter(a, t) : -1;
  const uint16_t* brow =
      pick(a.gb, g) + (static_cast<int64_t>(my_ad >= 0 ? my_ad : 0) * Ng + n) * a.r_max;
  u32x4 bv[kSteps][4];  // [8-column step][feature]
  if (my_ad >= 0) {
#pragma unroll
    for (int js = 0; js < kSteps; ++js)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        bv[js][i] = 8 * js < a.r_max ? ld_global<u32x4>(brow + i * a.r_max + 8 * js) : zero4;
  }

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int z = 0; z < KSB; ++z) acc += pv[z];

  if (lora) {
    // U_s of the tile's tokens, 4 rank rows per item: bf16(s_t * u), u the
    // sum of the shrink slices in slice order (batches of 8 loads)
    const int quads = a.r_max / 4;
    const int64_t slice = a.T * a.p_stride;
    for (int e = tid; e < kEpTokens * quads; e += kEpThreads) {
      const int et = e / quads, j = 4 * (e % quads);
      const int ad = token_adapter(a, t0 + et);
      f32x4 u = {0.f, 0.f, 0.f, 0.f};
      if (ad >= 0) {
        const float sc = a.scale[t0 + et];
        const int rk = rank_g(a, g, ad);
        const float* p = a.pout + (t0 + et) * a.p_stride +
                         (a.p_stacked ? static_cast<int64_t>(g) * a.R + ad * a.r_max
                                      : static_cast<int64_t>(g) * a.r_max) + j;
        for (int z0 = 0; z0 < a.up_ks; z0 += 8) {
          f32x4 sv[8];
#pragma unroll
          for (int zz = 0; zz < 8; ++zz)
            sv[zz] = z0 + zz < a.up_ks ? ld_global<f32x4>(p + (z0 + zz) * slice)
                                       : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int zz = 0; zz < 8; ++zz) u += sv[zz];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)  // rows at or past the rank are never written
          u[q] = j + q < rk ? bf16_to_f32(f32_to_bf16(sc * u[q])) : 0.f;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) us[et][j + q] = u[q];
    }
    __syncthreads();
    if (my_ad >= 0) {
      // delta of 4 features over the rank columns
      const int rk = rank_g(a, g, my_ad);
#pragma unroll
      for (int js = 0; js < kSteps; ++js)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = 8 * js + e;
          if (j < rk) {  // columns at or past the rank are never used
            const float u = us[tt][j];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t w = bv[js][i][e / 2];
              acc[i] += u * __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
            }
          }
        }
    }
  }
  if (!live) return;
  if (res) {
    acc[0] += __uint_as_float(rv.x << 16);
    acc[1] += __uint_as_float(rv.x & 0xffff0000u);
    acc[2] += __uint_as_float(rv.y << 16);
    acc[3] += __uint_as_float(rv.y & 0xffff0000u);
  }
  *reinterpret_cast<u32x2*>(pick(a.gy, g) + t * Ng + n) =
      u32x2{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
}

// r_max > kEpFewColumns.
template <int KSB>
__global__ __launch_bounds__(kEpThreads) void lora_epilogue_wide_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t us[kEpTokens * kEpUsRow];
  __shared__ __attribute__((aligned(16))) float delta[kEpTokens * (kEpFeatures + 4)];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane % 16, kgrp = lane / 16;
  const int tt = tid / (kEpFeatures / 4), ng = tid % (kEpFeatures / 4);
  const int64_t t0 = static_cast<int64_t>(blockIdx.y) * kEpTokens;
  const int64_t nv0 = static_cast<int64_t>(blockIdx.x) * kEpFeatures;  // virtual row
  const int64_t t = t0 + tt, nv = nv0 + 4 * ng;
  const bool live = t < a.T && nv < a.N;
  const bool lora = a.n_ad > 0;  // uniform
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  // the tile's projection (a 64-row tile lies in one) and its own row index
  const int g = group_of(a, nv0);
  const int64_t Ng = gstart_of(a, g + 1) - gstart_of(a, g);
  const int64_t n = nv - gstart_of(a, g);

  // Every load that needs no other load's result is issued first: the
  // adapter of token col of the tile, the base slices, the residual.
  const int my_ad = lora ? token_adapter(a, t0 + col) : -1;
  f32x4 pv[KSB];
#pragma unroll
  for (int z = 0; z < KSB; ++z)
    pv[z] = live ? ld_global<f32x4>(a.part + (static_cast<int64_t>(z) * a.T + t) * a.N + nv)
                 : f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* res = pick(a.gres, g);
  u32x2 rv = {0u, 0u};
  if (live && res) rv = ld_global<u32x2>(res + t * Ng + n);

  // ---- delta: for each adapter of the tile's tokens the product of its B
  // rows (16 of this wave's features) and every token's U_s, of which the
  // tokens of that adapter keep theirs. Items: (adapter, 32 rank columns).
  uint64_t pending = __ballot(my_ad >= 0) & 0xffffull;
  if (pending) {  // uniform over the workgroup (every wave holds the same 16 tokens)
    const int my_rk = my_ad >= 0 ? rank_g(a, g, my_ad) : 0;
    // lane i holds item i (at most 16 adapters x 4 steps of rank columns): its
    // first column and a token of its adapter. One step holds r_max <= 32
    // columns, whatever the rank: then the B rows need not wait for the ranks.
    int it_t = 0, it_j = 0, n_items = 0;
    while (pending) {
      const int l = __builtin_ctzll(pending);
      pending &= ~__ballot(my_ad == __builtin_amdgcn_readlane(my_ad, l));
      if (lane >= n_items) {
        it_t = l;
        it_j = 32 * (lane - n_items);
      }
      n_items += a.r_max <= 32 ? 1 : (__builtin_amdgcn_readlane(my_rk, l) + 31) / 32;
    }
    const uint16_t* brow = pick(a.gb, g) +  // (N_g is a multiple of 64)
                           (nv0 - gstart_of(a, g) + 16 * wave + col) * a.r_max;
    const int64_t ad_stride = Ng * a.r_max;
    u32x4 bv[kEpBatch];
    auto load_batch = [&](int base) {
#pragma unroll
      for (int i = 0; i < kEpBatch; ++i)
        if (base + i < n_items) {
          const int j = __builtin_amdgcn_readlane(it_j, base + i) + 8 * kgrp;
          const int ad =
              __builtin_amdgcn_readlane(my_ad, __builtin_amdgcn_readlane(it_t, base + i));
          bv[i] = ld_global<u32x4>(brow + ad * ad_stride + (j < a.r_max ? j : 0));
        }
    };
    load_batch(0);

    // U_s of the tile's tokens, 4 rank rows per item: bf16(s_t * u), u the
    // sum of the shrink slices in slice order (batches of 8 loads)
    const int quads = (a.r_max + 31) / 32 * 8;
    const int64_t slice = a.T * a.p_stride;
    for (int e = tid; e < kEpTokens * quads; e += kEpThreads) {
      const int et = e / quads, j = 4 * (e % quads);
      const int ead = token_adapter(a, t0 + et);
      f32x4 u = {0.f, 0.f, 0.f, 0.f};
      if (ead >= 0 && j < a.r_max) {
        const float sc = a.scale[t0 + et];
        const int erk = rank_g(a, g, ead);
        const float* p = a.pout + (t0 + et) * a.p_stride +
                         (a.p_stacked ? static_cast<int64_t>(g) * a.R + ead * a.r_max
                                      : static_cast<int64_t>(g) * a.r_max) + j;
        for (int z0 = 0; z0 < a.up_ks; z0 += 8) {
          f32x4 sv[8];
#pragma unroll
          for (int zz = 0; zz < 8; ++zz)
            sv[zz] = z0 + zz < a.up_ks ? ld_global<f32x4>(p + (z0 + zz) * slice)
                                       : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int zz = 0; zz < 8; ++zz) u += sv[zz];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)  // rows at or past the rank are never written
          u[q] = j + q < erk ? sc * u[q] : 0.f;
      }
      *reinterpret_cast<u32x2*>(us + et * kEpUsRow + j) =
          u32x2{pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3])};
    }
    __syncthreads();

    f32x4 mine = {0.f, 0.f, 0.f, 0.f}, prod = {0.f, 0.f, 0.f, 0.f};
    for (int base = 0; base < n_items; base += kEpBatch) {
      if (base) load_batch(base);
#pragma unroll
      for (int i = 0; i < kEpBatch; ++i)
        if (base + i < n_items) {
          const int at = __builtin_amdgcn_readlane(it_t, base + i);
          const int j0 = __builtin_amdgcn_readlane(it_j, base + i);
          const int ad = __builtin_amdgcn_readlane(my_ad, at);
          const int rk = __builtin_amdgcn_readlane(my_rk, at);
          const u32x4 b = keep_first8(bv[i], rk - j0 - 8 * kgrp);
          const u32x4 u = *reinterpret_cast<const u32x4*>(us + col * kEpUsRow + j0 + 8 * kgrp);
          if (j0 == 0) prod = f32x4{0.f, 0.f, 0.f, 0.f};
          prod = mfma16x16x32(as_bf16x8(b), as_bf16x8(u), prod);
          // the tokens of the adapter (after its last columns: the whole sum)
#pragma unroll
          for (int q = 0; q < 4; ++q) mine[q] = my_ad == ad ? prod[q] : mine[q];
        }
    }
    *reinterpret_cast<f32x4*>(delta + col * (kEpFeatures + 4) + 16 * wave + 4 * kgrp) = mine;
  }
  const bool any = lora && __ballot(my_ad >= 0) != 0ull;
  if (any) __syncthreads();
  if (!live) return;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int z = 0; z < KSB; ++z) acc += pv[z];
  if (any) acc += *reinterpret_cast<const f32x4*>(delta + tt * (kEpFeatures + 4) + 4 * ng);
  if (res) {
    acc[0] += __uint_as_float(rv.x << 16);
    acc[1] += __uint_as_float(rv.x & 0xffff0000u);
    acc[2] += __uint_as_float(rv.y << 16);
    acc[3] += __uint_as_float(rv.y & 0xffff0000u);
  }
  *reinterpret_cast<u32x2*>(pick(a.gy, g) + t * Ng + n) =
      u32x2{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
}

template <int KSB>
local_status_t launch_epilogue(const GemmArgs& a, hipStream_t s) {
  dim3 grid(static_cast<unsigned>((a.N + kEpFeatures - 1) / kEpFeatures),
            static_cast<unsigned>((a.T + kEpTokens - 1) / kEpTokens));
  if (a.n_ad > 0 && a.r_max > kEpFewColumns)
    lora_epilogue_wide_kernel<KSB><<<grid, kEpThreads, 0, s>>>(a);
  else if (a.n_ad > 0 && a.r_max > 16)
    lora_epilogue_kernel<KSB, 3><<<grid, kEpThreads, 0, s>>>(a);
  else
    lora_epilogue_kernel<KSB, 2><<<grid, kEpThreads, 0, s>>>(a);
  return local_check_launch("lora_linear (epilogue)");
}

local_status_t run_epilogue(const GemmArgs& a, hipStream_t s) {
  switch (a.ksplit) {
    case 1: return launch_epilogue<1>(a, s);
    case 2: return launch_epilogue<2>(a, s);
    case 4: return launch_epilogue<4>(a, s);
    case 8: return launch_epilogue<8>(a, s);
    default: return launch_epilogue<16>(a, s);
  }
}

// ----------------------------------------------------------------- prefill
// Long chunks (T > 256), the fused main product. Workgroup: tokens
// [m0, m0 + BM) x features [n0, n0 + BN), WM x WN waves. Both operands reach
// LDS by direct global-to-LDS loads (no staging registers, no LDS store
// instructions): a K-step of 64 is one stage (x: BM rows, W: BN rows, 128
// bytes each) of a ring of STAGES, so the loads of later steps are in flight
// while step s computes. Each load instruction moves 8 whole 128-byte rows
// (64 lanes x 16 bytes), so the vector memory path sees fully used lines.
// Inside a row the eight 16-byte chunks are stored XOR-swizzled by the row
// index (chunk c of row r at position c ^ (r % 8)): the MFMA operand reads
// (16 rows, one chunk column) then touch distinct banks. The loads name their
// own waits (the library waits on the load counter itself before each
// barrier). The LoRA delta runs first, as K-steps over 64 stacked columns of
// the adapters used in the token tile.
template <int BM, int BN, int WM_, int WN_, int STAGES>
struct PfShape {
  static constexpr int M = BM, N = BN, WM = WM_, WN = WN_;
  static constexpr int S = STAGES;                // ring stages
  static constexpr int WAVES = WM * WN, THREADS = WAVES * kWave;
  static constexpr int FT = BN / WN / 16;         // 16-feature MFMA tiles per wave
  static constexpr int TT = BM / WM / 16;         // 16-token MFMA tiles per wave
  static constexpr int X_BYTES = BM * 128;        // x rows of a stage
  static constexpr int STAGE = (BM + BN) * 128;   // bytes of a stage
  static constexpr int OUT_ROW = BN * 4 + 16;     // bytes of a token row of the output tile
  static constexpr int RING = S * STAGE;          // the U_s tile of the delta follows it
  static constexpr int LDS = RING + X_BYTES > BM * OUT_ROW ? RING + X_BYTES : BM * OUT_ROW;
  static constexpr int XD = BM / 8 / WAVES, WD = BN / 8 / WAVES;  // 1 KB loads per wave and step
  static constexpr int DMA = XD + WD;
  static constexpr int MFMAS = FT * TT;           // per wave and half step
  static_assert(BM % (8 * WAVES) == 0 && BN % (8 * WAVES) == 0 && LDS <= 163840, "tile");
  static_assert(DMA * (S - 1) < 64 && S >= 3, "ring");
};

template <class PF>
__global__ __launch_bounds__(PF::THREADS, 1) void lora_prefill_kernel(GemmArgs a) {
  constexpr int FT = PF::FT, TT = PF::TT, XD = PF::XD, WD = PF::WD, S = PF::S;
  extern __shared__ __attribute__((aligned(16))) uint8_t pf_lds[];

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // uniform: LDS bases in SGPRs
  const int col = lane % 16, kgrp = lane / 16;

  // ---- tile coordinates: XCD-aware grouped order (the blocks of one XCD
  // take an 8-tall column of tiles, so its L2 serves x and W rows in common)
  int mt, nt;
  {
    const int id = blockIdx.x;
    const int total = a.gm * a.gn;
    int lid = id;
    if (total % kNumXcd == 0) lid = (id % kNumXcd) * (total / kNumXcd) + id / kNumXcd;
    constexpr int GM = 8;
    const int group = lid / (GM * a.gn);
    const int first_m = group * GM;
    const int gsize = min(a.gm - first_m, GM);
    const int r = lid % (GM * a.gn);
    mt = first_m + r % gsize;
    nt = r / gsize;
  }
  const int64_t m0 = static_cast<int64_t>(mt) * PF::M;
  const int64_t n0 = static_cast<int64_t>(nt) * PF::N;
  // projection of the tile (a tile lies in one projection) and its operands;
  // feature indices below are virtual rows n0 + ...
  const int gq = group_of(a, n0);
  const int64_t gbase = gstart_of(a, gq), Ng = gstart_of(a, gq + 1) - gbase;
  const uint16_t* Wg = pick(a.gw, gq);
  const int wm = wave / PF::WN, wn = wave % PF::WN;
  const int tw0 = 16 * TT * wm;  // this wave's first token of the tile
  const int fw0 = 16 * FT * wn;  // ... and first feature

  const bool lora = a.n_ad > 0;  // uniform

  // ---- direct loads. Wave w moves BM / waves x rows and BN / waves W rows of
  // every stage; lane l writes 16 bytes at block + 16 l, i.e. row 8q + l/8,
  // position l%8, which holds chunk (l%8) ^ (l/8) of that row. Rows past T (N)
  // repeat row m0 (row 0): their accumulators are never stored.
  const int dchunk = (lane % 8) ^ (lane / 8);
  const uint16_t* xg[XD];
  const uint16_t* wg[WD];
  int64_t xt[XD];          // the x rows
  // the x rows' adapters and scales, and those of the whole tile (a token per
  // lane): loaded before the stage loads, so that they wait for nothing else
  int xad[XD], tad[PF::M / kWave];
  float xsc[XD];
#pragma unroll
  for (int h = 0; h < PF::M / kWave; ++h) {
    const int64_t t = m0 + kWave * h + lane;
    tad[h] = lora && t < a.T ? a.idx[t] : -1;
  }
#pragma unroll
  for (int q = 0; q < XD; ++q) {
    const int64_t t = m0 + 8 * (XD * wave + q) + lane / 8;
    xt[q] = t < a.T ? t : m0;
    xad[q] = lora && t < a.T ? a.idx[t] : -1;
    xsc[q] = lora && t < a.T ? a.scale[t] : 0.f;
    xg[q] = a.x + xt[q] * a.K + 8 * dchunk;
  }
#pragma unroll
  for (int q = 0; q < WD; ++q) {
    const int64_t nl = n0 - gbase + 8 * (WD * wave + q) + lane / 8;
    wg[q] = Wg + (nl < Ng ? nl : 0) * a.K + 8 * dchunk;
  }
  auto x_dst = [&](int stage, int q) {
    return pf_lds + stage * PF::STAGE + 1024 * (XD * wave + q);
  };
  auto w_dst = [&](int stage, int q) {
    return pf_lds + stage * PF::STAGE + PF::X_BYTES + 1024 * (WD * wave + q);
  };
  // loads of K-step s into stage `stage`
  auto issue = [&](int stage, int s) {
    const int64_t k = static_cast<int64_t>(s) * 64;
#pragma unroll
    for (int q = 0; q < XD; ++q) lds_load16(xg[q] + k, x_dst(stage, q));
#pragma unroll
    for (int q = 0; q < WD; ++q) lds_load16(wg[q] + k, w_dst(stage, q));
  };

  f32x4 acc[FT][TT];
#pragma unroll
  for (int i = 0; i < FT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // MFMA operand reads. K-group g of MFMA m holds k = 32m + 8g .. +8 of the
  // step (chunk 4m + g), the same for W and x; chunk c of row r sits at
  // position c ^ (r % 8), and r % 8 = col % 8 for every row a lane reads.
  const int rd0 = col * 128 + 16 * (kgrp ^ (col % 8));  // chunk kgrp
  const int rd1 = rd0 ^ 64;                              // chunk 4 + kgrp
  u32x4 xf[2][TT], wf[2][FT];
  auto read_half = [&](int stage, int m) {
    const uint8_t* st = pf_lds + stage * PF::STAGE + (m ? rd1 : rd0);
#pragma unroll
    for (int i = 0; i < FT; ++i)
      wf[m][i] = *reinterpret_cast<const u32x4*>(st + PF::X_BYTES + (fw0 + 16 * i) * 128);
#pragma unroll
    for (int j = 0; j < TT; ++j)
      xf[m][j] = *reinterpret_cast<const u32x4*>(st + (tw0 + 16 * j) * 128);
  };
  // MFMAs [b, e) of half m, in the order tile (i, j) = (idx / TT, idx % TT)
  auto mfma_range = [&](int m, int b, int e) {
#pragma unroll
    for (int idx = b; idx < e; ++idx) {
      const int i = idx / TT, j = idx % TT;
      acc[i][j] = mfma16x16x32(as_bf16x8(wf[m][i]), as_bf16x8(xf[m][j]), acc[i][j]);
    }
  };
  // instruction-group masks of the scheduler's group barriers, and the
  // group sizes of a step: R operand reads per half, Q MFMAs of the second
  // half before the barrier, the loads paired with MFMAs after the reads
  constexpr int kSgMfma = 0x8, kSgVmem = 0x10, kSgDsRead = 0x100;
  constexpr int kR = FT + TT;
  constexpr int kQ = PF::MFMAS / 4 < PF::MFMAS - kR ? PF::MFMAS / 4 : PF::MFMAS - kR;
  constexpr int kVPair = PF::DMA < PF::MFMAS - kQ - kR ? PF::DMA : PF::MFMAS - kQ - kR;
  static_assert(kQ >= 0 && kVPair >= 0, "step schedule");

  // Step s (stage s % S), first half: the m = 1 operands are read under the
  // m = 0 MFMAs. Then each wave waits for its own loads of step s + 1 (those
  // of later steps may stay in flight) and for its reads of stage s % S; after
  // the barrier every wave's loads of step s + 1 are visible and stage s % S
  // is free, so the loads of step s + S refill it. Second half: the m = 0
  // operands of step s + 1 are read under the m = 1 MFMAs of step s. The
  // body has no branch (a branch between the two halves makes the compiler
  // copy the accumulators around it): past the last step the loads
  // repeat the last step into the free stage and the reads fetch operands
  // that are never used, so every wait count holds at every step.
  const int steps = static_cast<int>(a.K / 64);
  const int last = steps - 1;
  // the loads of every stage go out before anything else waits
#pragma unroll
  for (int p = 0; p < S; ++p) issue(p, min(p, last));

  // ---- LoRA delta: K-steps of 64 stacked columns c = a*r_max + j, a tile of
  // U_s rows (laid out as x rows) against B rows loaded as operands, while the
  // first stages load. U_s[t][c] = bf16(s_t u) when a is token t's adapter and
  // j below its rank, else 0: as the shrink wrote it, by direct loads like
  // those of x (pieces of other adapters from 16 bytes of zeros), or formed
  // here from the sums of its K slices, in order. B's columns at or past the
  // rank, and those of adapters that no token of the tile uses, are zeroed on
  // their way into the product (they may hold anything). Adding the delta
  // first leaves a zero up-projection's result bit-identical (the MFMAs add
  // +0).
  if (lora) {
    const uint16_t* Bg = pick(a.gb, gq);
    const int32_t* ranksg = pick(a.granks, gq);
    uint8_t* ut = pf_lds + PF::RING;
#pragma unroll
    for (int h = 0; h < PF::M / kWave; ++h)
      if (tad[h] >= a.n_ad) tad[h] = -1;
#pragma unroll
    for (int q = 0; q < XD; ++q)
      if (xad[q] >= a.n_ad) xad[q] = -1;
    // the first chunk after chunk c with columns of an adapter that a token of
    // the tile uses, or -1
    auto next_chunk = [&](int c) {
      int first = INT_MAX;
#pragma unroll
      for (int h = 0; h < PF::M / kWave; ++h)
        if (tad[h] >= 0 && ((tad[h] + 1) * a.r_max - 1) / 64 > c)
          first = min(first, max(tad[h] * a.r_max / 64, c + 1));
      if (a.R <= 64) return __any(first == 0) ? 0 : -1;
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off));
      first = __builtin_amdgcn_readfirstlane(first);
      return first == INT_MAX ? -1 : first;
    };
    for (int c = next_chunk(-1); c >= 0;) {
      const int cl = c * 64 + 8 * dchunk;  // the stacked columns of this lane's pieces
      const int ca = cl / a.r_max, cj = cl % a.r_max;
      // B operands: features fw0 + 16 i + col, columns 64 c + 32 m + 8 kgrp ..
      // +8, and how many of those columns are used
      const int a_lo = c * 64 / a.r_max;
      uint32_t routed = 0u;  // bit i: a token of the tile uses adapter a_lo + i
      for (int i = 0; i <= (c * 64 + 63) / a.r_max - a_lo; ++i) {
        bool any = false;
#pragma unroll
        for (int h = 0; h < PF::M / kWave; ++h) any |= tad[h] == a_lo + i;
        routed |= __any(any) ? 1u << i : 0u;
      }
      u32x4 bw[2][FT];
      int keep[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int k0 = c * 64 + 32 * m + 8 * kgrp;
        const int ad = min(k0 / a.r_max, a.n_ad - 1), j = k0 % a.r_max;
        const int rk = ranksg ? min(max(ranksg[ad], 0), a.r_max) : a.r_max;
        keep[m] = k0 < a.R && (routed >> (ad - a_lo) & 1u) ? rk - j : 0;
#pragma unroll
        for (int i = 0; i < FT; ++i) {
          const int64_t nl = n0 - gbase + fw0 + 16 * i + col;
          bw[m][i] = ld_global<u32x4>(
              Bg + (static_cast<int64_t>(ad) * Ng + (nl < Ng ? nl : 0)) * a.r_max + j);
        }
      }
      if (a.us) {
        const uint16_t* Ug = a.us + gq * a.T * a.r_max;
#pragma unroll
        for (int q = 0; q < XD; ++q)
          lds_load16(xad[q] == ca ? Ug + xt[q] * a.r_max + cj : a.zero16,
                     ut + 1024 * (XD * wave + q));
      } else {
        // All loads go out before the first sum: clamped to valid addresses
        // instead of left out, four slices at a time.
        const float* Pg = a.pout + static_cast<int64_t>(gq) * a.up_ks * a.T * a.r_max;
        const int rk = ranksg ? min(max(ranksg[min(ca, a.n_ad - 1)], 0), a.r_max) : a.r_max;
        const int64_t slice = a.T * a.r_max;
        f32x4 sum[XD][2] = {};
        for (int z0 = 0; z0 < a.up_ks; z0 += 4) {
          f32x4 v[4][XD][2];
#pragma unroll
          for (int dz = 0; dz < 4; ++dz)
#pragma unroll
            for (int q = 0; q < XD; ++q) {
              const float* p = Pg + min(z0 + dz, a.up_ks - 1) * slice +
                               (xad[q] == ca ? xt[q] * a.r_max + cj : 0);
              v[dz][q][0] = ld_global<f32x4>(p);
              v[dz][q][1] = ld_global<f32x4>(p + 4);
            }
#pragma unroll
          for (int dz = 0; dz < 4; ++dz)
            if (z0 + dz < a.up_ks)
#pragma unroll
              for (int q = 0; q < XD; ++q) {
                sum[q][0] += v[dz][q][0];
                sum[q][1] += v[dz][q][1];
              }
        }
#pragma unroll
        for (int q = 0; q < XD; ++q) {
          const int keep = xad[q] == ca ? rk - cj : 0;
          float u[8];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            u[i] = i < keep ? xsc[q] * (i < 4 ? sum[q][0][i] : sum[q][1][i - 4]) : 0.f;
          *reinterpret_cast<u32x4*>(ut + 1024 * (XD * wave + q) + 16 * lane) =
              u32x4{pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3]), pack_bf16x2(u[4], u[5]),
                    pack_bf16x2(u[6], u[7])};
        }
      }
      wait_vmcnt<0>();
      wait_lgkm0_barrier();
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        u32x4 uv[TT];
#pragma unroll
        for (int j = 0; j < TT; ++j)
          uv[j] = *reinterpret_cast<const u32x4*>(ut + (tw0 + 16 * j) * 128 + (m ? rd1 : rd0));
#pragma unroll
        for (int i = 0; i < FT; ++i) {
          const bf16x8 b = as_bf16x8(keep_first8(bw[m][i], keep[m]));
#pragma unroll
          for (int j = 0; j < TT; ++j) acc[i][j] = mfma16x16x32(b, as_bf16x8(uv[j]), acc[i][j]);
        }
      }
      c = next_chunk(c);
      if (c >= 0) wait_lgkm0_barrier();  // the tile is rewritten
    }
  }
  wait_vmcnt<PF::DMA * (S - 1)>();
  wait_lgkm0_barrier();
  read_half(0, 0);
  // unrolled over the stage ring so that stage offsets are constants; the
  // tail leaves the loop (a branch out of the loop, not around work in it)
  for (int s0 = 0; s0 < steps; s0 += S) {
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int s = s0 + u;
      if (s >= steps) break;
      // first half: one operand read (m = 1) beside each of the first kR
      // MFMAs (m = 0)
      read_half(u, 1);
      mfma_range(0, 0, PF::MFMAS);
#pragma unroll
      for (int g = 0; g < kR; ++g) {
        __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 0);
      }
      if (PF::MFMAS > kR) __builtin_amdgcn_sched_group_barrier(kSgMfma, PF::MFMAS - kR, 0);
      __builtin_amdgcn_sched_barrier(0);
      // second half: kQ MFMAs (m = 1) before the barrier, then the operand
      // reads of the next step and the loads of step s + S beside the rest
      mfma_range(1, 0, kQ);
      __builtin_amdgcn_sched_barrier(0);
      wait_vmcnt<PF::DMA * (S - 2)>();
      wait_lgkm0_barrier();
      __builtin_amdgcn_sched_barrier(0);
      read_half((u + 1) % S, 0);
      issue(u, min(s + S, last));
      mfma_range(1, kQ, PF::MFMAS);
#pragma unroll
      for (int g = 0; g < kR; ++g) {
        __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 1);
        __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 1);
      }
#pragma unroll
      for (int g = 0; g < kVPair; ++g) {
        __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 1);
        __builtin_amdgcn_sched_group_barrier(kSgVmem, 1, 1);
      }
      if (PF::DMA > kVPair) __builtin_amdgcn_sched_group_barrier(kSgVmem, PF::DMA - kVPair, 1);
      if (PF::MFMAS - kQ - kR > kVPair)
        __builtin_amdgcn_sched_group_barrier(kSgMfma, PF::MFMAS - kQ - kR - kVPair, 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  wait_vmcnt<0>();

  // ---- output. The tile's fp32 sums go through LDS (the stages are free once
  // every wave's loads have landed and its reads are done), so that each
  // thread then finishes 8 consecutive features of one token: the residual
  // and the output move as coalesced 16-byte pieces. Token rows are
  // padded by 16 bytes, so the 16 tokens of one MFMA tile written
  // together fall in distinct banks.
  const uint16_t* res = pick(a.gres, gq);
  uint16_t* y = pick(a.gy, gq);
  wait_lgkm0_barrier();
#pragma unroll
  for (int j = 0; j < TT; ++j)
#pragma unroll
    for (int i = 0; i < FT; ++i)
      *reinterpret_cast<f32x4*>(pf_lds + (tw0 + 16 * j + col) * PF::OUT_ROW +
                                (fw0 + 16 * i + 4 * kgrp) * 4) = acc[i][j];
  wait_lgkm0_barrier();
  constexpr int kGroups = PF::N / 8;                     // 8-feature groups per token
  constexpr int kItems = PF::M * kGroups / PF::THREADS;  // per thread
  static_assert(PF::M * kGroups % PF::THREADS == 0, "output items");
  u32x4 rv[kItems];
#pragma unroll
  for (int e = 0; e < kItems; ++e) {
    const int item = tid + e * PF::THREADS, tl = item / kGroups, f = 8 * (item % kGroups);
    const int64_t t = m0 + tl, n = n0 - gbase + f;
    rv[e] = (res && t < a.T && n < Ng) ? ld_global<u32x4>(res + t * Ng + n) : u32x4{0u, 0u, 0u, 0u};
  }
#pragma unroll
  for (int e = 0; e < kItems; ++e) {
    const int item = tid + e * PF::THREADS, tl = item / kGroups, f = 8 * (item % kGroups);
    const int64_t t = m0 + tl, n = n0 - gbase + f;
    const uint8_t* src = pf_lds + tl * PF::OUT_ROW + f * 4;
    const f32x4 lo = *reinterpret_cast<const f32x4*>(src);
    const f32x4 hi = *reinterpret_cast<const f32x4*>(src + 16);
    float o[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    if (res) {
      const uint32_t r[4] = {rv[e].x, rv[e].y, rv[e].z, rv[e].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        o[2 * q] += __uint_as_float(r[q] << 16);
        o[2 * q + 1] += __uint_as_float(r[q] & 0xffff0000u);
      }
    }
    if (t < a.T && n < Ng)
      *reinterpret_cast<u32x4*>(y + t * Ng + n) =
          u32x4{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]),
                pack_bf16x2(o[6], o[7])};
  }
}

// One projection of a (grouped) call.
struct Proj {
  const uint16_t* W;
  int64_t N;
  const uint16_t* A;
  const uint16_t* B;
  const int32_t* ranks;
  const uint16_t* res;
  uint16_t* y;
};

template <typename Kernel>
void raise_lds_limit(Kernel k, size_t bytes, bool& done) {
  if (!done) {  // benign race: every caller sets the same value
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(bytes));
    done = true;
  }
}

template <class PF>
local_status_t launch_prefill(GemmArgs a, hipStream_t s) {
  a.gm = static_cast<int>((a.T + PF::M - 1) / PF::M);
  a.gn = static_cast<int>((a.N + PF::N - 1) / PF::N);
  static bool done = false;
  raise_lds_limit(lora_prefill_kernel<PF>, PF::LDS, done);
  lora_prefill_kernel<PF><<<a.gm * a.gn, PF::THREADS, PF::LDS, s>>>(a);
  return local_check_launch("lora_linear (prefill)");
}

using Pf128x256 = PfShape<128, 256, 2, 4, 3>;
using Pf128x128 = PfShape<128, 128, 2, 4, 4>;
using Pf64x128 = PfShape<64, 128, 2, 2, 3>;
using Pf64x64 = PfShape<64, 64, 2, 2, 4>;

// Tile shape of a long chunk's product over projections of N_g features, by
// the time its tiles take: whole rounds of `slots` workgroups (two per compute
// unit where the ring is at most half its LDS), then a last round of what is
// left. A workgroup takes `fixed` us and, per 64-k step, `few` us while a
// third of the chip or less is busy and `full` us when all of it is (the
// clock falls and the caches are shared). Measured at K = 4096 (tile: us of a
// round that is nearly empty / full): 128x256: 44 / 58, 128x128: 28 / 36,
// 64x128: 24 / 41, 64x64: 23 / 26; of one of several full rounds 66, 40, 48 and
// -, so 64x128 is priced at 43. So, at 4096 features, 2048 tokens take
// 128x256 (58 us; 128x128: 70), 1000 tokens 128x128 (37 us; 128x256: 49) and
// 300 tokens 64x128 (24 us; 128x256: 44); at 12288, 1300 tokens 128x256 (whole
// call 169 us; 64x128: 188). (Larger tiles are no faster where they would fill
// the chip: a full round of 256x256 takes twice that of 128x256, the clock being
// what gives.)
struct PfCost {
  int m, n, slots;
  double fixed, few, full, knee;  // knee: the load from which a step takes `full`
};
constexpr PfCost kPfCosts[] = {{128, 256, 256, 5.0, 0.62, 0.83, 1.0},
                               {128, 128, 256, 4.0, 0.37, 0.51, 1.0},
                               {64, 128, 512, 3.2, 0.32, 0.62, 0.75},
                               {64, 64, 512, 3.0, 0.31, 0.35, 1.0}};

int prefill_tile(int64_t T, int64_t K, int G, const Proj* p) {
  int64_t n_total = 0;
  for (int g = 0; g < G; ++g) n_total += p[g].N;
  int best = 3;  // every N_g is a multiple of 64
  double best_us = 0.0;
  for (int c = best; c >= 0; --c) {
    const PfCost& f = kPfCosts[c];
    bool ok = true;  // no tile straddles two projections
    for (int g = 0; g < G && G > 1; ++g) ok = ok && p[g].N % f.n == 0;
    if (!ok) continue;
    const int64_t tiles = ((T + f.m - 1) / f.m) * ((n_total + f.n - 1) / f.n);
    const int64_t rest = tiles % f.slots;
    const double steps = static_cast<double>(K / 64);
    double us = static_cast<double>(tiles / f.slots) * (f.fixed + steps * f.full);
    if (rest) {
      const double busy = static_cast<double>(rest) / f.slots;
      const double load = std::max(0.0, (busy - 0.35) / (f.knee - 0.35));
      us += f.fixed + steps * (f.few + (f.full - f.few) * std::min(load, 1.0));
    }
    if (c == 3 || us < best_us) {
      best = c;
      best_us = us;
    }
  }
  return best;
}

}  // namespace

// The tile of a long chunk's product that a call's sizes select: 0 to 3 = 128 x
// 256, 128 x 128, 64 x 128, 64 x 64 (for the tests, which name the tile that they
// mean; not in local.h).
extern "C" int32_t localk_prefill_tile(int64_t T, int64_t K, int32_t G, const int64_t* N) {
  Proj p[kMaxGroup] = {};
  for (int g = 0; g < G; ++g) p[g].N = N[g];
  return prefill_tile(T, K, G, p);
}

namespace {

local_status_t run_prefill(const GemmArgs& a, int tile, hipStream_t s) {
  switch (tile) {
    case 0: return launch_prefill<Pf128x256>(a, s);
    case 1: return launch_prefill<Pf128x128>(a, s);
    case 2: return launch_prefill<Pf64x128>(a, s);
    default: return launch_prefill<Pf64x64>(a, s);
  }
}

template <int FN, int FM, int XT>
local_status_t launch_stream(GemmArgs a, hipStream_t s) {
  using SS = StreamShape<FN, FM, XT>;
  static bool done = false;
  raise_lds_limit(lora_stream_kernel<FN, FM, XT>, kStLdsMax, done);
  dim3 grid(static_cast<unsigned>((a.N + 16 * FN - 1) / (16 * FN)),
            static_cast<unsigned>((a.T + 16 * FM - 1) / (16 * FM)),
            static_cast<unsigned>(a.ksplit));
  lora_stream_kernel<FN, FM, XT><<<grid, kStThreads, SS::S * SS::STAGE, s>>>(a);
  return local_check_launch("lora_linear (stream)");
}

// Decode sizes (T <= 256): base partial sums over K slices. Wider feature
// tiles cut the re-reads of x (every workgroup of a slice reads the slice of
// x for all its tokens); the shape is the widest tile (of 6, 4, 3 or 2 MFMA
// tiles; 6 up to 32 tokens and above 128) and K split that bring the grid closest
// to LOCAL_P_TARGET_WG workgroups from below. Above 64 tokens the re-reads of x
// bound the product (2 tiles: 16 KB of x a step for 4 KB of W) and the partial sums
// of more than 2 slices cost more than they bring, except with the smallest tile.
// Measured, whole calls with 2 / 3 / 4 / 6 tiles: 128 tokens x 6144 x 4096 35.4 / 28.9
// / 29.1 / 28.8 us, x 12288 (rank 64) 86 / 65 / 66 / 68; 256 tokens x 6144 67 / 48 / 49
// / 44, x 12288 132 / 132 / 126 / 103; 128 tokens x 1536 x 1024 with 4 slices 14.7 / 15.9.
#ifndef LOCAL_P_TARGET_WG
#define LOCAL_P_TARGET_WG 256  // aim: about one workgroup per compute unit
#endif
#ifndef LOCAL_P_WIDE
#define LOCAL_P_WIDE 6  // widest feature tile (MFMA tiles); 0 = none
#endif

struct PartialShape {
  int fn;   // 16-row MFMA tiles per workgroup
  int ksb;  // K slices
};

int token_tiles(int64_t T) { return T <= 16 ? 1 : T <= 32 ? 2 : T <= 64 ? 4 : 8; }

PartialShape partial_shape(int64_t T, int64_t N, int64_t K, bool allow_wide) {
  const int64_t fm = token_tiles(T);
  const int64_t ttiles = (T + 16 * fm - 1) / (16 * fm);
  PartialShape best{4, 1};
  int64_t best_wg = -1;
  const int fns[4] = {LOCAL_P_WIDE, 4, 3, 2};
  for (int fn : fns) {
    if (fn == 0 || (fn > 4 && ((T > 32 && T <= 128) || !allow_wide))) continue;
    const int64_t tiles = (N + 16 * fn - 1) / (16 * fn) * ttiles;
    const int most = T > 64 && fn > 2 ? 2 : 8;
    for (int ks = 1; ks <= most && ks <= K / 64; ks *= 2) {
      const int64_t wg = tiles * ks;
      if (wg <= LOCAL_P_TARGET_WG && wg > best_wg) {
        best = {fn, ks};
        best_wg = wg;
      }
    }
  }
  return best;
}

// The stream kernel for the planned shape: FM token tiles by batch size
// (16 / 32 / 64 / 256 tokens), only the combinations the planner produces.
template <int FN, int XT>
local_status_t run_partial_fn(const GemmArgs& a, hipStream_t s) {
  if (a.T <= 16) return launch_stream<FN, 1, XT>(a, s);
  if constexpr (FN <= 4) {
    if (a.T <= 32) return launch_stream<FN, 2, XT>(a, s);
    if (a.T <= 64) return launch_stream<FN, 4, XT>(a, s);
    return launch_stream<FN, 8, XT>(a, s);
  } else if constexpr (XT <= 2) {
    if (a.T <= 32) return launch_stream<FN, 2, XT>(a, s);
    if (a.T > 64) return launch_stream<FN, 8, XT>(a, s);
  }
  return local_fail(LOCAL_ERR_UNSUPPORTED, "lora_linear: tile of %d features, %d extra row tiles, "
                    "%lld tokens", 16 * FN, XT, static_cast<long long>(a.T));
}

template <int XT>
local_status_t run_partial_xt(const GemmArgs& a, int fn, hipStream_t s) {
#if LOCAL_P_WIDE > 4
  if (fn == LOCAL_P_WIDE) return run_partial_fn<LOCAL_P_WIDE, XT>(a, s);
#endif
  if (fn == 4) return run_partial_fn<4, XT>(a, s);
  if (fn == 3) return run_partial_fn<3, XT>(a, s);
  return run_partial_fn<2, XT>(a, s);
}

// Stacked-A rows each feature-tile workgroup takes with the base product
// (the shrink fused into it), or 0 when that would take more than 4 extra
// row tiles; then the SGMV shrink runs as its own kernel.
int partial_xrows(int64_t ftiles, int64_t rows) {
  if (rows == 0) return 0;
  const int64_t per = (rows + ftiles - 1) / ftiles;
  return per <= 64 ? static_cast<int>(per) : 0;
}

local_status_t run_partial(const GemmArgs& a, int fn, hipStream_t s) {
  if (a.xrows == 0) return run_partial_xt<0>(a, fn, s);
  if (a.xrows <= 16) return run_partial_xt<1>(a, fn, s);
  if (a.xrows <= 32) return run_partial_xt<2>(a, fn, s);
  if (a.xrows <= 64) return run_partial_xt<4>(a, fn, s);
  return local_fail(LOCAL_ERR_UNSUPPORTED, "lora_linear: %d stacked rows per tile", a.xrows);
}

size_t align256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

// Sets the group fields of `a` for projections p[0..G).
void set_groups(GemmArgs& a, int G, const Proj* p) {
  a.G = G;
  int64_t n = 0;
  for (int g = 0; g <= kMaxGroup; ++g) {
    a.gstart[g] = n;
    if (g < G) n += p[g].N;
  }
  for (int g = 0; g < kMaxGroup; ++g) {
    const Proj& q = p[g < G ? g : 0];
    a.gw[g] = q.W;
    a.ga[g] = q.A;
    a.gb[g] = q.B;
    a.granks[g] = q.ranks;
    a.gres[g] = q.res;
    a.gy[g] = q.y;
  }
  a.N = n;
}

// Decode-size plan of a call: tile shape, fused shrink rows, workspace.
struct DecodePlan {
  PartialShape shape;
  int xrows;      // stacked-A rows per workgroup (shrink fused), or 0
  int slices;     // SGMV shrink K slices (shrink not fused), or 0
  size_t part_bytes, shrink_bytes;
};

DecodePlan plan_decode(int64_t T, int64_t K, int G, const Proj* p, int n_ad, int r_max) {
  DecodePlan d{};
  int64_t n_total = 0;
  for (int g = 0; g < G; ++g) n_total += p[g].N;
  const int64_t R = n_ad > 0 ? static_cast<int64_t>(n_ad) * r_max : 0;
  d.shape = partial_shape(T, n_total, K, true);
  int64_t ftiles = (n_total + 16 * d.shape.fn - 1) / (16 * d.shape.fn);
  d.xrows = partial_xrows(ftiles, G * R);
  // the wide tile takes at most 2 extra row tiles
  if (d.shape.fn > 4 && (d.xrows > 32 || (T > 64 && R > 0 && d.xrows == 0))) {
    d.shape = partial_shape(T, n_total, K, false);
    ftiles = (n_total + 16 * d.shape.fn - 1) / (16 * d.shape.fn);
    d.xrows = partial_xrows(ftiles, G * R);
  }
  // (Measured at 64 tokens over 16 adapters padded from ranks 8..64 to 64:
  // taking the shrink out of the base product saves 6.8 us of streaming
  // there, and its own SGMV launch costs 10.3 us; so the shrink rides along
  // whenever it fits.)
  if (n_ad > 0 && d.xrows == 0) d.slices = sgmv_slices(K, r_max);
  d.part_bytes = align256(static_cast<size_t>(d.shape.ksb) * T * n_total * sizeof(float));
  d.shrink_bytes =
      d.xrows > 0 ? align256(static_cast<size_t>(d.shape.ksb) * T * G * R * sizeof(float))
                  : align256(static_cast<size_t>(d.slices) * T * G * r_max * sizeof(float));
  return d;
}

local_status_t lora_impl(const uint16_t* x, int64_t T, int64_t K, int G, const Proj* p,
                         int32_t n_adapters, int32_t r_max, const int32_t* adapter_idx,
                         const float* scale, void* ws, size_t* ws_bytes, hipStream_t s) {
  const int R = n_adapters > 0 ? n_adapters * r_max : 0;
  const bool decode = T <= kSgMaxTokens;
  DecodePlan d{};
  if (decode) d = plan_decode(T, K, G, p, n_adapters, r_max);
  // Workspace. Decode sizes (T <= kSgMaxTokens): the base partial sums
  // [ksb][T][N] fp32 (N over all projections), then the shrink's partial
  // sums: [ksb][T][G*R] fp32 when the shrink runs inside the base product,
  // [slices][T][r_max] after the SGMV shrink. Above: the shrink's sums
  // [G][ks][T][r_max] fp32 (at most long_slices K slices), or its U_s and 16
  // zero bytes; the size (with 32 bytes per 64 tokens, once bitmaps) is the
  // one that callers have always been told.
  const int slices = decode ? 0 : long_slices(T, K, r_max, G);
  size_t decode_need = d.part_bytes + d.shrink_bytes;
  if (decode && T > 128) {  // never less than 128 tokens, whose plan differs, take
    const DecodePlan h = plan_decode(128, K, G, p, n_adapters, r_max);
    decode_need = std::max(decode_need, h.part_bytes + h.shrink_bytes);
  }
  const size_t need =
      decode ? decode_need
      : n_adapters > 0
          ? align256(static_cast<size_t>(G) * slices * T * r_max * sizeof(float)) +
                align256(static_cast<size_t>((T + 63) / 64) * 32)
          : 0;
  if (!ws) {
    *ws_bytes = need;
    return LOCAL_OK;
  }
  if (*ws_bytes < need)
    return local_fail(LOCAL_ERR_WORKSPACE, "lora_linear: workspace %zu < %zu", *ws_bytes, need);
  if (T == 0) return LOCAL_OK;

  GemmArgs g{};
  g.x = x;
  g.T = T;
  g.K = K;
  g.idx = adapter_idx;
  g.scale = scale;
  g.n_ad = n_adapters;
  g.r_max = r_max;
  g.R = R;
  local_status_t st;

  if (decode) {
    float* part = static_cast<float*>(ws);
    float* sp = reinterpret_cast<float*>(static_cast<char*>(ws) + d.part_bytes);
    const bool fused = d.xrows > 0;
    if (n_adapters > 0 && !fused) {  // SGMV shrink of every projection: partial sums
      GemmArgs sh = g;
      set_groups(sh, G, p);
      sh.pout = sp;
      sh.up_ks = d.slices;
      sh.p_stride = G * r_max;
      if ((st = run_sgmv_shrink(sh, s)) != LOCAL_OK) return st;
    }
    GemmArgs m = g;  // base product (+ fused shrink): partial sums per K slice
    set_groups(m, G, p);
    m.part = part;
    m.ksplit = d.shape.ksb;
    m.xrows = d.xrows;
    m.pout = sp;
    if ((st = run_partial(m, d.shape.fn, s)) != LOCAL_OK) return st;
    m.up_ks = fused ? d.shape.ksb : d.slices;  // epilogue: sums, up-projection, residual
    m.p_stride = fused ? G * R : G * r_max;
    m.p_stacked = fused ? 1 : 0;
    m.ksplit = d.shape.ksb;
    return run_epilogue(m, s);
  }

  // long chunks: the shrink of every projection, then the main product over
  // the projections' tiles
  GemmArgs m = g;
  set_groups(m, G, p);
  if (n_adapters > 0) {
    // Few 16-token tiles leave compute units idle, and one unit reads no
    // faster than about 50 GB/s: below 128 of them K is cut into up to 4
    // slices (300 tokens, K = 4096: shrink 8.6 us in one slice, 4.3 in four;
    // with the product, which then forms U_s itself, 33.2 and 30.5 us). From
    // 128 on the slices save less than their sums cost the product (3 x 4096
    // features, 2048 tokens: 199 us with them, 194 without).
    const int64_t tiles = (T + 15) / 16 * G;
    int ks = 1;
    if (tiles < 128)
      while (2 * ks <= std::min(slices, 4) && tiles * ks < 256) ks *= 2;
    m.up_ks = ks;
    uint16_t* us = ks == 1 ? static_cast<uint16_t*>(ws) : nullptr;
    uint16_t* zero16 = us ? us + static_cast<int64_t>(G) * T * r_max : nullptr;
    m.us = us;
    m.zero16 = zero16;
    m.pout = static_cast<float*>(ws);
    ShrinkJob jobs[kMaxGroup];
    for (int q = 0; q < G; ++q)
      jobs[q] = us ? ShrinkJob{x, p[q].A, nullptr, K, us + static_cast<int64_t>(q) * T * r_max,
                               p[q].ranks}
                   : ShrinkJob{x, p[q].A, m.pout + static_cast<int64_t>(q) * ks * T * r_max, K,
                               nullptr, nullptr};
    if ((st = token_shrink(jobs, G, T, n_adapters, r_max, adapter_idx, ks, s, scale, zero16)) !=
        LOCAL_OK)
      return st;
  }
  return run_prefill(m, prefill_tile(T, K, G, p), s);
}

// Argument checks shared by the entry points (before any launch).
local_status_t check_args(const char* who, const uint16_t* x, int64_t T, int64_t K, int G,
                          const Proj* p, int32_t n_adapters, int32_t r_max,
                          const int32_t* adapter_idx, const float* scale, size_t* ws_bytes,
                          bool sizes_only) {
  if (!ws_bytes) return local_fail(LOCAL_ERR_WORKSPACE, "%s: ws_bytes is NULL", who);
  if (T < 0 || K <= 0 || n_adapters < 0)
    return local_fail(LOCAL_ERR_SHAPE, "%s: T=%lld K=%lld n_adapters=%d", who, (long long)T,
                      (long long)K, n_adapters);
  for (int g = 0; g < G; ++g)
    if (p[g].N <= 0)
      return local_fail(LOCAL_ERR_SHAPE, "%s: N=%lld (projection %d)", who, (long long)p[g].N, g);
  bool shapes_ok = K % 64 == 0 && n_adapters <= 256 &&
                   (n_adapters == 0 || (r_max >= 8 && r_max <= 128 && r_max % 8 == 0));
  for (int g = 0; g < G; ++g) shapes_ok = shapes_ok && p[g].N % 64 == 0;
  if (!shapes_ok)
    return local_fail(LOCAL_ERR_UNSUPPORTED,
                      "%s: K=%lld n_adapters=%d r_max=%d (need K and every N %% 64 == 0, "
                      "n_adapters <= 256, r_max in [8,128] and %% 8 == 0)",
                      who, (long long)K, n_adapters, r_max);
  if (sizes_only || T == 0) return LOCAL_OK;
  if (!x) return local_fail(LOCAL_ERR_NULL, "%s: NULL x", who);
  for (int g = 0; g < G; ++g) {
    if (!p[g].W || !p[g].y) return local_fail(LOCAL_ERR_NULL, "%s: NULL W or y", who);
    if (n_adapters > 0 && (!p[g].A || !p[g].B))
      return local_fail(LOCAL_ERR_NULL, "%s: NULL adapter argument", who);
  }
  if (n_adapters > 0 && (!adapter_idx || !scale))
    return local_fail(LOCAL_ERR_NULL, "%s: NULL adapter argument", who);
  return LOCAL_OK;
}

}  // namespace

}  // namespace localk

using namespace localk;

extern "C" local_status_t local_lora_linear(
    const uint16_t* x, int64_t T, int64_t K, const uint16_t* W, int64_t N, const uint16_t* A,
    const uint16_t* B, int32_t n_adapters, int32_t r_max, const int32_t* ranks,
    const int32_t* adapter_idx, const float* scale, const uint16_t* residual, uint16_t* y,
    void* ws, size_t* ws_bytes, void* stream) {
  const Proj p{W, N, A, B, ranks, residual, y};
  local_status_t st = check_args("lora_linear", x, T, K, 1, &p, n_adapters, r_max, adapter_idx,
                                 scale, ws_bytes, ws == nullptr);
  if (st != LOCAL_OK) return st;
  return lora_impl(x, T, K, 1, &p, n_adapters, r_max, adapter_idx, scale, ws, ws_bytes,
                   static_cast<hipStream_t>(stream));
}

extern "C" local_status_t local_lora_linear_grouped(
    const uint16_t* x, int64_t T, int64_t K, int32_t G, const uint16_t* const* W,
    const int64_t* N, const uint16_t* const* A, const uint16_t* const* B, int32_t n_adapters,
    int32_t r_max, const int32_t* const* ranks, const int32_t* adapter_idx, const float* scale,
    uint16_t* const* y, void* ws, size_t* ws_bytes, void* stream) {
  if (G < 1 || G > kMaxGroup)
    return local_fail(LOCAL_ERR_UNSUPPORTED, "lora_linear_grouped: G=%d (need 1..%d)", G,
                      kMaxGroup);
  if (!W || !N || !y || (n_adapters > 0 && (!A || !B)))
    return local_fail(LOCAL_ERR_NULL, "lora_linear_grouped: NULL argument array");
  Proj p[kMaxGroup];
  for (int g = 0; g < G; ++g)
    p[g] = Proj{W[g], N[g], n_adapters > 0 ? A[g] : nullptr, n_adapters > 0 ? B[g] : nullptr,
                (n_adapters > 0 && ranks) ? ranks[g] : nullptr, nullptr, y[g]};
  local_status_t st = check_args("lora_linear_grouped", x, T, K, G, p, n_adapters, r_max,
                                 adapter_idx, scale, ws_bytes, ws == nullptr);
  if (st != LOCAL_OK) return st;
  return lora_impl(x, T, K, G, p, n_adapters, r_max, adapter_idx, scale, ws, ws_bytes,
                   static_cast<hipStream_t>(stream));
}
