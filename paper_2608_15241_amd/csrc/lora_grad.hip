// local_lora_grad, local_lora_grad_input: the backward of the mixed-adapter
// LoRA projection, for the training chunks that update an agent's adapter
// while the frozen base serves (§2.2: adapters on a frozen base model; §4:
// background training in bounded chunks). With u_t = x_t A_a^T and
// g_t = s_t dy_t B_a (a = a_t, both over a's rank):
//   dB_a = sum_{t of a} s_t dy_t^T u_t,  dA_a = sum_{t of a} g_t^T x_t,
//   dx_t = dy_t W + g_t A_a.
//
// Design (HBM-bound for the adapter gradients: 4 T r (K + N) flop, shrinks
// included, against T (K + N) bf16 read), three launches (four above 2048 tokens):
//  * set-up: the tokens bucketed by adapter (a stable counting sort in one
//    workgroup, as in SGMV) while the other workgroups transpose B per
//    adapter to [r_max][N];
//  * u = x A^T and dy B for every projection in one launch (lora_shrink.hip);
//  * dB and dA as segmented outer products in one launch, each workgroup over
//    up to 2048 tokens of one adapter: sums of 64 tokens added in token order,
//    deterministic, no partial sums in memory, no atomics. A fourth launch adds
//    the sums of an adapter of more tokens.
//  dx runs the forward fused projection on the transposed weights: with
//  x := dy, W := W^T, A := B^T and B := A^T, its shrink is dy B and its
//  delta s (dy B) A, so dx needs no kernel of its own.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "lora_internal.hpp"

namespace localk {
namespace {

constexpr int kGrUnit = 64;      // tokens per unit of the segmented products
constexpr int kGrThreads = 256;
constexpr int kGrMaxAdapters = 256;
constexpr int kGrGroup = 4;            // projections of one x in a call
constexpr int kGrJobs = 2 * kGrGroup;  // (dB, dA) per projection

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

size_t al256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ int wave_incl_scan(int v) {
  const int lane = threadIdx.x % kWave;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int u = __shfl_up(v, off);
    if (lane >= off) v += u;
  }
  return v;
}

// ---- tokens bucketed by adapter, stable: perm[seg[a] .. seg[a+1]) holds the
// tokens of adapter a in ascending order, pscale their scales; tokens without
// one are left out.
// One workgroup of kPrepThreads: wave w owns a contiguous chunk of the
// tokens. It counts its chunk per adapter (ballots over equal adapters),
// then one prefix over (adapter, wave) gives every wave its own running
// offsets, and each wave places its chunk in order with no further barrier.
constexpr int kPrepThreads = 1024;
constexpr int kPrepWaves = kPrepThreads / kWave;

// The tokens of an adapter with more than few_tokens of them are also listed in
// spans of kGrSpan for the outer products: {adapter, first position, tokens,
// whether it is the adapter's only span}; an adapter of several spans in the
// list of those, {adapter, first span, spans, 0}.
constexpr int kGrSpan = 2048;

// Tokens up to which an adapter is not listed in spans (it does not change the
// result): one unit, or two in banks where adapters have fewer than two on average
// and the grid, which has room for every adapter that could be listed, matters
// more (with one unit / two: 512 tokens of 4 adapters at 1024 x 1024 18.0 / 21.7 us,
// 2048 of 64 at 4096 x 4096 97.5 / 95.2, 512 of 64 57.4 / 56.0).
int few_tokens(int64_t T, int n_ad) {
  return n_ad >= 16 && T < 2 * kGrUnit * n_ad ? 2 * kGrUnit : kGrUnit;
}

// The most entries of either list.
int64_t max_spans(int64_t T, int n_ad) {
  return T / kGrSpan + std::min<int64_t>(n_ad, T / (few_tokens(T, n_ad) + 1));
}
int64_t max_long(int64_t T, int n_ad) { return std::min<int64_t>(n_ad, T / (kGrSpan + 1)); }

struct Buckets {
  int32_t* perm;   // [T]
  float* pscale;   // [T]
  int32_t* seg;    // [n_ad + 1]
  int32_t* n_list; // entries of spans and of longs
  i32x4 *spans, *longs;
  int few;         // few_tokens
};

__device__ void bucket_tokens(const int32_t* __restrict__ idx, int64_t T, int n_ad,
                              const float* __restrict__ scale, const Buckets& bk) {
  int32_t* __restrict__ perm = bk.perm;
  float* __restrict__ pscale = bk.pscale;
  int32_t* __restrict__ seg = bk.seg;
  __shared__ int cnt[kPrepWaves][kGrMaxAdapters];  // per wave: count, then running offset
  __shared__ int tot[kGrMaxAdapters];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int64_t chunk = (T + kPrepWaves * kWave - 1) / (kPrepWaves * kWave) * kWave;
  const int64_t c0 = wave * chunk, c1 = min(T, c0 + chunk);
  auto adapter_at = [&](int64_t t) {
    const int32_t v = t < c1 ? idx[t] : -1;
    return (v >= 0 && v < n_ad) ? v : -1;
  };
  for (int a = lane; a < n_ad; a += kWave) cnt[wave][a] = 0;
  // 1. counts of the wave's chunk (lane 0 writes the wave's own row)
  for (int64_t t0 = c0; t0 < c1; t0 += kWave) {
    const int my = adapter_at(t0 + lane);
    uint64_t pending = __ballot(my >= 0);
    while (pending) {
      const int ad = __builtin_amdgcn_readlane(my, __ffsll(static_cast<long long>(pending)) - 1);
      const uint64_t m = __ballot(my == ad);
      if (lane == 0) cnt[wave][ad] += __popcll(m);
      pending &= ~m;
    }
  }
  __syncthreads();
  // 2. per adapter totals; prefixes over adapters (wave 0); each wave's
  //    first position per adapter
  for (int a = tid; a < n_ad; a += kPrepThreads) {
    int c = 0;
    for (int w = 0; w < kPrepWaves; ++w) c += cnt[w][a];
    tot[a] = c;
  }
  __syncthreads();
  if (wave == 0) {
    int run = 0, run_span = 0, run_long = 0;
    for (int a0 = 0; a0 < n_ad; a0 += kWave) {
      const int a = a0 + lane;
      const int c = a < n_ad ? tot[a] : 0;
      const int ic = wave_incl_scan(c);
      const int ns = c > bk.few ? (c + kGrSpan - 1) / kGrSpan : 0;
      const int is = wave_incl_scan(ns);
      const uint64_t several = __ballot(ns > 1);
      const int s0 = run + ic - c, sp0 = run_span + is - ns;
      if (a < n_ad) {
        seg[a] = s0;
        tot[a] = s0;
      }
      for (int i = 0; i < ns; ++i)
        bk.spans[sp0 + i] = i32x4{a, s0 + i * kGrSpan, min(kGrSpan, c - i * kGrSpan), ns == 1};
      if (ns > 1)
        bk.longs[run_long + __popcll(several & ((1ull << lane) - 1ull))] = i32x4{a, sp0, ns, 0};
      run += __shfl(ic, kWave - 1);
      run_span += __shfl(is, kWave - 1);
      run_long += __popcll(several);
    }
    if (lane == 0) {
      seg[n_ad] = run;
      bk.n_list[0] = run_span;
      bk.n_list[1] = run_long;
    }
  }
  __syncthreads();
  for (int a = tid; a < n_ad; a += kPrepThreads) {
    int off = tot[a];
    for (int w = 0; w < kPrepWaves; ++w) {
      const int c = cnt[w][a];
      cnt[w][a] = off;
      off += c;
    }
  }
  __syncthreads();
  // 3. the wave places its chunk in order
  for (int64_t t0 = c0; t0 < c1; t0 += kWave) {
    const int my = adapter_at(t0 + lane);
    const float sc = my >= 0 ? scale[t0 + lane] : 0.f;
    uint64_t pending = __ballot(my >= 0);
    while (pending) {
      const int ad = __builtin_amdgcn_readlane(my, __ffsll(static_cast<long long>(pending)) - 1);
      const uint64_t m = __ballot(my == ad);
      const int base = cnt[wave][ad];
      if (my == ad) {
        const int at = base + __popcll(m & ((1ull << lane) - 1ull));
        perm[at] = static_cast<int32_t>(t0 + lane);
        pscale[at] = sc;
      }
      if (lane == 0) cnt[wave][ad] = base + __popcll(m);
      pending &= ~m;
    }
  }
}

// ---- per-matrix transposes dst[i][c][r] = src[i][r][c] of n matrices of
// R x C bf16 (R and C multiples of 8). A tile of TR x TC (at most 2048
// elements) goes through LDS: 16-byte loads along the source rows, 16-byte
// stores along the destination rows.
struct TransposeJob {
  const uint16_t* src;
  uint16_t* dst;
  int64_t R, C;
  int TR, TC, tiles_c, tiles;
};

TransposeJob transpose_job(const uint16_t* src, uint16_t* dst, int64_t n, int64_t R,
                           int64_t C) {
  TransposeJob j{src, dst, R, C, 0, 0, 0, 0};
  if (R < C) {
    j.TR = static_cast<int>(std::min<int64_t>(R, 64));
    j.TC = 2048 / j.TR / 8 * 8;
  } else {
    j.TC = static_cast<int>(std::min<int64_t>(C, 64));
    j.TR = 2048 / j.TC / 8 * 8;
  }
  j.tiles_c = static_cast<int>((C + j.TC - 1) / j.TC);
  j.tiles = j.tiles_c * static_cast<int>((R + j.TR - 1) / j.TR) * static_cast<int>(n);
  return j;
}

// Tile k of job j (tiles of matrix 0 first, then of matrix 1, ...), by the
// 256 threads of quarter q of the workgroup; every thread of the workgroup
// calls it (the barrier is shared), a quarter without a tile with live false.
__device__ void transpose_tile(const TransposeJob& j, int k, bool live) {
  __shared__ __attribute__((aligned(16))) uint16_t tiles[kPrepThreads / kGrThreads][4096];
  const int q = threadIdx.x / kGrThreads;
  uint16_t* tile = tiles[q];  // TR x (TC + 8)
  const int TR = j.TR, TC = j.TC, ld = TC + 8;
  const int per_mat = j.tiles_c * static_cast<int>((j.R + TR - 1) / TR);
  const int64_t i = live ? k / per_mat : 0;
  const int kk = live ? k % per_mat : 0;
  const int64_t r0 = static_cast<int64_t>(kk / j.tiles_c) * TR;
  const int64_t c0 = static_cast<int64_t>(kk % j.tiles_c) * TC;
  const uint16_t* s = j.src + i * j.R * j.C;
  uint16_t* d = j.dst + i * j.R * j.C;
  const int e8 = (threadIdx.x % kGrThreads) * 8;
  if (live && e8 < TR * TC) {
    const int rr = e8 / TC, cc = e8 % TC;
    if (r0 + rr < j.R && c0 + cc < j.C)
      *reinterpret_cast<u32x4*>(tile + rr * ld + cc) =
          ld_global<u32x4>(s + (r0 + rr) * j.C + c0 + cc);
  }
  __syncthreads();
  if (live && e8 < TR * TC) {
    const int cc = e8 / TR, rr = e8 % TR;
    if (c0 + cc < j.C && r0 + rr < j.R) {
      uint32_t w[4];
#pragma unroll
      for (int h = 0; h < 4; ++h)
        w[h] = static_cast<uint32_t>(tile[(rr + 2 * h) * ld + cc]) |
               (static_cast<uint32_t>(tile[(rr + 2 * h + 1) * ld + cc]) << 16);
      *reinterpret_cast<u32x4*>(d + (c0 + cc) * j.R + r0 + rr) = u32x4{w[0], w[1], w[2], w[3]};
    }
  }
}

// One launch for the set-up work, workgroups of kPrepThreads: workgroup 0
// buckets the tokens (when idx is given); each other workgroup transposes
// four tiles (one per quarter) of one job, the jobs one after another.
struct PrepArgs {
  TransposeJob job[kGrGroup];
  int n_jobs;
  const int32_t* idx;
  const float* scale;
  int64_t T;
  int n_ad;
  Buckets bk;
};

__global__ __launch_bounds__(kPrepThreads) void grad_prep_kernel(PrepArgs a) {
  constexpr int per = kPrepThreads / kGrThreads;
  int wg = blockIdx.x;
  if (a.idx) {
    if (wg == 0) {
      bucket_tokens(a.idx, a.T, a.n_ad, a.scale, a.bk);
      return;
    }
    --wg;
  }
  // the job of this workgroup (each job's tiles fill whole workgroups)
  int q = 0;
  while (q + 1 < a.n_jobs && wg >= (a.job[q].tiles + per - 1) / per) {
    wg -= (a.job[q].tiles + per - 1) / per;
    ++q;
  }
  const int k = wg * per + static_cast<int>(threadIdx.x) / kGrThreads;
  transpose_tile(a.job[q], k, k < a.job[q].tiles);
}

local_status_t run_prep(hipStream_t s, const PrepArgs& a) {
  constexpr int per = kPrepThreads / kGrThreads;
  int wgs = a.idx ? 1 : 0;
  for (int q = 0; q < a.n_jobs; ++q) wgs += (a.job[q].tiles + per - 1) / per;
  if (wgs == 0) return LOCAL_OK;
  grad_prep_kernel<<<static_cast<unsigned>(wgs), kPrepThreads, 0, s>>>(a);
  return local_check_launch("lora_grad (prep)");
}

// ---- segmented outer products, every gradient of the call in one launch:
// blockIdx.y = job: 2g = dB of projection g (V = dy_g, P = N_g, coefficients
// s u_g, out [n_ad][P][r_max]), 2g + 1 = dA of projection g (V = x, P = K,
// coefficients g_g = s dy_g B_g, out [n_ad][r_max][P]).
//
// Bound by the reads of V. D[j][p] += c^T V on v_mfma_f32_16x16x32_bf16 over 32
// tokens: a lane loads 4 consecutive columns of its 8 tokens, and byte
// permutes turn the 8 rows into the operands of 4 columns. V is bf16; a
// float32 coefficient is cut by truncation into three bf16 parts that add up
// to it exactly, one product each: 6 MFMAs of 16 cycles per column tile and 64
// tokens, where v_mfma_f32_16x16x4_f32 takes 16 of 32 cycles (2048 tokens, q,
// k and v at 4096 x 4096 and rank 16: 24.0 us against 34.7). Every product is
// exact in float32 either way and the sums are float32; against float64 the
// gradients are 1.6e-7 off (2.1e-7 with the float32 instruction). The bf16
// instruction drops results below 2^-126, so the products run 2^24 times too
// large: what it drops is then less than half the smallest float32.
//
// A workgroup takes one span of an adapter's tokens for one column tile, its
// four waves every fourth unit of 64 tokens; after each round their tiles are
// added through LDS in unit order to sums that stay in registers until the
// span's last unit, so no partial sum goes through memory (with a workgroup per
// unit, the partial sums of 2048 tokens at 4096 x 4096 x 3 were 56 MB written and
// read back: 43 us and a 10.8 us reduce launch). An adapter of few tokens or none
// gives each wave a column tile instead, which keeps its sum in LDS (a bank's
// unused adapters only have zeros to write): 256 adapters in runs of 512 tokens
// 150 us, 199 with every workgroup on one tile. Which of the two follows from the
// adapter's own tokens, whatever the size of the bank: 2048 tokens of one adapter
// of 64 take 76 us (128 with the waves per tile chosen by the bank's tokens per
// adapter), and 33 at 1024 x 1024 (103).
//
// Spans of 2048 tokens: one workgroup over all of an adapter's tokens left the
// chip idle where the columns are few (32768 tokens of one adapter at 256 x 256 x 3:
// 24 workgroups, 257 us). The sums of an adapter of several spans go through
// memory, in 2048-token pieces, and a reduce launch adds them in order. Units
// are added in order within a span and spans in order, whatever the launch.
struct OuterArgs {
  const uint16_t* V[kGrJobs];
  const float* S[kGrJobs];  // low-rank products [T][r_max], unscaled
  float* out[kGrJobs];
  float* part[kGrJobs];     // sums of the spans of adapters with several
  int64_t P[kGrJobs];
  const int32_t* ranks[kGrJobs];  // the projection's ranks, or NULL
  Buckets bk;
  int n_jobs, n_ad;
  int tiles4;     // groups of four column tiles of the widest job
  int max_spans;  // items of spans; those of adapters of few tokens follow
  int r_max;
};

constexpr int kGrWaves = kGrThreads / kWave;
constexpr int kGrCols = 4;  // columns per lane (E below)
constexpr float kUp = 0x1p24f, kDown = 0x1p-24f;

template <int JT>
__global__ __launch_bounds__(kGrThreads) void grad_outer_kernel(OuterArgs args) {
  constexpr int E = kGrCols;
  constexpr int RJ = 16 * JT, CW = 16 * E;  // rank rows and columns of a tile
  constexpr int kLaneTok = kGrUnit / 4;  // tokens of a unit in a lane's group
  constexpr int kSums = JT * E / kGrWaves;  // f32x4 of sums per thread
  static_assert(JT * E % kGrWaves == 0, "sums per thread");
  // a wave's tile in LDS: [RJ][CW + 4] for dA, [CW][RJ + 4] for dB
  constexpr int TILE_A = RJ * (CW + 4), TILE_B = CW * (RJ + 4);
  constexpr int TILE = TILE_A > TILE_B ? TILE_A : TILE_B;
  __shared__ __attribute__((aligned(16))) float tl[kGrWaves][TILE];
  __shared__ __attribute__((aligned(16))) int tok[kGrWaves][2][kGrUnit];
  __shared__ __attribute__((aligned(16))) float tsc[kGrWaves][2][kGrUnit];  // times kUp
  __shared__ float tf[kGrWaves];  // what undoes that in a wave's tile
  using RowT = u32x2;

  // The workgroup's item: a span, or (`single`) an adapter of few tokens, four of
  // these in place of one span. Items vary slowest, so that those that turn out
  // empty come after those with work: between them they would leave the work
  // unevenly over the compute units (2048 tokens of one adapter 24.5 -> 29 us).
  // Every branch is uniform.
  const int jx = blockIdx.y, n_jobs = args.n_jobs;
  const int jbase = jx < n_jobs ? 0 : 64;  // ranks above 64: 64 rows at a time
  const int job = jx < n_jobs ? jx : jx - n_jobs;
  const bool single = static_cast<int>(blockIdx.z) >= args.max_spans;
  const int waves = single ? 1 : kGrWaves;  // that share a tile
  int i = blockIdx.z, tg = blockIdx.x;      // the span or adapter; its (group of) column tiles
  if (single) {
    const int t4 = args.tiles4, q = (tg >= t4) + (tg >= 2 * t4) + (tg >= 3 * t4);
    i = kGrWaves * (i - args.max_spans) + q;
    tg -= q * t4;
    if (i >= args.n_ad) return;
  }

  const int64_t P = args.P[job];
  const int r_max = args.r_max;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = lane % 16, k = lane / 16;
  // its tokens [s0, s0 + count) of adapter a, the wave's column tile and first
  // unit, and where the result goes
  const int64_t wcol = static_cast<int64_t>(single ? tg * kGrWaves + wave : tg) * CW;
  const int uw = single ? 0 : wave;
  int a, s0, count;
  float* out = args.out[job];
  if (single) {
    a = i;
    s0 = args.bk.seg[i];
    count = args.bk.seg[i + 1] - s0;
    if (count > args.bk.few || static_cast<int64_t>(tg) * kGrWaves * CW >= P) return;
    out += static_cast<int64_t>(a) * P * r_max;
  } else {
    const int n_spans = args.bk.n_list[0];
    const i32x4 e = args.bk.spans[i];  // (beside the count: not one after the other)
    if (i >= n_spans || wcol >= P) return;
    a = e[0];
    s0 = e[1];
    count = e[2];
    out = e[3] ? out + static_cast<int64_t>(a) * P * r_max
               : args.part[job] + static_cast<int64_t>(i) * P * r_max;
  }
  const int64_t col = wcol + E * n;  // this lane's columns
  const bool live = col < P;
  const int32_t* ranks = args.ranks[job];
  const int rk = ranks ? min(max(ranks[a], 0), r_max) : r_max;
  const int units = (count + kGrUnit - 1) / kGrUnit;
  const uint16_t* V = args.V[job];
  const float* S = args.S[job];

  f32x4 sum[kSums];
#pragma unroll
  for (int q = 0; q < kSums; ++q) sum[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // 4 consecutive floats of a tile from element e of the output order on
  auto lds_at = [&](int w, int e) {
    if (job & 1) return &tl[w][(e / CW) * (CW + 4) + e % CW];
    return &tl[w][(e / RJ) * (RJ + 4) + e % RJ];
  };

  // Token ids and scales of the wave's unit of round r, in slot r % 2. Past
  // the unit's tokens the last one repeats (masked below).
  auto unit_tokens = [&](int u0, int* tk, float* ts) {
    const int left = count - kGrUnit * (u0 + uw);
    if (left <= 0) return;
    const int at = s0 + kGrUnit * (u0 + uw) + min(lane, left - 1);
    *tk = args.bk.perm[at];
    *ts = args.bk.pscale[at];
  };
  auto put_tokens = [&](int slot, int tk, float ts) {
    tok[wave][slot][lane] = tk;
    tsc[wave][slot][lane] = ts * kUp;
  };
  const uint16_t* Vc = V + (live ? col : P - E);  // columns past P: never stored
  int jc[JT];
  bool jok[JT];  // at or past the rank: A's padding rows may hold anything
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    jc[jt] = min(jbase + 16 * jt + n, r_max - 1);
    jok[jt] = jbase + 16 * jt + n < rk;
  }
  // the lane's tokens of a unit: 32 h + 8 k + i (h < 2, i < 8) at 8 h + i
  RowT raw[kLaneTok];
  float c[JT][kLaneTok];
  auto load_half = [&](int slot, int h) {
#pragma unroll
    for (int i4 = 0; i4 < 8; i4 += 4) {
      const i32x4 tv = *reinterpret_cast<const i32x4*>(&tok[wave][slot][32 * h + 8 * k + i4]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t t = tv[q];
        raw[8 * h + i4 + q] = ld_global<RowT>(Vc + t * P);
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) c[jt][8 * h + i4 + q] = S[t * r_max + jc[jt]];
      }
    }
  };
  int tk = 0;
  float ts = 0.f;
  if (uw < units) {
    unit_tokens(0, &tk, &ts);
    put_tokens(0, tk, ts);
    unit_tokens(waves, &tk, &ts);
    load_half(0, 0);
    load_half(0, 1);
  }
  for (int u0 = 0, slot = 0; u0 < units; u0 += waves, slot ^= 1) {
    const int unit = u0 + uw;
    if (unit < units) {
      const int nt = min(kGrUnit, count - kGrUnit * unit);
      f32x4 acc[JT][E];
#pragma unroll
      for (int jt = 0; jt < JT; ++jt)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[jt][e] = f32x4{0.f, 0.f, 0.f, 0.f};
      const bool more = unit + waves < units;  // uniform
      if (more) {
        put_tokens(slot ^ 1, tk, ts);
        unit_tokens(u0 + 2 * waves, &tk, &ts);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // operands of the half's 32 tokens: element i of column e from the
        // i-th row; the coefficients' three bf16 parts
        if (nt < kGrUnit) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const bool in = 32 * h + 8 * k + i < nt;
            raw[8 * h + i] = in ? raw[8 * h + i] : u32x2{0u, 0u};
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) c[jt][8 * h + i] = in ? c[jt][8 * h + i] : 0.f;
          }
        }
        u32x4 vf[E];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
          for (int e = 0; e < E; ++e)
            vf[e][d] = __builtin_amdgcn_perm(raw[8 * h + 2 * d + 1][e / 2], raw[8 * h + 2 * d][e / 2],
                                             e & 1 ? 0x07060302u : 0x05040100u);
        float sv[8];
#pragma unroll
        for (int i = 0; i < 8; i += 4) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(&tsc[wave][slot][32 * h + 8 * k + i]);
#pragma unroll
          for (int q = 0; q < 4; ++q) sv[i + q] = v[q];
        }
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          u32x4 cf[3];
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            uint32_t part[2][3];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const float cs = jok[jt] ? c[jt][8 * h + 2 * d + q] * sv[2 * d + q] : 0.f;
              part[q][0] = __float_as_uint(cs);
              const float r1 = cs - __uint_as_float(part[q][0] & 0xffff0000u);
              part[q][1] = __float_as_uint(r1);
              part[q][2] =
                  __float_as_uint(r1 - __uint_as_float(part[q][1] & 0xffff0000u));
            }
#pragma unroll
            for (int m = 0; m < 3; ++m)
              cf[m][d] = __builtin_amdgcn_perm(part[1][m], part[0][m], 0x07060302u);
          }
#pragma unroll
          for (int m = 2; m >= 0; --m)
#pragma unroll
            for (int e = 0; e < E; ++e)
              acc[jt][e] = mfma16x16x32(as_bf16x8(cf[m]), as_bf16x8(vf[e]), acc[jt][e]);
        }
        if (more) load_half(slot ^ 1, h);
      }
      float zero[4] = {0.f, 0.f, 0.f, 0.f};  // NaN once a value is infinite or NaN
#pragma unroll
      for (int jt = 0; jt < JT; ++jt)
#pragma unroll
        for (int e = 0; e < E; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i) zero[i] += acc[jt][e][i] * 0.f;
      const float all = (zero[0] + zero[1]) + (zero[2] + zero[3]);
      float down = kDown;
      if (__any(all != all)) {
        // a value of the unit is not finite (the parts of a coefficient then
        // mix infinities with zeros) or too large to scale, so the unit runs
        // again as float32 products (16x16x4: lane l gives token l / 16)
        down = 1.f;
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
          for (int e = 0; e < E; ++e) acc[jt][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int i = k; i < kGrUnit; i += 4) {
          const bool in = i < nt;
          const int64_t t = tok[wave][slot][i];
          const float st = args.bk.pscale[s0 + kGrUnit * unit + min(i, nt - 1)];
          const RowT r = ld_global<RowT>(Vc + t * P);
#pragma unroll
          for (int jt = 0; jt < JT; ++jt) {
            const float cs = in && jok[jt] ? S[t * r_max + jc[jt]] * st : 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const uint32_t w = in ? r[e / 2] : 0u;
              const float v = __uint_as_float(e & 1 ? w & 0xffff0000u : w << 16);
              acc[jt][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs, v, acc[jt][e], 0, 0, 0);
            }
          }
        }
      }
      if (lane == 0) tf[wave] = down;
      float* w = tl[wave];
      // a wave that has the tile alone keeps the sum there
      auto put = [&](float* p, f32x4 v) {
        if (single) {
          v *= down;
          if (u0) v += *reinterpret_cast<const f32x4*>(p);
        }
        *reinterpret_cast<f32x4*>(p) = v;
      };
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const int j0 = 16 * jt + 4 * k;  // this lane's rows j0 .. j0 + 3
        if (job & 1) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < E; e += 4)
              put(w + (j0 + i) * (CW + 4) + E * n + e,
                  f32x4{acc[jt][e][i], acc[jt][e + 1][i], acc[jt][e + 2][i], acc[jt][e + 3][i]});
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e)
            put(w + (E * n + e) * (RJ + 4) + j0, acc[jt][e]);
        }
      }
    }
    __syncthreads();
    if (single) continue;
#pragma unroll
    for (int v = 0; v < kGrWaves; ++v)
      if (u0 + v < units) {
        const float f = tf[v];
#pragma unroll
        for (int q = 0; q < kSums; ++q)
          sum[q] += *reinterpret_cast<const f32x4*>(lds_at(v, 4 * (tid + q * kGrThreads))) * f;
      }
    if (u0 + waves < units) __syncthreads();  // the tiles are rewritten by the next round
  }

  // out: zero at or past the rank (and for an adapter without tokens)
  auto store = [&](int e, f32x4 v) {
    if (job & 1) {
      const int j = jbase + e / CW;
      const int64_t p = wcol + e % CW;
      if (j < r_max && p < P)
        *reinterpret_cast<f32x4*>(out + static_cast<int64_t>(j) * P + p) =
            j < rk ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
      const int j = jbase + e % RJ;
      const int64_t p = wcol + e / RJ;
      if (j < r_max && p < P) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (j + i >= rk) v[i] = 0.f;
        *reinterpret_cast<f32x4*>(out + p * r_max + j) = v;
      }
    }
  };
  if (single) {  // each wave its own tile
#pragma unroll
    for (int q = 0; q < JT * E; ++q) {
      const int e = 4 * (lane + q * kWave);
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (units) v = *reinterpret_cast<const f32x4*>(lds_at(wave, e));
      store(e, v);
    }
  } else {
#pragma unroll
    for (int q = 0; q < kSums; ++q) store(4 * (tid + q * kGrThreads), sum[q]);
  }
}

// The sums of an adapter's spans, added in order.
__global__ __launch_bounds__(kGrThreads) void grad_reduce_kernel(OuterArgs args) {
  if (static_cast<int>(blockIdx.y) >= args.bk.n_list[1]) return;
  const i32x4 l = args.bk.longs[blockIdx.y];
  const int job = blockIdx.z;
  const int64_t elems = args.P[job] * args.r_max;
  const int64_t e = 4 * (static_cast<int64_t>(blockIdx.x) * kGrThreads + threadIdx.x);
  if (e >= elems) return;
  const float* p = args.part[job] + l[1] * elems + e;
  f32x4 v = *reinterpret_cast<const f32x4*>(p);
  for (int i = 1; i < l[2]; ++i) v += *reinterpret_cast<const f32x4*>(p + i * elems);
  *reinterpret_cast<f32x4*>(args.out[job] + l[0] * elems + e) = v;
}

template <int JT>
local_status_t launch_outer_jt(OuterArgs o, int n_jobs, int64_t T, int n_ad, hipStream_t s) {
  int64_t pmax = 0;
  for (int q = 0; q < n_jobs; ++q) pmax = std::max(pmax, o.P[q]);
  constexpr int64_t cols = 16 * kGrCols;
  o.tiles4 = static_cast<int>((pmax + kGrWaves * cols - 1) / (kGrWaves * cols));
  o.n_jobs = n_jobs;
  o.n_ad = n_ad;
  o.max_spans = static_cast<int>(max_spans(T, n_ad));
  const dim3 grid(static_cast<unsigned>(kGrWaves * o.tiles4),
                  static_cast<unsigned>(n_jobs * ((o.r_max + 63) / 64)),
                  static_cast<unsigned>(o.max_spans + (n_ad + kGrWaves - 1) / kGrWaves));
  if (grid.z > 65535)
    return local_fail(LOCAL_ERR_UNSUPPORTED, "lora_grad: T=%lld", (long long)T);
  grad_outer_kernel<JT><<<grid, kGrThreads, 0, s>>>(o);
  const local_status_t st = local_check_launch("lora_grad (outer)");
  const int64_t longs = max_long(T, n_ad);
  if (st != LOCAL_OK || longs == 0) return st;
  const int64_t threads = pmax * o.r_max / 4;
  grad_reduce_kernel<<<dim3(static_cast<unsigned>((threads + kGrThreads - 1) / kGrThreads),
                            static_cast<unsigned>(longs), static_cast<unsigned>(n_jobs)),
                       kGrThreads, 0, s>>>(o);
  return local_check_launch("lora_grad (reduce)");
}

local_status_t launch_outer(const OuterArgs& o, int n_jobs, int64_t T, int n_ad,
                            hipStream_t s) {
  if (o.r_max <= 16) return launch_outer_jt<1>(o, n_jobs, T, n_ad, s);
  if (o.r_max <= 32) return launch_outer_jt<2>(o, n_jobs, T, n_ad, s);
  return launch_outer_jt<4>(o, n_jobs, T, n_ad, s);
}

local_status_t grad_checks(const char* who, int64_t T, int64_t K, int64_t N, int32_t n_ad,
                           int32_t r_max) {
  if (T < 0 || K <= 0 || N <= 0 || n_ad < 1)
    return local_fail(LOCAL_ERR_SHAPE, "%s: T=%lld K=%lld N=%lld n_adapters=%d", who,
                      (long long)T, (long long)K, (long long)N, n_ad);
  if (K % 64 || N % 64 || n_ad > kGrMaxAdapters || r_max < 8 || r_max > 128 || r_max % 8)
    return local_fail(LOCAL_ERR_UNSUPPORTED,
                      "%s: K=%lld N=%lld n_adapters=%d r_max=%d (need K, N %% 64 == 0, "
                      "n_adapters <= 256, r_max in [8,128] and %% 8 == 0)",
                      who, (long long)K, (long long)N, n_ad, r_max);
  return LOCAL_OK;
}

}  // namespace
}  // namespace localk

using namespace localk;

namespace localk {
namespace {

// Adapter gradients of G projections that share x (and the routing).
local_status_t grad_impl(const char* who, const uint16_t* x, int64_t T, int64_t K, int G,
                         const uint16_t* const* dy, const int64_t* N, const uint16_t* const* A,
                         const uint16_t* const* B, int32_t n_adapters, int32_t r_max,
                         const int32_t* const* ranks, const int32_t* adapter_idx,
                         const float* scale, float* const* dA, float* const* dB, void* ws,
                         size_t* ws_bytes, hipStream_t s) {
  if (!ws_bytes) return local_fail(LOCAL_ERR_WORKSPACE, "%s: ws_bytes is NULL", who);
  if (G < 1 || G > kGrGroup)
    return local_fail(LOCAL_ERR_UNSUPPORTED, "%s: G=%d (need 1..%d)", who, G, kGrGroup);
  local_status_t st;
  for (int g = 0; g < G; ++g)
    if ((st = grad_checks(who, T, K, N[g], n_adapters, r_max)) != LOCAL_OK) return st;
  const int64_t Tw = T > 0 ? T : 1;
  // workspace: token order, adapter offsets, the lists of spans, B_g^T, the
  // low-rank products u_g and dy_g B_g, the sums of spans
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += al256(bytes);
    return at;
  };
  const size_t o_perm = take(static_cast<size_t>(Tw) * 4);
  const size_t o_psc = take(static_cast<size_t>(Tw) * 4);
  const size_t o_seg = take(static_cast<size_t>(n_adapters + 1) * 4);
  const size_t o_list = take(2 * sizeof(int32_t));
  const int64_t n_spans = max_spans(Tw, n_adapters), n_longs = max_long(Tw, n_adapters);
  const size_t o_spans = take(static_cast<size_t>(n_spans) * sizeof(i32x4));
  const size_t o_longs = take(static_cast<size_t>(n_longs) * sizeof(i32x4));
  size_t o_bt[kGrGroup], o_u[kGrGroup], o_g[kGrGroup], o_pb[kGrGroup], o_pa[kGrGroup];
  for (int g = 0; g < G; ++g) {
    o_bt[g] = take(static_cast<size_t>(n_adapters) * r_max * N[g] * 2);
    o_u[g] = take(static_cast<size_t>(Tw) * r_max * 4);
    o_g[g] = take(static_cast<size_t>(Tw) * r_max * 4);
    o_pb[g] = take(n_longs > 0 ? static_cast<size_t>(n_spans) * N[g] * r_max * 4 : 0);
    o_pa[g] = take(n_longs > 0 ? static_cast<size_t>(n_spans) * K * r_max * 4 : 0);
  }
  // The size is the one that callers have always been told, which these parts
  // fit: token order, two lists of adapter offsets, 16 bytes for each of at
  // most T / 64 + n_adapters units, the B_g^T, the shrinks' sums over K slices,
  // and a partial product of every unit and gradient.
  const int64_t units = Tw / kGrUnit + n_adapters;
  auto sums = [&](int64_t k, int g) {
    return al256(static_cast<size_t>(g) * long_slices(Tw, k, r_max, g) * Tw * r_max * 4) +
           al256(static_cast<size_t>((Tw + 63) / 64) * 32);
  };
  size_t need = al256(static_cast<size_t>(Tw) * 4) +
                2 * al256(static_cast<size_t>(n_adapters + 1) * 4) + al256(units * 16) +
                al256(sums(K, G));
  for (int g = 0; g < G; ++g)
    need += al256(static_cast<size_t>(n_adapters) * r_max * N[g] * 2) + al256(sums(N[g], 1)) +
            al256(static_cast<size_t>(units) * N[g] * r_max * 4) +
            al256(static_cast<size_t>(units) * K * r_max * 4);
  need = std::max(need, o);
  if (!ws) {
    *ws_bytes = need;
    return LOCAL_OK;
  }
  if (*ws_bytes < need)
    return local_fail(LOCAL_ERR_WORKSPACE, "%s: workspace %zu < %zu", who, *ws_bytes, need);
  for (int g = 0; g < G; ++g) {
    if (!dA[g] || !dB[g]) return local_fail(LOCAL_ERR_NULL, "%s: NULL output", who);
    if (T > 0 && (!dy[g] || !A[g] || !B[g]))
      return local_fail(LOCAL_ERR_NULL, "%s: NULL pointer argument", who);
  }
  if (T > 0 && (!x || !adapter_idx || !scale))
    return local_fail(LOCAL_ERR_NULL, "%s: NULL pointer argument", who);
  char* w = static_cast<char*>(ws);
  const uint16_t* Bt[kGrGroup];
  // tokens bucketed by adapter and every B_g transposed per adapter to
  // [r_max][N_g], in one launch. T = 0: every adapter is empty and the outer
  // products write zero gradients (no memset: the call stays capturable)
  PrepArgs pr{};
  pr.n_jobs = T > 0 ? G : 0;
  for (int g = 0; g < G; ++g) {
    uint16_t* bt = reinterpret_cast<uint16_t*>(w + o_bt[g]);
    Bt[g] = bt;
    if (T > 0) pr.job[g] = transpose_job(B[g], bt, n_adapters, N[g], r_max);
  }
  pr.idx = adapter_idx ? adapter_idx : reinterpret_cast<const int32_t*>(w);  // not read if T = 0
  pr.T = T;
  pr.n_ad = n_adapters;
  pr.scale = scale;
  pr.bk = Buckets{reinterpret_cast<int32_t*>(w + o_perm), reinterpret_cast<float*>(w + o_psc),
                  reinterpret_cast<int32_t*>(w + o_seg), reinterpret_cast<int32_t*>(w + o_list),
                  reinterpret_cast<i32x4*>(w + o_spans), reinterpret_cast<i32x4*>(w + o_longs),
                  few_tokens(Tw, n_adapters)};
  if ((st = run_prep(s, pr)) != LOCAL_OK) return st;
  if (T > 0) {  // u_g = x A_g^T and dy_g B_g, one launch
    ShrinkJob jobs[kGrJobs];
    for (int g = 0; g < G; ++g) {
      jobs[g] = ShrinkJob{x, A[g], reinterpret_cast<float*>(w + o_u[g]), K, nullptr, nullptr};
      jobs[G + g] = ShrinkJob{dy[g], Bt[g], reinterpret_cast<float*>(w + o_g[g]), N[g], nullptr,
                              nullptr};
    }
    if ((st = token_shrink(jobs, 2 * G, T, n_adapters, r_max, adapter_idx, 1, s)) != LOCAL_OK)
      return st;
  }
  // dB_g from (dy_g, s u_g), dA_g from (x, s dy_g B_g)
  OuterArgs oa{};
  for (int g = 0; g < G; ++g) {
    const int32_t* rg = ranks ? ranks[g] : nullptr;
    oa.V[2 * g] = dy[g];
    oa.S[2 * g] = reinterpret_cast<const float*>(w + o_u[g]);
    oa.out[2 * g] = dB[g];
    oa.P[2 * g] = N[g];
    oa.ranks[2 * g] = rg;
    oa.part[2 * g] = reinterpret_cast<float*>(w + o_pb[g]);
    oa.part[2 * g + 1] = reinterpret_cast<float*>(w + o_pa[g]);
    oa.V[2 * g + 1] = x;
    oa.S[2 * g + 1] = reinterpret_cast<const float*>(w + o_g[g]);
    oa.out[2 * g + 1] = dA[g];
    oa.P[2 * g + 1] = K;
    oa.ranks[2 * g + 1] = rg;
  }
  oa.bk = pr.bk;
  oa.r_max = r_max;
  return launch_outer(oa, 2 * G, T, n_adapters, s);
}

}  // namespace
}  // namespace localk

extern "C" local_status_t local_lora_grad(
    const uint16_t* x, int64_t T, int64_t K, const uint16_t* dy, int64_t N, const uint16_t* A,
    const uint16_t* B, int32_t n_adapters, int32_t r_max, const int32_t* ranks,
    const int32_t* adapter_idx, const float* scale, float* dA, float* dB, void* ws,
    size_t* ws_bytes, void* stream) {
  return grad_impl("lora_grad", x, T, K, 1, &dy, &N, &A, &B, n_adapters, r_max, &ranks,
                   adapter_idx, scale, &dA, &dB, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

extern "C" local_status_t local_lora_grad_grouped(
    const uint16_t* x, int64_t T, int64_t K, int32_t G, const uint16_t* const* dy,
    const int64_t* N, const uint16_t* const* A, const uint16_t* const* B, int32_t n_adapters,
    int32_t r_max, const int32_t* const* ranks, const int32_t* adapter_idx, const float* scale,
    float* const* dA, float* const* dB, void* ws, size_t* ws_bytes, void* stream) {
  if (G < 1 || G > kGrGroup)
    return local_fail(LOCAL_ERR_UNSUPPORTED, "lora_grad_grouped: G=%d (need 1..%d)", G,
                      kGrGroup);
  if (!dy || !N || !A || !B || !dA || !dB)
    return local_fail(LOCAL_ERR_NULL, "lora_grad_grouped: NULL argument array");
  return grad_impl("lora_grad_grouped", x, T, K, G, dy, N, A, B, n_adapters, r_max, ranks,
                   adapter_idx, scale, dA, dB, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

extern "C" local_status_t local_lora_grad_input(
    const uint16_t* dy, int64_t T, int64_t N, const uint16_t* Wt, int64_t K, const uint16_t* A,
    const uint16_t* B, int32_t n_adapters, int32_t r_max, const int32_t* ranks,
    const int32_t* adapter_idx, const float* scale, uint16_t* dx, void* ws, size_t* ws_bytes,
    void* stream) {
  if (!ws_bytes) return local_fail(LOCAL_ERR_WORKSPACE, "lora_grad_input: ws_bytes is NULL");
  local_status_t st = grad_checks("lora_grad_input", T, K, N, n_adapters, r_max);
  if (st != LOCAL_OK) return st;
  // the forward projection of dy: x := dy [T][N], W := W^T [K][N],
  // A := B^T [n][r_max][N], B := A^T [n][K][r_max]
  const size_t o_bt = 0;
  const size_t o_at = o_bt + al256(static_cast<size_t>(n_adapters) * r_max * N * 2);
  const size_t o_fw = o_at + al256(static_cast<size_t>(n_adapters) * K * r_max * 2);
  size_t fw = 0;
  if ((st = local_lora_linear(nullptr, T, N, nullptr, K, nullptr, nullptr, n_adapters, r_max,
                              nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, &fw,
                              stream)) != LOCAL_OK)
    return st;
  const size_t need = o_fw + fw;
  if (!ws) {
    *ws_bytes = need;
    return LOCAL_OK;
  }
  if (*ws_bytes < need)
    return local_fail(LOCAL_ERR_WORKSPACE, "lora_grad_input: workspace %zu < %zu", *ws_bytes,
                      need);
  if (T == 0) return LOCAL_OK;
  if (!dy || !Wt || !A || !B || !adapter_idx || !scale || !dx)
    return local_fail(LOCAL_ERR_NULL, "lora_grad_input: NULL pointer argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* w = static_cast<char*>(ws);
  uint16_t* Bt = reinterpret_cast<uint16_t*>(w + o_bt);
  uint16_t* At = reinterpret_cast<uint16_t*>(w + o_at);
  PrepArgs pr{};
  pr.job[0] = transpose_job(B, Bt, n_adapters, N, r_max);
  pr.job[1] = transpose_job(A, At, n_adapters, r_max, K);
  pr.n_jobs = 2;
  if ((st = run_prep(s, pr)) != LOCAL_OK) return st;
  size_t rest = *ws_bytes - o_fw;
  return local_lora_linear(dy, T, N, Wt, K, Bt, At, n_adapters, r_max, ranks, adapter_idx,
                           scale, nullptr, dx, w + o_fw, &rest, stream);
}
