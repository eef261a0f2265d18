// Batched prefill of T tokens through one layer.
//
// The paper's measurements cover generated tokens only (Sec. 5.1); this path
// runs a prompt's tokens through the same MoE layer at once, with the same
// per-token arithmetic, and lets the cache see the whole batch's routing:
//
//   1. gate    Z = H W_g^T in fp64 (exact products, fp64 sums), top-K per
//              token, renormalised softmax weights, x = h / rms(h) in bf16
//   2. plan    histogram of the T*K (token, rank) pairs by expert, exclusive
//              scan, scatter into expert-sorted order; the cache table takes
//              the batch at once: counts += per-expert routings, the clock
//              ticks once per pair, then the S highest-ranked experts stay
//              resident (LFU: count; aged LFU: the count aged to the batch's
//              last tick; LRU: last use; ties: resident first, lower id);
//              kept experts keep their slots, newcomers take the
//              freed slots in ascending order
//   3. experts grouped GEMMs (MFMA bf16, fp32 accumulate) on experts resident
//              at the start, while the copy stream streams every other routed
//              expert (into its new slot, or a staging ring) followed by the
//              grouped GEMMs on those; the host schedules them from the plan,
//              except with a slot for every expert, where the plan kernel
//              writes the GEMM tiles itself
//   4. unpermute  h_t += sum_r g_tr Y[pos(t, r)] in rank order (no atomics)
//
// The gate GEMM and the grouped GEMMs are dense contractions, so they run on
// the matrix cores: the gate on the fp64 ones (exact products, fp64 sums),
// the expert GEMMs (rows = pairs routed to one expert) on bf16 ones: tiles of
// up to 256 rows (gemm.hip), or the small-M kernel here for groups of few
// rows.
#include "common.hpp"
#include "moe_offload.h"

#include <algorithm>
#include <cmath>

namespace moe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int kGateTok = kRouteTok;  // tokens per gate and route workgroup

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float silu(float v) { return v / (1.0f + __expf(-v)); }

// ---------------------------------------------------------------------------
// 1. gate logits, top-K, combine weights, normalised bf16 rows
//
// Z = H W_g^T is a dense T x E x d contraction kept in fp64 (every bf16 x fp32
// product is exact there), so it runs on the fp64 matrix cores:
// v_mfma_f64_16x16x4_f64, A = 16 tokens x 4 columns, B = 4 columns x 16
// experts; lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and gets
// back D[l / 16 + 4 v][l % 16], v = 0..3.
//
// A workgroup takes 16 tokens and one of `splits` ranges of columns, so that
// small batches still fill the chip, and leaves its partial logits in memory;
// the route kernel adds the ranges in order.  Its eight waves are the groups
// of 16 experts times cw shares of the columns: lane (i, kq) = (lane % 16,
// lane / 16) of a wave loads columns 8 kq .. + 7 of token row i and of expert
// row 16 g + i of each 32-column block, and MFMA step s uses column 8 kq + s
// of both, so A and B always pair the same column.  The column shares of a
// group meet in LDS and are added in order.
//
// Bound by latency below some 500 tokens and by the fp64 matrix rate (13.7 us
// at 4096 tokens) above.  d 2048, 64 experts, us in the trace, one kernel of a
// workgroup per 16 tokens before / gate + route now: 32 tokens 35.8 / 5.3 +
// 11.6, 509 tokens 37 / 9.3 + 12.1, 4096 tokens 40-47 / 29-39 + 12-16.  A whole
// batch with d_ff 64 (plan and GEMMs included): 86, 131, 282 before, 51, 73,
// 233 now.
constexpr int kGateWaves = 8;
constexpr int kGateThreads = kGateWaves * kWave;
constexpr int kGateAhead = 4;      // 32-column blocks in flight per wave
constexpr int kGateCols = 32;      // columns of a block

struct GateBlock {
  float4 h[2];  // 8 columns of this lane's token row
  uint4 w;      // 8 bf16 columns of its expert row
};

// (batches run on bf16 models only, so the gate is bf16)
template <bool RAGGED>
__global__ __launch_bounds__(kGateThreads) void prefill_gate_kernel(PrefillArgs a) {
  __shared__ double zp[kGateWaves][kGateTok][16];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int d = a.d, E = a.E;
  const int i = lane % 16, kq = lane / 16;
  const int t0 = blockIdx.x * kGateTok, split = blockIdx.y;
  const int ng = (E + 15) / 16, cw = kGateWaves / ng;  // expert groups, column shares
  const int g = wave % ng, cs = wave / ng;
  // blocks of this range, dealt round-robin to the column shares
  const int nb = (d + kGateCols - 1) / kGateCols;
  const int b0 = nb * split / a.splits, b1 = nb * (split + 1) / a.splits;
  const bool live = cs < cw;
  double4_t acc[2] = {};
  if (live) {
    // rows past T and experts past E read the last valid one: logits nobody reads
    const float *hrow = a.H + (size_t)min(t0 + i, a.T - 1) * d;
    const uint8_t *wrow = static_cast<const uint8_t *>(a.gate) + (size_t)min(16 * g + i, E - 1) * d * 2;
    GateBlock buf[kGateAhead];
    auto load = [&](GateBlock &b, int blk) {
      // unconditional (past the range: its last block again, unused); a
      // ragged d reads its last 8 columns instead of columns past the end
      const int k = min(min(blk, b1 - 1) * kGateCols + 8 * kq, RAGGED ? d - 8 : d);
      b.h[0] = *reinterpret_cast<const float4 *>(hrow + k);
      b.h[1] = *reinterpret_cast<const float4 *>(hrow + k + 4);
      b.w = *reinterpret_cast<const uint4 *>(wrow + (size_t)k * 2);
    };
    auto mul = [&](const GateBlock &b, int blk) {
      const bool in = !RAGGED || blk * kGateCols + 8 * kq < d;
      float h[8] = {b.h[0].x, b.h[0].y, b.h[0].z, b.h[0].w, b.h[1].x, b.h[1].y, b.h[1].z, b.h[1].w}, w[8];
      bf16x8_to_f32(b.w, w);
#pragma unroll
      for (int s = 0; s < 8; ++s)
        acc[s & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)h[s] : 0.0, in ? (double)w[s] : 0.0, acc[s & 1], 0, 0, 0);
    };
    // this wave's blocks: first, first + cw, ...; straight-line main loop, the
    // last blocks, which load nothing, peeled off
    const int first = b0 + cs, n = first < b1 ? (b1 - first + cw - 1) / cw : 0;
#pragma unroll
    for (int u = 0; u < kGateAhead; ++u) load(buf[u], first + u * cw);
    int j = 0;
    for (; j + kGateAhead < n; j += kGateAhead) {
#pragma unroll
      for (int u = 0; u < kGateAhead; ++u) {
        mul(buf[u], first + (j + u) * cw);
        load(buf[u], first + (j + u + kGateAhead) * cw);
        __builtin_amdgcn_sched_barrier(0);  // keep each refill next to its block
      }
    }
#pragma unroll
    for (int u = 0; u < kGateAhead; ++u)
      if (j + u < n) mul(buf[u], first + (j + u) * cw);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) zp[wave][kq + 4 * v][i] = acc[0][v] + acc[1][v];
  __syncthreads();
  for (int x = tid; x < kGateTok * kMaxE; x += kGateThreads) {
    const int r = x / kMaxE, e = x % kMaxE;
    if (e < E && t0 + r < a.T) {
      double z = zp[e / 16][r][e % 16];
      for (int c = 1; c < cw; ++c) z += zp[c * ng + e / 16][r][e % 16];
      a.zpart[((size_t)split * a.T + t0 + r) * kMaxE + e] = z;
    }
  }
}

// One wave per token of a block: the partial logits added in order, rms in
// fp64, top-K by rank counting, renormalised softmax weights and the
// normalised bf16 row; a block's 16 tokens also leave how many of them chose
// each expert and the last (token, rank) pair that did, from which the plan
// kernel's workgroups find their places without passing over all pairs.  The
// row's loads are issued first and stay in registers up to 256 * NV columns.
// With TB blocks a wave takes one token of each, side by side: the chain of a
// token's steps is latency, which the other fills.
template <int TB>
struct RouteShared {
  double zs[TB][kGateTok][kMaxE];
  int top[TB][kGateTok][kMaxK];
  int cnt[TB][kMaxE], last[TB][kMaxE];
};

template <int NV, int TB>
__device__ __forceinline__ void route_blocks(const PrefillArgs &a, int blk0, RouteShared<TB> &sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int d = a.d, E = a.E, K = a.K;
  for (int x = tid; x < TB * kMaxE; x += kGateTok * kWave) {
    sh.cnt[x / kMaxE][x % kMaxE] = 0;
    sh.last[x / kMaxE][x % kMaxE] = 0;
  }
  __syncthreads();
  int t[TB];
  bool live[TB];  // the same for the whole wave
  const float *row[TB];
#pragma unroll
  for (int q = 0; q < TB; ++q) {
    t[q] = (blk0 + q) * kGateTok + wave;
    live[q] = t[q] < a.T;
    row[q] = a.H + (size_t)min(t[q], a.T - 1) * d;  // past T: the last token again, unused
  }
  if (live[0]) {  // blocks are in token order: with none in the first there is none in the second
    float4 v[TB][NV];
#pragma unroll
    for (int q = 0; q < TB; ++q)
#pragma unroll
      for (int u = 0; u < NV; ++u) v[q][u] = *reinterpret_cast<const float4 *>(row[q] + min(u * 256 + lane * 4, d - 4));
    const size_t zstride = (size_t)a.T * kMaxE;
    constexpr int kAhead = 8;  // partial logits in flight (clamped past the last, unused)
    const double *zr0[TB];
    double zv[TB][kAhead], z[TB];
#pragma unroll
    for (int q = 0; q < TB; ++q) {
      zr0[q] = a.zpart + (size_t)min(t[q], a.T - 1) * kMaxE + min(lane, E - 1);
#pragma unroll
      for (int u = 0; u < kAhead; ++u) zv[q][u] = zr0[q][min(u, a.splits - 1) * zstride];
      z[q] = zv[q][0];
    }
    for (int s0 = 0; s0 < a.splits; s0 += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
#pragma unroll
        for (int q = 0; q < TB; ++q) {
          if (s0 + u > 0) z[q] += s0 + u < a.splits ? zv[q][u] : 0.0;
          zv[q][u] = zr0[q][min(s0 + u + kAhead, a.splits - 1) * zstride];
        }
    }
#pragma unroll
    for (int q = 0; q < TB; ++q) sh.zs[q][wave][lane] = z[q];
    auto square = [](double &sq, const float4 &x) {
      sq = fma((double)x.x, (double)x.x, sq);
      sq = fma((double)x.y, (double)x.y, sq);
      sq = fma((double)x.z, (double)x.z, sq);
      sq = fma((double)x.w, (double)x.w, sq);
    };
    double rr[TB];
#pragma unroll
    for (int q = 0; q < TB; ++q) {
      double sq = 0.0;
#pragma unroll
      for (int u = 0; u < NV; ++u)
        if (u * 256 + lane * 4 < d) square(sq, v[q][u]);
      for (int c = NV * 256 + lane * 4; c < d; c += 256) square(sq, *reinterpret_cast<const float4 *>(row[q] + c));
      rr[q] = sqrt(lane_value_d(wave_sum_d_to_lane63(sq), kWave - 1) / (double)d + 1e-5);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const double *zq[TB];
    int *tq[TB], mine[TB];
#pragma unroll
    for (int q = 0; q < TB; ++q) {
      zq[q] = sh.zs[q][wave];
      tq[q] = sh.top[q][wave];
    }
    wave_topk_lds<TB>(zq, E, K, lane, tq, mine);
#pragma unroll
    for (int q = 0; q < TB; ++q) {
      const double zr = lane < K ? zq[q][mine[q]] : 0.0;
      const double z0 = lane_value_d(zr, 0);
      const double ex = lane < K ? exp((zr - z0) / rr[q]) : 0.0;
      const double den = lane_value_d(wave_sum_d_to_lane63(ex), kWave - 1);
      if (live[q] && lane < K) {
        a.ids[(size_t)t[q] * K + lane] = mine[q];
        a.g[(size_t)t[q] * K + lane] = (float)(ex / den);
        atomicAdd(&sh.cnt[q][mine[q]], 1);
        atomicMax(&sh.last[q][mine[q]], wave * K + lane);
      }
    }
#pragma unroll
    for (int q = 0; q < TB; ++q) {
      if (!live[q]) continue;
      const float inv = (float)(1.0 / rr[q]);
      uint16_t *xr = a.xn + (size_t)t[q] * d;
      auto put = [&](const float4 &x, int c) {
        uint2 o;
        o.x = (uint32_t)f32_to_bf16_rne(x.x * inv) | ((uint32_t)f32_to_bf16_rne(x.y * inv) << 16);
        o.y = (uint32_t)f32_to_bf16_rne(x.z * inv) | ((uint32_t)f32_to_bf16_rne(x.w * inv) << 16);
        *reinterpret_cast<uint2 *>(xr + c) = o;
      };
#pragma unroll
      for (int u = 0; u < NV; ++u)
        if (u * 256 + lane * 4 < d) put(v[q][u], u * 256 + lane * 4);
      for (int c = NV * 256 + lane * 4; c < d; c += 256) put(*reinterpret_cast<const float4 *>(row[q] + c), c);
    }
  }
  __syncthreads();
  for (int x = tid; x < TB * kMaxE; x += kGateTok * kWave) {
    const int q = x / kMaxE, e = x % kMaxE;
    if ((blk0 + q) * kGateTok >= a.T) break;
    a.blk_cnt[(size_t)(blk0 + q) * kMaxE + e] = (uint8_t)sh.cnt[q][e];   // at most 16: a token names an expert once
    a.blk_last[(size_t)(blk0 + q) * kMaxE + e] = (uint8_t)sh.last[q][e];  // below 16 * 16
  }
}

template <int NV>
__global__ __launch_bounds__(kGateTok *kWave) void prefill_route_kernel(PrefillArgs a) {
  __shared__ RouteShared<1> sh;
  route_blocks<NV, 1>(a, blockIdx.x, sh);
}

// ---------------------------------------------------------------------------
// 2. sort by expert and update the layer's table for the whole batch
//
// A counting sort over the route kernel's per-block counts.  Every workgroup
// adds up all of them (64 bytes a block of 16 tokens), which gives it the
// experts' totals and how many pairs of each lie before its own blocks, and
// then places its own pairs (LDS atomics that return the position).  Positions
// within a workgroup's share follow the atomics' order, which varies from run
// to run; nothing downstream depends on it, since every row of the grouped
// GEMMs is computed alone and the combine reads each (token, rank) pair
// through pos_of.  Workgroup 0 also updates the table.  32768 pairs of 64
// experts: 26-32 us by one workgroup passing twice
// over the pairs, 12-15 so.
constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kPlanAhead = 8;  // blocks' counts in flight per wave

struct PlanShared {
  int part[3][kPlanWaves][kMaxE];  // totals, totals before this share, last pair + 1
  int cnt[kMaxE], cur[kMaxE], lastp[kMaxE], offs[kMaxE];
  // tile lists (when a.ntiles): cost of each row-block size, the expert's
  // first tile and rows per tile in each list, the lists' lengths
  float tcost[2][kWideRows / 32];
  int tfirst[2][kMaxE], trows[2][kMaxE], tlen[2];
  const uint16_t *tw[kMaxE];  // the experts' weights (when a.tiles)
  int bad;
};

// Lane e's view of the layer's table, and the trace's length: what the plan
// needs that no other kernel of the batch writes.
struct PlanTable {
  int slot0, pf;
  uint32_t count;
  int64_t last, clock0, token0;
  uint64_t tbase;
};

__device__ __forceinline__ PlanTable plan_table(const PlanArgs &a, bool keeper) {
  const LayerTable *T = a.table;
  const int le = min((int)(threadIdx.x & (kWave - 1)), a.E - 1);
  PlanTable p{};
  p.slot0 = T->expert_slot[le];
  if (keeper) {
    p.count = T->count[le];
    p.last = T->last[le];
    p.pf = T->pf[le];
    p.clock0 = T->clock;
    p.token0 = T->lookups;
    p.tbase = *a.trace_in;
  }
  return p;
}

// Share g of G of the plan; pt loaded before (keeper: g == 0, first wave).
__device__ __forceinline__ void plan_share(const PlanArgs &a, int g, int G, const PlanTable &pt, PlanShared &sh) {
  auto &part = sh.part;
  auto &cnt = sh.cnt;
  auto &cur = sh.cur;
  auto &lastp = sh.lastp;
  auto &offs = sh.offs;
  auto &tcost = sh.tcost;
  auto &tfirst = sh.tfirst;
  auto &trows = sh.trows;
  auto &tlen = sh.tlen;
  auto &tw = sh.tw;
  int &bad = sh.bad;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int E = a.E, P = a.T * a.K;
  const int nblk = (a.T + kGateTok - 1) / kGateTok;
  const int b0 = (int)((long)nblk * g / G), b1 = (int)((long)nblk * (g + 1) / G);
  LayerTable *T = a.table;
  const bool in_range = lane < E;
  const bool keeper = wave == 0 && g == 0;  // the wave that updates the table
  int slot0 = pt.slot0, pf = pt.pf;
  uint32_t count = pt.count;
  int64_t last = pt.last;
  const int64_t clock0 = pt.clock0, token0 = pt.token0;
  const uint64_t tbase = pt.tbase;
  // the first of this share's ids and the blocks' counts
  const int p_lo = b0 * kGateTok * a.K, p_hi = min(P, b1 * kGateTok * a.K);
  const int id0 = p_lo < p_hi ? a.ids[min(p_lo + tid, p_hi - 1)] : 0;
  if (tid == 0) bad = 0;
  int tot = 0, before = 0, lp = 0;
  for (int b = wave; b < nblk; b += kPlanAhead * kPlanWaves) {
    int c[kPlanAhead], l[kPlanAhead];
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
      const size_t at = (size_t)min(b + u * kPlanWaves, nblk - 1) * kMaxE + lane;
      c[u] = a.blk_cnt[at];
      l[u] = g == 0 ? a.blk_last[at] : 0;  // only the table needs it
    }
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
      const int bu = b + u * kPlanWaves;
      const int n = bu < nblk ? c[u] : 0;
      tot += n;
      before += bu < b0 ? n : 0;
      lp = n > 0 ? max(lp, bu * kGateTok * a.K + l[u] + 1) : lp;
    }
  }
  part[0][wave][lane] = tot;
  part[1][wave][lane] = before;
  part[2][wave][lane] = lp;
  __syncthreads();
  if (wave == 0) {
    int n = 0, bf = 0, l = 0;
#pragma unroll
    for (int w = 0; w < kPlanWaves; ++w) {
      n += part[0][w][lane];
      bf += part[1][w][lane];
      l = max(l, part[2][w][lane]);
    }
    int incl = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int v = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += v;
    }
    cnt[lane] = n;
    lastp[lane] = l;
    offs[lane] = incl - n;
    cur[lane] = incl - n + bf;
    if (a.tiles) {
      // every expert has a slot from the warm start on, so its slot is the
      // same before and after the batch; no tile is ever made without one
      const bool ok = !in_range || (slot0 >= 0 && slot0 < a.S);
      tw[lane] = in_range && ok ? reinterpret_cast<const uint16_t *>(a.arena_layer + (size_t)slot0 * a.slot_bytes) : nullptr;
      if (!ok) bad = 1;
    }
  }
  __syncthreads();
  // place this share's pairs
  for (int p = p_lo + tid; p < p_hi; p += kPlanThreads) {
    const int e = p == p_lo + tid ? id0 : a.ids[p];
    if (e < 0 || e >= E) {  // cannot happen: the route kernel ranks experts 0 .. E - 1
      *a.err = ERR_BAD_LIST;
      continue;
    }
    const int pos = atomicAdd(&cur[e], 1);
    a.perm_tok[pos] = p / a.K;
    a.pos_of[p] = pos;
  }
  if (a.ntiles) {
    if (wave >= 1 && wave <= kWideRows / 32) {
      // wave w: what the lists cost with row blocks of at most 32 w rows
      const int n = in_range ? cnt[lane] : 0;
      const int per = n > 0 ? tile_rows(n, 32 * wave) : 32;
      int nt = (n + per - 1) / per, blocks = nt * (per / 32);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        nt += __shfl_xor(nt, o, kWave);
        blocks += __shfl_xor(blocks, o, kWave);
      }
      if (lane < 2) {
        const TileList &tl = lane == 0 ? a.up : a.dn;
        const int r = 32 * wave;
        tcost[lane][wave - 1] = r >= tl.lo && r <= tl.hi ? tile_cost(tl, nt, blocks) : __builtin_inff();
      }
    }
    __syncthreads();
    if (wave < 2) {
      // wave li: expert e's tiles of list li, nt row blocks in each column
      // block, and the list's first tile of each expert
      const int li = wave;
      const TileList &tl = li == 0 ? a.up : a.dn;
      const int c = in_range ? cnt[lane] : 0;
      int best = kWideRows / 32 - 1;
      for (int w = kWideRows / 32 - 2; w >= 0; --w) best = tcost[li][w] < tcost[li][best] ? w : best;
      const int per = c > 0 ? tile_rows(c, 32 * (best + 1)) : 32;
      const int mine = (c + per - 1) / per * tl.cb;
      int it = mine;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int v = __shfl_up(it, o, kWave);
        if (lane >= o) it += v;
      }
      trows[li][lane] = per;
      tfirst[li][lane] = it - mine;
      if (lane == kWave - 1) {
        const bool fits = it <= tl.cap && !bad;  // the host's bound holds for any counts
        tlen[li] = fits ? it : 0;
        if (g == 0) {
          a.ntiles[li] = tlen[li];
          if (!fits) *a.err = ERR_BAD_LIST;
        }
      }
    }
    __syncthreads();
    // tile i of a list belongs to the last expert whose first tile is <= i
    const int nup = tlen[0], n_all = tlen[0] + tlen[1];
    for (int i = g * kPlanThreads + tid; i < n_all; i += G * kPlanThreads) {
      const int list = i < nup ? 0 : 1;
      const int li = list == 0 ? i : i - nup;
      int lo = 0, hi = E - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (tfirst[list][mid] <= li)
          lo = mid;
        else
          hi = mid - 1;
      }
      const int per = trows[list][lo], nt = (cnt[lo] + per - 1) / per;
      const int k = li - tfirst[list][lo];
      const int cb = k / nt, mb = k - cb * nt;
      a.tiles[(list == 0 ? a.up.first : a.dn.first) + li] =
          GemmTile{tw[lo], offs[lo] + mb * per, min(per, cnt[lo] - mb * per), cb * (list == 0 ? a.up.cols : a.dn.cols),
                   nt == 1};
    }
  }
  if (a.tiles && a.small && keeper && in_range) {
    a.tiles[lane] = GemmTile{tw[lane], offs[lane], bad ? 0 : cnt[lane], 0, 1};
    if (bad) *a.err = ERR_BAD_LIST;
  }
  if (!keeper) return;

  // table update: lane e = expert e
  if (!in_range) {
    slot0 = -1;
    count = 0;
    last = 0;
    pf = 0;
  }
  const int n = in_range ? cnt[lane] : 0;
  const bool res_start = slot0 >= 0;
  count += (uint32_t)n;
  if (in_range && lastp[lane] > 0) last = clock0 + lastp[lane];
  const int64_t clock1 = clock0 + (int64_t)P;  // the batch's last tick

  // R*: the S highest-ranked experts, by the policy's value, then residency
  // at the batch's start, then the lower id.  Lane e counts the experts that
  // rank above it (a strict order, so the ranks are 0 .. E - 1 and S <= E of
  // them are kept).
  const uint64_t k1 = a.policy == 1   ? (uint64_t)count
                      : a.policy == 2 ? (uint64_t)aged_count(count, last, clock1, a.aging)
                                      : (uint64_t)(last + (1ll << 40));
  const int k2 = res_start ? 1 : 0;
  int above = 0;
  for (int j = 0; j < (a.S < E ? E : 0); ++j) {  // with a slot for every expert all are kept
    const uint64_t o1 = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(k1 >> 32), j) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)k1, j);
    const int o2 = __builtin_amdgcn_readlane(k2, j);
    above += (o1 > k1 || (o1 == k1 && (o2 > k2 || (o2 == k2 && j < lane)))) ? 1 : 0;
  }
  const bool chosen = in_range && above < a.S;
  const bool newcomer = chosen && !res_start;
  const bool evicted = res_start && !chosen;
  // freed slots (ascending) are handed to newcomers (ascending id)
  unsigned long long freed = evicted ? (1ull << slot0) : 0ull;
  if (a.S < E)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) freed |= __shfl_xor(freed, o, kWave);
  const unsigned long long newmask = __ballot(newcomer);
  int slot1 = evicted ? -1 : slot0;
  int victim = -1;
  const int n_new = __popcll(newmask);
  unsigned long long fm = freed, nm = newmask;
  for (int i = 0; i < n_new; ++i) {
    const int s = __ffsll((long long)fm) - 1;
    const int e = __ffsll((long long)nm) - 1;
    fm &= fm - 1;
    nm &= nm - 1;
    const unsigned long long owner = __ballot(slot0 == s);
    if (lane == e) {
      slot1 = s;
      victim = owner ? __ffsll((long long)owner) - 1 : -1;
    }
  }
  const bool fetched = in_range && ((n > 0 && !res_start) || newcomer);
  int useful = 0, wasted = 0;
  if (pf) {
    if (n > 0)
      useful = 1;
    else
      wasted = 1;
  }
  const int hits = res_start ? n : 0;
  int all_hits = hits;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) all_hits += __shfl_xor(all_hits, o, kWave);
  const int sm = P - all_hits;  // every pair is a hit or a miss
  const int su = __popcll(__ballot(useful)), sw = __popcll(__ballot(wasted)), sf = __popcll(__ballot(fetched));
  if (in_range) {
    T->expert_slot[lane] = slot1;
    T->count[lane] = count;
    T->last[lane] = last;
    T->pf[lane] = 0;
    if (newcomer) T->slot_expert[slot1] = lane;
    PrefillPlan pl;
    pl.n = n;
    pl.off = offs[lane];
    pl.slot_start = slot0;
    pl.slot_after = slot1;
    pl.newcomer = newcomer ? 1 : 0;
    pl.pad[0] = pl.pad[1] = pl.pad[2] = 0;
    a.plan[lane] = pl;
    if (a.trace && a.trace_cap) {
      TraceRec r;
      r.kind = REC_PREFILL;
      r.token = (int32_t)token0;
      r.layer = a.layer;
      r.rank = n;
      r.expert = lane;
      r.flags = (res_start ? 1 : 0) | (chosen ? 2 : 0) | (fetched ? 4 : 0);
      r.slot = slot1;
      r.victim = newcomer ? victim : -1;
      a.trace[(tbase + lane) % a.trace_cap] = r;
    }
  }
  if (lane == 0) {
    T->clock = clock1;
    T->lookups = token0 + a.T;
    *a.trace_out = tbase + (a.trace && a.trace_cap ? (uint64_t)E : 0);
    LayerStats *st = a.stats;
    st->v[ST_HITS] += all_hits;
    st->v[ST_MISSES] += sm;
    st->v[ST_EVICT] += n_new;
    st->v[ST_PF_USEFUL] += su;
    st->v[ST_PF_WASTED] += sw;
    st->v[ST_LOOKUPS] += a.T;
    st->v[ST_BYTES] += (uint64_t)sf * a.expert_bytes;
  }
}

__global__ __launch_bounds__(kPlanThreads) void prefill_plan_kernel(PlanArgs a) {
  __shared__ PlanShared sh;
  const PlanTable pt = plan_table(a, threadIdx.x < kWave && blockIdx.x == 0);
  plan_share(a, blockIdx.x, gridDim.x, pt, sh);
}

// Both for a batch of one or two blocks of a narrow model, in one workgroup:
// such batches are bound by launches.  us with one launch / two: 16 tokens of
// 15 experts of d 256 40.8 / 42.2, of 32 of d 1024 45.7 / 47.0, of 64 of d 2048
// 82.8 / 83.4; 24 tokens of 4 experts of d 1024 34.7 / 42.1, of 32 of d 256
// 38.9 / 42.6.  Two blocks cost more there than in workgroups of their own
// (eight layers in turn, where the host keeps ahead: 4 experts of d 1024 238 /
// 231 us, 32 of d 256 268 / 253), with many experts more than the launch saves
// (64 of d 256 44.2 / 42.4 and 330 / 297); one after the other they cost 48.7
// and 364 there.  Rows of more than 2048 columns do not fit
// the registers of a 1024-thread workgroup: held all the same they spill (16
// tokens of 8 experts of d 4096 66.4 us), read again they cost more than the
// launch saves (57.9 / 56.8; d 8192 89.8 / 87.9).  Two blocks of 1025 to 2048
// columns cost 2 to 4 us more in one launch, which only pays where the experts
// are so small that the host is behind (24 tokens: 4 experts of 1440 x 864, 28
// MiB, 40.0 / 41.8; 8 of 2048 x 1024, 96 MiB, 49.2 / 46.9).
constexpr bool route_plan_in_one(int blocks, int d, int E, uint64_t expert_bytes) {
  return (blocks == 1 && d <= 2048) ||
         (blocks == 2 && E <= 32 && (d <= 1024 || (d <= 2048 && E * expert_bytes <= (32u << 20))));
}
static_assert(kPlanThreads == kGateTok * kWave, "one workgroup does both");

template <int NV, int TB>
__global__ __launch_bounds__(kPlanThreads) void prefill_route_plan_kernel(PrefillArgs a, PlanArgs p) {
  __shared__ RouteShared<TB> rs;
  __shared__ PlanShared ps;
  const PlanTable pt = plan_table(p, threadIdx.x < kWave);
  route_blocks<NV, TB>(a, 0, rs);
  __syncthreads();  // the blocks' ids and counts are written
  plan_share(p, 0, 1, pt, ps);
}

// ---------------------------------------------------------------------------
// 3. grouped GEMMs.  A rows come from the sorted pair order; B = expert
// weights stored out x in (K contiguous), so both operands are K-major.

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const uint16_t *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, bytes, 0x00020000);
}

typedef uint32_t gemm_u32x4 __attribute__((ext_vector_type(4)));  // a 16-byte slice as a register value

__device__ __forceinline__ gemm_u32x4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(gemm_u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 0));
}

// Small-M grouped GEMM: launches whose experts have few rows (batched decode;
// which ones: small_m in the engine).  A workgroup owns 16 output features of
// one expert for all of its rows: one 16-row MFMA block, or two where it has 17
// to 32 rows.  Its four waves split K in four; each streams its quarter of the
// 16 weight rows (of W1 and W3 in the up projection) from global memory
// straight into v_mfma_f32_16x16x32_bf16 fragments, several 32-deep steps
// ahead, with the rows' activations read alongside (from L2: every workgroup of
// the expert reads them).  A row or feature past the end reads a valid row
// instead (its outputs are not written); only a K tail that is not a multiple
// of 32 is zeroed.  The four partial products meet in LDS and are added in wave
// order.
constexpr int kSkinnyAheadUp = 8, kSkinnyAheadDown = 8;  // steps in flight per wave

__device__ __forceinline__ bf16x8 load_frag(const uint16_t *p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const gemm_u32x4 *>(p));
}

__device__ __forceinline__ bf16x8 load_frag(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(bf16x8, buffer_load16(r, byte_off));
}

// One tile of at most 16 * RB rows by the 16 features of block fb.
template <bool UP, int AHEAD, int RB>
__device__ __forceinline__ void skinny_tile(const GemmTile &t, int fb, const uint16_t *a_src, const int32_t *perm_tok,
                                            void *out, int d, int d_ff, floatx4 (*red)[UP ? 2 : 1][RB][kWave]) {
  constexpr int NB = UP ? 2 : 1;  // B matrices: W1 and W3, or W2
  const int K = UP ? d : d_ff;  // reduction length
  const int N = UP ? d_ff : d;  // output features
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int M = min(t.rows, 16 * RB);
  const int kg = (lane / 16) * 8;  // this lane's 8 elements of a 32-deep step
  // A rows (tokens of the expert) and B row (feature) of this lane, clamped
  const uint16_t *ap[RB];
#pragma unroll
  for (int x = 0; x < RB; ++x) {
    const int m = t.row + min(16 * x + lane % 16, M - 1);
    ap[x] = (UP ? a_src + (size_t)perm_tok[m] * d : a_src + (size_t)m * d_ff) + kg;
  }
  // B rows: features fb * 16 .. + nf - 1 of each weight matrix, read with
  // buffer loads (the pointer comes from the tile list; flat loads would make
  // every wait drain all the loads in flight)
  const int nf = min(16, N - fb * 16);
  __amdgpu_buffer_rsrc_t brs[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
    brs[b] = rows_rsrc(t.w + (UP ? (size_t)b * d_ff * d : 2 * (size_t)d_ff * d) + (size_t)fb * 16 * K,
                       (uint32_t)nf * K * 2);
  const uint32_t boff = ((uint32_t)min(lane % 16, nf - 1) * K + kg) * 2;

  floatx4 c[NB][RB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int x = 0; x < RB; ++x) c[b][x] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

  // this wave's full 32-deep steps
  const int full = K / 32;
  const int q = (full + 3) / 4;
  const int s0 = min(wave * q, full), s1 = min(s0 + q, full);
  const int n = s1 - s0;
  bf16x8 wa[AHEAD][NB], xa[AHEAD][RB];
  // no load is conditional, so the compiler can count the loads in flight
  auto load = [&](int slot, int step) {
    const int k = step * 32;
#pragma unroll
    for (int b = 0; b < NB; ++b) wa[slot][b] = load_frag(brs[b], boff + 2 * k);
#pragma unroll
    for (int x = 0; x < RB; ++x) xa[slot][x] = load_frag(ap[x] + k);
  };
  auto mma = [&](int slot) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int x = 0; x < RB; ++x)
        c[b][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[slot][x], wa[slot][b], c[b][x], 0, 0, 0);
  };
  // straight-line main loop: a step past the wave's last reloads that step
  // (in bounds, never used); the last steps, which load nothing, are peeled
  if (n > 0) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load(u, s0 + min(u, n - 1));
    int i = 0;
    for (; i + AHEAD < n; i += AHEAD) {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        mma(u);
        load(u, s0 + min(i + u + AHEAD, n - 1));
        __builtin_amdgcn_sched_barrier(0);  // keep each refill next to its step, not batched at the end
      }
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (i + u < n) mma(u);
  }
  // K tail (K not a multiple of 32): the last wave adds it, zeroing past K
  if (K % 32 && wave == 3) {
    const bool in = full * 32 + kg < K;
    const int k = in ? full * 32 : 0;  // lanes past K read their row's start, then take zeros
    const bf16x8 z = {};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bf16x8 v = load_frag(brs[b], boff + 2 * k);
      wa[0][b] = in ? v : z;
    }
#pragma unroll
    for (int x = 0; x < RB; ++x) {
      const bf16x8 v = load_frag(ap[x] + k);
      xa[0][x] = in ? v : z;
    }
    mma(0);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int x = 0; x < RB; ++x) red[wave][b][x][lane] = c[b][x];
  __syncthreads();
  if (wave == 0) {
    floatx4 r[NB][RB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int x = 0; x < RB; ++x) {
        r[b][x] = red[0][b][x][lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) r[b][x] += red[w][b][x][lane];
      }
    const int n_out = fb * 16 + lane % 16;
    if (n_out < N) {
#pragma unroll
      for (int x = 0; x < RB; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int mo = 16 * x + (lane / 16) * 4 + i;
          if (mo >= M) continue;
          if (UP)
            static_cast<uint16_t *>(out)[(size_t)(t.row + mo) * N + n_out] =
                f32_to_bf16_rne(silu(r[0][x][i]) * r[NB - 1][x][i]);
          else
            static_cast<float *>(out)[(size_t)(t.row + mo) * N + n_out] = r[0][x][i];
        }
    }
  }
}

template <bool UP, int AHEAD, int RB>
__global__ __launch_bounds__(256) void prefill_skinny_kernel(const GemmTile *tiles, const uint16_t *a_src,
                                                             const int32_t *perm_tok, void *out, int d, int d_ff) {
  constexpr int NB = UP ? 2 : 1;
  __shared__ floatx4 red[4 * NB * RB * kWave];
  const int N = UP ? d_ff : d;  // output features
  const int nfb = (N + 15) / 16;
  const int ti = blockIdx.x / nfb, fb = blockIdx.x - ti * nfb;
  const GemmTile t = tiles[ti];
  if (t.rows <= 0) return;  // an expert without rows
  if (RB == 1 || t.rows <= 16)
    skinny_tile<UP, AHEAD, 1>(t, fb, a_src, perm_tok, out, d, d_ff, reinterpret_cast<floatx4 (*)[NB][1][kWave]>(red));
  else
    skinny_tile<UP, AHEAD, RB>(t, fb, a_src, perm_tok, out, d, d_ff, reinterpret_cast<floatx4 (*)[NB][RB][kWave]>(red));
}

// ---------------------------------------------------------------------------
// 4. h_t += sum_r g_tr Y[pos(t, r)], ranks in order
constexpr int kUnpermRanks = 8;  // ranks whose rows are loaded before the first is added
constexpr int kUnpermSteps = 2;  // four-column steps per lane and pass

__global__ __launch_bounds__(256) void prefill_unpermute_kernel(float *H, const float *Y, const float *g,
                                                                const int32_t *pos_of, int T, int d, int K) {
  const int t = blockIdx.x;
  if (t >= T) return;
  // A workgroup per token.  Every rank's row is loaded before the first is
  // added, so a pass waits for its positions once and for the rows once (one
  // rank after another, each wait was two trips to memory).  Loads are
  // clamped to a valid rank and column, so none waits behind a branch; ranks
  // are added in order, and a rank past K adds nothing (selected, not
  // multiplied by zero).
  for (int c0 = threadIdx.x * 4; c0 < d; c0 += kUnpermSteps * 256 * 4) {
    float4 y[kUnpermSteps], h[kUnpermSteps];
#pragma unroll
    for (int u = 0; u < kUnpermSteps; ++u) {
      y[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      h[u] = *reinterpret_cast<const float4 *>(H + (size_t)t * d + min(c0 + u * 1024, d - 4));
    }
    for (int r0 = 0; r0 < K; r0 += kUnpermRanks) {
      float4 v[kUnpermRanks][kUnpermSteps];
      float gr[kUnpermRanks];
#pragma unroll
      for (int i = 0; i < kUnpermRanks; ++i) {
        const int r = min(r0 + i, K - 1);
        gr[i] = g[(size_t)t * K + r];
        const float *yr = Y + (size_t)pos_of[(size_t)t * K + r] * d;
#pragma unroll
        for (int u = 0; u < kUnpermSteps; ++u)
          v[i][u] = *reinterpret_cast<const float4 *>(yr + min(c0 + u * 1024, d - 4));
      }
#pragma unroll
      for (int i = 0; i < kUnpermRanks; ++i) {
        const bool live = r0 + i < K;
#pragma unroll
        for (int u = 0; u < kUnpermSteps; ++u) {
          y[u].x = live ? fmaf(gr[i], v[i][u].x, y[u].x) : y[u].x;
          y[u].y = live ? fmaf(gr[i], v[i][u].y, y[u].y) : y[u].y;
          y[u].z = live ? fmaf(gr[i], v[i][u].z, y[u].z) : y[u].z;
          y[u].w = live ? fmaf(gr[i], v[i][u].w, y[u].w) : y[u].w;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kUnpermSteps; ++u) {
      const int c = c0 + u * 1024;
      if (c < d) {
        float4 o = h[u];
        o.x += y[u].x;
        o.y += y[u].y;
        o.z += y[u].z;
        o.w += y[u].w;
        *reinterpret_cast<float4 *>(H + (size_t)t * d + c) = o;
      }
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers used by the host engine
int prefill_gate_splits(int T, int d) {
  // about two workgroups a compute unit, each with at least 128 columns
  const int blocks = (T + kGateTok - 1) / kGateTok;
  return std::max(1, std::min((512 + blocks - 1) / blocks, d / 128));
}

hipError_t launch_prefill_gate(const PrefillArgs &a, const Launch &l) {
  const dim3 grid((a.T + kGateTok - 1) / kGateTok, a.splits);
  if (a.d % kGateCols != 0)
    MOE_LAUNCH((prefill_gate_kernel<true>), grid, dim3(kGateThreads), 0, l, a);
  else
    MOE_LAUNCH((prefill_gate_kernel<false>), grid, dim3(kGateThreads), 0, l, a);
  return hipGetLastError();
}

hipError_t launch_prefill_route_plan(const PrefillArgs &a, const PlanArgs &p, const Launch &l) {
  const int blocks = (a.T + kGateTok - 1) / kGateTok;
  if (route_plan_in_one(blocks, a.d, a.E, p.slot_bytes)) {
#define MOE_ROUTE(NV, TB) MOE_LAUNCH((prefill_route_plan_kernel<NV, TB>), dim3(1), dim3(kPlanThreads), 0, l, a, p)
    if (blocks == 2 && a.d <= 512)
      MOE_ROUTE(2, 2);
    else if (blocks == 2)
      MOE_ROUTE(4, 2);  // (columns past 1024 are read again: two rows of 2048 do not fit the registers)
    else if (a.d <= 512)
      MOE_ROUTE(2, 1);
    else if (a.d <= 1024)
      MOE_ROUTE(4, 1);
    else
      MOE_ROUTE(8, 1);
#undef MOE_ROUTE
    return hipGetLastError();
  }
#define MOE_ROUTE(NV) MOE_LAUNCH((prefill_route_kernel<NV>), dim3(blocks), dim3(kGateTok * kWave), 0, l, a)
  if (a.d <= 512)
    MOE_ROUTE(2);
  else if (a.d <= 1024)
    MOE_ROUTE(4);
  else if (a.d <= 2048)
    MOE_ROUTE(8);
  else
    MOE_ROUTE(16);
#undef MOE_ROUTE
  // one pair a thread or less in most batches; each workgroup of the plan
  // reads every block's counts, so there are at most 64
  const long pairs = (long)a.T * a.K;
  const int shares = (int)std::min<long>(64, (pairs + kPlanThreads - 1) / kPlanThreads);
  MOE_LAUNCH(prefill_plan_kernel, dim3(shares), dim3(kPlanThreads), 0, l, p);
  return hipGetLastError();
}

hipError_t launch_prefill_skinny_up(const GemmTile *tiles, int ntiles, int max_rows, const uint16_t *xn,
                                    const int32_t *perm_tok, uint16_t *act, int d, int d_ff, const Launch &l) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid(ntiles * ((d_ff + 15) / 16));
  if (max_rows > 16)
    MOE_LAUNCH((prefill_skinny_kernel<true, kSkinnyAheadUp, 2>), grid, dim3(256), 0, l, tiles, xn, perm_tok, (void *)act, d, d_ff);
  else
    MOE_LAUNCH((prefill_skinny_kernel<true, kSkinnyAheadUp, 1>), grid, dim3(256), 0, l, tiles, xn, perm_tok, (void *)act, d, d_ff);
  return hipGetLastError();
}

hipError_t launch_prefill_skinny_down(const GemmTile *tiles, int ntiles, int max_rows, const uint16_t *act, float *Y, int d,
                                      int d_ff, const Launch &l) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid(ntiles * ((d + 15) / 16));
  if (max_rows > 16)
    MOE_LAUNCH((prefill_skinny_kernel<false, kSkinnyAheadDown, 2>), grid, dim3(256), 0, l, tiles, act, nullptr, (void *)Y, d, d_ff);
  else
    MOE_LAUNCH((prefill_skinny_kernel<false, kSkinnyAheadDown, 1>), grid, dim3(256), 0, l, tiles, act, nullptr, (void *)Y, d, d_ff);
  return hipGetLastError();
}

hipError_t launch_prefill_unpermute(float *H, const float *Y, const float *g, const int32_t *pos_of, int T,
                                    int d, int K, const Launch &l) {
  MOE_LAUNCH(prefill_unpermute_kernel, dim3(T), dim3(256), 0, l, H, Y, g, pos_of, T, d, K);
  return hipGetLastError();
}

}  // namespace moe
