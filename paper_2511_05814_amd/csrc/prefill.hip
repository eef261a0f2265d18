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
//              writes the GEMM jobs and tiles itself
//   4. unpermute  h_t += sum_r g_tr Y[pos(t, r)] in rank order (no atomics)
//
// The gate GEMM and the grouped GEMMs are dense contractions, so they run on
// the matrix cores: the gate on the fp64 ones (exact products, fp64 sums),
// the expert GEMMs (rows = pairs routed to one expert) on bf16 ones: tiles of
// up to 256 rows (gemm.hip), or the small-M kernel here for groups of at most
// 16 rows.
#include "common.hpp"
#include "moe_offload.h"

#include <cmath>

namespace moe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int kGateTok = 16;     // tokens per gate workgroup

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
// A workgroup holds 16 tokens and all experts.  The columns are cut into
// 16-wide blocks dealt round-robin to the eight waves (two a SIMD, so one
// wave's loads and conversions overlap the other's products), so each wave
// reads a distinct eighth of H.  In a block, lane (i, kq) = (lane % 16, lane / 16)
// loads columns 4kq .. 4kq+3 of token row i and of expert row 16g + i for
// each expert group g, and MFMA step s uses column 4kq + s of both, so A and
// B always pair the same column.  The waves' partial sums meet in LDS and
// are added in wave order.
// At 4096 tokens, d 2048, 64 experts: four waves with eight blocks ahead
// 54.6 us, eight waves with two ahead 40.3 (four ahead: 43.3), sixteen with
// one 40.6.
constexpr int kGateWaves = 8;
constexpr int kGateThreads = kGateWaves * kWave;
constexpr int kGateAhead = 2;  // blocks in flight per wave

struct GateBlock {
  float4 h;              // 4 columns of this lane's token row
  uint2 w[kMaxE / 16];   // 4 bf16 columns of this lane's row in each expert group
  float4 wf[kMaxE / 16]; // fp32 gate weights instead (dtype 0)
};

// FAST (d a multiple of 16 * kGateWaves * kGateAhead): every block the loop
// multiplies lies inside d, so loads are unconditional; the look-ahead past
// the end reads the row's last columns and is never used, and rows past T or
// experts past E (clamped to the last valid one) only feed logits nobody reads.
// A guarded load would be waited for on the spot.
template <int DT, bool FAST>
__device__ __forceinline__ void gate_load(GateBlock &b, const float *hrow, const uint8_t *wbase, int ng, int k,
                                          int d, int E, int i) {
  if (FAST) {
    const int kk = min(k, d - 4);
    b.h = *reinterpret_cast<const float4 *>(hrow + kk);
#pragma unroll
    for (int g = 0; g < kMaxE / 16; ++g) {
      if (g >= ng) break;
      const int e = min(16 * g + i, E - 1);
      if (DT == 1)
        b.w[g] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(wbase) + (size_t)e * d + kk);
      else
        b.wf[g] = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(wbase) + (size_t)e * d + kk);
    }
    return;
  }
  b.h = make_float4(0.f, 0.f, 0.f, 0.f);
  if (hrow && k < d) b.h = *reinterpret_cast<const float4 *>(hrow + k);
#pragma unroll
  for (int g = 0; g < kMaxE / 16; ++g) {
    const int e = 16 * g + i;
    if (DT == 1) {
      b.w[g] = make_uint2(0, 0);
      if (g < ng && e < E && k < d)
        b.w[g] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(wbase) + (size_t)e * d + k);
    } else {
      b.wf[g] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (g < ng && e < E && k < d)
        b.wf[g] = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(wbase) + (size_t)e * d + k);
    }
  }
}

template <int DT>
__device__ __forceinline__ void gate_mfma(const GateBlock &b, int ng, double4_t *acc, double &sq) {
  const double h4[4] = {b.h.x, b.h.y, b.h.z, b.h.w};
#pragma unroll
  for (int s = 0; s < 4; ++s) sq = fma(h4[s], h4[s], sq);
#pragma unroll
  for (int g = 0; g < kMaxE / 16; ++g) {
    if (g >= ng) break;
    double w4[4];
    if (DT == 1) {
      w4[0] = __uint_as_float(b.w[g].x << 16);
      w4[1] = __uint_as_float(b.w[g].x & 0xFFFF0000u);
      w4[2] = __uint_as_float(b.w[g].y << 16);
      w4[3] = __uint_as_float(b.w[g].y & 0xFFFF0000u);
    } else {
      w4[0] = b.wf[g].x;
      w4[1] = b.wf[g].y;
      w4[2] = b.wf[g].z;
      w4[3] = b.wf[g].w;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(h4[s], w4[s], acc[g], 0, 0, 0);
  }
}

template <int DT, bool FAST>
__device__ __forceinline__ void gate_partial(const PrefillArgs &a, int t0, int wave, int lane,
                                             double (*zp)[kGateTok][kMaxE], double (*rp)[kGateTok]) {
  const int d = a.d, E = a.E;
  const int i = lane % 16, kq = lane / 16;
  const int ng = (E + 15) / 16;
  const float *hrow = FAST ? a.H + (size_t)min(t0 + i, a.T - 1) * d
                           : (t0 + i < a.T ? a.H + (size_t)(t0 + i) * d : nullptr);
  const uint8_t *wbase = static_cast<const uint8_t *>(a.gate);
  double4_t acc[kMaxE / 16];
#pragma unroll
  for (int g = 0; g < kMaxE / 16; ++g) acc[g] = double4_t{0.0, 0.0, 0.0, 0.0};
  double sq = 0.0;
  const int stride = 16 * kGateWaves;
  GateBlock buf[kGateAhead];
#pragma unroll
  for (int j = 0; j < kGateAhead; ++j) gate_load<DT, FAST>(buf[j], hrow, wbase, ng, (wave + j * kGateWaves) * 16 + 4 * kq, d, E, i);
  for (int k0 = wave * 16; k0 < d; k0 += stride * kGateAhead) {
#pragma unroll
    for (int j = 0; j < kGateAhead; ++j) {
      const GateBlock cur = buf[j];
      gate_load<DT, FAST>(buf[j], hrow, wbase, ng, k0 + (j + kGateAhead) * stride + 4 * kq, d, E, i);
      gate_mfma<DT>(cur, ng, acc, sq);
    }
  }
#pragma unroll
  for (int g = 0; g < kMaxE / 16; ++g)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * g + i < E) zp[wave][kq + 4 * v][16 * g + i] = acc[g][v];
  sq += __shfl_xor(sq, 16, kWave);
  sq += __shfl_xor(sq, 32, kWave);
  if (kq == 0) rp[wave][i] = sq;
}

__global__ __launch_bounds__(kGateThreads) void prefill_gate_kernel(PrefillArgs a) {
  __shared__ double zp[kGateWaves][kGateTok][kMaxE];
  __shared__ double rp[kGateWaves][kGateTok];
  __shared__ int s_top[kGateWaves][kMaxK];
  __shared__ float s_inv[kGateTok];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int t0 = blockIdx.x * kGateTok;
  const int E = a.E, d = a.d;
  const bool fast = d % (16 * kGateWaves * kGateAhead) == 0;
  if (a.dtype == 1) {
    if (fast)
      gate_partial<1, true>(a, t0, wave, lane, zp, rp);
    else
      gate_partial<1, false>(a, t0, wave, lane, zp, rp);
  } else {
    if (fast)
      gate_partial<0, true>(a, t0, wave, lane, zp, rp);
    else
      gate_partial<0, false>(a, t0, wave, lane, zp, rp);
  }
  __syncthreads();
  // zs = zp[0] + zp[1] + ... in wave order, kept in zp[0]
  for (int x = tid; x < kGateTok * kMaxE; x += kGateThreads) {
    const int r = x / kMaxE, e = x % kMaxE;
    if (e < E) {
      double z = zp[0][r][e];
#pragma unroll
      for (int w = 1; w < kGateWaves; ++w) z += zp[w][r][e];
      zp[0][r][e] = z;
    }
  }
  if (tid < kGateTok) {
    double r = rp[0][tid];
#pragma unroll
    for (int w = 1; w < kGateWaves; ++w) r += rp[w][tid];
    rp[0][tid] = r;
    const float inv = (float)(1.0 / sqrt(r / (double)d + 1e-5));
    s_inv[tid] = inv;
    if (t0 + tid < a.T) a.inv_r[t0 + tid] = inv;
  }
  __syncthreads();
  double (*zs)[kMaxE] = zp[0];
  double *rs = rp[0];

  // top-K per token: wave w handles tokens TW w .. TW w + TW - 1
  constexpr int TW = kGateTok / kGateWaves;
  static_assert(kGateTok % kGateWaves == 0, "whole tokens per wave");
  for (int q = 0; q < TW; ++q) {
    const int r = wave * TW + q;
    const int t = t0 + r;
    if (t >= a.T) break;
    const int mine = wave_topk_lds(zs[r], E, a.K, lane, s_top[wave]);
    const double rr = sqrt(rs[r] / (double)d + 1e-5);
    const double zr = (lane < a.K) ? zs[r][mine] : 0.0;
    const double z0 = __shfl(zr, 0, kWave);
    const double ex = (lane < a.K) ? exp((zr - z0) / rr) : 0.0;
    double den = ex;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) den += __shfl_xor(den, o, kWave);
    if (lane < a.K) {
      a.ids[(size_t)t * a.K + lane] = mine;
      a.g[(size_t)t * a.K + lane] = (float)(ex / den);
    }
  }
  // normalised bf16 rows of all the workgroup's tokens, every thread taking
  // part, eight loads in flight (clamped, so none waits behind a branch); a
  // wave starts on them as soon as its tokens' top-K is written (1/r was set
  // with the sums)
  constexpr int kRowAhead = 8;
  const int nt = min(kGateTok, a.T - t0);
  const int q4 = d / 4;  // float4 per row
  const int total = nt * q4;
  for (int i0 = tid; i0 < total; i0 += kRowAhead * kGateThreads) {
    float4 v[kRowAhead];
#pragma unroll
    for (int u = 0; u < kRowAhead; ++u) {
      const int i = min(i0 + u * kGateThreads, total - 1);
      const int r = i / q4, c = (i - r * q4) * 4;
      v[u] = *reinterpret_cast<const float4 *>(a.H + (size_t)(t0 + r) * d + c);
    }
#pragma unroll
    for (int u = 0; u < kRowAhead; ++u) {
      const int i = i0 + u * kGateThreads;
      if (i < total) {
        const int r = i / q4, c = (i - r * q4) * 4;
        const float inv = s_inv[r];
        uint2 o;
        o.x = (uint32_t)f32_to_bf16_rne(v[u].x * inv) | ((uint32_t)f32_to_bf16_rne(v[u].y * inv) << 16);
        o.y = (uint32_t)f32_to_bf16_rne(v[u].z * inv) | ((uint32_t)f32_to_bf16_rne(v[u].w * inv) << 16);
        *reinterpret_cast<uint2 *>(a.xn + (size_t)(t0 + r) * d + c) = o;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// 2. sort by expert and update the layer's table for the whole batch
//
// A counting sort in one workgroup: count the pairs of each expert (LDS
// atomics that return nothing), take offsets, then give each pair the next
// position of its expert (atomics that return it).  Positions within an
// expert follow the atomics' order, which varies from run to run; nothing
// downstream depends on it, since every row of the grouped GEMMs is computed
// alone and the combine reads each (token, rank) pair through pos_of.  Each
// thread loads kPlanAhead ids before using the first.  (Placing each pair
// after the earlier pairs of its expert, with one wave's lanes of an expert
// found by ballots so no two lanes met on one counter, took 39 us against
// 22 us for these two passes at 4096 tokens of top-8 over 64 experts.)
constexpr int kPlanThreads = 1024;
constexpr int kPlanAhead = 8;

__global__ __launch_bounds__(kPlanThreads) void prefill_plan_kernel(PlanArgs a) {
  __shared__ int cnt[kMaxE], cur[kMaxE], lastp[kMaxE], offs[kMaxE];
  // tile lists (when a.ntiles): cost of each row-block size, the expert's
  // first tile and rows per tile in each list, the lists' lengths
  __shared__ float tcost[2][kWideRows / 32];
  __shared__ int tfirst[2][kMaxE], trows[2][kMaxE], tlen[2];
  __shared__ const uint16_t *tw[kMaxE];  // the experts' weights (when a.tiles)
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int E = a.E, P = a.T * a.K;
  if (tid < kMaxE) {
    cnt[tid] = 0;
    cur[tid] = 0;
    lastp[tid] = 0;
  }
  if (tid == 0) bad = 0;
  __syncthreads();
  if (a.tiles && tid < E) {
    // every expert has a slot from the warm start on, so its slot is the same
    // before and after the batch; no tile is ever made without one
    const int slot = a.table->expert_slot[tid];
    tw[tid] = slot >= 0 && slot < a.S ? reinterpret_cast<const uint16_t *>(a.arena_layer + (size_t)slot * a.slot_bytes) : nullptr;
    if (!tw[tid]) bad = 1;
    // an invalid batch leaves empty tiles
    if (!a.ntiles) a.tiles[tid] = GemmTile{nullptr, 0, 0, 0, 0};
    if (a.ntiles && tid < 2) a.ntiles[tid] = 0;
  }
  __syncthreads();
  for (int p0 = tid; p0 < P; p0 += kPlanAhead * kPlanThreads) {
    int ev[kPlanAhead];
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
      const int p = p0 + u * kPlanThreads;
      ev[u] = p < P ? a.ids[p] : 0;
    }
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
      const int p = p0 + u * kPlanThreads;
      if (p < P) {
        if (ev[u] < 0 || ev[u] >= E) {
          bad = 1;
        } else {
          atomicAdd(&cnt[ev[u]], 1);
          atomicMax(&lastp[ev[u]], p + 1);
        }
      }
    }
  }
  __syncthreads();
  if (bad) {
    if (tid == 0) {
      *a.err = ERR_BAD_LIST;
      *a.trace_out = *a.trace_in;
    }
    return;
  }
  if (a.ntiles && wave < kWideRows / 32) {
    // wave w: what the lists cost with row blocks of at most 32 (w + 1) rows
    const int n = lane < E ? cnt[lane] : 0;
    const int per = n > 0 ? tile_rows(n, 32 * (wave + 1)) : 32;
    int nt = (n + per - 1) / per, blocks = nt * (per / 32);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      nt += __shfl_xor(nt, o, kWave);
      blocks += __shfl_xor(blocks, o, kWave);
    }
    if (lane < 2) {
      const TileList &tl = lane == 0 ? a.up : a.dn;
      const int r = 32 * (wave + 1);
      tcost[lane][wave] = r >= tl.lo && r <= tl.hi ? tile_cost(tl.cb * nt, tl.cb * blocks, a.cus) : __builtin_inff();
    }
  }
  __syncthreads();
  if (wave == 0) {
    const int c = lane < E ? cnt[lane] : 0;
    int incl = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int v = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += v;
    }
    if (lane < E) offs[lane] = incl - c;
    if (a.ntiles) {
      // expert e's tiles: nt row blocks in each column block; the lists' first
      // tile of each expert by the same scan
#pragma unroll
      for (int li = 0; li < 2; ++li) {
        const TileList &tl = li == 0 ? a.up : a.dn;
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
        if (lane < E) {
          trows[li][lane] = per;
          tfirst[li][lane] = it - mine;
        }
        if (lane == kWave - 1) {
          const bool fits = it <= tl.cap;  // the host's bound holds for any counts
          tlen[li] = fits ? it : 0;
          a.ntiles[li] = tlen[li];
          if (!fits) *a.err = ERR_BAD_LIST;
        }
      }
    } else if (a.tiles && lane < E) {
      a.tiles[lane] = GemmTile{tw[lane], incl - c, c, 0, 0};
    }
  }
  __syncthreads();
  if (a.ntiles) {
    // tile i of a list belongs to the last expert whose first tile is <= i
    const int nup = tlen[0], n_all = tlen[0] + tlen[1];
    for (int i = tid; i < n_all; i += kPlanThreads) {
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
          GemmTile{tw[lo], offs[lo] + mb * per, min(per, cnt[lo] - mb * per), cb * (list == 0 ? a.up.cols : a.dn.cols), 0};
    }
  }
  for (int p0 = tid; p0 < P; p0 += kPlanAhead * kPlanThreads) {
    int ev[kPlanAhead];
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
      const int p = p0 + u * kPlanThreads;
      ev[u] = p < P ? a.ids[p] : 0;
    }
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
      const int p = p0 + u * kPlanThreads;
      if (p < P) {
        const int pos = offs[ev[u]] + atomicAdd(&cur[ev[u]], 1);
        a.perm_tok[pos] = p / a.K;
        a.pos_of[p] = pos;
      }
    }
  }
  if (wave != 0) return;

  // table update: lane e = expert e
  LayerTable *T = a.table;
  const uint64_t tbase = *a.trace_in;
  const bool in_range = lane < E;
  const int slot0 = in_range ? T->expert_slot[lane] : -1;
  uint32_t count = in_range ? T->count[lane] : 0u;
  int64_t last = in_range ? T->last[lane] : 0;
  int pf = in_range ? T->pf[lane] : 0;
  const int64_t clock0 = T->clock;
  const int64_t token0 = T->lookups;
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
  for (int j = 0; j < E; ++j) {
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
  const int misses = res_start ? 0 : n;
  int sh = hits, sm = misses, su = useful, sw = wasted, sf = fetched ? 1 : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sh += __shfl_xor(sh, o, kWave);
    sm += __shfl_xor(sm, o, kWave);
    su += __shfl_xor(su, o, kWave);
    sw += __shfl_xor(sw, o, kWave);
    sf += __shfl_xor(sf, o, kWave);
  }
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
    st->v[ST_HITS] += sh;
    st->v[ST_MISSES] += sm;
    st->v[ST_EVICT] += n_new;
    st->v[ST_PF_USEFUL] += su;
    st->v[ST_PF_WASTED] += sw;
    st->v[ST_LOOKUPS] += a.T;
    st->v[ST_BYTES] += (uint64_t)sf * a.expert_bytes;
  }
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

// Small-M grouped GEMM: launches whose experts have at most kSkinnyRows rows
// (batched decode).  A workgroup owns 16 output features of one expert for all
// of its rows (one 16-row MFMA block).  Its four
// waves split K in four; each streams its quarter of the 16 weight rows (of W1
// and W3 in the up projection) from global memory straight into
// v_mfma_f32_16x16x32_bf16 fragments, several 32-deep steps ahead, with
// the rows' activations read alongside (from L2: every workgroup of the expert
// reads them).  A row or feature past the end reads a valid row instead (its
// outputs are not written); only a K tail that is not a multiple of 32 is
// zeroed.  The four partial products meet in LDS and are added in wave order.
// Batches of more than 16 tokens take the tiled kernels: with a second row
// block here 32 tokens of top-8 over 64 experts took 126 / 103 us (up / down)
// and 32 tokens of top-2 over 8 experts 373 / 221, the tiles 126 / 66 and 329 / 174.
constexpr int kSkinnyAheadUp = 8, kSkinnyAheadDown = 8;  // steps in flight per wave

__device__ __forceinline__ bf16x8 load_frag(const uint16_t *p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const gemm_u32x4 *>(p));
}

__device__ __forceinline__ bf16x8 load_frag(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(bf16x8, buffer_load16(r, byte_off));
}

template <bool UP, int AHEAD>
__global__ __launch_bounds__(256) void prefill_skinny_kernel(const GemmTile *tiles, const uint16_t *a_src,
                                                             const int32_t *perm_tok, void *out, int d, int d_ff) {
  constexpr int NB = UP ? 2 : 1;  // B matrices: W1 and W3, or W2
  __shared__ floatx4 red[4][NB][kWave];
  const int K = UP ? d : d_ff;  // reduction length
  const int N = UP ? d_ff : d;  // output features
  const int nfb = (N + 15) / 16;
  const int ti = blockIdx.x / nfb, fb = blockIdx.x - ti * nfb;
  const GemmTile t = tiles[ti];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int M = min(t.rows, kSkinnyRows);
  if (M <= 0) return;              // an expert without rows
  const int kg = (lane / 16) * 8;  // this lane's 8 elements of a 32-deep step
  // A row (token of the expert) and B row (feature) of this lane, clamped
  const int m = t.row + min(lane % 16, M - 1);
  const uint16_t *ap = (UP ? a_src + (size_t)perm_tok[m] * d : a_src + (size_t)m * d_ff) + kg;
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

  floatx4 c[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) c[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

  // this wave's full 32-deep steps
  const int full = K / 32;
  const int q = (full + 3) / 4;
  const int s0 = min(wave * q, full), s1 = min(s0 + q, full);
  const int n = s1 - s0;
  bf16x8 wa[AHEAD][NB], xa[AHEAD];
  // no load is conditional, so the compiler can count the loads in flight
  auto load = [&](int slot, int step) {
    const int k = step * 32;
#pragma unroll
    for (int b = 0; b < NB; ++b) wa[slot][b] = load_frag(brs[b], boff + 2 * k);
    xa[slot] = load_frag(ap + k);
  };
  auto mma = [&](int slot) {
#pragma unroll
    for (int b = 0; b < NB; ++b) c[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[slot], wa[slot][b], c[b], 0, 0, 0);
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
    const bf16x8 x0 = load_frag(ap + k);
    xa[0] = in ? x0 : z;
    mma(0);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) red[wave][b][lane] = c[b];
  __syncthreads();
  if (wave == 0) {
    floatx4 r[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      r[b] = red[0][b][lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) r[b] += red[w][b][lane];
    }
    const int n_out = fb * 16 + lane % 16;
    if (n_out < N) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int mo = (lane / 16) * 4 + i;
        if (mo >= M) continue;
        if (UP)
          static_cast<uint16_t *>(out)[(size_t)(t.row + mo) * N + n_out] = f32_to_bf16_rne(silu(r[0][i]) * r[NB - 1][i]);
        else
          static_cast<float *>(out)[(size_t)(t.row + mo) * N + n_out] = r[0][i];
      }
    }
  }
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
hipError_t launch_prefill_gate(const PrefillArgs &a, const Launch &l) {
  MOE_LAUNCH(prefill_gate_kernel, dim3((a.T + kGateTok - 1) / kGateTok), dim3(kGateThreads), 0, l, a);
  return hipGetLastError();
}

hipError_t launch_prefill_plan(const PlanArgs &a, const Launch &l) {
  MOE_LAUNCH(prefill_plan_kernel, dim3(1), dim3(kPlanThreads), 0, l, a);
  return hipGetLastError();
}

hipError_t launch_prefill_skinny_up(const GemmTile *tiles, int ntiles, const uint16_t *xn, const int32_t *perm_tok,
                                    uint16_t *act, int d, int d_ff, const Launch &l) {
  if (ntiles <= 0) return hipSuccess;
  MOE_LAUNCH((prefill_skinny_kernel<true, kSkinnyAheadUp>), dim3(ntiles * ((d_ff + 15) / 16)), dim3(256), 0, l, tiles, xn,
             perm_tok, (void *)act, d, d_ff);
  return hipGetLastError();
}

hipError_t launch_prefill_skinny_down(const GemmTile *tiles, int ntiles, const uint16_t *act, float *Y, int d, int d_ff,
                                      const Launch &l) {
  if (ntiles <= 0) return hipSuccess;
  MOE_LAUNCH((prefill_skinny_kernel<false, kSkinnyAheadDown>), dim3(ntiles * ((d + 15) / 16)), dim3(256), 0, l, tiles, act,
             nullptr, (void *)Y, d, d_ff);
  return hipGetLastError();
}

hipError_t launch_prefill_unpermute(float *H, const float *Y, const float *g, const int32_t *pos_of, int T,
                                    int d, int K, const Launch &l) {
  MOE_LAUNCH(prefill_unpermute_kernel, dim3(T), dim3(256), 0, l, H, Y, g, pos_of, T, d, K);
  return hipGetLastError();
}

}  // namespace moe
