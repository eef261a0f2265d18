// Internal layout shared by the kernels and the host engine of the MoE
// offloading library.  Everything here lives in the caller's device
// workspace; the host engine carves the workspace into these regions.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe {

constexpr int kMaxE = 64;   // experts per layer: one lane per expert in the table wave
constexpr int kMaxK = 16;   // experts per token
constexpr int kWave = 64;   // CDNA wavefront

// One layer's cache table.  slot_expert[s] = expert held by slot s;
// expert_slot[e] = slot of expert e or -1; count = LFU use count (persists
// across eviction); last = clock tick of the last use or insertion;
// pf = 1 while a prefetched expert has not yet been used.
struct LayerTable {
  int64_t clock;
  int64_t lookups;
  int32_t slot_expert[kMaxE];
  int32_t expert_slot[kMaxE];
  uint32_t count[kMaxE];
  int32_t pf[kMaxE];
  int64_t last[kMaxE];
};

enum StatIdx {
  ST_HITS = 0, ST_MISSES, ST_EVICT, ST_PF_GUESS, ST_PF_ISSUED, ST_PF_USEFUL,
  ST_PF_WASTED, ST_LOOKUPS, ST_BYTES, ST_COUNT
};
struct LayerStats {
  uint64_t v[16];
};

// Copies the router decided: expert e of `layer` from the host store into
// slot s of `layer` in the arena.
struct FetchList {
  int32_t n;
  int32_t layer;
  int32_t expert[kMaxK];
  int32_t slot[kMaxK];
  int32_t pad[2];
};

// Router output consumed by the decode FFN on the compute stream.
struct RouteOut {
  int32_t ids[kMaxK];
  int32_t slot[kMaxK];
  int32_t hit[kMaxK];
  float g[kMaxK];
  float inv_r;
  int32_t k;
  int32_t pad[2];
};

struct TraceRec {
  int32_t kind, token, layer, rank, expert, flags, slot, victim;
};

enum { REC_ACCESS = 0, REC_PREFETCH = 1, REC_PREFILL = 2 };
enum { ERR_NONE = 0, ERR_BAD_IDS = 1, ERR_BAD_LIST = 2, ERR_BAD_PACK = 3 };

struct RouterArgs {
  const void *gate;        // [L][E][d]
  const float *h;          // [d]
  const int32_t *inj_ids;  // injected routing (test hook) or nullptr
  LayerTable *tables;
  LayerStats *stats;
  FetchList *dlists;       // demand list of each layer
  FetchList *plists;       // prefetch list targeting each layer
  RouteOut *route;
  TraceRec *trace;
  int32_t *err;
  // Records written so far (ring position = count % cap).  A launch reads
  // trace_in and writes the new count to trace_out, a second word, so that
  // the workgroups of one launch never see a count another of them updated.
  const uint64_t *trace_in;
  uint64_t *trace_out;
  uint64_t trace_cap;
  uint64_t expert_bytes;
  int layer, L, E, S, K, d, dtype, policy;
  int aging;               // aged LFU: lookup-clock ticks per halving of a count
  int demand;              // 1: route + look up `layer`
  int spec_layer;          // >= 0: guess that layer's experts from h and prefetch
  int pmax;                // prefetch at most this many guesses
};

struct FfnArgs {
  const uint8_t *arena;
  const RouteOut *route;
  float *h;                // in/out [d]
  float *act;              // [K][d_ff]
  float *part;             // [chunks][d]
  uint64_t expert_bytes;
  int layer, S, K, d, d_ff;
};

// ---- batched prefill ------------------------------------------------------
struct PrefillPlan {
  int32_t n;           // pairs routed to the expert
  int32_t off;         // first sorted position
  int32_t slot_start;  // slot before the batch, -1 if not resident
  int32_t slot_after;  // slot after the batch, -1 if not resident
  int32_t newcomer;    // became resident in this batch
  int32_t pad[3];
};

// A tile of a grouped GEMM: `rows` sorted rows from `row` on, all of the
// expert whose weights are at w, by the output columns from n0 on.
struct GemmTile {
  const uint16_t *w;  // expert base (W1 | W3 | W2), bf16
  int32_t row, rows, n0;
  int32_t once;       // these are all of the expert's rows: the launch reads its weights once
};
constexpr int kWideRows = 256, kNarrowRows = 64;  // most rows of a wide and of a narrow tile

// How a launch's tiles are cut: column blocks of `cols` output columns, row
// blocks of 32 * k rows with lo <= 32 * k <= hi (the plan chooses k), at most
// `cap` tiles in all, `slots` of them at a time.  staging: what a tile's weights
// cost, in 32-row blocks.
struct TileList {
  int cols, cb, lo, hi, first, cap, slots;
  float staging;
};

// Relative cost of a launch whose experts are cut into `row_blocks` row blocks
// of `blocks` 32-row blocks in all.  A tile costs its staging of the weights
// (2.6 blocks' worth of wide tiles' 256 weight rows; of narrow ones' 128 rows 2
// where they start on 128-byte lines, else 2.6) and its blocks; a last round
// that fills only part of the chip costs half a round and half its share.
// Fitted on MI355X: wide to 2048 tokens of top-2 over 8 experts (down, d_ff
// 14336), rows a tile 96 .. 256: 592, 638, 538, 579, 615, 622 us measured, 610,
// 638, 543, 574, 584, 635 by the model; narrow to which of 32 and 64 rows a pass
// is faster with (us, 64 / 32): 4 experts of 2048 x 2048, 96 tokens of top-2
// 66.5 / 53.1, 64 tokens 63.5 / 61.4; 64 of 512 x 256, 300 of top-8 50.1 / 47.0;
// 16 of 1024 x 1024, 192 of top-4 57.6 / 53.2; 12 of 3072 x 1536, 200 of top-2
// 118.8 / 113.9; 8 of 4096 x 4096, 200 of top-1 182.7 / 193.3; 8 of 4096 x 14336,
// 128 of top-2 495 / 567; 17 of 1832 x 3248, 136 of top-4 190 / 202 (so chosen
// all eight).
__host__ __device__ inline float tile_cost(const TileList &t, int row_blocks, int blocks) {
  const int tiles = t.cb * row_blocks;
  if (tiles <= 0) return 0.0f;
  const float n = (float)tiles / (float)t.slots;
  const float rounds = 0.5f * ((float)((tiles + t.slots - 1) / t.slots) + n);
  return rounds / n * (t.staging * (float)tiles + (float)(t.cb * blocks));
}

// Rows of an expert's tiles when its n > 0 rows are cut into blocks of at most
// r rows: equal blocks, rounded up to 32.
__host__ __device__ inline int tile_rows(int n, int r) {
  const int nt = (n + r - 1) / r;
  return ((n + nt - 1) / nt + 31) / 32 * 32;
}

struct PrefillArgs {
  const void *gate;  // layer's gate [E][d], bf16
  const float *H;    // [T][d]
  int32_t *ids;      // [T][K]
  float *g;          // [T][K]
  uint16_t *xn;      // [T][d] bf16
  double *zpart;     // [splits][T][kMaxE] partial logits of the column ranges
  uint8_t *blk_cnt;  // [blocks of kRouteTok tokens][kMaxE] tokens that chose the expert
  uint8_t *blk_last; // and the last pair (token in block * K + rank) that did
  int T, d, E, K, splits;
};
constexpr int kRouteTok = 16;

struct PlanArgs {
  const int32_t *ids;
  const uint8_t *blk_cnt, *blk_last;  // as in PrefillArgs
  int32_t *perm_tok;  // [T*K] sorted position -> token
  int32_t *pos_of;    // [T*K] (token, rank) -> sorted position
  PrefillPlan *plan;  // [E]
  LayerTable *table;
  LayerStats *stats;
  TraceRec *trace;
  const uint64_t *trace_in;  // record count before / after, as in RouterArgs
  uint64_t *trace_out;
  uint64_t trace_cap;
  int32_t *err;
  uint64_t expert_bytes;
  int T, K, E, S, layer, policy;
  int aging;  // aged LFU: lookup-clock ticks per halving of a count
  // Batches planned on the device (a slot for every expert): the kernel also
  // writes the GEMM tiles; nullptr otherwise.  Small-M launches take one tile
  // per expert, at tiles[0 ..] (when small).  Others (when ntiles is not
  // nullptr) take lists ordered (expert, column block, row block) at
  // tiles[up.first ..] and tiles[dn.first ..], their lengths written to
  // ntiles[0] and [1]; a list that no launch reads has cb == 0.
  GemmTile *tiles;
  int32_t *ntiles;
  int small;
  TileList up, dn;
  const uint8_t *arena_layer;  // this layer's slots
  uint64_t slot_bytes;
};

// Where a kernel goes: its stream and, when kernel timing is on, two events
// the dispatch itself stamps at the kernel's start and end.
struct Launch {
  hipStream_t s = nullptr;
  hipEvent_t start = nullptr, stop = nullptr;
};
#define MOE_LAUNCH(kernel, grid, block, shmem, L, ...) \
  hipExtLaunchKernelGGL(kernel, grid, block, shmem, (L).s, (L).start, (L).stop, 0, __VA_ARGS__)

// launchers (one per translation unit that owns the kernel)
// Streaming read of bytes (a multiple of 16) at buf with the given number of
// workgroups; reads only.
hipError_t launch_hbm_read_probe(const void *buf, size_t bytes, int workgroups, hipStream_t s);
// Copy bytes (a multiple of 16) from src_dev (the device address of mapped
// pinned host memory) to dst with the fetch kernel's access pattern.
hipError_t launch_h2d_copy_probe(const void *src_dev, void *dst, size_t bytes, int workgroups, hipStream_t s);
// Register-only bf16 MFMA loop; returns the flops the launch performs.
double launch_mfma_bf16_probe(int shape, int workgroups, int iters, hipStream_t s);
hipError_t launch_router(const RouterArgs &a, const Launch &l);
// Copies of a fetch list: expert e of the list's layer from its host store
// (stride src_stride) into its HBM slot (stride expert_bytes), or, when
// staging is non-NULL, entry i into staging + i * src_stride.
hipError_t launch_fetch(const FetchList *list, const uint8_t *const *layers, uint8_t *arena, int L, int E,
                        int S, int K, uint64_t expert_bytes, uint64_t src_stride, uint8_t *staging,
                        int32_t *err, const Launch &l);
// Packed experts of a fetch list, entry i at staging + i * 3 * mat_cap, rebuilt
// as bf16 into their slots; n = weights per matrix.
hipError_t launch_unpack(const FetchList *list, const uint8_t *staging, uint8_t *arena, int L, int S, int K,
                         uint64_t mat_cap, uint64_t expert_bytes, uint64_t n, int32_t *err, const Launch &l);
// Entropy-coded experts (host format 2): the same, from the entropy layout
// with cap_words stream words per matrix.
hipError_t launch_entropy_unpack(const FetchList *list, const uint8_t *staging, uint8_t *arena, int L, int S, int K,
                                 uint64_t mat_cap, uint64_t expert_bytes, uint64_t n, uint64_t cap_words,
                                 int32_t *err, const Launch &l);
// Bytes of one entropy-coded matrix (0 unless n is a positive multiple of 512)
// and the host encoder (0, or -1 with *why set).
uint64_t entropy_matrix_bytes(uint64_t n, uint64_t cap_words);
int entropy_pack(const uint16_t *w, uint64_t n, uint64_t cap_words, uint8_t *out, uint64_t *used, const char **why);
hipError_t launch_ffn_up(const FfnArgs &a, int dtype, const Launch &l);
hipError_t launch_ffn_down(const FfnArgs &a, int dtype, const Launch &l);
// Adds the partial row sums that the down launch left (ffn_down_chunks rows of
// them; with 0 the down launch adds into h itself and there is nothing to do).
hipError_t launch_ffn_reduce(const FfnArgs &a, int dtype, const Launch &l);
int ffn_down_chunks(int K, int d, int d_ff, int dtype);
// group-quantised experts (dtype 2)
hipError_t launch_ffnq_up(const FfnArgs &a, const Launch &l);
hipError_t launch_ffnq_down(const FfnArgs &a, const Launch &l);
int ffnq_down_chunks(int K, int d_ff);
hipError_t launch_prefill_gate(const PrefillArgs &a, const Launch &l);
int prefill_gate_splits(int T, int d);  // column ranges of a batch's gate launch
// Top-K, weights and rows of every token, then the batch's plan.
hipError_t launch_prefill_route_plan(const PrefillArgs &a, const PlanArgs &p, const Launch &l);
// Grouped GEMMs over a tile list (wide tiles: up to kWideRows rows by
// prefill_tile_cols(up, true) output columns; narrow ones up to kNarrowRows by
// half as many).  With ntiles the list's length is read on the device (at most
// `grid`; the surplus workgroups exit), otherwise it is `grid`.
hipError_t launch_prefill_up(const GemmTile *tiles, const int32_t *ntiles, int grid, bool wide, const uint16_t *xn,
                             const int32_t *perm_tok, uint16_t *act, int d, int d_ff, const Launch &l);
hipError_t launch_prefill_down(const GemmTile *tiles, const int32_t *ntiles, int grid, bool wide, const uint16_t *act,
                               float *Y, int d, int d_ff, const Launch &l);
constexpr int prefill_tile_cols(bool up, bool wide) { return (up ? 128 : 256) / (wide ? 1 : 2); }
// Small-M grouped GEMMs: one tile per expert, each with at most max_rows <=
// kSkinnyRows rows; a workgroup per (tile, 16 output features).
constexpr int kSkinnyRows = 32;
hipError_t launch_prefill_skinny_up(const GemmTile *tiles, int ntiles, int max_rows, const uint16_t *xn, const int32_t *perm_tok,
                                    uint16_t *act, int d, int d_ff, const Launch &l);
hipError_t launch_prefill_skinny_down(const GemmTile *tiles, int ntiles, int max_rows, const uint16_t *act, float *Y, int d, int d_ff,
                                      const Launch &l);
hipError_t launch_prefill_unpermute(float *H, const float *Y, const float *g, const int32_t *pos_of, int T,
                                    int d, int K, const Launch &l);

// ---------------------------------------------------------------------------
// device helpers

// 8 bf16 (one 16-byte load) -> 8 fp32; bf16 is the top half of an fp32.
__device__ __forceinline__ void bf16x8_to_f32(const uint4 v, float *f) {
  f[0] = __uint_as_float(v.x << 16);
  f[1] = __uint_as_float(v.x & 0xFFFF0000u);
  f[2] = __uint_as_float(v.y << 16);
  f[3] = __uint_as_float(v.y & 0xFFFF0000u);
  f[4] = __uint_as_float(v.z << 16);
  f[5] = __uint_as_float(v.z & 0xFFFF0000u);
  f[6] = __uint_as_float(v.w << 16);
  f[7] = __uint_as_float(v.w & 0xFFFF0000u);
}

// Aged LFU key: the usage count halved (rounding down) once per `aging` ticks
// between the expert's last use and `clock`.
__device__ __forceinline__ uint32_t aged_count(uint32_t count, int64_t last, int64_t clock, int aging) {
  const int64_t halvings = (clock - last) / aging;
  return halvings >= 32 ? 0u : count >> (int)halvings;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Sum over the 64 lanes of a wave, left in lane 63, through DPP moves (no LDS
// round trips): running sums within each row of 16 lanes (row_shr 1, 2, 4,
// 8), then lane 15 of rows 0 and 2 into rows 1 and 3 (row_bcast:15) and lane
// 31 into rows 2 and 3 (row_bcast:31).  Lanes whose DPP source lies outside
// the pattern add the 0 passed as the old value.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK,
                                                                   0xF, false));
}
__device__ __forceinline__ float wave_sum_to_lane63(float v) {
  v = dpp_add<0x111, 0xF>(v);  // row_shr:1
  v = dpp_add<0x112, 0xF>(v);  // row_shr:2
  v = dpp_add<0x114, 0xF>(v);  // row_shr:4
  v = dpp_add<0x118, 0xF>(v);  // row_shr:8
  v = dpp_add<0x142, 0xA>(v);  // row_bcast:15
  v = dpp_add<0x143, 0xC>(v);  // row_bcast:31
  return v;
}

// fp64 sum over a wave's lanes, left in lane 63: running sums within rows of
// 16 lanes (row_shr 1, 2, 4, 8), then row_bcast:15 and row_bcast:31; lanes
// whose DPP source lies outside the pattern add 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add_d(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xF, false);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_d_to_lane63(double v) {
  v = dpp_add_d<0x111, 0xF>(v);
  v = dpp_add_d<0x112, 0xF>(v);
  v = dpp_add_d<0x114, 0xF>(v);
  v = dpp_add_d<0x118, 0xF>(v);
  v = dpp_add_d<0x142, 0xA>(v);
  v = dpp_add_d<0x143, 0xC>(v);
  return v;
}

// Value of x on lane src, for a src the whole wave agrees on (a scalar read,
// not an LDS round trip like a general shuffle).
__device__ __forceinline__ int lane_value(int x, int src) { return __builtin_amdgcn_readlane(x, src); }
__device__ __forceinline__ double lane_value_d(double x, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), src),
                          __builtin_amdgcn_readlane(__double2loint(x), src));
}

// Top-K of E <= 64 logits held in LDS, in rank order: larger z first, lower
// id on ties, NaN ranked as -inf.  Lane e < E counts the entries that come
// before its own in that order, which is its rank, and rank r < K writes its
// id to out[r]; id is out[lane] on lanes < K and -1 elsewhere.  N independent
// sets at once.  Called by one whole wave; `out` is LDS owned by that wave.
__device__ __forceinline__ double rank_key(double z) { return z != z ? -__builtin_inf() : z; }

template <int N>
__device__ inline void wave_topk_lds(const double *const (&z)[N], int E, int K, int lane, int *const (&out)[N],
                                     int (&id)[N]) {
  if (lane < E) {
    double mine[N];
    int rank[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      mine[q] = rank_key(z[q][lane]);
      rank[q] = 0;
    }
#pragma unroll 8
    for (int o = 0; o < E; ++o)
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const double zo = rank_key(z[q][o]);
        rank[q] += (zo > mine[q] || (zo == mine[q] && o < lane)) ? 1 : 0;
      }
#pragma unroll
    for (int q = 0; q < N; ++q)
      if (rank[q] < K) out[q][rank[q]] = lane;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int q = 0; q < N; ++q) id[q] = lane < K ? out[q][lane] : -1;
}

}  // namespace moe
