// Grouped GEMMs of the batched paths (prefill and batched decode of more than
// a handful of rows): rows sorted by expert times that expert's weights.
//
//   up    act[row] = SiLU(W1 x) * (W3 x), x = xn[perm_tok[row]]   (bf16 out)
//   down  Y[row]   = W2 act[row]                                   (fp32 out)
//
// Weights are stored out x in, so both operands are K-major.  A tile is up to
// 256 sorted rows of one expert by 256 weight rows (128 output features of W1
// and of W3 in the up projection, 256 of W2 in the down projection; half as
// many in the narrow form).  Four waves, one a SIMD, share its products; the
// number of 32-row blocks (MX = 1 .. 8) is a template parameter, so a tile
// costs what its rows need, to 32 rows.
//
// Both operands are staged by the memory system (loads straight into LDS) in
// slices of 64 columns, whole 128-byte lines, into rings of three slices (two
// of weights when the tile has more than 160 rows: 160 KB of LDS).  A wave
// keeps the fragments of the next 16-deep part in registers while it
// multiplies the current one, and the one barrier per slice stands before the
// last part's products, so the matrix cores have work queued while the waves
// meet.  The loads are dealt out between the products, one every two to four:
// issued back to back they fill the address path and stall the wave.
//
// Measured on MI355X, us a launch in the trace (up / down, average of 12 in a row
// and the fastest): 4096 tokens of top-8 over 64 experts, d 2048, d_ff 1408: 436 /
// 268, 362 / 227; 2048 tokens of top-2 over 8 experts, d 4096, d_ff 14336: 1021 /
// 592, 855 / 514.  A pass through each, against eight waves of 64-row slabs with two
// slices and no fragment prefetch, in turn on one card: 784 -> 726 and 1877 ->
// 1543.
#include "common.hpp"

#include <type_traits>

namespace moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kThreads = 256;
constexpr int kOnceBlocks = 5;     // most row blocks of a tile with a non-temporal form
constexpr int kKs = 64;            // columns of a slice
constexpr int kRowB = kKs * 2;     // bytes of a slice row: one 128-byte line
constexpr int kBlockB = 32 * kRowB;  // bytes of 32 slice rows
// Byte offset for a chunk that must read zeros: at or past every weight
// resource's record count (all below 2^31), which the hardware turns into
// zeros.  The range check admits any dword that starts below the record
// count, so the offset must clear it, not merely approach it.
constexpr uint32_t kOobOffset = 0x80000000u;

__device__ const uint4 g_zeros[1] = {};  // what rows of A read past the end of K

__device__ __forceinline__ uint32_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// v / (1 + e^-v).  The quotient is v times the hardware's reciprocal (one ulp)
// with one step of refinement, which rounds as the division does but for one
// quotient in some 2^22; div_fixup sets the infinite and NaN cases.  4096 tokens
// of top-8 over 64 experts: 720 us a pass with the reciprocal alone and so; the
// compiler's division took 1.5% more.
__device__ __forceinline__ float silu(float v) {
  const float x = 1.0f + __expf(-v), r = __builtin_amdgcn_rcpf(x), q = v * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-x, q, v), r, q), x, v);
}

// One wave-wide 16-byte-a-lane load into LDS at m0 + 16 * lane.  Written as
// instructions of their own rather than the compiler's builtin: the compiler
// tracks loads in flight into LDS per array, loses track across a ring's loop
// and then waits for all of them before reading any slice; here the kernel's
// own waits (wait_vm) are the only ones.  M0 carries the LDS address.  It is a
// reserved register, which a clobber list cannot name: the compiler keeps
// nothing in it and sets it before any instruction of its own that reads it
// (none in this kernel: gfx9 LDS instructions do not use it).
// ONCE: non-temporal.
template <bool ONCE>
__device__ __forceinline__ void dma_weights(__amdgpu_buffer_rsrc_t r, uint32_t m0, uint32_t voff, uint32_t soff) {
  if constexpr (ONCE)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 : : "s"(__builtin_amdgcn_readfirstlane(m0)), "v"(voff), "s"(r), "s"(__builtin_amdgcn_readfirstlane(soff)) : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(__builtin_amdgcn_readfirstlane(m0)), "v"(voff), "s"(r), "s"(__builtin_amdgcn_readfirstlane(soff)) : "memory");
}
__device__ __forceinline__ void dma_rows(const void *p, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               : : "s"(__builtin_amdgcn_readfirstlane(m0)), "v"(p) : "memory");
}

// s_waitcnt with vmcnt = N, or lgkmcnt = 0, and the other counters left alone
// (gfx9 encoding)
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (0x7 << 4)); }

__device__ __forceinline__ bf16x8 frag(const uint8_t *p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

// One tile of MX 32-row blocks by NY * 128 weight rows, in an LDS area of
// LDS bytes.  A slice row holds eight 16-byte chunks; chunk c of row r sits at
// c ^ ((r / 2) % 8), so the 16 lanes the LDS serves at once in a fragment read
// (16 rows at one chunk) touch all 64 banks once.  A load instruction fills
// eight rows, lane i fetching the chunk that the swizzle puts at its place.
// ONCE: the tile has all of its expert's rows, so no other reads its weights
// and they are loaded non-temporally: 32 tokens of top-8 over 64 experts 176 ->
// 152 us, 509 tokens 250 -> 232.  Weights that several tiles share in L2 lose by
// it: with every load so 4096 tokens take 740 us instead of 704, 2048 tokens of
// top-2 over 8 experts 1523 instead of 1477.
template <bool UP, bool RAGGED, int MX, bool ONCE, int NY, int LDS>
__device__ __forceinline__ void gemm_tile(const GemmTile &t, const uint16_t *a_src, const int32_t *perm_tok, void *out,
                                          int d, int d_ff, uint8_t *lds) {
  constexpr int AB = MX * kBlockB, BB = NY * 4 * kBlockB;  // bytes of an A and of a B slice
  constexpr int NA = 3, NB = 3 * (AB + BB) <= LDS ? 3 : 2;  // slices in the rings
  static_assert(NA * AB + NB * BB <= LDS, "the rings fit");
  constexpr int BN = (UP ? 64 : 128) * NY;           // output features of the tile
  // The waves form a WM x (4 / WM) grid over (row blocks, weight rows): XW row
  // blocks by YW 32-row weight blocks each, in the up projection YM of W1 and
  // the same features' YM of W3.
  // Two by two where the tile is tall (XW, YW 4, 4 instead of 8, 2: eight
  // fragment reads per sixteen products instead of ten), else every wave has
  // all row blocks, so that a tile costs what its rows need; 4096 tokens of
  // top-8 over 64 experts 709 / 704 us, of top-4 over 16 (d_ff 4096) 863 / 858.
  constexpr int WM = NY == 2 && MX % 2 == 0 && MX >= 6 ? 2 : 1;
  constexpr int XW = MX / WM, YW = NY * WM, YM = UP && NY == 2 ? YW / 2 : YW;
  constexpr int IA = MX, IB = 4 * NY;                // a wave's load instructions per slice
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int wm = wave % WM, wn = wave / WM;
  const int K = UP ? d : d_ff, N = UP ? d_ff : d;

  // sources: load instruction i of the wave fills slice rows 8 (4 i + wave) ..
  // + 7.  Rows past the tile's end read its last row and columns past N the
  // last one (their results are not written).  perm_tok names a token of the
  // batch at every position below its pair count: the plan writes them all, from
  // ids and counts that the route kernel takes from one register (a clamp here
  // costs 1%: 4096 tokens of top-8 over 64 experts 720 -> 728 us).
  const int lr = lane / 8, lc = (lane & 7) ^ ((4 * (wave & 1) + lane / 16) & 7);
  const uint8_t *ap[IA];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int m = t.row + min(8 * (4 * i + wave) + lr, t.rows - 1);
    ap[i] = reinterpret_cast<const uint8_t *>(a_src + (UP ? (size_t)perm_tok[m] : (size_t)m) * K + 8 * lc);
  }
  const int nb = min(BN, N - t.n0);
  __amdgpu_buffer_rsrc_t brs[UP ? 2 : 1];
#pragma unroll
  for (int b = 0; b < (UP ? 2 : 1); ++b)
    brs[b] = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(t.w + (UP ? (size_t)b * d_ff * d : 2 * (size_t)d_ff * d) + (size_t)t.n0 * K), 0,
        (uint32_t)nb * K * 2, 0x00020000);
  uint32_t boff[IB];
#pragma unroll
  for (int i = 0; i < IB; ++i) boff[i] = (uint32_t)min((8 * (4 * i + wave) + lr) % BN, nb - 1) * K * 2 + 16 * lc;
  const uint32_t m0a = (uint32_t)(uintptr_t)(lds_void_t *)lds + wave * (8 * kRowB), m0b = m0a + NA * AB;
  auto load_a = [&](int i, int s, uint32_t at) {
    const uint8_t *p = ap[i] + (size_t)s * kRowB;
    if (RAGGED && s * kKs + 8 * lc >= K) p = reinterpret_cast<const uint8_t *>(g_zeros);
    dma_rows(p, m0a + at + i * kBlockB);
  };
  auto load_b = [&](int i, int s, uint32_t at) {
    const uint32_t so = (uint32_t)s * kRowB;
    const __amdgpu_buffer_rsrc_t r = brs[UP ? i / (IB / 2) : 0];
    if (RAGGED)
      dma_weights<ONCE>(r, m0b + at + i * kBlockB, s * kKs + 8 * lc >= K ? kOobOffset : boff[i] + so, 0);
    else
      dma_weights<ONCE>(r, m0b + at + i * kBlockB, boff[i], so);
  };

  // fragments: lane i holds row i % 32 of a block, columns 16 h + 8 (i / 32) .. + 7
  // of part h.  (Narrow up tiles: 16 rows of W1 and 16 of W3 in one block.)
  const int r32 = lane & 31, hi = lane >> 5, sw = (r32 >> 1) & 7;
  const uint32_t fa = (wm * XW * 32 + r32) * kRowB + ((hi ^ sw) << 4);
  constexpr bool kMixed = UP && NY == 1;
  const int brow = kMixed ? (r32 < 16 ? 16 * wn + r32 : 64 + 16 * wn + r32 - 16) : 32 * YM * wn + r32;
  const uint32_t fb = NA * AB + brow * kRowB + ((hi ^ ((brow >> 1) & 7)) << 4);
  struct Frags {
    bf16x8 a[XW], b[YW];
  };
  constexpr int NF = XW + YW;
  auto rd = [&](Frags &f, int i, uint32_t at_a, uint32_t at_b, int h) {
    if (i < YW)
      f.b[i] = frag(lds + ((fb + at_b) ^ (h << 5)) + (i / YM * 128 + i % YM * 32) * kRowB);
    else
      f.a[i - YW] = frag(lds + ((fa + at_a) ^ (h << 5)) + (i - YW) * kBlockB);
  };

  floatx16 c[XW][YW];
#pragma unroll
  for (int x = 0; x < XW; ++x)
#pragma unroll
    for (int y = 0; y < YW; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i) c[x][y][i] = 0.0f;

  const int nk = (K + kKs - 1) / kKs;
  // fill the rings, oldest slice first, and read the first part
#pragma unroll
  for (int s = 0; s < NA; ++s) {
    if (s < nk) {
      if (s < NB) {
#pragma unroll
        for (int i = 0; i < IB; ++i) load_b(i, s, s * BB);
      }
#pragma unroll
      for (int i = 0; i < IA; ++i) load_a(i, s, s * AB);
    }
  }
  Frags P, Q;
  if (nk >= NA)
    wait_vm<IA *(NA - 1) + IB *(NB - 1)>();
  else
    wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < NF; ++i) rd(P, i, 0, 0, 0);

  // The products of part F, with the reads of part H into G (two a product)
  // and COUNT loads spread evenly between them.  The weights are the MFMA's
  // first operand: a lane's results are then four consecutive features of one
  // row, one wide store.
  constexpr int M2 = MX * NY;
#define MOE_PART(F, G, ATA, ATB, H, COUNT, LOAD)                                                         \
  _Pragma("unroll") for (int m = 0; m < M2; ++m) {                                                       \
    _Pragma("unroll") for (int i = 0; i < NF; ++i) if (i / 2 == m || (m == M2 - 1 && i / 2 > m)) rd(G, i, ATA, ATB, H); \
    c[m / YW][m % YW] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F.b[m % YW], F.a[m / YW], c[m / YW][m % YW], 0, 0, 0);  \
    __builtin_amdgcn_sched_barrier(0);                                                                   \
    _Pragma("unroll") for (int q = 0; q < (COUNT); ++q)                                                  \
      if (q * M2 / max((COUNT), 1) == m) {                                                               \
        LOAD;                                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                                               \
      }                                                                                                  \
  }
  // Step s multiplies slice s.  Loads of A slice s + 2 go, in its first two
  // parts, to the place of slice s - 1 (every wave has read it: the barrier of
  // step s - 1), and loads of B slice s + NB, after the barrier, to the place
  // of slice s.  At the barrier slice s + 1 has landed: younger than it are A
  // slices up to s + 2 and B slices up to s + NB - 1.
  constexpr int A0 = (IA + 1) / 2, A1 = IA - A0;
  uint32_t at_a = 0, at_b = 0, old_a = 0;
  for (int s = 0; s < nk; ++s) {
    const uint32_t next_a = at_a + AB == NA * AB ? 0 : at_a + AB;
    const uint32_t next_b = at_b + BB == NB * BB ? 0 : at_b + BB;
    const bool more_a = s > 0 && s + NA - 1 < nk, more_b = s + NB < nk;
    __builtin_amdgcn_sched_barrier(0);
    MOE_PART(P, Q, at_a, at_b, 1, A0, if (more_a) load_a(q, s + NA - 1, old_a))
    MOE_PART(Q, P, at_a, at_b, 2, A1, if (more_a) load_a(A0 + q, s + NA - 1, old_a))
    MOE_PART(P, Q, at_a, at_b, 3, 0, )
    if (s + NA - 1 < nk)
      wait_vm<IA *(NA - 2) + IB *(NB - 2)>();
    else
      wait_vm<0>();
    wait_lds();  // this wave's reads of slice s are done
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    MOE_PART(Q, P, next_a, next_b, 0, IB, if (more_b) load_b(q, s + NB, at_b))  // past the last slice: unused bytes
    old_a = at_a;
    at_a = next_a;
    at_b = next_b;
  }
#undef MOE_PART

  // a lane holds row lane % 32 of each block and its features 8 g + 4 (lane / 32) + 0 .. 3
#pragma unroll
  for (int x = 0; x < XW; ++x) {
    const int m = (wm * XW + x) * 32 + r32;
    if (m >= t.rows) continue;
    const size_t row = (size_t)(t.row + m) * N;
    if (UP) {
      uint16_t *o = static_cast<uint16_t *>(out) + row;
      constexpr int G = kMixed ? 2 : 4;  // groups of four features a block of W1 rows makes
#pragma unroll
      for (int y = 0; y < (kMixed ? 1 : YM); ++y)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int n = t.n0 + 8 * G * (wn * (kMixed ? 1 : YM) + y) + 8 * g + 4 * hi;
          if (n < N) {
            uint32_t v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              v[i] = bf16_rne(silu(c[x][y][4 * g + i]) * (kMixed ? c[x][0][8 + 4 * g + i] : c[x][YW - YM + y][4 * g + i]));
            *reinterpret_cast<u32x2 *>(o + n) = u32x2{v[0] | (v[1] << 16), v[2] | (v[3] << 16)};
          }
        }
    } else {
      float *o = static_cast<float *>(out) + row;
#pragma unroll
      for (int y = 0; y < YW; ++y)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = t.n0 + 32 * (YW * wn + y) + 8 * g + 4 * hi;
          if (n < N)
            *reinterpret_cast<floatx4 *>(o + n) =
                floatx4{c[x][y][4 * g], c[x][y][4 * g + 1], c[x][y][4 * g + 2], c[x][y][4 * g + 3]};
        }
    }
  }
}

// Workgroup i runs on XCD i % 8, and tiles that run together on an XCD should
// share their A and B panels in its L2, so each XCD works through contiguous
// stretches of the list.  Short lists (below four tiles a CU) are cut into one
// stretch an XCD: they are bound by streaming weights, and XCDs that read
// different experts' do that faster.  Long lists are dealt in runs of as many
// tiles as an XCD multiplies at once, so that every XCD gets its part of each
// expert (tiles of different experts differ in height), with the last,
// incomplete deal spread over all.  us a pass with one stretch always / so /
// runs from 256 tiles on: 32 tokens of top-8 over 64 experts 222 / 222 / 229, 509
// tokens 253 / 252 / 277, 4096 tokens 735 / 722 / 720, 2048 tokens of top-2 over 8
// experts 1518 / 1484 / 1473.
constexpr int kXcds = 8, kXcdRun = 32, kLongList = 4 * kXcds * kXcdRun;

__device__ __forceinline__ int xcd_tile(int b, int n) {
  const int x = b % kXcds, i = b / kXcds, deals = n >= kLongList ? n / (kXcds * kXcdRun) : 0;
  const int dealt = deals * kXcdRun;  // of each XCD
  if (i < dealt) return (i / kXcdRun * kXcds + x) * kXcdRun + i % kXcdRun;
  const int left = n - dealt * kXcds, per = left / kXcds, rem = left % kXcds;
  return dealt * kXcds + x * per + min(x, rem) + i - dealt;
}

// Wide tiles: up to 256 rows by 256 weight rows, one workgroup a CU.  Narrow
// ones: up to 64 rows by 128, two workgroups a CU.  list: where the launch's
// tiles start and how many there are (never more than the grid; the surplus
// workgroups exit).
template <bool UP, bool RAGGED, bool WIDE>
__global__ __launch_bounds__(kThreads, WIDE ? 1 : 2) void prefill_gemm_kernel(const GemmTile *tiles, const int32_t *ntiles,
                                                                             const uint16_t *a_src, const int32_t *perm_tok,
                                                                             void *out, int d, int d_ff) {
  constexpr int LDS = WIDE ? 160 * 1024 : 72 * 1024;
  __shared__ __align__(1024) uint8_t lds[LDS];
  const int nt = ntiles ? min(*ntiles, (int)gridDim.x) : (int)gridDim.x;
  if ((int)blockIdx.x >= nt) return;
  const GemmTile t = tiles[xcd_tile(blockIdx.x, nt)];
  if (t.rows <= 0 || t.rows > (WIDE ? kWideRows : kNarrowRows)) return;  // the planners make no such tiles
  // (from six row blocks on a tile is bound by its products either way)
#define MOE_CASE(M)                                                                                      \
  case M:                                                                                                \
    if (M <= kOnceBlocks && t.once)                                                                      \
      gemm_tile<UP, RAGGED, M, M <= kOnceBlocks, WIDE ? 2 : 1, LDS>(t, a_src, perm_tok, out, d, d_ff, lds); \
    else                                                                                                 \
      gemm_tile<UP, RAGGED, M, false, WIDE ? 2 : 1, LDS>(t, a_src, perm_tok, out, d, d_ff, lds);         \
    break;
  if constexpr (WIDE) {
    switch ((t.rows + 31) / 32) {
      MOE_CASE(1) MOE_CASE(2) MOE_CASE(3) MOE_CASE(4) MOE_CASE(5) MOE_CASE(6) MOE_CASE(7) MOE_CASE(8)
    }
  } else {
    switch ((t.rows + 31) / 32) { MOE_CASE(1) MOE_CASE(2) }
  }
#undef MOE_CASE
}

template <bool UP>
hipError_t launch_gemm(const GemmTile *tiles, const int32_t *ntiles, int grid, bool wide, const uint16_t *a_src,
                       const int32_t *perm_tok, void *out, int d, int d_ff, const Launch &l) {
  if (grid <= 0) return hipSuccess;
  const bool ragged = (UP ? d : d_ff) % kKs != 0;
#define MOE_GEMM(R, W) \
  MOE_LAUNCH((prefill_gemm_kernel<UP, R, W>), dim3(grid), dim3(kThreads), 0, l, tiles, ntiles, a_src, perm_tok, out, d, d_ff)
  if (wide) {
    if (ragged) MOE_GEMM(true, true); else MOE_GEMM(false, true);
  } else {
    if (ragged) MOE_GEMM(true, false); else MOE_GEMM(false, false);
  }
#undef MOE_GEMM
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_up(const GemmTile *tiles, const int32_t *ntiles, int grid, bool wide, const uint16_t *xn,
                             const int32_t *perm_tok, uint16_t *act, int d, int d_ff, const Launch &l) {
  return launch_gemm<true>(tiles, ntiles, grid, wide, xn, perm_tok, act, d, d_ff, l);
}

hipError_t launch_prefill_down(const GemmTile *tiles, const int32_t *ntiles, int grid, bool wide, const uint16_t *act,
                               float *Y, int d, int d_ff, const Launch &l) {
  return launch_gemm<false>(tiles, ntiles, grid, wide, act, nullptr, Y, d, d_ff, l);
}

}  // namespace moe
