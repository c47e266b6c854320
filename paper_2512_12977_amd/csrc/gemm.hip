// GEMMs of the recomputed rows: C[M,N] = epilogue(A[M,K] * W[N,K]^T), both operands K-contiguous.
//   bf16: MFMA (v_mfma_f32_16x16x32_bf16), LDS-tiled, float accumulation.
//   f32 : MFMA (v_mfma_f32_16x16x4_f32) from registers (the small fp32 configuration).
// Epilogues: + bias, + residual (optionally gathered through a row map), SwiGLU of a gate|up pair.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rope_device.h"
#include "vlc_internal.h"

namespace vlc {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // a 16-byte chunk (native vector: stays in registers)

__device__ __forceinline__ float bf16_to_f32(uint16_t u) { return __uint_as_float(((uint32_t)u) << 16); }
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {   // round to nearest, ties to even
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
// two floats -> packed bf16 pair with the hardware conversion (round to nearest even), one instruction
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// x * sigmoid(x) with the hardware reciprocal (1 ulp) instead of an IEEE division (a dozen instructions per
// element in an epilogue during which the MFMAs are idle); the result is rounded to bf16 anyway
__device__ __forceinline__ float silu_f(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// ---------------------------------------------------------------------------------------------
// tile id -> (tile_m, tile_n).  Workgroups are dealt round-robin to the 8 XCDs, each with its own
// L2; the remap hands every XCD one contiguous range of tile ids, and inside a range tiles are
// walked in groups of GROUP_M row-tiles so that concurrently resident tiles share A and W panels.
// ---------------------------------------------------------------------------------------------
constexpr int kXcds = 8;
constexpr int kGroupM = 8;

__device__ __forceinline__ int xcd_contiguous(int pid, int total) {
  const int per = total / kXcds;
  return pid < per * kXcds ? (pid % kXcds) * per + pid / kXcds : pid;
}

template <bool REMAP = true>
__device__ __forceinline__ void tile_coords(int pid, int total, int tiles_m, int tiles_n, int* tm, int* tn) {
  const int vid = REMAP ? xcd_contiguous(pid, total) : pid;
  const int in_group = kGroupM * tiles_n;
  const int group = vid / in_group;
  const int first_m = group * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int r = vid - group * in_group;
  *tm = first_m + r % gm;
  *tn = r / gm;
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA kernel
// ---------------------------------------------------------------------------------------------
// Workgroup tile BM x BN, WGM x WGN wavefronts, wavefront tile (BM/WGM) x (BN/WGN) made of 16x16
// MFMA tiles.  The MFMA "A" operand is the W fragment and the "B" operand the activation fragment,
// so an accumulator tile is indexed [n][m]: lane l holds, for m = l % 16, the outputs
// n = 4*(l/16) + j (j = register index): four consecutive n per lane, i.e. 8 contiguous bytes of a bf16 C row.
//
// 16x16x32 and not 32x32x16: the large products run at the power limit of the card, and a loop of nothing but MFMAs on
// random operands reaches 2.04 (one wavefront per SIMD) to 2.18 PFLOP/s with 16x16x32 there (vlc_probe_mfma_bf16), 1.70 to 1.82
// with 32x32x16 (2.4 both on constants).  7B at 18944 rows, before /
// after: gate|up 3944 / 3782 us, down 2086 / 1957; at 5824 rows gate|up 1258 / 1211.
//
// Operands reach LDS straight from global memory (global_load_lds, 16 bytes per lane, no register
// staging) through a ring of STAGES k-tiles of 64 columns, so the next k-tiles are in flight while
// the current one is consumed.  The instruction stream of a k-tile is laid out in groups of MFMAs, each preceded by its share
// of fragment reads and of the loads that refill a stage; sched_barrier keeps the compiler from regrouping them.  A
// wavefront-level load writes 64 consecutive 16-byte chunks of LDS in lane order (whole 128-byte lines of 8 rows: loads of
// 64-byte pieces, which a 32-wide k-tile would need, reach half the rate, 18 against 35 TB/s from L2); the XOR swizzle of the
// fragment reads is therefore applied on the global side (which chunk of its row each lane
// fetches).  Fragments are double-buffered in registers across the two 32-wide k-steps.
//
// SPLIT > 1 (few output tiles): each workgroup reduces one contiguous range of k-tiles and
// writes float partials; splitk_epilogue_kernel sums them and applies the epilogue.
//
// Tail split: when the tile count is not a multiple of the workgroups the chip holds at once, the
// last, partly filled round would cost as much as a full one.  The tiles of that round (ids from
// full_tiles on) are then shared out over tail_splits workgroups each, along k; these write their
// accumulators as float blocks to tail_ws and tail_reduce_kernel sums them and applies the epilogue.
//
// RESIDENT: one round of workgroups stays for all tiles and asks for the next tile's first k-tiles under the last k-step of
// this one (tile_may_stay, gemm_stays): no workgroup starts, reads its arguments and waits for its first k-tiles in
// between.  Products of few k-tiles gain most: gate|up / down of 128 experts (2048 x 768) at 444 rows each 378 -> 361 and 260 -> 248
// us, at 4000 2654 -> 2644 and 1853 -> 1780; 7B gate|up at 5824 rows 1157 -> 1131.  The next tile's place costs scalar registers: all
// are taken, and 16 ... 62 spilled to lanes of a vector register outside the k-loop.  Products that stream their weights
// through small tiles are no faster (37 rows per expert) or slower.  The tiles are dealt once and for all, so a workgroup that
// another stream's kernel keeps waiting holds up its whole share of them.
//
// The epilogue reads its residual rows (and bias) ahead of the stores, and whole tiles store without a condition: each
// 16 x 16 output tile under a condition of its own is a memory round trip, the compiler waits for its load in front of its store.
// q|k|v at 5824 rows (7B, 320 x 192) 189 -> 168 us, O 165 -> 153; O at 900 rows (128 x 128) 37.4 -> 35.7, q|k|v 43 -> 40.5.
constexpr int BK = 64;

// A fragment read takes 16 bytes of 16 consecutive rows in four neighbouring chunks of 8 elements.  The LDS serves it in
// four turns of 16 lanes (0-3, 12-15, 20-27; 4-11, 16-19, 28-31; the same + 32), 256 bytes each: with chunk ^ (row % 8) every turn
// touches all 64 banks once.  (With one more bit of the row in it, which suits rows 0-31 of one chunk, every turn takes two.)
__device__ __forceinline__ int fswz(int row) { return row & 7; }

// One wavefront-level global -> LDS copy of 64 x 16 bytes: lane l's 16 bytes land at lds_byte_addr + 16*l.
// Written as inline assembly rather than through the builtin because the compiler, seeing an LDS
// write it cannot order against the fragment reads, waits for every outstanding LDS access before
// each k-step; issued this way the loads are tracked only by the explicit vmcnt waits below (the
// loop contains no other vector-memory instruction).  M0 holds the LDS address; the compiler never
// keeps a live value in M0 across statements (it is reserved and written right before each use).
// The global address is a wavefront-uniform base (scalar registers) plus a 32-bit byte offset per lane: the lane
// offsets never change, the base moves along k with scalar adds, so the k-loop holds no vector address arithmetic
// (a wavefront's own vector instructions run under its MFMAs, but an MFMA lasts only 16 cycles, four instructions).
__device__ __forceinline__ void dma16(const void* uniform_base, uint32_t lane_byte_off, uint32_t lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_byte_addr), "v"(lane_byte_off), "s"(uniform_base)
               : "memory");
}

// acc += W fragment x activation fragment, in place.  Written as an instruction because the compiler, free to give the result
// of the builtin other registers than the addend, moved half of the accumulators once per k-tile (452 moves beside 240
// MFMAs in the loop of 320 x 192).  accumulation_regs is a constant of the unrolled code.
// The compiler's own waits know nothing of these instructions.  One takes 4 passes, and what is no MFMA that adds to its result
// may touch that only 8 wait states later; inside the loop nothing does, and the last k-step of a workgroup takes
// mfma_add_last, whose wait is part of the same statement: a copy or a spill of an accumulator, which the compiler may
// place right behind the statement that wrote it, comes after the wait.  (One wait behind the loop left room in front of it:
// in 256 x 256 on four wavefronts and in 320 x 256, 2 to 14 accumulators were spilled there.)
__device__ __forceinline__ void mfma_add(f32x4& acc, const bf16x8& w, const bf16x8& a, bool accumulation_regs) {
  if (accumulation_regs)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(a));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(a));
}
// N of them and one wait, about 20 cycles per statement over the MFMAs' own.  In statements of 8 that hardly shows (7B prefill of
// 596 rows 1248 / 1245 and 1271 / 1275 us, before / after, on two cards); in statements of 4 it was 1275 / 1283.
template <int N>
__device__ __forceinline__ void mfma_add_last(f32x4* const (&c)[N], const bf16x8* const (&w)[N], const bf16x8* const (&a)[N],
                                              bool accumulation_regs) {
  static_assert(N == 8 || N == 4 || N == 1, "statements of 8, 4 or 1 tiles");
#define VLC_MFMA(C, W, A) "v_mfma_f32_16x16x32_bf16 %" #C ", %" #W ", %" #A ", %" #C "\n\t"
#define VLC_LAST_1(R) asm volatile("s_nop 1\n\t" VLC_MFMA(0, 1, 2) "s_nop 7" : "+" R(*c[0]) : "v"(*w[0]), "v"(*a[0]))
#define VLC_LAST_4(R)                                                                                              \
  asm volatile("s_nop 1\n\t" VLC_MFMA(0, 4, 8) VLC_MFMA(1, 5, 9) VLC_MFMA(2, 6, 10) VLC_MFMA(3, 7, 11) "s_nop 7"                  \
               : "+" R(*c[0]), "+" R(*c[1]), "+" R(*c[2]), "+" R(*c[3])                                            \
               : "v"(*w[0]), "v"(*w[1]), "v"(*w[2]), "v"(*w[3]), "v"(*a[0]), "v"(*a[1]), "v"(*a[2]), "v"(*a[3]))
#define VLC_LAST_8(R)                                                                                              \
  asm volatile("s_nop 1\n\t" VLC_MFMA(0, 8, 16) VLC_MFMA(1, 9, 17) VLC_MFMA(2, 10, 18) VLC_MFMA(3, 11, 19)                       \
               VLC_MFMA(4, 12, 20) VLC_MFMA(5, 13, 21) VLC_MFMA(6, 14, 22) VLC_MFMA(7, 15, 23) "s_nop 7"           \
               : "+" R(*c[0]), "+" R(*c[1]), "+" R(*c[2]), "+" R(*c[3]), "+" R(*c[4]), "+" R(*c[5]), "+" R(*c[6]),  \
                 "+" R(*c[7])                                                                                      \
               : "v"(*w[0]), "v"(*w[1]), "v"(*w[2]), "v"(*w[3]), "v"(*w[4]), "v"(*w[5]), "v"(*w[6]), "v"(*w[7]),    \
                 "v"(*a[0]), "v"(*a[1]), "v"(*a[2]), "v"(*a[3]), "v"(*a[4]), "v"(*a[5]), "v"(*a[6]), "v"(*a[7]))
  if constexpr (N == 8) {
    if (accumulation_regs) VLC_LAST_8("a");
    else VLC_LAST_8("v");
  } else if constexpr (N == 4) {
    if (accumulation_regs) VLC_LAST_4("a");
    else VLC_LAST_4("v");
  } else {
    if (accumulation_regs) VLC_LAST_1("a");
    else VLC_LAST_1("v");
  }
#undef VLC_LAST_8
#undef VLC_LAST_4
#undef VLC_LAST_1
#undef VLC_MFMA
}
// A vector instruction's result may be read by an MFMA two wait states later: the zeroed accumulators pass through here
// before the wait in front of the loop.
__device__ __forceinline__ void mfma_operand(f32x4& acc, bool accumulation_regs) {
  if (accumulation_regs)
    asm volatile("" : "+a"(acc));
  else
    asm volatile("" : "+v"(acc));
}

enum { EPI_PARTIAL = 100 };   // internal: float partial sums of one k-range (split-K)

#define VLC_WAITCNT_VM(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (7 << 4) | (15 << 8) | (((N) >> 4) << 14))

// Whether the workgroups of a kernel can stay for several tiles (RESIDENT; tile_may_stay): tiles of 160 x 256 outputs and more on four
// wavefronts, where products of more than kStayRounds rounds land on them (over 240000 products of decoder proportions, up to 60000
// rows, residuals on two tiles only).  Not 320 x 256, whose sums and fragments leave no registers for the next tile's addresses, nor
// eight wavefronts, two per SIMD, which fill each other's waits (and spill).  Not float outputs either: the waits for the next tile's
// k-tiles also wait for the stores in front of them, twice the bytes here.  q|k|v at K = 1536 ... 5120 in 3.5 to 7 rounds is slower by
// staying in 77 of 84 products, 1.8 % on average and up to 5.4, going / staying: 320 x 192 at K = 2048 in 7 rounds 356 / 377 us, 320 x 160 at K = 4096 in 4 rounds
// 323 / 327, 192 x 256 at K = 3584 in 5.5 rounds 405 / 413.
constexpr int kStayRounds = 3, kStayManyRounds = 20;
constexpr int64_t kStayOperands = 400000000;   // bytes of A and W
// Whether the workgroups of a product stay: from more than kStayRounds rounds on (items: tiles, and the k ranges of a split last
// round's; between 3 and 4 rounds SwiGLU and residuals gain 3 ... 6 % at K = 1024, 1 ... 2 % at 3584, 0 ... 1 % at 8192, and not much less from
// 1.5 rounds on), and over more than kStayManyRounds only if the operands are not much more than the memory-side cache holds (256 MB).
// The tiles are dealt once and for all, so nothing keeps the XCDs in step over many of them; one that is behind would fetch from HBM
// again what the others have used.  Gate|up of eight shapes, 5200 ... 38000 rows, going / staying, us: up to 20 rounds staying gains 1.7 % on
// average whatever the operands (-0.4 ... 4.1; 72B at 5200 rows, 19 rounds, 1054 MB: 3543 / 3503), beyond them 1.6 % up to 400 MB (0.2 ... 4.4;
// 1.5B at 31000, 33 rounds, 150 MB: 1349 / 1314; 7B at 16500, 38 rounds, 390 MB: 3150 / 3127) and loses 2.6 % over more (0.8 ... -8.3; 7B at
// 18944, 43 rounds, 408 MB: 3706 / 3759; 13824 x 5120 at 38000, 63 rounds: 7918 / 8637; 72B at 7500, 27 rounds: 5269 / 5560).
bool gemm_stays(bool may, int64_t items, int slots, int64_t operand_bytes) {
  return may && items > kStayRounds * slots && (items <= kStayManyRounds * slots || operand_bytes <= kStayOperands);
}

//
// GROUPED (mixture-of-experts): the row tiles come from a device-resident table; entry t holds an
// expert and the range [m0, m_end) of rows it owns (at most BM of them); the tile multiplies these
// rows - fetched through amap when given - with that expert's matrix W + expert * w_stride.
// Workgroups beyond the table's length (only known on the device) exit at once, and the XCDs share out the tiles that
// are there (dealt by the largest possible length, 37 rows per expert left two of the eight XCDs idle).
template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, bool RESIDENT, bool GROUPED>
__device__ __forceinline__ void gemm_bf16_items(
    const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ W, uint16_t* __restrict__ C,
    int64_t ldc, int M, int N, int K, const uint16_t* __restrict__ bias, const uint16_t* __restrict__ resid,
    int64_t ldr, const int32_t* __restrict__ rmap, int tiles_m, int tiles_n, int kt_per_split, int full_tiles,
    int tail_splits, int items, float* __restrict__ tail_ws, const GroupTile* __restrict__ gtab,
    const int32_t* __restrict__ g_ntiles, const int32_t* __restrict__ amap, int64_t w_stride) {
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;      // wavefront tile
  constexpr int MT = WM / 16, NT = WN / 16;        // MFMA tiles per wavefront
  constexpr int STAGE_CHUNKS = (BM + BN) * 8;      // 16-byte chunks per stage
  constexpr int A_INSTR = BM * 8 / 64 / NW, W_INSTR = BN * 8 / 64 / NW;   // wavefront loads per k-tile
  constexpr int LOADS = A_INSTR + W_INSTR;
  constexpr int KS = BK / 32;
  constexpr bool TAIL = !GROUPED && EPI != EPI_PARTIAL;
  static_assert(KS == 2, "two k-steps per k-tile");
  // columns of C covered by this tile: SwiGLU consumes a gate and an up row per output column
  constexpr int CN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  static_assert(STAGES >= 2 && STAGES <= 6, "ring depth");
  // SwiGLU pairs a gate and an up column inside a lane: the first half of the tile's W rows (= LDS rows) are gate rows, the
  // others the up rows of the same outputs, N rows further in the matrix; a wavefront's first NT/2 tiles are gate columns.
  static_assert(EPI != EPI_SWIGLU || NT % 2 == 0, "gate and up tiles come in pairs");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* lds = reinterpret_cast<u32x4*>(smem);

  if constexpr (GROUPED) {   // the table's real length: every XCD gets its share of what is there, the rest leaves
    tiles_m = *g_ntiles;
    items = full_tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= items) return;
  }
  const int tiles = tiles_m * tiles_n;
  // what a workgroup multiplies next: a tile of C, one k range of it, or one k range of a tail tile (tail_block >= 0)
  struct Item {
    int split, tail_block, tn, m0, m_end, n0, expert;
  };
  auto locate = [&](int item) {
    Item t = {0, -1, 0, 0, M, 0, 0};
    int pid = item;
    if constexpr (EPI == EPI_PARTIAL) {
      // all items (k range major) are dealt to the XCDs in contiguous pieces: an XCD then works on one or two
      // k ranges and its L2 holds only their slices of A, instead of every XCD streaming all of A
      const int b = xcd_contiguous(item, items);
      t.split = b / tiles;
      pid = b - t.split * tiles;
    } else if (item >= full_tiles) {
      t.tail_block = item - full_tiles;
      const int tail = t.tail_block / tail_splits;
      t.split = t.tail_block - tail * tail_splits;
      pid = full_tiles + tail;
    }
    int tm;
    tile_coords<EPI != EPI_PARTIAL>(pid, tiles, tiles_m, tiles_n, &tm, &t.tn);
    t.m0 = tm * BM;
    t.n0 = t.tn * CN;
    if constexpr (GROUPED) {
      const GroupTile g = gtab[tm];
      t.m0 = g.m0;
      t.m_end = g.m_end;
      t.expert = g.expert;
    }
    return t;
  };

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lane = tid & 63;
  const int wm = wave / WGN, wn = wave % WGN;

  // Experts with few rows read their weights once: the column tiles start at different k-tiles and walk around the end of the
  // range.  In step, all of them ask for the same 128 bytes out of 4 KiB at a time (rows of 2048 are 4 KiB apart), which few
  // channels hold.  The start depends on the column tile and the expert alone, so that a row's sums do not depend on its place in
  // the table.  Us per pass of
  // three layers (128 experts, 2048 x 768), before / after: 6 rows per expert 883 / 865, 37 rows 1073 / 1051.  Not for the
  // dense products: the wrap costs them 0.4 ... 1 % where several row tiles share the weights (7B at 596 rows), and
  // with one row tile the gain is 0.5 % (rows of 3584; the heads: none).
  constexpr bool WRAP = GROUPED && STAGES > 2;
  int KT = 0, k_first = 0;
  auto k_tile = [&](int kt) { return WRAP ? kt + (kt + k_first < KT ? k_first : k_first - KT) : kt; };

  // ---- global source of each of this wavefront's loads: a uniform base (first row of the tile, first k-tile) and a
  // per-lane byte offset.  Rows fetched through amap are offsets from A itself.
  uint32_t a_lane[A_INSTR], w_lane[W_INSTR];
  const uint16_t *a_base = nullptr, *w_base = nullptr;
  const bool mapped = GROUPED && amap != nullptr;
  int a_row[A_INSTR];                                      // mapped: rows of A behind this lane's rows of the tile
  auto fetch_rows = [&](const Item& t) {
    if constexpr (GROUPED) {
      if (mapped) {
#pragma unroll
        for (int i = 0; i < A_INSTR; ++i) a_row[i] = amap[min(t.m0 + (((wave * A_INSTR + i) * 64 + lane) >> 3), t.m_end - 1)];
      }
    }
  };
  auto aim = [&](const Item& t) {
    const int kt_begin = t.split * kt_per_split;
    KT = ((EPI == EPI_PARTIAL || t.tail_block >= 0) ? min(K / BK, kt_begin + kt_per_split) : K / BK) - kt_begin;
    k_first = WRAP ? (t.tn + 5 * t.expert) % KT : 0;
    a_base = A + (mapped ? (int64_t)0 : (int64_t)t.m0 * lda) + (int64_t)kt_begin * BK;
    w_base = W + (int64_t)t.expert * w_stride + (int64_t)t.n0 * K + (int64_t)kt_begin * BK;
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
      const int p = (wave * A_INSTR + i) * 64 + lane;        // LDS chunk this lane fills
      const int r = p >> 3, c = (p & 7) ^ fswz(r);
      int64_t rel = min(r, t.m_end - 1 - t.m0);              // ragged tail: re-read the last row
      if constexpr (GROUPED) {
        if (mapped) rel = a_row[i];
      }
      a_lane[i] = (uint32_t)((rel * lda + c * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < W_INSTR; ++i) {
      const int p = (wave * W_INSTR + i) * 64 + lane;
      const int r = p >> 3, c = (p & 7) ^ fswz(r);
      const int row = EPI == EPI_SWIGLU && r >= BN / 2 ? N + r - BN / 2 : r;
      const int last = (EPI == EPI_SWIGLU ? 2 * N : N) - 1 - t.n0;
      w_lane[i] = (uint32_t)(((int64_t)min(row, last) * K + c * 8) * 2);
    }
  };
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  // LDS byte address of this wavefront's i-th load of a stage (A part first, then W)
#define VLC_LDS_DST(stage_, i_)                                                                              \
  (lds_base + (uint32_t)(((stage_) * STAGE_CHUNKS +                                                           \
                          ((i_) < A_INSTR ? wave * A_INSTR * 64 + (i_) * 64                                  \
                                          : BM * 8 + wave * W_INSTR * 64 + ((i_) - A_INSTR) * 64)) * 16))
#define VLC_DMA(kt_, i_, stage_)                                                                              \
  dma16(((i_) < A_INSTR ? a_base : w_base) + k_tile(kt_) * BK,                                              \
        (i_) < A_INSTR ? a_lane[(i_) < A_INSTR ? (i_) : 0] : w_lane[(i_) >= A_INSTR ? (i_) - A_INSTR : 0],     \
        VLC_LDS_DST(stage_, i_))
#define VLC_ISSUE(kt_, stage_) _Pragma("unroll") for (int i = 0; i < LOADS; ++i) VLC_DMA(kt_, i, stage_);

  // Fragment positions inside a stage (chunk units) for every 32-wide k-step: one address per operand and k-step, the
  // tiles of a wavefront are whole multiples of 16 rows apart (the swizzle repeats every 16 rows) and sit in the
  // immediate offset of the read.
  constexpr int WR = (EPI == EPI_SWIGLU) ? WN / 2 : WN;
  static_assert(WR % 16 == 0 && WM % 16 == 0, "wavefront tiles start at multiples of 16 rows");
  auto w_row = [](int nt) { return (EPI == EPI_SWIGLU && nt >= NT / 2) ? BN / 2 + (nt - NT / 2) * 16 : nt * 16; };
  int w_off[KS], a_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int l16 = lane & 15, c = (4 * ks + (lane >> 4)) ^ fswz(l16);
    w_off[ks] = BM * 8 + (wn * WR + l16) * 8 + c;
    a_off[ks] = (wm * WM + l16) * 8 + c;
  }

  // one wavefront per SIMD: the first 64 tiles in accumulation registers, what is over in vector registers.  A multiple of
  // 8: mfma_add_last takes tiles of one kind.  Of 64 tiles 56, or the compiler, left with no free accumulation register, moves one
  // in the middle of the last k-tile.
  constexpr int ACC = OCC * NW > 4 ? 0 : RESIDENT && NT * MT == 64 ? 56 : 64;
  f32x4 acc[NT][MT];

  // One k-tile: two k-steps of G groups of MFMAs, the fragment reads of the next k-step spread over groups of this one.
  // ONE BARRIER, before the second k-step: every wavefront holds the fragments of that k-step by then, so the tile's stage
  // is free and is refilled under it, and the next k-tile (whose loads every wavefront has waited for) can be read: its
  // first fragments arrive under the second k-step's MFMAs.  The loads have STAGES - 1 k-tiles to arrive.
  // TWO barriers (rings of two stages on four wavefronts, where one k-tile is less than a miss takes): the reads of the
  // second k-step are pulled into the first RN groups of the first, the stage is refilled from there on, and the next k-tile is
  // waited for only before the last RN groups of the second k-step: half a k-tile more for the loads to arrive.
  // 7B gate|up at 900 rows on 192 x 256: 214 -> 202 us, O at 5824 rows 156 -> 140, gate|up at 18944 rows on 320 x 192 3735 -> 3700;
  // on eight wavefronts (256 x 256) the second barrier costs what the time gains, and two workgroups per CU fill each
  // other's waits.
  constexpr bool TWO = STAGES == 2 && OCC == 1 && NW == 4;
  constexpr int TILES = NT * MT;
  constexpr int MPG = TILES % 8 == 0 ? 8 : TILES % 6 == 0 ? 6 : TILES % 5 == 0 ? 5 : TILES % 4 == 0 ? 4 : TILES % 2 == 0 ? 2 : 1;   // MFMAs per group
  constexpr int G = TILES / MPG;               // groups per k-step
  constexpr int NF = NT + MT;                  // fragments per k-step
  bf16x8 wf[2][NT], af[2][MT];
#define VLC_READ_FRAGS(st_, ks_, buf_, g_)                                                                    \
  _Pragma("unroll") for (int f = 0; f < NF; ++f) {                                                            \
    if ((g_) < 0 || f * RN / NF == (g_)) {                                                                    \
      if (f < NT) wf[buf_][f < NT ? f : 0] = __builtin_bit_cast(bf16x8, (st_)[w_off[ks_] + w_row(f < NT ? f : 0) * 8]); \
      else af[buf_][f >= NT ? f - NT : 0] = __builtin_bit_cast(bf16x8, (st_)[a_off[ks_] + (f >= NT ? f - NT : 0) * 128]); \
    }                                                                                                         \
  }
  constexpr int RN = TWO ? (2 * G + 4) / 5 : G;            // groups that read the fragments of a k-step
  constexpr int L0 = TWO ? RN : G, LN = TWO ? 2 * (G - RN) : G;   // groups that refill the stage: LN from L0 on
  // The MFMAs of a k-step walk its tiles in a snake: one operand changes at a time.
  auto nt_of = [](int t) { return t / MT; };
  auto mt_of = [](int t) { return (t / MT & 1) ? MT - 1 - t % MT : t % MT; };
  // cst_ / nst_: stages of this and the next k-tile.  LOAD_: refill this tile's stage with k-tile lkt_; WAIT_: the wait that
  // leaves only the loads of the tiles after the next one in flight; NEXT_: there is a next tile.  GROUPS_: groups to run, 2 G or,
  // without the second k-step, G.
#define VLC_COMPUTE_TILE(cst_, nst_, LOAD_, lkt_, NEXT_, WAIT_, GROUPS_)                                      \
  {                                                                                                           \
    const u32x4* st_ = lds + (cst_) * STAGE_CHUNKS;                                                           \
    const u32x4* sn_ = lds + (nst_) * STAGE_CHUNKS;                                                           \
    _Pragma("unroll") for (int g = 0; g < (GROUPS_); ++g) {                                                   \
      if (TWO && g == L0 && (LOAD_)) __syncthreads();                                                         \
      if (g == 2 * G - RN && (NEXT_)) {                                                                       \
        WAIT_;                                                                                                \
        __syncthreads();                                                                                      \
      }                                                                                                       \
      if ((LOAD_) && g >= L0) {                                                                               \
        _Pragma("unroll") for (int i = 0; i < LOADS; ++i) if (i * LN / LOADS == g - L0) VLC_DMA(lkt_, i, cst_);   \
      }                                                                                                       \
      if (g < RN) { VLC_READ_FRAGS(st_, 1, 1, g) }                                                             \
      else if (g >= 2 * G - RN && (NEXT_)) { VLC_READ_FRAGS(sn_, 0, 0, g - (2 * G - RN)) }                     \
      __builtin_amdgcn_sched_barrier(0);                                                                      \
      _Pragma("unroll") for (int j = 0; j < MPG; ++j) {                                                       \
        const int t_ = g % G * MPG + j, nt_ = nt_of(t_), mt_ = mt_of(t_);                                      \
        mfma_add(acc[nt_][mt_], wf[g / G][nt_], af[g / G][mt_], t_ < ACC);                                     \
      }                                                                                                       \
      __builtin_amdgcn_sched_barrier(0);                                                                      \
    }                                                                                                         \
  }

  // One item after the other.  The next one's first k-tiles are asked for under the last k-step of this one, when its ring
  // is free, and arrive under that and the epilogue.
  int item = blockIdx.x;
  Item cur = locate(item);
  fetch_rows(cur);
  aim(cur);
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < KT) { VLC_ISSUE(s, s) }
  for (;;) {
  asm volatile("" : "+v"(lane));         // what follows from the lane is worked out anew for every item, not kept
  const bool more = RESIDENT && item + (int)gridDim.x < items;
  Item nxt = cur;
  if (more) {
    nxt = locate(item + (int)gridDim.x);
    fetch_rows(nxt);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < TILES; ++t) mfma_operand(acc[nt_of(t)][mt_of(t)], t < ACC);
  asm volatile("s_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  if (KT >= STAGES) { VLC_WAITCNT_VM((STAGES - 1) * LOADS); } else { VLC_WAITCNT_VM(0); }
  __syncthreads();
  VLC_READ_FRAGS(lds, 0, 0, -1)
  int kt = 0;
  // steady state: under the last k-step of k-tile kt its stage is refilled with k-tile kt + STAGES
  if constexpr (STAGES == 2) {
    // two k-tiles per trip, so that the stage every fragment address refers to is a constant of the code
    // and the addresses of both stages stay in registers (no address arithmetic inside the loop)
    for (; kt + 3 < KT; kt += 2) {
      VLC_COMPUTE_TILE(0, 1, true, kt + 2, true, VLC_WAITCNT_VM(TWO ? LOADS : 0), 2 * G)
      VLC_COMPUTE_TILE(1, 0, true, kt + 3, true, VLC_WAITCNT_VM(TWO ? LOADS : 0), 2 * G)
    }
    if (kt + 2 < KT) {
      VLC_COMPUTE_TILE(0, 1, true, kt + 2, true, VLC_WAITCNT_VM(TWO ? LOADS : 0), 2 * G)
      ++kt;
    }
  } else {
    for (; kt + STAGES < KT; ++kt)
      VLC_COMPUTE_TILE(kt % STAGES, (kt + 1) % STAGES, true, kt + STAGES, true, VLC_WAITCNT_VM((STAGES - 2) * LOADS), 2 * G)
  }
  for (; kt + 1 < KT; ++kt) {            // drain
    const int later = min(KT - 2 - kt, STAGES - 2);   // tiles after the next one still in flight
    VLC_COMPUTE_TILE(kt % STAGES, (kt + 1) % STAGES, false, 0, true,
                     { if (later >= 4) { VLC_WAITCNT_VM(4 * LOADS); } else if (later == 3) { VLC_WAITCNT_VM(3 * LOADS); } else if (later == 2) { VLC_WAITCNT_VM(2 * LOADS); } else if (later == 1) { VLC_WAITCNT_VM(LOADS); } else { VLC_WAITCNT_VM(0); } }, 2 * G)
  }
  // The last k-tile: nothing is left to read ahead.  Its MFMAs in front of a branch wait for their own results: the last group
  // of the first k-step, and all of the second.
#define VLC_ACC(t_) &acc[nt_of(t_)][mt_of(t_)]
#define VLC_W(b_, t_) &wf[b_][nt_of(t_)]
#define VLC_A(b_, t_) &af[b_][mt_of(t_)]
  // tiles [first_, first_ + count_) with the fragments of buffer b_; BEFORE_(j): in front of statement j
#define VLC_LAST(b_, first_, count_, BEFORE_)                                                                 \
  {                                                                                                           \
    _Pragma("unroll") for (int j = 0; j + 8 <= (count_); j += 8) {                                            \
      const int t = (first_) + j;                                                                             \
      BEFORE_(j / 8)                                                                                          \
      mfma_add_last<8>({VLC_ACC(t), VLC_ACC(t + 1), VLC_ACC(t + 2), VLC_ACC(t + 3), VLC_ACC(t + 4), VLC_ACC(t + 5), VLC_ACC(t + 6), VLC_ACC(t + 7)},  \
                       {VLC_W(b_, t), VLC_W(b_, t + 1), VLC_W(b_, t + 2), VLC_W(b_, t + 3), VLC_W(b_, t + 4), VLC_W(b_, t + 5), VLC_W(b_, t + 6), VLC_W(b_, t + 7)}, \
                       {VLC_A(b_, t), VLC_A(b_, t + 1), VLC_A(b_, t + 2), VLC_A(b_, t + 3), VLC_A(b_, t + 4), VLC_A(b_, t + 5), VLC_A(b_, t + 6), VLC_A(b_, t + 7)}, t < ACC); \
    }                                                                                                         \
    if constexpr ((count_) % 8 >= 4) {                                                                        \
      constexpr int t = (first_) + (count_) / 8 * 8;                                                          \
      BEFORE_((count_) / 8)                                                                                   \
      mfma_add_last<4>({VLC_ACC(t), VLC_ACC(t + 1), VLC_ACC(t + 2), VLC_ACC(t + 3)},                          \
                       {VLC_W(b_, t), VLC_W(b_, t + 1), VLC_W(b_, t + 2), VLC_W(b_, t + 3)},                  \
                       {VLC_A(b_, t), VLC_A(b_, t + 1), VLC_A(b_, t + 2), VLC_A(b_, t + 3)}, t < ACC);        \
    }                                                                                                         \
    _Pragma("unroll") for (int j = 0; j < (count_) % 4; ++j) {                                                \
      const int t = (first_) + (count_) / 4 * 4 + j;                                                          \
      BEFORE_((count_) / 8 + ((count_) % 8 >= 4 ? 1 : 0) + j)                                                 \
      mfma_add_last<1>({VLC_ACC(t)}, {VLC_W(b_, t)}, {VLC_A(b_, t)}, t < ACC);                                \
    }                                                                                                         \
  }
  VLC_COMPUTE_TILE(kt % STAGES, 0, false, 0, false, , G - 1)
  {
    const u32x4* st_ = lds + kt % STAGES * STAGE_CHUNKS;
    if (G - 1 < RN) { VLC_READ_FRAGS(st_, 1, 1, G - 1) }
    __builtin_amdgcn_sched_barrier(0);
  }
#define VLC_NOTHING(j_)
  VLC_LAST(0, TILES - MPG, MPG, VLC_NOTHING)
  __builtin_amdgcn_sched_barrier(0);
  int fill = 0;                          // stages of the next item to ask for
  if (more) {
    __syncthreads();                     // every wavefront holds its last fragments
    aim(nxt);
    fill = min(STAGES, KT);
  }
  __builtin_amdgcn_sched_barrier(0);
  constexpr int STATEMENTS = TILES / 8 + (TILES % 8 >= 4 ? 1 : 0) + TILES % 4;
  // its share of the next item's loads before statement j_
#define VLC_FILL(j_)                                                                                          \
  _Pragma("unroll") for (int s = 0; s < STAGES; ++s) {                                                        \
    if (s < fill) {                                                                                           \
      _Pragma("unroll") for (int i = 0; i < LOADS; ++i) if ((s * LOADS + i) * STATEMENTS / (STAGES * LOADS) == (j_)) VLC_DMA(s, i, s); \
    }                                                                                                         \
  }                                                                                                           \
  __builtin_amdgcn_sched_barrier(0);
  VLC_LAST(1, 0, TILES, VLC_FILL)
#undef VLC_FILL
#undef VLC_NOTHING
#undef VLC_LAST
#undef VLC_ACC
#undef VLC_W
#undef VLC_A
  __builtin_amdgcn_sched_barrier(0);

  // ---- epilogue ---------------------------------------------------------------------------------
  constexpr int ONT = (EPI == EPI_SWIGLU) ? NT / 2 : NT;   // output tiles along n per wavefront
  constexpr int OWN = (EPI == EPI_SWIGLU) ? WN / 2 : WN;   // output columns per wavefront
  const int l16 = lane & 15, lg = lane >> 4;
  // EDGE: rows or columns of the tile are past the end.  Bias and residual are read ahead of the stores (the bias once, the
  // residual of the next 16 rows before these are stored), past the end from the last valid place.
  // Every path takes the sums through mfma_operand first, so that the compiler does not copy all of them out of their registers
  // ahead of the paths.
  auto own = [&](int nt, int mt) { mfma_operand(acc[nt][mt], nt * MT + ((nt & 1) ? MT - 1 - mt : mt) < ACC); };
  auto finish = [&](auto edge) {
    constexpr bool EDGE = decltype(edge)::value;
    const int m_last = cur.m_end - 1;
    const int n_first = cur.n0 + wn * OWN + 4 * lg;        // + 16 * nt; N is a multiple of 4
    auto column = [&](int nt) { return EDGE ? min(n_first + nt * 16, N - 4) : n_first + nt * 16; };
    constexpr bool WITH_BIAS = EPI == EPI_BIAS_F32 /* EPI_BIAS: the experts' products, without one */, RESID = EPI == EPI_RESIDUAL;
    uint2 bias_q[WITH_BIAS ? NT : 1], resid_q[2][RESID ? NT : 1];
    int r_row[RESID ? MT : 1];
    if constexpr (WITH_BIAS) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) bias_q[nt] = make_uint2(0x80008000u, 0x80008000u);   // -0: adds nothing
      if (bias) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bias_q[nt] = *reinterpret_cast<const uint2*>(bias + column(nt));
      }
    }
    auto read_resid = [&](int mt) {
      const uint16_t* r = resid + (int64_t)r_row[RESID ? mt : 0] * ldr;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) resid_q[mt & 1][RESID ? nt : 0] = *reinterpret_cast<const uint2*>(r + column(nt));
    };
    if constexpr (RESID) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) r_row[mt] = EDGE ? min(cur.m0 + wm * WM + mt * 16 + l16, m_last) : cur.m0 + wm * WM + mt * 16 + l16;
      if (rmap) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) r_row[mt] = rmap[r_row[mt]];
      }
      read_resid(0);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = cur.m0 + wm * WM + mt * 16 + l16;
      if constexpr (RESID) {
        if (mt + 1 < MT) read_resid(mt + 1);
      }
      __builtin_amdgcn_sched_barrier(0);                   // one row of tiles after the other: few registers beside the sums
#pragma unroll
      for (int nt = 0; nt < ONT; ++nt) {
        const int n = n_first + nt * 16;
        if (EDGE && (m > m_last || n >= N)) continue;
        float v[4];
        own(nt, mt);
        if constexpr (EPI == EPI_SWIGLU) own(nt + NT / 2, mt);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[nt][mt][e];
        if constexpr (WITH_BIAS || RESID) {
          const uint2 b = WITH_BIAS ? bias_q[WITH_BIAS ? nt : 0] : resid_q[mt & 1][RESID ? nt : 0];
          v[0] += __uint_as_float(b.x << 16); v[1] += __uint_as_float(b.x & 0xffff0000u);
          v[2] += __uint_as_float(b.y << 16); v[3] += __uint_as_float(b.y & 0xffff0000u);
        } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = silu_f(v[e]) * acc[nt + NT / 2][mt][e];
        }
        if constexpr (EPI == EPI_PARTIAL) {
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + ((int64_t)cur.split * M + m) * ldc + n) =
              make_float4(v[0], v[1], v[2], v[3]);
        } else if constexpr (EPI == EPI_BIAS_F32) {        // unrounded float output (C is a float matrix)
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + (int64_t)m * ldc + n) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
          uint2 o;
          o.x = pack_bf16x2(v[0], v[1]);
          o.y = pack_bf16x2(v[2], v[3]);
          *reinterpret_cast<uint2*>(C + (int64_t)m * ldc + n) = o;
        }
      }
    }
  };
  if (TAIL && cur.tail_block >= 0) {
    // raw accumulators as a float block [BN/4][BM][4] (lanes of consecutive m write 512 contiguous bytes)
    float* P = tail_ws + (int64_t)cur.tail_block * (BM * BN);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        own(nt, mt);
        const int j = wn * WR + w_row(nt) + 4 * lg;        // SwiGLU: gate columns of the tile first, then its up columns
        *reinterpret_cast<float4*>(P + ((int64_t)(j >> 2) * BM + wm * WM + mt * 16 + l16) * 4) =
            make_float4(acc[nt][mt][0], acc[nt][mt][1], acc[nt][mt][2], acc[nt][mt][3]);
      }
    }
  } else if (cur.m0 + BM <= cur.m_end && cur.n0 + CN <= N) {
    finish(std::false_type{});
  } else {
    finish(std::true_type{});
  }
  if (!more) return;
  cur = nxt;
  item += (int)gridDim.x;
  }
#undef VLC_READ_FRAGS
#undef VLC_ISSUE
#undef VLC_DMA
#undef VLC_LDS_DST
#undef VLC_COMPUTE_TILE
}

// The entries.  What a workgroup needs for its first loads comes first: 14 words of arguments are in scalar registers when a
// workgroup starts (see build.py), the others it has to fetch.
template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, bool RESIDENT>
__global__ __launch_bounds__(WGM * WGN * 64, OCC) void gemm_bf16_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ W, int K, int N, int lda, int tiles_n, int M, int tiles_m,
    int kt_per_split, int full_tiles, int tail_splits, int items, uint16_t* __restrict__ C, int64_t ldc,
    const uint16_t* __restrict__ bias, const uint16_t* __restrict__ resid, int64_t ldr, const int32_t* __restrict__ rmap,
    float* __restrict__ tail_ws) {
  gemm_bf16_items<BM, BN, WGM, WGN, STAGES, OCC, EPI, RESIDENT, false>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, tiles_m,
                                                                       tiles_n, kt_per_split, full_tiles, tail_splits, items, tail_ws,
                                                                       nullptr, nullptr, nullptr, 0);
}
template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, bool RESIDENT, bool GROUPED>
__global__ __launch_bounds__(WGM * WGN * 64, OCC) void gemm_bf16_kernel(
    const int32_t* __restrict__ g_ntiles, const GroupTile* __restrict__ gtab, const int32_t* __restrict__ amap,
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ W, int K, int N, int lda, int tiles_n, int64_t w_stride,
    uint16_t* __restrict__ C, int64_t ldc) {
  static_assert(GROUPED, "the other entry");
  gemm_bf16_items<BM, BN, WGM, WGN, STAGES, OCC, EPI, RESIDENT, true>(A, lda, W, C, ldc, 0, N, K, nullptr, nullptr, 0, nullptr, 0,
                                                                      tiles_n, K / BK, 0, 1, 0, nullptr, gtab, g_ntiles, amap, w_stride);
}

// Sum of the split-K partials [splits][M][N] (float) + epilogue; one thread per 4 columns.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_epilogue_kernel(const float* __restrict__ P, int splits, int M, int N,
                                                              const uint16_t* __restrict__ resid, int64_t ldr,
                                                              const int32_t* __restrict__ rmap,
                                                              const uint16_t* __restrict__ bias,
                                                              uint16_t* __restrict__ C, int64_t ldc) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int nq = N / 4;
  const int64_t m = id / nq;
  const int n = (int)(id - m * nq) * 4;
  if (m >= M) return;
  // all loads first (independent), then the sum in split order
  float4 part[8];
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (k < splits) part[k] = *reinterpret_cast<const float4*>(P + ((int64_t)k * M + m) * N + n);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (k < splits) { s.x += part[k].x; s.y += part[k].y; s.z += part[k].z; s.w += part[k].w; }
  if constexpr (EPI == EPI_BIAS_F32) {
    if (bias) {
      const uint2 b = *reinterpret_cast<const uint2*>(bias + n);
      s.x += __uint_as_float(b.x << 16); s.y += __uint_as_float(b.x & 0xffff0000u);
      s.z += __uint_as_float(b.y << 16); s.w += __uint_as_float(b.y & 0xffff0000u);
    }
  } else if constexpr (EPI == EPI_RESIDUAL) {
    const int64_t rrow = rmap ? (int64_t)rmap[m] : m;
    const uint2 b = *reinterpret_cast<const uint2*>(resid + rrow * ldr + n);
    s.x += __uint_as_float(b.x << 16); s.y += __uint_as_float(b.x & 0xffff0000u);
    s.z += __uint_as_float(b.y << 16); s.w += __uint_as_float(b.y & 0xffff0000u);
  }
  if constexpr (EPI == EPI_BIAS_F32) {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + m * ldc + n) = s;
  } else {
    uint2 o;
    o.x = pack_bf16x2(s.x, s.y);
    o.y = pack_bf16x2(s.z, s.w);
    *reinterpret_cast<uint2*>(C + m * ldc + n) = o;
  }
}

// Sum over k-ranges of the tail tiles' float blocks + epilogue.  grid ((BM / 32) * ceil(QN / 16), tail tiles), QN = quads
// of output columns per tile; a workgroup owns 32 rows x 16 quads.  It reads the blocks as they lie (lanes: consecutive
// rows of a quad) and turns the sums around in LDS, so that residual and output are touched in pieces of whole rows
// (64 columns at a time): 66 tiles of 256 x 256 in three ranges 32 -> 13 us, against lanes that each stored
// 8 bytes of another row.
template <int BM, int BN, int EPI>
__global__ __launch_bounds__(256) void tail_reduce_kernel(const float* __restrict__ P, int splits, int full_tiles,
                                                          int tiles_m, int tiles_n, uint16_t* __restrict__ C,
                                                          int64_t ldc, int M, int N,
                                                          const uint16_t* __restrict__ bias,
                                                          const uint16_t* __restrict__ resid, int64_t ldr,
                                                          const int32_t* __restrict__ rmap) {
  constexpr int CN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int QN = CN / 4, QB = (QN + 15) / 16;
  __shared__ float4 turned[32][17];
  const int t = blockIdx.y;
  int tm, tn;
  tile_coords(full_tiles + t, tiles_m * tiles_n, tiles_m, tiles_n, &tm, &tn);
  const int r0 = (int)(blockIdx.x / QB) * 32, q0 = (int)(blockIdx.x % QB) * 16;
  const float* base = P + (int64_t)t * splits * (BM * BN);
  {
    const int ml = threadIdx.x & 31;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int ql = (threadIdx.x >> 5) + 8 * i, jq = q0 + ql;
      if (jq >= QN) break;
      const float* p = base + ((int64_t)jq * BM + r0 + ml) * 4;
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f), u = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int k0 = 0; k0 < splits; k0 += 4) {   // four ranges' loads together
        float4 a[4], b[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          a[k] = b[k] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (k0 + k < splits) {
            a[k] = *reinterpret_cast<const float4*>(p + (int64_t)(k0 + k) * (BM * BN));
            if constexpr (EPI == EPI_SWIGLU)
              b[k] = *reinterpret_cast<const float4*>(p + (int64_t)(k0 + k) * (BM * BN) + (int64_t)(BN / 8) * BM * 4);
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          s.x += a[k].x; s.y += a[k].y; s.z += a[k].z; s.w += a[k].w;
          if constexpr (EPI == EPI_SWIGLU) { u.x += b[k].x; u.y += b[k].y; u.z += b[k].z; u.w += b[k].w; }
        }
      }
      if constexpr (EPI == EPI_SWIGLU) {
        s.x = silu_f(s.x) * u.x; s.y = silu_f(s.y) * u.y; s.z = silu_f(s.z) * u.z; s.w = silu_f(s.w) * u.w;
      }
      turned[ml][ql] = s;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int id = i * 256 + (int)threadIdx.x, ml = id >> 4, ql = id & 15;
    const int m = tm * BM + r0 + ml, n = tn * CN + 4 * (q0 + ql);
    if (m >= M || n >= N || q0 + ql >= QN) continue;
    float4 s = turned[ml][ql];
    if constexpr (EPI == EPI_BIAS_F32) {
      if (bias) {
        const uint2 b = *reinterpret_cast<const uint2*>(bias + n);
        s.x += __uint_as_float(b.x << 16); s.y += __uint_as_float(b.x & 0xffff0000u);
        s.z += __uint_as_float(b.y << 16); s.w += __uint_as_float(b.y & 0xffff0000u);
      }
    } else if constexpr (EPI == EPI_RESIDUAL) {
      const int64_t rrow = rmap ? (int64_t)rmap[m] : (int64_t)m;
      const uint2 b = *reinterpret_cast<const uint2*>(resid + rrow * ldr + n);
      s.x += __uint_as_float(b.x << 16); s.y += __uint_as_float(b.x & 0xffff0000u);
      s.z += __uint_as_float(b.y << 16); s.w += __uint_as_float(b.y & 0xffff0000u);
    }
    if constexpr (EPI == EPI_BIAS_F32) {
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + (int64_t)m * ldc + n) = s;
    } else {
      uint2 o;
      o.x = pack_bf16x2(s.x, s.y);
      o.y = pack_bf16x2(s.z, s.w);
      *reinterpret_cast<uint2*>(C + (int64_t)m * ldc + n) = o;
    }
  }
}

// Four consecutive columns n ... n + 3 of row m (v; up: SwiGLU's second factor) through the epilogue.  resid_row: its first element.
template <int EPI>
__device__ __forceinline__ void store_f32(f32x4 v, const f32x4& up, int m, int n, int N, const float* __restrict__ bias,
                                          const float* __restrict__ resid, int64_t resid_row, float* __restrict__ C, int64_t ldc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (EPI == EPI_BIAS) {
      if (bias && n + e < N) v[e] += bias[n + e];
    } else if (EPI == EPI_RESIDUAL) {
      if (n + e < N) v[e] += resid[resid_row + n + e];
    } else {
      v[e] = v[e] / (1.0f + expf(-v[e])) * up[e];
    }
  }
  float* c = C + (int64_t)m * ldc + n;
  if (N % 4 == 0 && ldc % 4 == 0) {        // four columns of a row in one store
    if (n < N) *reinterpret_cast<f32x4*>(c) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < N) c[e] = v[e];
  }
}

// ---------------------------------------------------------------------------------------------
// f32 kernel: v_mfma_f32_16x16x4_f32 (exact fp32 products and sums) on operands loaded straight into registers
// ---------------------------------------------------------------------------------------------
// A wavefront owns MT x WT tiles of 16 x 16.  The W fragment is the MFMA "A" operand, so a lane ends up with four
// consecutive output columns of one row.  Lane l loads 16 bytes of row l % 16 at k = 16 * step + 4 * (l / 16): element
// e of all lanes is one k-slice of four for MFMA e (the order of k inside a step does not matter as long as both
// operands use the same).  Nothing is staged through LDS: the fp32 configuration is small, its time is latency.
//
// KW = 4 (few output tiles): the four wavefronts of a workgroup share one 16 x 16 output tile (two W tiles for
// SwiGLU) and take every fourth k-step each; their sums meet in LDS.  With 61 rows of the tiny decoder (K = 256 or
// 512) a product is 64 ... 128 workgroups and 4 ... 5 us, one memory latency and the launch; 64 x 64 tiles on vector
// instructions, 4 ... 8 workgroups walking k in 16-wide steps behind barriers, took 43 ... 98 us.
// KW = 1 (enough tiles for the chip): 2 x 2 wavefronts, each with its own output tiles; up to 106 TFLOP/s (47 before).
template <int MT, int NT, int WGM, int WGN, int KW, int EPI, bool GROUPED = false>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W, int K, int M,
                                                       int N, int lda, const float* __restrict__ bias,
                                                       const float* __restrict__ resid, const int32_t* __restrict__ rmap,
                                                       float* __restrict__ C, int64_t ldc, int64_t ldr,
                                                       const GroupTile* __restrict__ gtab,
                                                       const int32_t* __restrict__ g_ntiles,
                                                       const int32_t* __restrict__ amap, int64_t w_stride) {
  static_assert(WGM * WGN * KW == 4, "four wavefronts");
  constexpr int WT = (EPI == EPI_SWIGLU) ? 2 * NT : NT;   // W tiles: gate tiles, then the up tiles of the same columns
  constexpr int BM = WGM * MT * 16, BN = WGN * NT * 16;   // rows, output columns per workgroup
  constexpr int U = KW > 1 ? 4 : 1;                       // k-steps loaded together
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int kw = wave % KW, wm = wave / KW / WGN, wn = wave / KW % WGN;
  int m0 = blockIdx.y * BM;
  const int n0 = blockIdx.x * BN;
  if constexpr (GROUPED) {       // see gemm_bf16_kernel; a 64-row entry of the table is 64 / BM workgroups here
    constexpr int SUB = 64 / BM;
    if ((int)blockIdx.y / SUB >= *g_ntiles) return;
    const GroupTile g = gtab[blockIdx.y / SUB];
    m0 = g.m0 + (int)(blockIdx.y % SUB) * BM;
    M = min(g.m_end, g.m0 + 64);
    if (m0 >= M) return;
    W += (int64_t)g.expert * w_stride;
  }
  const float* ap[MT];
  const float* wp[WT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = min(m0 + (wm * MT + i) * 16 + l16, M - 1);   // ragged edges: re-read the last row
    int64_t row = m;
    if constexpr (GROUPED) {
      if (amap) row = amap[m];
    }
    ap[i] = A + row * lda + 4 * lk;
  }
#pragma unroll
  for (int j = 0; j < WT; ++j) {
    const int n = min(n0 + (wn * NT + j % NT) * 16 + l16, N - 1);
    wp[j] = W + (int64_t)(j < NT ? n : N + n) * K + 4 * lk;
  }
  f32x4 acc[WT][MT];
#pragma unroll
  for (int j = 0; j < WT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int steps = K / 16;      // K is a multiple of 16
  f32x4 ab[2][U][MT], wb[2][U][WT];
  // a step past the end loads the last one again and is left out of the sum
#define VLC_F32_LOAD(b_, s_)                                                                       \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                                   \
    const int k_ = min((s_) + u * KW, steps - 1) * 16;                                              \
    _Pragma("unroll") for (int i = 0; i < MT; ++i) ab[b_][u][i] = *reinterpret_cast<const f32x4*>(ap[i] + k_); \
    _Pragma("unroll") for (int j = 0; j < WT; ++j) wb[b_][u][j] = *reinterpret_cast<const f32x4*>(wp[j] + k_); \
  }
#define VLC_F32_MULTIPLY(b_, s_)                                                                   \
  _Pragma("unroll") for (int u = 0; u < U; ++u)                                                     \
    if ((s_) + u * KW < steps) {                                                                    \
      _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                 \
        _Pragma("unroll") for (int j = 0; j < WT; ++j)                                              \
          _Pragma("unroll") for (int i = 0; i < MT; ++i)                                            \
            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wb[b_][u][j][e], ab[b_][u][i][e], acc[j][i], 0, 0, 0); \
    }
  VLC_F32_LOAD(0, kw)
  for (int s = kw; s < steps; s += 2 * U * KW) {
    if (s + U * KW < steps) { VLC_F32_LOAD(1, s + U * KW) }
    VLC_F32_MULTIPLY(0, s)
    if (s + 2 * U * KW < steps) { VLC_F32_LOAD(0, s + 2 * U * KW) }
    VLC_F32_MULTIPLY(1, s + U * KW)
  }
#undef VLC_F32_LOAD
#undef VLC_F32_MULTIPLY

  if constexpr (KW > 1) {        // the wavefronts' sums over their k-steps, added in wavefront order
    __shared__ f32x4 part[KW - 1][WT * MT][64];
    if (kw > 0) {
#pragma unroll
      for (int t = 0; t < WT * MT; ++t) part[kw - 1][t][lane] = acc[t / MT][t % MT];
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int t = 0; t < WT * MT; ++t)
#pragma unroll
      for (int w = 0; w < KW - 1; ++w) acc[t / MT][t % MT] += part[w][t][lane];
  }

#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = m0 + (wm * MT + i) * 16 + l16;
    if (m >= M) continue;
    const int64_t rr = (EPI == EPI_RESIDUAL && rmap) ? (int64_t)rmap[m] : (int64_t)m;
#pragma unroll
    for (int j = 0; j < NT; ++j)
      store_f32<EPI>(acc[j][i], acc[(EPI == EPI_SWIGLU ? NT : 0) + j][i], m, n0 + (wn * NT + j) * 16 + 4 * lk, N, bias, resid, rr * ldr, C, ldc);
  }
}

// ---------------------------------------------------------------------------------------------
// f32 products that take the RMSNorm of their input rows with them (K <= kF32NormK): one launch instead of two, and with the
// heads of q|k|v also the rotation and the scatter of the fresh rows
// ---------------------------------------------------------------------------------------------
// Bound by latency and launches: a layer of the tiny decoder (61 rows) was eight kernels of 2.5 ... 10 us, it is five.
// Layout as in gemm_f32_kernel with KW = 4: 16 rows, WT tiles of 16 columns, wavefront kw takes k-steps kw, kw + 4, ...  Its
// pieces of the rows stay in registers (at most 8 steps of 16), the squares meet in LDS, and every workgroup norms its rows for
// itself; the first of a row tile also leaves them in y.  The sums are taken in the order of rmsnorm_kernel (a tree over
// the row's 16-byte pieces, whose number is 16 i + 4 kw + lk here) and the products in the order of gemm_f32_kernel: the same bits as the two kernels.
// w_norm = nullptr: the rows are normed already.
constexpr int kF32NormK = 512;

// meanwhile(): what the caller has to do while the first loads are on their way.
template <int WT, typename F>
__device__ __forceinline__ void normed_sums_f32(const float* __restrict__ x, const int32_t* __restrict__ map,
                                                const float* __restrict__ w_norm, int K, int M, float inv_h, float eps,
                                                float* __restrict__ y, int m0, const float* const (&wp)[WT], f32x4 (&acc)[WT], F meanwhile) {
  constexpr int KW = 4, NS = kF32NormK / 16 / KW, U = WT > 4 ? 2 : 4;   // U: k-steps of W in flight
  __shared__ float squares[NS / 4][KW][64];
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int m = min(m0 + l16, M - 1), steps = K / 16;
  const float* xp = x + (map ? (int64_t)map[m] : (int64_t)m) * K + 4 * lk;
  f32x4 a[NS], nw[NS], wb[2][U][WT];
  // a step past the end loads the last one again and is left out of the sums
#define VLC_STEP(i_) (min(kw + (i_) * KW, steps - 1) * 16)
#define VLC_NORM_LOAD_W(b_, i0_)                                                                                \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                                               \
    _Pragma("unroll") for (int j = 0; j < WT; ++j) wb[b_][u][j] = *reinterpret_cast<const f32x4*>(wp[j] + VLC_STEP((i0_) + u)); \
  }
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (kw + (i & ~3) * KW < steps) a[i] = *reinterpret_cast<const f32x4*>(xp + VLC_STEP(i));
  if (w_norm) {
#pragma unroll
    for (int i = 0; i < NS; ++i)
      if (kw + (i & ~3) * KW < steps) nw[i] = *reinterpret_cast<const f32x4*>(w_norm + VLC_STEP(i) + 4 * lk);
  }
  VLC_NORM_LOAD_W(0, 0)
  __builtin_amdgcn_sched_barrier(0);
  meanwhile();
  if (w_norm) {
#pragma unroll
    for (int q = 0; q < NS / 4; ++q) {
      float p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) ss += a[4 * q + i][e] * a[4 * q + i][e];
        p[i] = kw + (4 * q + i) * KW < steps ? ss : 0.f;
      }
      squares[q][kw][lane] = (p[0] + p[2]) + (p[1] + p[3]);
    }
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int q = 0; q < NS / 4; ++q) {
      float ss = (squares[q][0][lane] + squares[q][2][lane]) + (squares[q][1][lane] + squares[q][3][lane]);
      ss += __shfl_xor(ss, 32);
      ss += __shfl_xor(ss, 16);
      tot += ss;
    }
    const float r = 1.0f / sqrtf(tot * inv_h + eps);
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[i][e] = a[i][e] * r * nw[i][e];
    if (y && m0 + l16 < M) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
        if (kw + i * KW < steps) *reinterpret_cast<f32x4*>(y + (int64_t)m * K + VLC_STEP(i) + 4 * lk) = a[i];
    }
  }
#pragma unroll
  for (int j = 0; j < WT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i0 = 0; i0 < NS; i0 += U) {
    if (kw + i0 * KW < steps) {
      if (i0 + U < NS && kw + (i0 + U) * KW < steps) { VLC_NORM_LOAD_W((i0 / U + 1) & 1, i0 + U) }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (kw + (i0 + u) * KW < steps) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < WT; ++j)
              acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wb[i0 / U & 1][u][j][e], a[i0 + u][e], acc[j], 0, 0, 0);
        }
    }
  }
#undef VLC_NORM_LOAD_W
#undef VLC_STEP
}

template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_normed_kernel(const float* __restrict__ x, const float* __restrict__ w_norm,
                                                              const float* __restrict__ W, int K, int M, int N, float inv_h,
                                                              float eps, float* __restrict__ y, float* __restrict__ C,
                                                              int64_t ldc) {
  constexpr int WT = EPI == EPI_SWIGLU ? 2 : 1;
  __shared__ f32x4 part[3][WT][64];
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lk = lane >> 4, m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
  const int n = min(n0 + l16, N - 1);
  const float* wp[WT];
#pragma unroll
  for (int j = 0; j < WT; ++j) wp[j] = W + (int64_t)(j ? N + n : n) * K + 4 * lk;
  f32x4 acc[WT];
  normed_sums_f32<WT>(x, nullptr, w_norm, K, M, inv_h, eps, blockIdx.x == 0 ? y : nullptr, m0, wp, acc, [] {});
  if (kw > 0) {
#pragma unroll
    for (int t = 0; t < WT; ++t) part[kw - 1][t][lane] = acc[t];
  }
  __syncthreads();
  if (kw > 0) return;
#pragma unroll
  for (int t = 0; t < WT; ++t)
#pragma unroll
    for (int w = 0; w < 3; ++w) acc[t] += part[w][t][lane];
  const int m = m0 + l16;
  if (m < M) store_f32<EPI>(acc[0], acc[WT - 1], m, n0 + 4 * lk, N, nullptr, nullptr, 0, C, ldc);
}

// One head of q|k|v per workgroup: its D columns are D / 16 tiles, of which wavefront j rotates j and j + D / 32 (pairs i, i + D / 2).
// Sines and cosines are worked out while the first loads are on their way.  As rope_qk_scatter_kernel otherwise; the unrounded
// projection is left in qkv for the caller.
template <int D>
__global__ __launch_bounds__(256) void qkv_rope_f32_kernel(
    const float* __restrict__ x, const int32_t* __restrict__ map, const float* __restrict__ w_norm, const float* __restrict__ W,
    int K, int M, float inv_h, float eps, const int32_t* __restrict__ pos, const int32_t* __restrict__ pos3,
    const int32_t* __restrict__ slot, int Hq, int Hkv, const float* __restrict__ bias, const float* __restrict__ w_qn,
    const float* __restrict__ w_kn, float* __restrict__ y, float* __restrict__ qkv, float* __restrict__ q_out,
    float* __restrict__ k_cache, float* __restrict__ v_cache, RopeFreq freq) {
  constexpr int WT = D / 16, PT = WT / 2;
  __shared__ f32x4 part[4][WT][64];
  __shared__ float head_squares[PT][16];
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lk = lane >> 4, m0 = blockIdx.y * 16, h = blockIdx.x;
  const int m = min(m0 + l16, M - 1), c = 16 * kw + 4 * lk;   // first of this lane's four pairs
  const bool rotates = kw < PT, is_v = h >= Hq + Hkv;
  const float* wp[WT];
#pragma unroll
  for (int j = 0; j < WT; ++j) wp[j] = W + (int64_t)(h * D + 16 * j + l16) * K + 4 * lk;
  const int row_slot = slot[m];
  int p[4] = {0, 0, 0, 0};
  double f[4] = {0.0, 0.0, 0.0, 0.0};
  if (rotates && !is_v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[i] = freq.inv_freq[c + i];
      p[i] = pos3 ? pos3[3 * (int64_t)m + freq.axis[c + i]] : pos[m];
    }
  }
  float sn[4], cs[4];
  f32x4 acc[WT];
  normed_sums_f32<WT>(x, map, w_norm, K, M, inv_h, eps, h == 0 ? y : nullptr, m0, wp, acc, [&] {
    if (rotates && !is_v) {
#pragma unroll
      for (int i = 0; i < 4; ++i) rope_sincos<false>(f[i], p[i], &sn[i], &cs[i]);
    }
  });
#pragma unroll
  for (int t = 0; t < WT; ++t) part[kw][t][lane] = acc[t];
  __syncthreads();
  f32x4 lo, hi;
  if (rotates) {
    lo = part[0][kw][lane];
    hi = part[0][kw + PT][lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {          // in wavefront order
      lo += part[w][kw][lane];
      hi += part[w][kw + PT][lane];
    }
    if (bias) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lo[i] += bias[h * D + c + i];
        hi[i] += bias[h * D + D / 2 + c + i];
      }
    }
  }
  const bool ok = rotates && m0 + l16 < M;
  if (ok) {
    float* r = qkv + (int64_t)m * ((Hq + 2 * Hkv) * D) + h * D + c;
    *reinterpret_cast<f32x4*>(r) = lo;
    *reinterpret_cast<f32x4*>(r + D / 2) = hi;
  }
  if (is_v) {                              // the same for the whole workgroup
    if (ok && row_slot >= 0) {
      float* d = v_cache + ((int64_t)row_slot * Hkv + h - Hq - Hkv) * D + c;
      *reinterpret_cast<f32x4*>(d) = lo;
      *reinterpret_cast<f32x4*>(d + D / 2) = hi;
    }
    return;
  }
  if (w_qn) {
    if (rotates) {
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) ss += lo[i] * lo[i] + hi[i] * hi[i];
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (lk == 0) head_squares[kw][l16] = ss;
    }
    __syncthreads();
    if (rotates) {
      float ss = head_squares[0][l16] + head_squares[1][l16];
      if constexpr (PT == 4) ss += head_squares[2][l16] + head_squares[3][l16];
      const float rn = 1.0f / sqrtf(ss * (1.0f / (float)D) + eps);
      const float* wn = (h < Hq ? w_qn : w_kn) + c;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lo[i] = lo[i] * rn * wn[i];
        hi[i] = hi[i] * rn * wn[D / 2 + i];
      }
    }
  }
  if (!ok) return;
  f32x4 olo, ohi;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    olo[i] = lo[i] * cs[i] - hi[i] * sn[i];
    ohi[i] = hi[i] * cs[i] + lo[i] * sn[i];
  }
  float* d = h < Hq ? q_out + ((int64_t)m * Hq + h) * D + c : k_cache + ((int64_t)row_slot * Hkv + h - Hq) * D + c;
  if (h < Hq || row_slot >= 0) {           // a negative slot: the row is computed, its k and v are not stored
    *reinterpret_cast<f32x4*>(d) = olo;
    *reinterpret_cast<f32x4*>(d + D / 2) = ohi;
  }
}

// Tail split: the chip holds `slots` workgroups at once; the tiles of the last, partly filled round are shared out over as
// many k ranges as fit into the idle slots and the scratch, at least 8 k-tiles each.  ways = 1: not split.
struct LastRound {
  int tiles, ways, kt;   // tiles of the last round, k ranges per tile, k-tiles per range
};
LastRound split_last_round(int64_t tiles, int slots, int KT, int64_t block_bytes, int64_t ws_bytes) {
  LastRound r = {(int)(tiles % slots), 1, KT};
  if (r.tiles == 0 || tiles < slots) return r;
  int64_t ways = slots / r.tiles;
  if (ways > KT / 8) ways = KT / 8;
  if (ways > ws_bytes / (r.tiles * block_bytes)) ways = ws_bytes / (r.tiles * block_bytes);
  if (ways < 2) return r;
  r.kt = (int)((KT + ways - 1) / ways);
  r.ways = (KT + r.kt - 1) / r.kt;
  return r;
}

template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, bool MAY_STAY>
int launch_bf16(const void* A, int64_t lda, const void* W, void* C, int64_t ldc, int64_t M, int64_t N,
                int64_t K, const void* bias, const void* resid, int64_t ldr, const int32_t* rmap, int splits,
                int kt_per_split, void* tail_ws, int64_t tail_ws_bytes, hipStream_t st) {
  constexpr int CN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((N + CN - 1) / CN);
  const int tiles = tiles_m * tiles_n;
  const size_t lds = (size_t)STAGES * (BM + BN) * BK * 2;
  const int KT = (int)(K / BK);
  int full = tiles * splits, tail = 0, tsp = 1, tkt = kt_per_split;
  if constexpr (EPI != EPI_PARTIAL) {
    const LastRound r = split_last_round(tiles, 256 * OCC, KT, (int64_t)BM * BN * 4, tail_ws ? tail_ws_bytes : 0);
    if (r.ways > 1) {
      tail = r.tiles;
      tsp = r.ways;
      tkt = r.kt;
      full = tiles - tail;
    }
  }
  const int items = full + tail * tsp;
  const bool stay = gemm_stays(MAY_STAY, items, 256 * OCC, (M + (EPI == EPI_SWIGLU ? 2 : 1) * N) * K * 2);
  auto kern = stay ? gemm_bf16_kernel<BM, BN, WGM, WGN, STAGES, OCC, EPI, MAY_STAY> : gemm_bf16_kernel<BM, BN, WGM, WGN, STAGES, OCC, EPI, false>;
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds)) return rc;
  hipLaunchKernelGGL(kern, dim3(stay ? 256 * OCC : items), dim3(WGM * WGN * 64), lds, st, (const uint16_t*)A, (const uint16_t*)W,
                     (int)K, (int)N, (int)lda, tiles_n, (int)M, tiles_m, tkt, full, tsp, items, (uint16_t*)C, ldc,
                     (const uint16_t*)bias, (const uint16_t*)resid, ldr, rmap, (float*)tail_ws);
  VLC_CHECK_LAUNCH("gemm_bf16");
  if constexpr (EPI != EPI_PARTIAL) {
    if (tail > 0) {
      hipLaunchKernelGGL((tail_reduce_kernel<BM, BN, EPI>), dim3(BM / 32 * ((CN / 4 + 15) / 16), tail), dim3(256), 0, st,
                         (const float*)tail_ws, tsp, full, tiles_m, tiles_n, (uint16_t*)C, ldc, (int)M, (int)N,
                         (const uint16_t*)bias, (const uint16_t*)resid, ldr, rmap);
      VLC_CHECK_LAUNCH("gemm_tail_reduce");
    }
  }
  return VLC_OK;
}

// Tile choice.  Every configuration runs its k-loop at 1.2 ... 1.5 PFLOP/s when the chip is full of its workgroups, so
// what decides is how well the product's tiles fill whole rounds of the 256 CUs and how much of them is padding; with few
// rows, how many bytes of W are in flight.  The list therefore spans the tile areas from 64 x 128 to 320 x 256, and the
// cheapest by the model below is launched.  Rings of three to five stages where the LDS holds them (an HBM miss takes longer
// than a small k-tile); above 426 rows + columns two stages, with the later wait (TWO above).  With 16-wide MFMA tiles a
// wavefront's rows and columns are any multiples of 16: 320 x 160 (7B gate|up at 596 rows, 474 tiles = 1.85 rounds: 134 us; 128 x 192
// two per CU 150, 320 x 192 152), 224 x 192 (8B gate|up at 446 rows 75, best of the others 79), 128 x 96 (8B gate|up at
// 97 rows, 256 tiles: 47 against 53), 256 x 192, 160 x 160, 160 x 192, 320 x 256 (7B down at 5824 rows 599 against 630).
//
// Per configuration: time of one k-tile (us) with few workgroups on the chip, with one full round of them and with many
// rounds (power).  All numbers of the model were fitted together, to the times of 700 products of 2 ... 24000 rows in
// five decoder shapes and of heads, with every tile, every number of k ranges and both ends of a last round (27000 times, cold
// weights), so that its choice is as little slower as possible than the best of them: 0.5 % on average, 36 products more
// than 3 % (left out of the fit, the fifth shape is at 1.2 %).  That was with the kernels of that time: 534 products of 8 ... 24000 rows timed
// with the present ones, which end sooner (residuals and float outputs above all) and may stay, are 2.0 % slower than the best of the 14
// cheapest on average, 111 of them more than 3 %: q|k|v of K = 2048 at 60 ... 110 rows takes one k range where three to five are 20 ... 45 %
// faster, residuals and q|k|v from 6000 rows on 256 x 256 on eight wavefronts where 320 x 256 or 320 x 192 is 6 ... 8 % faster.  A list without one of the tiles costs 0.1 ... 1.3 % more.
// These are numbers of a fit and no measured times (192 x 128 is priced lower over many rounds than in one), and they miss: at
// 8192 columns and K = 29568, 320 x 256 takes 8469 us where 256 x 256 is chosen with 8833 (24000 rows), 12655 against 13745 (36000).
// USE: 0 all epilogues, 1 all but SwiGLU (an odd number of column tiles per wavefront, or never the fastest there), 3 float
// output without scratch (the heads; in the layers never the fastest).  256 x 256 on 8 wavefronts of
// 64 x 128 over many rounds, on 4 of 128 x 128 over few.
// STAY: the products whose workgroups can stay, 0 none, 1 SwiGLU, 2 residuals too.
//     BM   BN  WGM WGN STAGES OCC USE STAY light  full  many
#define VLC_GEMM_TILES(X)                             \
  X(64, 128, 2, 2, 4, 1, 0, 0, 0.247f, 0.375f, 0.378f)     \
  X(128, 96, 4, 1, 5, 1, 0, 0, 0.338f, 0.422f, 0.422f)     \
  X(128, 128, 2, 2, 4, 1, 0, 0, 0.477f, 0.522f, 0.652f)    \
  X(128, 160, 4, 1, 4, 1, 0, 0, 0.422f, 0.616f, 0.763f)    \
  X(160, 160, 2, 2, 4, 1, 1, 0, 0.350f, 0.725f, 0.799f)    \
  X(128, 256, 2, 2, 3, 1, 0, 0, 0.580f, 0.860f, 1.049f)    \
  X(192, 128, 2, 2, 4, 1, 1, 0, 0.541f, 0.645f, 0.581f)    \
  X(160, 192, 2, 2, 3, 1, 0, 0, 0.687f, 0.740f, 0.894f)    \
  X(192, 192, 2, 2, 3, 1, 0, 0, 0.431f, 0.859f, 1.073f)    \
  X(224, 192, 2, 2, 3, 1, 0, 1, 0.570f, 1.018f, 1.036f)    \
  X(160, 256, 2, 2, 3, 1, 0, 1, 0.783f, 0.990f, 1.036f)    \
  X(192, 256, 2, 2, 2, 1, 0, 1, 0.777f, 1.097f, 1.093f)    \
  X(256, 192, 2, 2, 2, 1, 0, 0, 0.644f, 1.062f, 1.289f)    \
  X(320, 160, 4, 1, 2, 1, 0, 2, 0.536f, 1.108f, 1.146f)    \
  X(320, 192, 2, 2, 2, 1, 0, 2, 0.970f, 1.339f, 1.333f)    \
  X(256, 256, 4, 2, 2, 1, 1, 0, 0.797f, 1.458f, 1.366f)    \
  X(256, 256, 2, 2, 2, 1, 0, 1, 0.733f, 1.493f, 1.418f)    \
  X(320, 256, 2, 2, 2, 1, 1, 0, 1.313f, 1.674f, 1.734f)    \
  X(128, 160, 4, 1, 2, 2, 3, 0, 0.701f, 0.838f, 0.991f)
constexpr bool tile_serves(int use, int epi) {
  return use == 0 || (use == 1 && epi != EPI_SWIGLU) || (use == 3 && epi == EPI_BIAS_F32);
}
constexpr bool tile_may_stay(int stay, int epi) { return (stay >= 1 && epi == EPI_SWIGLU) || (stay == 2 && epi == EPI_RESIDUAL); }

struct TileChoice {
  int index;        // into VLC_GEMM_TILES
  int splits;       // k ranges (> 1: float partials)
  bool split_tail;  // share the last round's tiles out along k
};

// Price (us) of a product: rounds of resident workgroups, each its k-tiles plus a start and an end.  A k-tile takes the
// longer of its multiplication and of the arrival of the weights that the resident workgroups ask for in that time (HBM), and
// a little of the other.  A split k range costs the kernel that sums the partials its reading (the RoPE kernel more than
// the norms); as a kernel of its own also a launch.  A split last round costs tail_reduce_kernel.
constexpr float kPriceHbm = 6.98e6f;          // bytes per us of weights
constexpr float kPriceHbmAligned = 0.85f;     // share of it left when all k ranges start at multiples of 4 KiB (one channel)
constexpr float kPriceOther = 0.275f;         // share of the shorter of the two that shows
constexpr float kPriceRounds = 1.83f;         // rounds past the first after which a k-tile takes its "many" time
constexpr float kPriceEnds = 1.91f, kPriceEndsArea = 8.13f;            // start and end: per workgroup, per 256 x 256 outputs
constexpr float kPriceEndsFloat = 2.08f;                               // more of the latter for float output
constexpr float kPriceEnds8 = 0.64f, kPriceEndsFloat8 = 2.44f;         // the last two on eight wavefronts, as shares
constexpr float kPriceTail = 3.80f, kPriceTailElem = 0.77e-6f;         // split last round: launch, per float of its blocks
constexpr float kPriceSumQkv = 1.58f, kPriceSumQkvElem = 1.47e-6f;     // split k range: per launch, per partial sum
constexpr float kPriceSum = 1.40f, kPriceSumElem = 1.01e-6f;
constexpr float kPriceSumLaunch = 2.5f;       // not deferred to the caller's next kernel

TileChoice choose_tile(int64_t M, int64_t N, int64_t K, int epi, bool deferred, int64_t ws_bytes) {
  struct Tile { int bm, bn, waves, occ, use; float light, full, many; };
#define X(BM, BN, WGM, WGN, S, OCC, USE, STAY, L, F, MA) {BM, BN, WGM * WGN, OCC, USE, L, F, MA},
  static constexpr Tile kTiles[] = {VLC_GEMM_TILES(X)};
#undef X
  constexpr int kCount = (int)(sizeof(kTiles) / sizeof(kTiles[0]));
  const int KT = (int)(K / BK);
  const bool float_out = epi == EPI_BIAS_F32, may_split = epi != EPI_SWIGLU && ws_bytes > 0;
  TileChoice best = {-1, 1, false};
  float best_us = 0.f;
  for (int i = 0; i < kCount; ++i) {
    const Tile& t = kTiles[i];
    if (!tile_serves(t.use, epi) || (t.use == 3 && ws_bytes > 0)) continue;
    const int cn = epi == EPI_SWIGLU ? t.bn / 2 : t.bn;
    const int64_t tiles_m = (M + t.bm - 1) / t.bm, tiles = tiles_m * ((N + cn - 1) / cn);
    const int slots = 256 * t.occ;
    const float area = (float)(t.bm * t.bn), area_share = (float)t.occ * area / 65536.0f;
    const bool eight = t.waves == 8;
    for (int sp = 1; sp <= (may_split ? 8 : 1); ++sp) {
      if (sp > 1 && (KT / sp < 4 || (int64_t)sp * M * N * 4 > ws_bytes)) break;
      const int per = (KT + sp - 1) / sp;
      const int64_t wgs = tiles * ((KT + per - 1) / per), full = wgs / slots, tail = wgs % slots;
      float ends = kPriceEnds + kPriceEndsArea * (eight ? kPriceEnds8 : 1.0f) * area_share;
      if (float_out || sp > 1) ends += kPriceEndsFloat * (eight ? kPriceEndsFloat8 : 1.0f) * area_share;
      float later = ((float)wgs / (float)slots - 1.0f) / kPriceRounds;
      later = later < 0.f ? 0.f : (later > 1.f ? 1.f : later);
      const float busy = t.full + (t.many - t.full) * later;
      // weights asked for per k-tile by n workgroups: those of a column tile (and k range) share them
      const float hbm_us = (float)t.bn * (float)(BK * 2) / (float)tiles_m / (kPriceHbm * (sp > 1 && per % 32 == 0 ? kPriceHbmAligned : 1.0f));
      auto round_us = [&](int64_t n, int kt) {   // one round of n <= slots workgroups of kt k-tiles
        const float m = t.light + (busy - t.light) * (float)n / (float)slots, h = (float)n * hbm_us;
        return (float)kt * (m > h ? m + kPriceOther * h : h + kPriceOther * m) + ends;
      };
      float us = (float)full * round_us(slots, per);
      bool split_tail = false;
      if (tail > 0) {
        float tail_us = round_us(tail, per);
        if (sp == 1) {
          const LastRound r = split_last_round(tiles, slots, KT, (int64_t)t.bm * t.bn * 4, ws_bytes);
          if (r.ways > 1) {
            const int64_t blocks = (int64_t)r.tiles * r.ways;
            const float shared = round_us(blocks, r.kt) + kPriceTail + (float)blocks * area * kPriceTailElem;
            if (shared < tail_us) {
              tail_us = shared;
              split_tail = true;
            }
          }
        }
        us += tail_us;
      }
      if (sp > 1)
        us += (float_out ? kPriceSumQkv : kPriceSum) + (deferred ? 0.f : kPriceSumLaunch) +
              (float)sp * (float)M * (float)N * (float_out ? kPriceSumQkvElem : kPriceSumElem);
      if (best.index < 0 || us < best_us) {
        best_us = us;
        best = {i, sp, split_tail};
      }
    }
  }
  return best;
}

template <int EPI>
int dispatch_bf16(const void* A, int64_t lda, const void* W, void* C, int64_t ldc, int64_t M, int64_t N,
                  int64_t K, const void* bias, const void* resid, int64_t ldr, const int32_t* rmap,
                  void* splitk_ws, int64_t splitk_ws_bytes, int* deferred, hipStream_t st) {
  const int KT = (int)(K / BK);
  const TileChoice c = choose_tile(M, N, K, EPI, deferred != nullptr, splitk_ws ? splitk_ws_bytes : 0);
  if (c.splits > 1) {
    if constexpr (EPI != EPI_SWIGLU) {
      const int per = (KT + c.splits - 1) / c.splits, splits = (KT + per - 1) / per;
      int rc = VLC_OK, i = 0;
#define X(BM, BN, WGM, WGN, S, OCC, USE, STAY, L, F, MA)                                                              \
  if (c.index == i++) {                                                                                              \
    if constexpr (USE != 3 && tile_serves(USE, EPI))                                                                 \
      rc = launch_bf16<BM, BN, WGM, WGN, S, OCC, EPI_PARTIAL, false>(A, lda, W, splitk_ws, N, M, N, K, nullptr, nullptr,  \
                                                                     0, nullptr, splits, per, nullptr, 0, st);       \
  }
      VLC_GEMM_TILES(X)
#undef X
      if (rc) return rc;
      if (deferred) {   // the caller's next kernel sums the partials and applies the epilogue
        *deferred = splits;
        return VLC_OK;
      }
      const int64_t threads = M * (N / 4);
      hipLaunchKernelGGL(splitk_epilogue_kernel<EPI>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                         (const float*)splitk_ws, splits, (int)M, (int)N, (const uint16_t*)resid, ldr, rmap,
                         (const uint16_t*)bias, (uint16_t*)C, ldc);
      VLC_CHECK_LAUNCH("splitk_epilogue");
      return VLC_OK;
    }
  }
  void* tail_ws = c.split_tail ? splitk_ws : nullptr;
  int i = 0;
#define X(BM, BN, WGM, WGN, S, OCC, USE, STAY, L, F, MA)                                                                \
  if (c.index == i++) {                                                                                                \
    if constexpr (tile_serves(USE, EPI))                                                                               \
      return launch_bf16<BM, BN, WGM, WGN, S, OCC, EPI, tile_may_stay(STAY, EPI)>(A, lda, W, C, ldc, M, N, K, bias, resid,  \
                                                                                  ldr, rmap, 1, KT, tail_ws, splitk_ws_bytes, st);  \
  }
  VLC_GEMM_TILES(X)
#undef X
  return fail(VLC_ERR_SHAPE, "gemm(bf16): no tile");
}

// Output tiles of 128 rows (grouped: 64) x 128 columns (SwiGLU: 64) from 96 of them on, else 16 x 16 tiles with the k
// range shared by the workgroup's four wavefronts.  Large against small tiles, 128 rows: 64 tiles 38 / 34 us (K = 256)
// and 161 / 131 us (K = 2048), 128 tiles 41 / 49 and 163 / 244 us (vector instructions: 67 and 407 us); with 2048 tiles
// 106 against 37 TFLOP/s.
constexpr int64_t kF32LargeTiles = 96;
bool f32_large_tiles(int64_t M, int64_t N, int epi) {
  const int64_t columns = epi == EPI_SWIGLU ? 64 : 128;
  return (M + 127) / 128 * ((N + columns - 1) / columns) >= kF32LargeTiles;
}

template <int EPI>
int launch_f32(const void* A, int64_t lda, const void* W, void* C, int64_t ldc, int64_t M, int64_t N,
               int64_t K, const void* bias, const void* resid, int64_t ldr, const int32_t* rmap,
               hipStream_t st) {
  constexpr int NT = EPI == EPI_SWIGLU ? 2 : 4;
  const int64_t lm = (M + 127) / 128, ln = (N + 32 * NT - 1) / (32 * NT);
  const bool large = f32_large_tiles(M, N, EPI);
  const int64_t gy = large ? lm : (M + 15) / 16;
  const dim3 grid((unsigned)(large ? ln : (N + 15) / 16), (unsigned)gy);
#define VLC_LAUNCH_F32(...)                                                                                        \
  hipLaunchKernelGGL((gemm_f32_kernel<__VA_ARGS__, EPI>), grid, dim3(256), 0, st, (const float*)A, (const float*)W, \
                     (int)K, (int)M, (int)N, (int)lda, (const float*)bias, (const float*)resid, rmap, (float*)C, ldc, ldr, \
                     (const GroupTile*)nullptr, (const int32_t*)nullptr, (const int32_t*)nullptr, (int64_t)0)
  if (large) VLC_LAUNCH_F32(4, NT, 2, 2, 1);
  else VLC_LAUNCH_F32(1, 1, 1, 1, 4);
#undef VLC_LAUNCH_F32
  VLC_CHECK_LAUNCH("gemm_f32");
  return VLC_OK;
}

// Grouped launches: the grid covers the largest number of row tiles the table can hold.
template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, bool STAY = false>
int launch_bf16_grouped(const void* A, int64_t lda, const int32_t* amap, const void* W, int64_t w_stride, void* C,
                        int64_t ldc, int64_t N, int64_t K, const GroupTile* gtab, const int32_t* g_ntiles,
                        int max_tiles_m, hipStream_t st) {
  constexpr int CN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  const int tiles_n = (int)((N + CN - 1) / CN);
  const size_t lds = (size_t)STAGES * (BM + BN) * BK * 2;
  auto kern = gemm_bf16_kernel<BM, BN, WGM, WGN, STAGES, OCC, EPI, STAY, true>;
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds)) return rc;
  const int most = max_tiles_m * tiles_n, grid = STAY && most > 256 * OCC ? 256 * OCC : most;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WGM * WGN * 64), lds, st, g_ntiles, gtab, amap, (const uint16_t*)A, (const uint16_t*)W,
                     (int)K, (int)N, (int)lda, tiles_n, w_stride, (uint16_t*)C, ldc);
  VLC_CHECK_LAUNCH("gemm_bf16_grouped");
  return VLC_OK;
}

template <int EPI>
int launch_f32_grouped(const void* A, int64_t lda, const int32_t* amap, const void* W, int64_t w_stride, void* C,
                       int64_t ldc, int64_t N, int64_t K, const GroupTile* gtab, const int32_t* g_ntiles,
                       int max_tiles_m, hipStream_t st) {
  constexpr int NT = EPI == EPI_SWIGLU ? 2 : 4;
  const int64_t ln = (N + 32 * NT - 1) / (32 * NT);
  const bool large = max_tiles_m * ln >= kF32LargeTiles;
  const int64_t gy = large ? max_tiles_m : (int64_t)max_tiles_m * 4;
  const dim3 grid((unsigned)(large ? ln : (N + 15) / 16), (unsigned)gy);
#define VLC_LAUNCH_F32(...)                                                                                       \
  hipLaunchKernelGGL((gemm_f32_kernel<__VA_ARGS__, EPI, true>), grid, dim3(256), 0, st, (const float*)A,          \
                     (const float*)W, (int)K, 0, (int)N, (int)lda, (const float*)nullptr, (const float*)nullptr, \
                     (const int32_t*)nullptr, (float*)C, ldc, (int64_t)0, gtab, g_ntiles, amap, w_stride)
  if (large) VLC_LAUNCH_F32(2, NT, 2, 2, 1);
  else VLC_LAUNCH_F32(1, 1, 1, 1, 4);
#undef VLC_LAUNCH_F32
  VLC_CHECK_LAUNCH("gemm_f32_grouped");
  return VLC_OK;
}

}  // namespace

// The products that norm their rows themselves are those on small tiles whose rows fit the registers: on large tiles the
// norm is read by few workgroups and its launch is a small part.
bool gemm_f32_norms(int64_t M, int64_t N, int64_t K, int epilogue) {
  return K % 16 == 0 && K <= kF32NormK && !f32_large_tiles(M, N, epilogue);
}

// q|k|v with rotation and scatter takes a head per workgroup, whose k-steps are those of four wavefronts in turn: at D = 128 eight column
// tiles each.  With few workgroups that is longer than the three launches it saves: us per layer, one kernel | three | before both:
//   columns x heads     512 x 8                             384 x 8             256 x 8             512 x 24
//   rows    16    32.2 | 27.6 | 30.7    29.2 | 27.1 | 30.0  25.2 | 24.5 | 27.4  36.3 | 31.9 | 35.2
//           64    33.5 | 29.3 | 35.3    30.8 | 28.6 | 34.2  25.9 | 25.4 | 30.9  39.7 | 39.2 | 42.4
//          192    46.4 | 45.2 | 53.4    43.3 | 44.4 | 52.5  36.1 | 37.2 | 45.7  61.1 | 59.9 | 80.8
//          512    64.7 | 71.5 | 141.6   58.8 | 68.1 | 139   50.2 | 55.6 | 127   113 | 113 | 265
// The two are level at some 110 workgroups with 512 columns, 60 with 384, 30 with 256; with 128 columns, and at D = 64, the one is faster or level
// (tiny_f32's shape 5 ... 15 %).
bool qkv_rope_f32_pays(int64_t M, int heads, int D, int64_t K) {
  return gemm_f32_norms(M, (int64_t)heads * D, K, EPI_BIAS) && (D == 64 || (M + 15) / 16 * heads >= (K - 192) / 3);
}

int launch_gemm_f32_normed(const void* x, const void* w_norm, const void* W, void* y, void* C, int64_t ldc, int64_t M, int64_t N,
                           int64_t K, float eps, int epilogue, hipStream_t st) {
  if (M <= 0 || N <= 0) return VLC_OK;
  if (!gemm_f32_norms(M, N, K, epilogue) || M > INT32_MAX || N > INT32_MAX / 2)
    return fail(VLC_ERR_SHAPE, "normed gemm(f32): M=%lld N=%lld K=%lld", (long long)M, (long long)N, (long long)K);
  const dim3 grid((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16));
  if (epilogue == EPI_SWIGLU)
    hipLaunchKernelGGL(gemm_f32_normed_kernel<EPI_SWIGLU>, grid, dim3(256), 0, st, (const float*)x, (const float*)w_norm, (const float*)W,
                       (int)K, (int)M, (int)N, 1.0f / (float)K, eps, (float*)y, (float*)C, ldc);
  else if (epilogue == EPI_BIAS)
    hipLaunchKernelGGL(gemm_f32_normed_kernel<EPI_BIAS>, grid, dim3(256), 0, st, (const float*)x, (const float*)w_norm, (const float*)W,
                       (int)K, (int)M, (int)N, 1.0f / (float)K, eps, (float*)y, (float*)C, ldc);
  else
    return fail(VLC_ERR_SHAPE, "normed gemm(f32): epilogue=%d", epilogue);
  VLC_CHECK_LAUNCH("gemm_f32_normed");
  return VLC_OK;
}

int launch_qkv_rope_f32(const void* x, const int32_t* map, const void* w_norm, const void* W, const void* bias, int64_t M, int64_t K,
                        float eps, const int32_t* pos, const int32_t* pos3, const int32_t* slot, int Hq, int Hkv, int D,
                        const RopeFreq& f, const void* w_qnorm, const void* w_knorm, void* y, float* qkv32, void* q_out, void* k_cache,
                        void* v_cache, hipStream_t st) {
  if (M <= 0) return VLC_OK;
  if (!gemm_f32_norms(M, (int64_t)(Hq + 2 * Hkv) * D, K, EPI_BIAS) || M > INT32_MAX || (D != 64 && D != 128))
    return fail(VLC_ERR_SHAPE, "q|k|v + rope(f32): M=%lld K=%lld D=%d", (long long)M, (long long)K, D);
  const dim3 grid((unsigned)(Hq + 2 * Hkv), (unsigned)((M + 15) / 16));
#define VLC_LAUNCH_QKV(D_)                                                                                            \
  hipLaunchKernelGGL(qkv_rope_f32_kernel<D_>, grid, dim3(256), 0, st, (const float*)x, map, (const float*)w_norm, (const float*)W, \
                     (int)K, (int)M, 1.0f / (float)K, eps, pos, pos3, slot, Hq, Hkv, (const float*)bias, (const float*)w_qnorm, \
                     (const float*)w_knorm, (float*)y, qkv32, (float*)q_out, (float*)k_cache, (float*)v_cache, f)
  if (D == 64) VLC_LAUNCH_QKV(64);
  else VLC_LAUNCH_QKV(128);
#undef VLC_LAUNCH_QKV
  VLC_CHECK_LAUNCH("qkv_rope_f32");
  return VLC_OK;
}

// Float scratch of the split k ranges and of the split tiles of a last round: choose_tile and launch_bf16 split only
// what fits.  64 MB is one float block per resident workgroup at 256 x 256; of 320 x 256 it holds 204 blocks, which caps the k
// ranges of such a last round.
int64_t gemm_splitk_ws_bytes(int64_t n_rows, int64_t max_n) {
  (void)max_n;
  return n_rows > 0 ? (int64_t)64 << 20 : 0;
}

// Rows per tile of the grouped GEMMs, from the mean number of rows per group.  Few rows per group: every
// matrix is streamed from HBM exactly once and nothing is reused, so the tile is small (64 x 128, below 9 rows per
// group 32 x 128) and the ring three (four) stages deep - with two workgroups per CU that keeps 64 (96) KB of matrix data
// in flight per CU, what the HBM latency needs; a two-stage ring of 128 x 128 tiles stalls at half of that.  More rows: an expert's
// rows cost their tiles, so the lines lie where most experts begin to need one tile more (192 rows per tile hold an expert of up to 190
// or so on average, 256 one of up to 250, and then two of 192 do better than two of 256).  Two layers of 128 experts (2048 x 768), a
// random router's loads, us of both layers with every tile, the chosen one in brackets:
//   rows per expert    9     37     56     81    106    138    175    219    269    325    394    469    562
//   32              (579)
//   64               581   (703)   793    944   1060
//   128                     706  (767)  (847)  (983)  1157   1217   1387   1682   1886   2185   2508   2909
//   192                     763    830    910   970  (1019) (1178)  1481 (1586) (1750)  2110   2372   2734
//   256                     816    857    963   1045   1061   1195 (1340)  1697   1885 (2030) (2288) (2819)
// (Lines at 56, 140 and 320, for 128, 192 and 256 rows: 3 % slower than the best on average, 13 % at 138; these 0.4 %, 3 % at 562.)
// That is where the tiles are several rounds (128 experts x 6 column tiles of gate|up).  Where all of gate|up is within one, a product takes as long as one tile, and the smaller is the
// faster: us of two layers, top 2 or 8, the smaller | the larger of two heights:
//   experts x column tiles of gate|up     8 x 6           16 x 6        32 x 6        64 x 6        128 x 6       16 x 12       32 x 12
//   128 | 192 rows, 105 on average        184 | 183       232 | 251     288 | 321     445 | 512     796 | 825     457 | 461     696 | 775
//                   120                   187 | 211       249 | 257     316 | 325     490 | 519     841 | 845     491 | 470     763 | 787
//                   135                   192 | 216       252 | 260     390 | 327     546 | 521     915 | 870     596 | 475     853 | 796
//   192 | 256 rows, 220                   236 | 260       312 | 313     468 | 418     687 | 628     1255 | 1137   739 | 578     1129 | 966
//                   245                   239 | 265       320 | 325     462 | 450     705 | 661     1254 | 1170   748 | 684     1146 | 1034
//                   330                   253 | 279       350 | 373     526 | 554     771 | 844     1424 | 1565   769 | 887     1159 | 1360
// The lines miss where one height just fills whole rounds: 32 and 64 experts x 4 column tiles are 4 and 9 % slower on 256 rows at 245, 11 and 6 % on
// 192 at 355 (two tiles of each of 32 experts are the round of 256; a third starts another).
int gemm_group_tile_rows(int64_t rows, int n_groups, int64_t width, int dtype) {
  if (dtype != VLC_BF16) return 64;
  const int64_t mean = rows / (n_groups > 0 ? n_groups : 1), columns = n_groups * ((2 * width + 255) / 256);
  if (mean < 56) return mean < 9 ? 32 : 64;
  if (mean < (columns >= 192 ? 128 : 140)) return 128;
  if (mean < 185) return 192;
  if (mean < 250) return columns >= 128 ? 256 : 192;
  return mean < 360 ? 192 : 256;
}

int launch_gemm_grouped(const void* A, int64_t lda, const int32_t* amap, const void* W, int64_t w_stride, void* C,
                        int64_t ldc, int64_t rows, int n_groups, int64_t N, int64_t K, int epilogue,
                        const GroupTile* tiles, const int32_t* n_tiles, int tile_rows, int dtype, hipStream_t st,
                        int64_t a_rows) {
  if (rows <= 0 || N <= 0) return VLC_OK;
  if (K <= 0 || n_groups <= 0) return fail(VLC_ERR_SHAPE, "grouped gemm: K=%lld groups=%d", (long long)K, n_groups);
  if (rows > INT32_MAX || N > INT32_MAX / 2 || K > INT32_MAX)
    return fail(VLC_ERR_SHAPE, "grouped gemm: dimension exceeds 32-bit tile indexing");
  if (tile_rows != gemm_group_tile_rows(rows, n_groups, epilogue == EPI_SWIGLU ? N : K, dtype))
    return fail(VLC_ERR_SHAPE, "grouped gemm: the tile table was built for %d rows per tile", tile_rows);
  const int max_tiles = (int)(rows / tile_rows) + n_groups;
  if (epilogue != EPI_BIAS && epilogue != EPI_SWIGLU)
    return fail(VLC_ERR_SHAPE, "grouped gemm: epilogue=%d", epilogue);
  if (dtype == VLC_BF16) {
    if (K % BK || N % 4 || lda % 8 || ldc % 4)
      return fail(VLC_ERR_SHAPE, "grouped gemm(bf16): K=%lld must be a multiple of %d, N, lda, ldc aligned", (long long)K, BK);
    // 32-bit lane offsets: rows fetched through amap are offsets from A itself (amap values are below a_rows)
    if ((amap ? a_rows : 256) * lda * 2 >= ((int64_t)1 << 31) || ((epilogue == EPI_SWIGLU ? N : 0) + 256) * K * 2 >= ((int64_t)1 << 31))
      return fail(VLC_ERR_SHAPE, "grouped gemm(bf16): operand rows span more than 2 GiB");
    if (tile_rows == 256) {
      if (epilogue == EPI_SWIGLU)
        return launch_bf16_grouped<256, 256, 2, 2, 2, 1, EPI_SWIGLU, true>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
      return launch_bf16_grouped<256, 256, 2, 2, 2, 1, EPI_BIAS, true>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
    }
    if (tile_rows == 192) {
      if (epilogue == EPI_SWIGLU)
        return launch_bf16_grouped<192, 256, 2, 2, 2, 1, EPI_SWIGLU, true>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
      return launch_bf16_grouped<192, 256, 2, 2, 2, 1, EPI_BIAS, true>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
    }
    if (tile_rows == 64) {
      if (epilogue == EPI_SWIGLU)
        return launch_bf16_grouped<64, 128, 1, 4, 3, 2, EPI_SWIGLU>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
      return launch_bf16_grouped<64, 128, 2, 2, 3, 2, EPI_BIAS>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
    }
    if (tile_rows == 32) {
      if (epilogue == EPI_SWIGLU)
        return launch_bf16_grouped<32, 128, 1, 4, 4, 2, EPI_SWIGLU>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
      return launch_bf16_grouped<32, 128, 1, 4, 4, 2, EPI_BIAS>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
    }
    if (epilogue == EPI_SWIGLU)
      return launch_bf16_grouped<128, 256, 2, 2, 3, 1, EPI_SWIGLU>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
    return launch_bf16_grouped<128, 128, 2, 2, 2, 2, EPI_BIAS>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
  }
  if (dtype == VLC_F32) {
    if (K % 16) return fail(VLC_ERR_SHAPE, "grouped gemm(f32): K=%lld must be a multiple of 16", (long long)K);
    if (epilogue == EPI_SWIGLU)
      return launch_f32_grouped<EPI_SWIGLU>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
    return launch_f32_grouped<EPI_BIAS>(A, lda, amap, W, w_stride, C, ldc, N, K, tiles, n_tiles, max_tiles, st);
  }
  return fail(VLC_ERR_DTYPE, "grouped gemm: dtype=%d", dtype);
}

int launch_gemm(const void* A, int64_t lda, const void* W, void* C, int64_t ldc, int64_t M, int64_t N,
                int64_t K, int epilogue, const void* bias, const void* resid, int64_t ldr,
                const int32_t* rmap, int dtype, void* splitk_ws, int64_t splitk_ws_bytes, hipStream_t st,
                int* deferred) {
  if (deferred) *deferred = 0;
  if (M <= 0 || N <= 0) return VLC_OK;
  if (K <= 0) return fail(VLC_ERR_SHAPE, "gemm: K=%lld", (long long)K);
  if (M > INT32_MAX || N > INT32_MAX / 2 || K > INT32_MAX)
    return fail(VLC_ERR_SHAPE, "gemm: dimension exceeds 32-bit tile indexing");
  if (dtype == VLC_BF16) {
    if (K % BK) return fail(VLC_ERR_SHAPE, "gemm(bf16): K=%lld must be a multiple of %d", (long long)K, BK);
    if (N % 4 || lda % 8 || ldc % 4 || (epilogue == EPI_RESIDUAL && ldr % 4))
      return fail(VLC_ERR_SHAPE, "gemm(bf16): N, lda, ldc, ldr must keep 8-byte (A: 16-byte) alignment");
    // lane offsets of the loads are unsigned 32-bit byte offsets from the tile's first row (SwiGLU: up rows sit N rows
    // on); below 2 GiB for 256 rows they are below 4 GiB for the largest tile
    if (256 * lda * 2 >= ((int64_t)1 << 31) || ((epilogue == EPI_SWIGLU ? N : 0) + 256) * K * 2 >= ((int64_t)1 << 31))
      return fail(VLC_ERR_SHAPE, "gemm(bf16): a tile's rows span more than 2 GiB (lda=%lld N=%lld K=%lld)",
                  (long long)lda, (long long)N, (long long)K);
    switch (epilogue) {
      case EPI_BIAS_F32: return dispatch_bf16<EPI_BIAS_F32>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, splitk_ws, splitk_ws_bytes, deferred, st);
      case EPI_RESIDUAL: return dispatch_bf16<EPI_RESIDUAL>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, splitk_ws, splitk_ws_bytes, deferred, st);
      case EPI_SWIGLU: return dispatch_bf16<EPI_SWIGLU>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, splitk_ws, splitk_ws_bytes, deferred, st);
    }
  } else if (dtype == VLC_F32) {
    if (K % 16) return fail(VLC_ERR_SHAPE, "gemm(f32): K=%lld must be a multiple of 16", (long long)K);
    switch (epilogue) {
      case EPI_BIAS:
      case EPI_BIAS_F32: return launch_f32<EPI_BIAS>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, st);
      case EPI_RESIDUAL: return launch_f32<EPI_RESIDUAL>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, st);
      case EPI_SWIGLU: return launch_f32<EPI_SWIGLU>(A, lda, W, C, ldc, M, N, K, bias, resid, ldr, rmap, st);
    }
  }
  return fail(VLC_ERR_DTYPE, "gemm: dtype=%d epilogue=%d", dtype, epilogue);
}

}  // namespace vlc

extern "C" int vlc_probe_gemm_choice(int epilogue, int64_t M, int64_t N, int64_t K, int scratch, int deferred, int32_t* out) {
  if (M <= 0 || N <= 0 || K < vlc::BK || K % vlc::BK || !out) return VLC_ERR_SHAPE;
  const int64_t ws = scratch ? vlc::gemm_splitk_ws_bytes(M, N) : 0;
  const vlc::TileChoice c = vlc::choose_tile(M, N, K, epilogue, deferred != 0, ws);
  int i = 0;
#define X(BM, BN, WGM, WGN, S, OCC, USE, STAY, L, F, MA)                                                         \
  if (c.index == i++) {                                                                                          \
    const int64_t cn = epilogue == vlc::EPI_SWIGLU ? BN / 2 : BN;                                                \
    const int64_t tiles = ((M + BM - 1) / BM) * ((N + cn - 1) / cn);                                             \
    const vlc::LastRound r = vlc::split_last_round(tiles, 256 * OCC, (int)(K / vlc::BK), (int64_t)BM * BN * 4, ws); \
    const int32_t o[5] = {BM, BN, OCC, c.splits, c.splits == 1 && c.split_tail ? r.ways : 1};                    \
    for (int e = 0; e < 5; ++e) out[e] = o[e];                                                                   \
  }
  VLC_GEMM_TILES(X)
#undef X
  return VLC_OK;
}

extern "C" int vlc_probe_gemm_waves(int epilogue, int64_t M, int64_t N, int64_t K, int scratch, int deferred) {
  if (M <= 0 || N <= 0 || K < vlc::BK || K % vlc::BK) return 0;
  const vlc::TileChoice c =
      vlc::choose_tile(M, N, K, epilogue, deferred != 0, scratch ? vlc::gemm_splitk_ws_bytes(M, N) : 0);
#define X(BM, BN, WGM, WGN, S, OCC, USE, STAY, L, F, MA) WGM * WGN,
  static constexpr int kWaves[] = {VLC_GEMM_TILES(X)};
#undef X
  return kWaves[c.index];
}

extern "C" int vlc_probe_gemm_stays(int epilogue, int64_t M, int64_t N, int64_t K, int scratch, int deferred) {
  int32_t o[5];   // rows, columns, workgroups per CU, k ranges, k ranges of the last round's tiles
  if (vlc_probe_gemm_choice(epilogue, M, N, K, scratch, deferred, o) || o[3] > 1) return 0;
  const int64_t cn = epilogue == vlc::EPI_SWIGLU ? o[1] / 2 : o[1], slots = 256 * o[2];
  const int64_t tiles = ((M + o[0] - 1) / o[0]) * ((N + cn - 1) / cn);
  const vlc::TileChoice c = vlc::choose_tile(M, N, K, epilogue, deferred != 0, scratch ? vlc::gemm_splitk_ws_bytes(M, N) : 0);
#define X(BM, BN, WGM, WGN, S, OCC, USE, STAY, L, F, MA) STAY,
  static constexpr int kStays[] = {VLC_GEMM_TILES(X)};
#undef X
  const bool may = vlc::tile_may_stay(kStays[c.index], epilogue);
  return vlc::gemm_stays(may, tiles + (o[4] - 1) * (tiles % slots), (int)slots, (M + (epilogue == vlc::EPI_SWIGLU ? 2 : 1) * N) * K * 2);
}

extern "C" int vlc_probe_group_tile_rows(int64_t pairs, int n_experts, int64_t width, int dtype) {
  return vlc::gemm_group_tile_rows(pairs, n_experts, width, dtype);
}
