// Attention for the recomputed query rows only, over the whole blended K/V of their request
// (Fig. 4 of the paper: row blocks of the recomputed tokens, each spanning its full causal key range).
//   bf16: MFMA flash-style kernel, one workgroup per (block of query rows, kv head); the g = Hq/Hkv
//         query heads that share a kv head are stacked into the same tile so K/V are streamed once
//         for all of them.
//   f32 : few (row, head) pairs: one workgroup each, on vector instructions; many: MFMA tiles of 16 pairs of one kv head.
#include <hip/hip_runtime.h>

#include "attention_shares.h"

namespace vlc {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

__device__ __forceinline__ uint32_t f32_to_bf16(float f) {   // round to nearest, ties to even
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) { return f32_to_bf16(a) | (f32_to_bf16(b) << 16); }

// ---------------------------------------------------------------------------------------------
// bf16 MFMA kernel, D = 128
// ---------------------------------------------------------------------------------------------
// Tile: VR = 128 "virtual rows" = (query row, head of the kv group) pairs, head fastest; 4 wavefronts
// of 32 virtual rows (two tiles of 16) each, two workgroups per CU.  Keys are consumed in blocks of 64.
//
// Both products are computed transposed so that a lane's accumulators belong to two virtual rows only:
//   S^T[key, vr] = K[key, :] . Q[vr, :]      MFMA A = K fragment (LDS), B = Q fragment (registers)
//   O^T[d,  vr] += V^T[d, key] P^T[key, vr]  MFMA A = V^T fragment (LDS), B = P^T (from S^T registers)
// In the 16x16 accumulator layout lane l holds column vr = l % 16 and rows 4*(l/16) + j, so running max, sum and rescale
// factor of a row are per-lane scalars and the only cross-lane step is one exchange between the four lanes of a row.  The S^T
// accumulators of two key tiles feed the second MFMA directly: its contraction index is just a relabeling of keys, as long as the
// V^T fragment uses the same relabeling, which is how it is read from LDS.
//
// 16x16x32 and not 32x32x16: from some thousand rows on the kernel runs at the power limit of the card (18944 rows: 1.64 of 2.4 GHz with up to
// 18432 keys a row on one card, matrix pipe busy 57 % of the cycles; with 32x32x16 1.53 GHz and 59 % there), and a loop of
// MFMAs on random operands reaches 1.70 ... 1.82 PFLOP/s with 32x32x16 there, 2.04 ... 2.18 with 16x16x32.  The K and V fragments are
// as large and feed as many products.  By itself at 18944 rows (28 / 4 heads, 3.9 TFLOP) 3631 -> 3474 us and, on a card that
// throttles more, 4230 -> 4029; inside the layer 3754 -> 3683; 7104 rows (32 / 4 heads) 741 -> 710, inside the layer 795 -> 778; 5824 rows 248 -> 238.
//
// K/V blocks go through a two-stage LDS ring: while block kb is consumed, the K and V tiles of block
// kb+1 are copied global -> LDS directly, both row-major [key][d] (the XOR swizzles are applied by
// permuting which 16-byte chunk each lane fetches).  The V^T fragments are read with the transposing
// LDS load (ds_read_b64_tr_b16): inside a group of 16 lanes, lane i receives element i%4 of the four
// 8-byte chunks addressed by lanes i/4, i/4+4, i/4+8, i/4+12; with lane s of the group pointing at
// row key0 + s/4, columns d0 + 4*(s%4), lane i ends up with V[key0 .. key0+3][d0 + i].
constexpr int ATT_D = 128;
constexpr int KB = ATT_KB;    // keys per block
constexpr int VR = 128;       // virtual rows per workgroup
constexpr int K_TILE_CHUNKS = KB * 16;      // [64 keys][16 chunks of 8 d]
constexpr int V_TILE_CHUNKS = KB * 16;      // same shape
constexpr int ATT_STAGE_CHUNKS = K_TILE_CHUNKS + V_TILE_CHUNKS;   // one K tile + one V tile

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

// K tile: chunk XOR key%16 (a 16-byte fragment read takes 16 keys x 4 chunks; each of its four turns touches every bank once).
// V tile: chunk XOR (key%8)*2 (a transposing read takes 16 keys x 32 bytes).
__device__ __forceinline__ int k_swz(int key, int c) { return c ^ (key & 15); }
__device__ __forceinline__ int v_swz(int key, int c) { return c ^ ((key & 7) << 1); }

// One wavefront-level global -> LDS copy of 64 x 16 bytes (lane l's 16 bytes land at dst + l).  Issued
// as inline assembly: through the builtin the compiler, unable to tell the LDS write apart from the
// fragment reads that follow, waits for every outstanding copy (vmcnt(0)) before the first of them,
// which serialises the prefetch with the block it was meant to overlap.  This way the copies are
// tracked only by the explicit waits at the end of each key block (the key loop has no other
// vector-memory instruction).  M0 holds the LDS address and is written right before each use.
// The global address is a wavefront-uniform base (scalar registers) plus a 32-bit byte offset per lane, so a copy
// needs no vector address arithmetic.
__device__ __forceinline__ void dma16(const void* uniform_base, uint32_t lane_byte_off, u32x4* lds_dst) {
  const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_dst;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(a), "v"(lane_byte_off), "s"(uniform_base)
               : "memory");
}

// Max / sum over the four lanes (l, l ^ 16, l ^ 32, l ^ 48) that share a virtual row, of both rows of a lane, in all of them: the
// swaps put one half's values beside the other's without an LDS round trip (a ds_bpermute here would also make the
// wavefront wait for every fragment read in flight)
__device__ __forceinline__ float2 row_max(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const float m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));          // a's in the lower half, b's in the upper
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  const float t = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return make_float2(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float2 row_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const float m = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  const float t = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return make_float2(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

#define VLC_ATT_WAIT_VM0() __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8) | (0 << 14))

// Block id -> (kv head, row tile); tile < 0: none.  XCD = id % 8.  With share = 8 / Hkv XCDs per kv head (Hkv divides 8)
// XCD x works on head x / share and takes tiles x % share, x % share + share, ...; otherwise the (head, tile) pairs in
// head order are dealt to the XCDs in contiguous pieces.
__host__ __device__ inline int att_grid(int tiles, int Hkv) {
  const int share = Hkv <= 8 && 8 % Hkv == 0 ? 8 / Hkv : 0;
  return share ? 8 * ((tiles + share - 1) / share) : tiles * Hkv;
}
__device__ __forceinline__ void att_tile(int id, int tiles, int Hkv, int* kvh, int* tile) {
  int t;
  if (Hkv <= 8 && 8 % Hkv == 0) {
    const int share = 8 / Hkv, xcd = id % 8;
    *kvh = xcd / share;
    t = id / 8 * share + xcd % share;
  } else {
    const int total = tiles * Hkv, per = total / 8;
    const int vid = id < per * 8 ? (id % 8) * per + id / 8 : id;
    *kvh = vid / tiles;
    t = vid - *kvh * tiles;
  }
  *tile = tiles - 1 - t;
}

// workgroups per kv head of a launch with shares, and block id -> (kv head, piece); XCDs as in att_tile
__host__ __device__ inline int att_slots(int Hkv) { return 512 / Hkv; }
__device__ __forceinline__ void att_piece(int id, int Hkv, int* kvh, int* piece) {
  if (Hkv <= 8 && 8 % Hkv == 0) {
    const int share = 8 / Hkv, xcd = id % 8;
    *kvh = xcd / share;
    *piece = id / 8 * share + xcd % share;
  } else {
    *kvh = id / att_slots(Hkv);
    *piece = id - *kvh * att_slots(Hkv);
  }
}

// SPLIT: the workgroup handles one share of the keys of a row tile (plan_attention_shares) and leaves an un-normalised partial (O as
// float, running max, running sum) for attention_merge_kernel.
template <bool SPLIT>
__global__ __launch_bounds__(256, 2) void attention_bf16_kernel(
    const int4* __restrict__ pieces, const int32_t* __restrict__ row_kv_start, const int32_t* __restrict__ row_kv_len,
    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, int n, int Hkv, int g, int rows_per_tile,
    const uint16_t* __restrict__ q, int64_t q_stride, int Hq, float scale_log2, uint16_t* __restrict__ out,
    float* __restrict__ part_o, float* __restrict__ part_ml) {
  __shared__ u32x4 lds[2 * ATT_STAGE_CHUNKS];     // 64 KB: K ring (2 tiles), then V ring (2 tiles)
  __shared__ int s_start[VR];
  __shared__ int s_len[VR];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, x = lane >> 4;
  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Every XCD works on one kv head at a time, so
  // that the workgroups resident on it stream the same K/V; XCDs that share a kv head (fewer than 8) take its row tiles
  // in turn, because later tiles see more keys: contiguous halves leave the XCD with the early rows idle a third of
  // the time.  Late tiles come first, so that the last workgroups to start are short ones.
  const int tiles = (n + rows_per_tile - 1) / rows_per_tile;
  int kvh, tile;
  int4 share = make_int4(0, 0, 0, 0);   // row tile, share, first key block, end
  if constexpr (SPLIT) {
    int piece;
    att_piece(blockIdx.x, Hkv, &kvh, &piece);
    share = pieces[piece];
    tile = share.x;
    if (tile < 0) return;
  } else {
    att_tile(blockIdx.x, tiles, Hkv, &kvh, &tile);
    if (tile < 0) return;
  }
  const int row0 = tile * rows_per_tile;
  const int rows_here = min(rows_per_tile, n - row0);

  if (tid < rows_per_tile) {                       // rows_per_tile <= 128 threads
    const bool ok = tid < rows_here;
    s_start[tid] = ok ? row_kv_start[row0 + tid] : -1;
    s_len[tid] = ok ? row_kv_len[row0 + tid] : 0;
  }
  __syncthreads();
  // rows lane, lane + 64, ... of the tile in registers: runs and maxima are found by ballots and wavefront maxima (walking
  // the rows through LDS costs a launch of few key blocks 2 us of its 15)
  constexpr int RL = VR / 64;
  int row_start[RL], row_len[RL];
#pragma unroll
  for (int i = 0; i < RL; ++i) {
    const bool ok = lane + 64 * i < rows_here;
    row_start[i] = ok ? s_start[lane + 64 * i] : -1;
    row_len[i] = ok ? s_len[lane + 64 * i] : 0;
  }

  // this lane's virtual rows
  int r_local[2], head[2], my_len[2];
  bool vr_ok[2];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int vr = wave * 32 + v * 16 + l16;
    r_local[v] = vr / g;
    head[v] = kvh * g + (vr - r_local[v] * g);
    vr_ok[v] = r_local[v] < rows_here;
    my_len[v] = vr_ok[v] ? s_len[r_local[v]] : 0;
  }

  // Q fragments: Q[vr][32*ks + 8*x .. +8).  They are fetched together with the first K and V tiles of the first
  // run of rows (one memory latency instead of two, which counts when a workgroup has only a few key blocks).
  bf16x8 qf[2][ATT_D / 32];
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int ks = 0; ks < ATT_D / 32; ++ks) qf[v][ks] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  bool q_loaded = false;

  f32x4 o_acc[ATT_D / 16][2];
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < ATT_D / 16; ++i)
#pragma unroll
    for (int v = 0; v < 2; ++v) o_acc[i][v] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int64_t kv_row_elems = (int64_t)Hkv * ATT_D;

  // K and V tiles: this lane fills LDS chunks (wave*4 + i)*64 + lane, i < 4, of each tile, i.e.
  // key = chunk / 16 and the logical 8-element chunk that the tile's swizzle places there.  Its
  // byte offset from the block's first row is loop-invariant; the block base is wavefront-uniform.
  const uint32_t kv_row_bytes = (uint32_t)Hkv * ATT_D * 2;
  int t_key[4], k_c[4], v_c[4];
  uint32_t k_go[4], v_go[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = (wave * 4 + i) * 64 + lane;
    t_key[i] = p >> 4;
    k_c[i] = k_swz(t_key[i], p & 15);
    v_c[i] = v_swz(t_key[i], p & 15);
    k_go[i] = (uint32_t)t_key[i] * kv_row_bytes + k_c[i] * 16;
    v_go[i] = (uint32_t)t_key[i] * kv_row_bytes + v_c[i] * 16;
  }
  // K fragment reads: key 16*kt + l16, chunk (4*ks + x) ^ (key % 16); byte offset for kt = 0, stage 0
  int k_rd[ATT_D / 32];
#pragma unroll
  for (int ks = 0; ks < ATT_D / 32; ++ks) k_rd[ks] = (l16 * 16 + k_swz(l16, 4 * ks + x)) * 16;
  // transposing V reads: lane s of 16-lane group x points at key 4*x + s/4, columns 4*(s%4) of a 16-wide d tile
  const int tr_key = 4 * x + (l16 >> 2);                 // + 32*t + 16*h
  int v_rd[ATT_D / 16];
#pragma unroll
  for (int dt = 0; dt < ATT_D / 16; ++dt)
    v_rd[dt] = (tr_key * 16 + v_swz(tr_key, 2 * dt + ((l16 & 3) >> 1))) * 16 + (l16 & 1) * 8;

  // Rows of different requests (different row_kv_start) may share a tile: handle one run of equal
  // start at a time; lanes outside the run see every key masked.
  int seg_begin = 0;
  while (seg_begin < rows_here) {
    const int seg_start = __builtin_amdgcn_readfirstlane(s_start[seg_begin]);
    int seg_end = rows_here;                        // first later row of another request
#pragma unroll
    for (int i = RL - 1; i >= 0; --i) {
      const int r = lane + 64 * i;
      const uint64_t other = __ballot(r > seg_begin && r < rows_here && row_start[i] != seg_start);
      if (other) seg_end = 64 * i + __builtin_ctzll(other);
    }
    int seg_max = 0;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      const int r = lane + 64 * i;
      if (r >= seg_begin && r < seg_end) seg_max = max(seg_max, row_len[i]);
    }
    seg_max = wave_max(seg_max);
    seg_max = __builtin_amdgcn_readfirstlane(seg_max);

    int len[2], longest = 0, shortest = -0x7fffffff;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const bool in_seg = vr_ok[v] && r_local[v] >= seg_begin && r_local[v] < seg_end;
      len[v] = in_seg ? my_len[v] : 0;
      longest = max(longest, len[v]);
      if (vr_ok[v]) shortest = max(shortest, -len[v]);
    }
    // longest / shortest visible range among this wavefront's rows (uniform per wavefront); padding lanes (no row behind
    // them) are left out of the shortest: nothing of theirs is stored, so they need no
    // masking - otherwise the wavefront that holds the tile's padding would mask every block
    const int w_max = __builtin_amdgcn_readfirstlane(wave_max(longest));
    const int w_min = -__builtin_amdgcn_readfirstlane(wave_max(shortest));

    const uint16_t* kbase = kc + (int64_t)seg_start * kv_row_elems + (int64_t)kvh * ATT_D;
    const uint16_t* vbase = vc + (int64_t)seg_start * kv_row_elems + (int64_t)kvh * ATT_D;
    const int all_blocks = (seg_max + KB - 1) / KB;
    int kb_first = 0, n_blocks = all_blocks;        // this workgroup's share of the run's key blocks
    if (SPLIT) {
      kb_first = min(all_blocks, share.z);
      n_blocks = min(all_blocks, share.w) - kb_first;
    }
    const int last_key = seg_max - 1;               // loads never leave the run's key range

    // LDS: K ring = chunks [0, 2*K_TILE), V ring = the next 2*V_TILE.
#define VLC_ATT_ISSUE_TILE(base_, go_, c_, kb_, lds_chunk0_)                                                   \
  {                                                                                                            \
    const int key0_ = (kb_) * KB;                                                                              \
    u32x4* dst_ = lds + (lds_chunk0_) + wave * 256;                                                            \
    const char* blk_ = reinterpret_cast<const char*>(base_) + (int64_t)key0_ * kv_row_bytes;                   \
    if (key0_ + KB <= seg_max) { /* whole block inside the run: uniform base + invariant lane offset */        \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) dma16(blk_, go_[i], dst_ + i * 64);                        \
    } else { /* last block of the run: rows past the end re-read the last row */                               \
      _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                            \
        dma16(blk_, (uint32_t)min(t_key[i], last_key - key0_) * kv_row_bytes + c_[i] * 16, dst_ + i * 64);     \
    }                                                                                                          \
  }
#define VLC_ATT_ISSUE_K(kb_, stage_) VLC_ATT_ISSUE_TILE(kbase, k_go, k_c, kb_, (stage_) * K_TILE_CHUNKS)
#define VLC_ATT_ISSUE_V(kb_, stage_) VLC_ATT_ISSUE_TILE(vbase, v_go, v_c, kb_, 2 * K_TILE_CHUNKS + (stage_) * V_TILE_CHUNKS)
    // S^T of one key block: ST[kt][v] = K Q^T from K ring stage kst_; a K fragment serves both row tiles
#define VLC_ATT_QK(ST, kst_)                                                                                   \
  {                                                                                                            \
    const unsigned char* sk_ = reinterpret_cast<const unsigned char*>(lds) + (kst_) * (K_TILE_CHUNKS * 16);    \
    _Pragma("unroll") for (int i = 0; i < 8; ++i) ST[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};               \
    u32x4 kf_[4];   /* four fragments are read ahead */                                                        \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                              \
      kf_[i] = *reinterpret_cast<const u32x4*>(sk_ + k_rd[0] + i * (16 * 256));                                \
    _Pragma("unroll") for (int i = 0; i < 16; ++i) {                                                           \
      _Pragma("unroll") for (int v = 0; v < 2; ++v)                                                            \
        ST[i & 3][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf_[i & 3]), qf[v][i >> 2], ST[i & 3][v], 0, 0, 0); \
      if (i + 4 < 16) kf_[i & 3] = *reinterpret_cast<const u32x4*>(sk_ + k_rd[(i + 4) >> 2] + (i & 3) * (16 * 256));  \
    }                                                                                                          \
  }
    // keys of the block beyond a lane's visible range are masked (only where the block crosses it)
#define VLC_ATT_MASK(ST, key0_)                                                                                \
  {                                                                                                            \
    if ((key0_) + KB > w_min) {                                                                                \
      _Pragma("unroll") for (int v = 0; v < 2; ++v)                                                            \
        _Pragma("unroll") for (int i = 0; i < 16; ++i) {                                                       \
          const int key_ = (key0_) + 16 * (i >> 2) + 4 * x + (i & 3);                                          \
          ST[i >> 2][v][i & 3] = key_ < len[v] ? ST[i >> 2][v][i & 3] : -INFINITY;                             \
        }                                                                                                      \
    }                                                                                                          \
  }
    // online softmax (base 2), first part: the new references of the rows and the rescale factors
#define VLC_ATT_REFERENCE(ST)                                                                                  \
    float mx_[2] = {-INFINITY, -INFINITY};                                                                     \
    _Pragma("unroll") for (int v = 0; v < 2; ++v)                                                              \
      _Pragma("unroll") for (int i = 0; i < 16; ++i) mx_[v] = fmaxf(mx_[v], ST[i >> 2][v][i & 3]);             \
    const float2 both_ = row_max(mx_[0], mx_[1]);   /* scale > 0: max commutes with it */                      \
    const float m_new_[2] = {fmaxf(m_run[0], both_.x * scale_log2), fmaxf(m_run[1], both_.y * scale_log2)};    \
    const float m_use_[2] = {m_new_[0] == -INFINITY ? 0.f : m_new_[0], m_new_[1] == -INFINITY ? 0.f : m_new_[1]}; \
    const float alpha_[2] = {__builtin_amdgcn_exp2f(m_run[0] - m_use_[0]),   /* m_run = -inf -> 0 */           \
                             __builtin_amdgcn_exp2f(m_run[1] - m_use_[1])};                                    \
    const bool grew_ = m_new_[0] > m_run[0] || m_new_[1] > m_run[1];                                           \
    m_run[0] = m_new_[0];                                                                                      \
    m_run[1] = m_new_[1];
    // second part: the probabilities of key tiles [first_, last_), in place
#define VLC_ATT_EXP(ST, first_, last_)                                                                         \
    _Pragma("unroll") for (int i = 4 * (first_); i < 4 * (last_); ++i)                                         \
      _Pragma("unroll") for (int v = 0; v < 2; ++v)                                                            \
        ST[i >> 2][v][i & 3] = __builtin_amdgcn_exp2f(fmaf(ST[i >> 2][v][i & 3], scale_log2, -m_use_[v]));
    // order template for the block of the next block's S^T: four K fragment reads up front, then per fragment two MFMAs, vector
    // work of this block's softmax behind each, and a read
#define VLC_ATT_INTERLEAVE()                                                                                   \
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);                                                         \
    _Pragma("unroll") for (int g_ = 0; g_ < 16; ++g_) {                                                        \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                       \
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);                                                       \
      __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);                                                       \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                       \
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);                                                       \
      __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);                                                       \
      if (g_ < 12) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                          \
    }
    // O rescale (only when some row's maximum moved)
#define VLC_ATT_RESCALE()                                                                                      \
    if (__any(grew_)) {                                                                                        \
      _Pragma("unroll") for (int v = 0; v < 2; ++v) {                                                          \
        _Pragma("unroll") for (int i = 0; i < ATT_D / 16; ++i)                                                 \
          _Pragma("unroll") for (int e = 0; e < 4; ++e) o_acc[i][v][e] *= alpha_[v];                           \
        l_run[v] *= alpha_[v];                                                                                 \
      }                                                                                                        \
    }
    // row sums and O^T += V^T P^T from V ring stage vst_; a V^T fragment (32 keys x 16 d) serves both row tiles
#define VLC_ATT_PV(ST, vst_)                                                                                   \
  {                                                                                                            \
    const unsigned char* sv_ = reinterpret_cast<const unsigned char*>(lds + 2 * K_TILE_CHUNKS + (vst_) * V_TILE_CHUNKS); \
    float psum_[2] = {0.f, 0.f};                                                                               \
    _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                                            \
      bf16x8 pf_[2];                                                                                           \
      _Pragma("unroll") for (int v = 0; v < 2; ++v)                                                            \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                        \
          f32x2 pr_ = {ST[2 * t + (e >> 1)][v][2 * (e & 1)], ST[2 * t + (e >> 1)][v][2 * (e & 1) + 1]};        \
          const bf16x2 pb_ = __builtin_convertvector(pr_, bf16x2);                                             \
          pf_[v][2 * e] = pb_[0];                                                                              \
          pf_[v][2 * e + 1] = pb_[1];                                                                          \
        }                                                                                                      \
      _Pragma("unroll") for (int dt = 0; dt < ATT_D / 16; ++dt) {                                              \
        s16x4 vh_[2];                                                                                          \
        _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                          \
          vh_[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(         \
              const_cast<unsigned char*>(sv_) + v_rd[dt] + (32 * t + 16 * h) * 256));                          \
        const s16x8 vv_ = __builtin_shufflevector(vh_[0], vh_[1], 0, 1, 2, 3, 4, 5, 6, 7);                     \
        _Pragma("unroll") for (int v = 0; v < 2; ++v) {                                                        \
          o_acc[dt][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv_), pf_[v], o_acc[dt][v], 0, 0, 0); \
          psum_[v] += ST[2 * t + (dt >> 2)][v][dt & 3];                                                        \
        }                                                                                                      \
      }                                                                                                        \
    }                                                                                                          \
    l_run[0] += psum_[0];                                                                                      \
    l_run[1] += psum_[1];                                                                                      \
  }
    // One key block j (S^T already in CUR): fetch ahead, start the next block's S^T into NXT (its MFMAs
    // are independent of this block's softmax arithmetic, so the two interleave), finish this block.
    // Half of the probabilities are taken under the S^T MFMAs and held there (the compiler moves what only the PV block uses behind the
    // rescale branch, where all 32 stood before: 3651 -> 3617 us at 18944 rows), half under the PV MFMAs.
    // The PV product runs at a raised wave priority: two wavefronts share a SIMD, and the matrix pipe is only kept busy when one
    // multiplies while the other does its softmax arithmetic.  With equal priorities two wavefronts that reach
    // their MFMA phases together alternate instruction by instruction and stay in step; the priority lets the
    // one already in its PV phase run ahead, which puts the pair out of step (4176 -> 4029 us).
#define VLC_ATT_BLOCK(j_, PAR, CUR, NXT)                                                                       \
  {                                                                                                            \
    if ((j_) + 2 < n_blocks) VLC_ATT_ISSUE_K(kb_first + (j_) + 2, PAR)                                         \
    if ((j_) + 1 < n_blocks) VLC_ATT_ISSUE_V(kb_first + (j_) + 1, (PAR) ^ 1)                                   \
    const int key0b_ = (kb_first + (j_)) * KB;                                                                 \
    if (key0b_ < w_max) { /* something visible for this wavefront in this block */                             \
      VLC_ATT_MASK(CUR, key0b_)                                                                                \
      VLC_ATT_QK(NXT, (PAR) ^ 1)   /* past the last block this reads a stale tile; the result is unused */     \
      VLC_ATT_REFERENCE(CUR)                                                                                   \
      VLC_ATT_EXP(CUR, 0, 2)                                                                                   \
      VLC_ATT_INTERLEAVE()                                                                                     \
      asm volatile("" : "+v"(CUR[0][0]), "+v"(CUR[0][1]), "+v"(CUR[1][0]), "+v"(CUR[1][1]));   /* see above */ \
      __builtin_amdgcn_s_setprio(1);   /* see above */                                                         \
      VLC_ATT_RESCALE()                                                                                        \
      VLC_ATT_EXP(CUR, 2, 4)                                                                                   \
      VLC_ATT_PV(CUR, PAR)                                                                                     \
      __builtin_amdgcn_s_setprio(0);                                                                           \
    }                                                                                                          \
    VLC_ATT_WAIT_VM0();   /* this wavefront's shares of the tiles fetched above have landed */                 \
    __syncthreads();                                                                                           \
  }

    __syncthreads();                 // the rings are free (previous run finished reading them)
    f32x4 st_a[4][2], st_b[4][2];
    if (n_blocks > 0) {
      VLC_ATT_ISSUE_K(kb_first, 0)
      VLC_ATT_ISSUE_V(kb_first, 0)
      if (n_blocks > 1) VLC_ATT_ISSUE_K(kb_first + 1, 1)
    }
    if (!q_loaded) {
      q_loaded = true;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const u32x4* qp = reinterpret_cast<const u32x4*>(q + (int64_t)(row0 + (vr_ok[v] ? r_local[v] : 0)) * q_stride +
                                                         (int64_t)head[v] * ATT_D);
#pragma unroll
        for (int ks = 0; ks < ATT_D / 32; ++ks)
          if (vr_ok[v]) qf[v][ks] = __builtin_bit_cast(bf16x8, qp[4 * ks + x]);
      }
    }
    // The Q loads are the only vector-memory reads the compiler knows of; completing them here, together with
    // this wavefront's shares of the tiles fetched above, keeps it from placing a vmcnt(0) wait (which would
    // also wait for freshly issued K/V copies) at their first use inside the key loop.
    VLC_ATT_WAIT_VM0();
    __syncthreads();
    if (n_blocks > 0 && kb_first * KB < w_max) VLC_ATT_QK(st_a, 0)
    __syncthreads();                 // K stage 0 may be refilled from here on
    for (int j = 0; j < n_blocks; j += 2) {
      VLC_ATT_BLOCK(j, 0, st_a, st_b)
      if (j + 1 < n_blocks) VLC_ATT_BLOCK(j + 1, 1, st_b, st_a)
    }
#undef VLC_ATT_ISSUE_TILE
#undef VLC_ATT_ISSUE_K
#undef VLC_ATT_ISSUE_V
#undef VLC_ATT_QK
#undef VLC_ATT_MASK
#undef VLC_ATT_REFERENCE
#undef VLC_ATT_EXP
#undef VLC_ATT_INTERLEAVE
#undef VLC_ATT_RESCALE
#undef VLC_ATT_PV
#undef VLC_ATT_BLOCK
    seg_begin = seg_end;
  }

  // ---- normalise and store: lane holds d = 16*dt + 4*x + j of its virtual rows ------------------
  const float2 l_both = row_sum(l_run[0], l_run[1]);
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const float l_tot = v ? l_both.y : l_both.x;
    if (!vr_ok[v]) continue;
    if (SPLIT) {
      const int64_t rh = ((int64_t)share.y * n + (row0 + r_local[v])) * Hq + head[v];
      float* po = part_o + rh * ATT_D + 4 * x;
#pragma unroll
      for (int dt = 0; dt < ATT_D / 16; ++dt)
        *reinterpret_cast<float4*>(po + 16 * dt) = make_float4(o_acc[dt][v][0], o_acc[dt][v][1], o_acc[dt][v][2], o_acc[dt][v][3]);
      if (x == 0) {
        part_ml[2 * rh] = m_run[v];
        part_ml[2 * rh + 1] = l_tot;
      }
    } else {
      const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
      uint16_t* op = out + ((int64_t)(row0 + r_local[v]) * Hq + head[v]) * ATT_D + 4 * x;
#pragma unroll
      for (int dt = 0; dt < ATT_D / 16; ++dt) {
        f32x2 a0 = {o_acc[dt][v][0] * inv, o_acc[dt][v][1] * inv};
        f32x2 a1 = {o_acc[dt][v][2] * inv, o_acc[dt][v][3] * inv};
        u32x2 w;
        w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(a0, bf16x2));
        w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(a1, bf16x2));
        *reinterpret_cast<u32x2*>(op + 16 * dt) = w;
      }
    }
  }
}

// Merge of the split partials: out = sum_z O_z 2^(m_z - m) / sum_z l_z 2^(m_z - m), m = max_z m_z, over the
// shares of the row's tile.  One thread per 8 output elements.
__global__ __launch_bounds__(256) void attention_merge_kernel(const float* __restrict__ part_o,
                                                              const float* __restrict__ part_ml,
                                                              const int32_t* __restrict__ tile_shares,
                                                              const int32_t* __restrict__ row_kv_len, int64_t rows_heads,
                                                              int rows_per_tile, int Hq, uint16_t* __restrict__ out) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t rh = id / (ATT_D / 8);
  const int c = (int)(id - rh * (ATT_D / 8));
  if (rh >= rows_heads) return;
  const uint32_t row = (uint32_t)rh / (uint32_t)Hq;
  // a tile whose rows see no key has no share
  const int nsplit = row_kv_len[row] > 0 ? tile_shares[row / (uint32_t)rows_per_tile] : 0;
  // all loads of a pass are issued together (at most ATT_MAX_SHARES shares): running maxima and sums first, then the outputs
  constexpr int MAXZ = ATT_MAX_SHARES;
  float mz[MAXZ], lz[MAXZ];
#pragma unroll
  for (int z = 0; z < MAXZ; ++z) {
    mz[z] = -INFINITY;
    lz[z] = 0.f;
    if (z < nsplit) {
      const float2 ml = *reinterpret_cast<const float2*>(part_ml + 2 * (z * rows_heads + rh));
      mz[z] = ml.x;
      lz[z] = ml.y;
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int z = 0; z < MAXZ; ++z) m = fmaxf(m, mz[z]);
  float4 pa[MAXZ], pb[MAXZ];
  float wz[MAXZ];
#pragma unroll
  for (int z = 0; z < MAXZ; ++z) {
    wz[z] = mz[z] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mz[z] - m);   // -inf: this share saw no visible key
    pa[z] = pb[z] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (z < nsplit && mz[z] != -INFINITY) {
      const float4* po = reinterpret_cast<const float4*>(part_o + (z * rows_heads + rh) * ATT_D + 8 * c);
      pa[z] = po[0];
      pb[z] = po[1];
    }
  }
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float l = 0.f;
#pragma unroll
  for (int z = 0; z < MAXZ; ++z) {      // in share order, as before
    l += lz[z] * wz[z];
    acc[0] += pa[z].x * wz[z]; acc[1] += pa[z].y * wz[z]; acc[2] += pa[z].z * wz[z]; acc[3] += pa[z].w * wz[z];
    acc[4] += pb[z].x * wz[z]; acc[5] += pb[z].y * wz[z]; acc[6] += pb[z].z * wz[z]; acc[7] += pb[z].w * wz[z];
  }
  const float inv = l == 0.f ? 0.f : 1.0f / l;   // a NaN sum stays NaN, as in the whole form
  u32x4 w4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f32x2 pr = {acc[2 * e] * inv, acc[2 * e + 1] * inv};
    w4[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
  }
  *reinterpret_cast<u32x4*>(out + rh * ATT_D + 8 * c) = w4;
}

// ---------------------------------------------------------------------------------------------
// f32 kernels (the small fp32 configuration)
// ---------------------------------------------------------------------------------------------
// From kF32PairsPerTile (row, head) pairs on 16 of them share a workgroup of four wavefronts, from kF32OneWavePairs on one wavefront.
// 4 / 2 heads, us, at 304 keys (in brackets at 1000), one workgroup per pair | 16 pairs on four wavefronts | on one:
//   pairs        244           512           768           1200          4800           12000          32000
//   D = 64    5.2 | 8.8      7.9 | 8.8     9.9 | 8.8    13.5 | 8.9     44 | 11.4    16.5 | 21.6    36.8 | 37.5 (83.8 | 102.9)
//   D = 128   6.6 | 14.7    11.5 | 15.0   15.5 | 15.0   22.9 | 15.1    79 | 25.1    39.3 | 34.1    93.4 | 66.4 (196 | 202)
// The kernel before, one or eight wavefronts per pair that read K and V for themselves: 55, 105 and 250 us at D = 64 and 4800, 12000 and
// 32000 pairs over 304 keys.  Four wavefronts of which each asks for the next step's pieces ahead take 186 registers instead of
// 136: 3 % faster up to 2400 pairs, 30 % slower at 12000.
// The line at 640 holds from 16 to 1000 keys; the one at 32768 is a mean: one wavefront per tile is faster there by 40 % at 16 keys (D = 128:
// by 60 %) and level at 304 (15 % faster), and slower by 25 % (15 %) at 1000.
constexpr int64_t kF32PairsPerTile = 640, kF32OneWavePairs = 32768;
// Tiles with rows of several requests: what a step of such a run costs, in steps of a pair on its own (estimated from the MFMAs of
// a step).  Rows that are all of other requests, one head per kv head, us at 16 / 304 / 1000 keys, runs | pairs | the kernel before
// (which took every pair by itself):
//   640 pairs, D = 64    40 | 7 | 8      126 | 20 | 20     399 | 71 | 62       D = 128    65 | 7 | 8      224 | 31 | 36     727 | 128 | 156
//   4800                 45 | 12 | 10    208 | 145 | 136   553 | 466 | 433                146 | 23 | 17   561 | 332 | 323   1517 | 1072 | 999
//   33000                92 | 58 | 48    934 | 896 | 843                                  271 | 153 | 123
// Of four requests per tile: 640 pairs 12 | 7 | 8, 31 | 13 | 20, 87 | 46 | 53; 4800 pairs 13 | 11 | 12, and from 64 keys on the runs.
template <int D> constexpr int kF32RunSteps = D == 64 ? 2 : 3;

__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// sum over the 16 lanes of a DPP row, in all of them
__device__ __forceinline__ float sum16(float v) {
  v += __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0xb1, 0xf, 0xf, true));    // quad_perm [1,0,3,2]
  v += __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x4e, 0xf, 0xf, true));    // quad_perm [2,3,0,1]
  v += __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x141, 0xf, 0xf, true));   // row_half_mirror
  v += __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x140, 0xf, 0xf, true));   // row_mirror
  return v;
}
// max / sum over lanes l, l ^ 16, l ^ 32, l ^ 48, in all of them
__device__ __forceinline__ float max_rows(float a) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  const float t = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float sum_rows(float a) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  const float t = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Few (row, head) pairs: one workgroup of 16 wavefronts per pair, bound by latency.  Sixteen lanes share a key, 16 bytes of it
// each, so that a load touches whole lines of four keys; a wavefront takes 32 keys at a time, the workgroup 512.  At D = 64 all K and V
// of a step are asked for together; at D = 128 they do not fit the 128 registers of 1024 threads, and part of V is loaded behind the
// scores.  D = 64, 61 rows x 4 heads over 304 / 1000 keys 5.2 / 8.9 us (one lane per key, whose load touched 64 lines, and V only behind
// the softmax: 7.7 / 17.2).
template <int D>
__global__ __launch_bounds__(1024) void attention_f32_pair_kernel(
    const float* __restrict__ q, const int32_t* __restrict__ row_kv_len, const int32_t* __restrict__ row_kv_start,
    const float* __restrict__ kc, const float* __restrict__ vc, int q_stride, int Hkv, int g, float scale, int Hq,
    float* __restrict__ out) {
  constexpr int W = 16, U = 8, P = D / 64;          // wavefronts, keys per lane, 16-byte pieces per lane and key
  __shared__ float red_m[W], red_l[W];
  __shared__ f32x4 red_o[W][D / 4];
  const int row = blockIdx.x, head = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, x = lane >> 4, kvh = head / g;
  const int len = row_kv_len[row];
  const int64_t start = row_kv_start[row], kv_row = (int64_t)Hkv * D;
  const float* qp = q + (int64_t)row * q_stride + (int64_t)head * D + 4 * l16;
  f32x4 qv[P];
#pragma unroll
  for (int p = 0; p < P; ++p) qv[p] = *reinterpret_cast<const f32x4*>(qp + 64 * p) * scale;
  const float* kbase = kc + start * kv_row + (int64_t)kvh * D + 4 * l16;
  const float* vbase = vc + start * kv_row + (int64_t)kvh * D + 4 * l16;
  float m = -INFINITY, l = 0.f;
  f32x4 acc[P];
#pragma unroll
  for (int p = 0; p < P; ++p) acc[p] = zero4();
  for (int c0 = 32 * wave; c0 < len; c0 += 32 * W) {
    f32x4 kv[U][P], vv[U][P];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p)                   // past the end: the last visible row again, left out below
        kv[u][p] = *reinterpret_cast<const f32x4*>(kbase + (int64_t)min(c0 + 4 * u + x, len - 1) * kv_row + 64 * p);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p)
        vv[u][p] = *reinterpret_cast<const f32x4*>(vbase + (int64_t)min(c0 + 4 * u + x, len - 1) * kv_row + 64 * p);
    float s[U], mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      f32x4 t = kv[u][0] * qv[0];
#pragma unroll
      for (int p = 1; p < P; ++p) t += kv[u][p] * qv[p];
      s[u] = sum16((t[0] + t[1]) + (t[2] + t[3]));
      if (c0 + 4 * u + x >= len) s[u] = -INFINITY;
      mx = fmaxf(mx, s[u]);
    }
    const float m_new = fmaxf(m, max_rows(mx));     // -inf only if every score so far is -inf or NaN
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m - m_use);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float e = expf(s[u] - m_use);
      l += e;
      const bool seen = c0 + 4 * u + x < len;       // a value past the end (it may be an infinity) does not count
#pragma unroll
      for (int p = 0; p < P; ++p) acc[p] += e * (seen ? vv[u][p] : zero4());
    }
  }
  l = sum_rows(l);
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[p][e] = sum_rows(acc[p][e]);
  if (lane < 16) {
#pragma unroll
    for (int p = 0; p < P; ++p) red_o[wave][16 * p + l16] = acc[p];
    if (lane == 0) {
      red_m[wave] = m;
      red_l[wave] = l;
    }
  }
  __syncthreads();
  if (tid >= D) return;
  float top = -INFINITY, lt = 0.f, o = 0.f;
#pragma unroll
  for (int w = 0; w < W; ++w) top = fmaxf(top, red_m[w]);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const float f = red_m[w] == -INFINITY ? 0.f : expf(red_m[w] - top);
    lt += red_l[w] * f;
    o += reinterpret_cast<const float*>(red_o[w])[tid] * f;
  }
  out[((int64_t)row * Hq + head) * D + tid] = len > 0 ? o / lt : 0.f;   // a NaN sum stays NaN
}

// One (row, head) pair by one wavefront, in the manner of the kernel above: 512 / D groups of four keys per step.  qp, kp, vp, op: at this
// lane's first piece of the row.  (As the body of the kernel above too, it waited for K more often: 5 % slower at 600 pairs.)
template <int D>
__device__ __forceinline__ void attend_pair_f32(const float* __restrict__ qp, const float* __restrict__ kp, const float* __restrict__ vp,
                                                int64_t kv_row, int len, float scale, float* __restrict__ op) {
  constexpr int U = 512 / D, P = D / 64;
  const int lane = threadIdx.x & 63, x = lane >> 4;
  f32x4 qv[P], acc[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    qv[p] = *reinterpret_cast<const f32x4*>(qp + 64 * p) * scale;
    acc[p] = zero4();
  }
  float m = -INFINITY, l = 0.f;
  for (int c0 = 0; c0 < len; c0 += 4 * U) {
    f32x4 kv[U][P], vv[U][P];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p)                   // past the end: the last visible row again, left out below
        kv[u][p] = *reinterpret_cast<const f32x4*>(kp + (int64_t)min(c0 + 4 * u + x, len - 1) * kv_row + 64 * p);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p)
        vv[u][p] = *reinterpret_cast<const f32x4*>(vp + (int64_t)min(c0 + 4 * u + x, len - 1) * kv_row + 64 * p);
    float s[U], mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      f32x4 t = kv[u][0] * qv[0];
#pragma unroll
      for (int p = 1; p < P; ++p) t += kv[u][p] * qv[p];
      s[u] = sum16((t[0] + t[1]) + (t[2] + t[3]));
      if (c0 + 4 * u + x >= len) s[u] = -INFINITY;
      mx = fmaxf(mx, s[u]);
    }
    const float m_new = fmaxf(m, max_rows(mx));     // -inf only if every score so far is -inf or NaN
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m - m_use);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float e = expf(s[u] - m_use);
      l += e;
      const bool seen = c0 + 4 * u + x < len;       // a value past the end (it may be an infinity) does not count
#pragma unroll
      for (int p = 0; p < P; ++p) acc[p] += e * (seen ? vv[u][p] : zero4());
    }
  }
  l = sum_rows(l);
#pragma unroll
  for (int p = 0; p < P; ++p) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[p][e] = len > 0 ? sum_rows(acc[p][e]) / l : 0.f;   // a NaN sum stays NaN
    if (lane < 16) *reinterpret_cast<f32x4*>(op + 64 * p) = acc[p];
  }
}

// Many pairs: 16 "virtual rows" (row, head of the kv group), head fastest, per workgroup, both products on
// v_mfma_f32_16x16x4_f32 (exact products, float sums), transposed as in the bf16 kernel: a lane's accumulators belong to one virtual
// row, and S^T feeds the second product from its registers.  Fragments come straight from global memory in 16-byte pieces: element e
// of a K piece is the k-slice of MFMA e; element e of a V piece belongs to the MFMA of output columns 4i + e.  The W wavefronts
// take every W-th step of 32 keys and meet in LDS.  K and V are read once per 16 pairs instead of once per pair.
template <int D, int W>
__global__ __launch_bounds__(64 * W) void attention_f32_tile_kernel(
    const float* __restrict__ q, const int32_t* __restrict__ row_kv_len, const int32_t* __restrict__ row_kv_start,
    const float* __restrict__ kc, const float* __restrict__ vc, int64_t pairs, int q_stride, int Hkv, int g, float scale, int Hq,
    float* __restrict__ out, int shares) {
  constexpr int DS = D / 16, DH = D / 64;
  __shared__ float red_m[W][16], red_l[W][16];
  __shared__ f32x4 red_o[W > 1 ? W : 1][W > 1 ? D / 4 : 1][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  const int l16 = lane & 15, x = lane >> 4, kvh = blockIdx.y;
  // z: a share of the tiles, or (few tiles) a workgroup among several of every tile; pairs: n * g of one kv head
  const int share = shares > 1 ? blockIdx.z : 0;
  const int64_t vr0 = ((int64_t)(shares > 1 ? 0 : blockIdx.z) * gridDim.x + blockIdx.x) * 16;
  if (vr0 >= pairs) return;
  const int64_t vr = vr0 + l16;
  const bool ok = vr < pairs;
  const int64_t row = (ok ? vr : pairs - 1) / g;
  const int head = kvh * g + (int)((ok ? vr : pairs - 1) - row * g);
  const int my_start = row_kv_start[row], my_len = ok ? row_kv_len[row] : 0;
  const int64_t kv_row = (int64_t)Hkv * D;

  // Rows of several requests: a run of equal first slots uses one of `runs` parts of the MFMAs, one run after the other.  Where that takes
  // longer than the pairs one by one, shared out over the wavefronts of all workgroups of the tile, these do it.
  const int next_start = __shfl(my_start, l16 < 15 ? l16 + 1 : l16);
  const int runs = 1 + __builtin_popcountll(__ballot(lane < 15 && next_start != my_start));
  if (runs > 1) {
    const int top = __builtin_amdgcn_readfirstlane(wave_max(my_len));
    const int tile_steps = runs * ((top + 32 * W - 1) / (32 * W));
    const int pair_steps = (16 + shares * W - 1) / (shares * W) * ((top + 2048 / D - 1) / (2048 / D));
    if (tile_steps * kF32RunSteps<D> > pair_steps) {
      for (int i = share * W + wave; i < 16; i += shares * W) {
        const int64_t v = vr0 + i;
        if (v >= pairs) return;
        const int64_t r = v / g;
        const int h = kvh * g + (int)(v - r * g);
        const int64_t at = (int64_t)row_kv_start[r] * kv_row + (int64_t)kvh * D + 4 * l16;
        attend_pair_f32<D>(q + r * q_stride + (int64_t)h * D + 4 * l16, kc + at, vc + at, kv_row, row_kv_len[r], scale,
                           out + (r * Hq + h) * D + 4 * l16);
      }
      return;                                       // the same for the whole workgroup
    }
  }
  if (share) return;
  f32x4 qf[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s)
    qf[s] = *reinterpret_cast<const f32x4*>(q + row * q_stride + (int64_t)head * D + 16 * s + 4 * x) * scale;
  float m = -INFINITY, l = 0.f;
  f32x4 o[DH][4];
#pragma unroll
  for (int h = 0; h < DH; ++h)
#pragma unroll
    for (int t = 0; t < 4; ++t) o[h][t] = zero4();

  // rows of different requests may share a tile: one run of equal first slots after the other
  int run = 0;
  while (run < 16) {
    const int start = __builtin_amdgcn_readlane(my_start, run);
    const uint64_t others = __ballot(lane < 16 && lane > run && my_start != start);
    const int run_end = others ? __builtin_ctzll(others) : 16;
    const int len = l16 >= run && l16 < run_end ? my_len : 0;
    const int longest = __builtin_amdgcn_readfirstlane(wave_max(len));
    const int shortest = -__builtin_amdgcn_readfirstlane(wave_max(ok ? -len : -0x7fffffff));
    run = run_end;
    const float* kbase = kc + (int64_t)start * kv_row + (int64_t)kvh * D + 4 * x;
    const float* vbase = vc + (int64_t)start * kv_row + (int64_t)kvh * D + 4 * l16;
    for (int c0 = 32 * wave; c0 < longest; c0 += 32 * W) {
      f32x4 kf[2][DS], vf[2][4][DH];
#pragma unroll
      for (int t = 0; t < 2; ++t)                   // past the end: the last row of the run again
#pragma unroll
        for (int s = 0; s < DS; ++s)
          kf[t][s] = *reinterpret_cast<const f32x4*>(kbase + (int64_t)min(c0 + 16 * t + l16, longest - 1) * kv_row + 16 * s);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < DH; ++h)
            vf[t][e][h] = *reinterpret_cast<const f32x4*>(vbase + (int64_t)min(c0 + 16 * t + 4 * x + e, longest - 1) * kv_row + 64 * h);
      f32x4 st[2] = {zero4(), zero4()};
#pragma unroll
      for (int s = 0; s < DS; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < 2; ++t)
            st[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][s][e], qf[s][e], st[t], 0, 0, 0);
      const bool partly = c0 + 32 > shortest;       // some row does not see all of these keys
      if (partly) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (c0 + 16 * t + 4 * x + j >= len) st[t][j] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) mx = fmaxf(mx, st[t][j]);
      const float m_new = fmaxf(m, max_rows(mx));
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = expf(m - m_use);          // m = -inf: 0
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int h = 0; h < DH; ++h)
#pragma unroll
        for (int t = 0; t < 4; ++t) o[h][t] *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          st[t][j] = expf(st[t][j] - m_use);
          l += st[t][j];
        }
      // A probability of zero times an infinity is a NaN: where a key that some row does not see has such a value, the
      // products are formed one by one, for the rows that see it.
      bool odd = false;
      if (partly) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < DH; ++h)
#pragma unroll
              for (int i = 0; i < 4; ++i) odd |= !(fabsf(vf[t][e][h][i]) < INFINITY);
      }
      if (__ballot(odd) == 0) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < DH; ++h)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                o[h][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][e][h][i], st[t][e], o[h][i], 0, 0, 0);
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            for (int y = 0; y < 4; ++y) {
              const int key = c0 + 16 * t + 4 * y + e;
              const float p = __shfl(st[t][e], l16 + 16 * y);
              if (key < len) {
                const float* vp = vc + ((int64_t)start + key) * kv_row + (int64_t)kvh * D + 16 * x;
#pragma unroll
                for (int h = 0; h < DH; ++h)
#pragma unroll
                  for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[h][i][j] = fmaf(p, vp[64 * h + 4 * j + i], o[h][i][j]);
              }
            }
      }
    }
  }
  l = sum_rows(l);
  // lane: columns 64 h + 16 x + 4 j + i of its row
  if constexpr (W > 1) {
#pragma unroll
    for (int h = 0; h < DH; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) red_o[wave][16 * h + 4 * x + j][l16] = f32x4{o[h][0][j], o[h][1][j], o[h][2][j], o[h][3][j]};
    if (x == 0) {
      red_m[wave][l16] = m;
      red_l[wave][l16] = l;
    }
    __syncthreads();
    // thread: virtual row id / (D / 4), four columns
    for (int id = tid; id < 16 * (D / 4); id += 64 * W) {
      const int r = id / (D / 4), c = id % (D / 4);
      const int64_t v = vr0 + r;
      if (v >= pairs) break;
      float top = -INFINITY, lt = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w) top = fmaxf(top, red_m[w][r]);
      f32x4 sum = zero4();
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float f = red_m[w][r] == -INFINITY ? 0.f : expf(red_m[w][r] - top);
        lt += red_l[w][r] * f;
        sum += red_o[w][c][r] * f;
      }
      const int64_t orow = v / g;
      const int ohead = kvh * g + (int)(v - orow * g);
      f32x4 res;
#pragma unroll
      for (int i = 0; i < 4; ++i) res[i] = row_kv_len[orow] > 0 ? sum[i] / lt : 0.f;   // a NaN sum stays NaN
      *reinterpret_cast<f32x4*>(out + (orow * Hq + ohead) * D + 4 * c) = res;
    }
  } else if (ok) {
#pragma unroll
    for (int h = 0; h < DH; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f32x4 res;
#pragma unroll
        for (int i = 0; i < 4; ++i) res[i] = my_len > 0 ? o[h][i][j] / l : 0.f;
        *reinterpret_cast<f32x4*>(out + (row * Hq + head) * D + 64 * h + 16 * x + 4 * j) = res;
      }
  }
}

}  // namespace

static int64_t ml_bytes(int64_t shares, int64_t n, int Hq) { return (shares * n * Hq * 2 * 4 + 15) / 16 * 16; }
// partial outputs, running maxima and sums, then the pieces of a head and every tile's number of shares
static int64_t share_bytes(int64_t shares, int64_t n, int Hq, int Hkv, int64_t tiles) {
  return shares * n * Hq * ATT_D * 4 + ml_bytes(shares, n, Hq) + att_slots(Hkv) * (int64_t)sizeof(int4) + tiles * 4;
}

int64_t attention_ws_bytes(int64_t n, int Hq, int Hkv, int D, int dtype) {
  if (dtype != VLC_BF16 || D != ATT_D || Hq % Hkv || Hq / Hkv > VR) return 0;
  const int64_t tiles = (n + VR / (Hq / Hkv) - 1) / (VR / (Hq / Hkv));
  if (tiles * Hkv >= 512 || n <= 0) return 0;          // enough workgroups without splitting
  return share_bytes(ATT_MAX_SHARES, n, Hq, Hkv, tiles);
}

// The most key shares that a row tile may take (1: none).  512 workgroups are resident at once, two per CU: with `pairs`
// (row tile, kv head) pairs a tile has 512 / pairs of them on average, and the longest one sees about twice the mean.
int attention_key_shares(int64_t n, int Hq, int Hkv, int64_t max_kv_len, int64_t ws_bytes) {
  const int rows_per_tile = VR / (Hq / Hkv);
  const int64_t tiles = (n + rows_per_tile - 1) / rows_per_tile, pairs = tiles * Hkv;
  if (pairs >= 512) return 1;
  int shares = (int)(1024 / pairs);
  if (shares > ATT_MAX_SHARES) shares = ATT_MAX_SHARES;
  while (shares > 1 && share_bytes(shares, n, Hq, Hkv, tiles) > ws_bytes) --shares;
  if (max_kv_len > 0) {
    const int64_t blocks = (max_kv_len + KB - 1) / KB, longest = (blocks + ATT_MIN_BLOCKS - 1) / ATT_MIN_BLOCKS;
    if (shares > longest) shares = (int)longest;
  }
  return shares;
}

AttentionShares attention_shares(int64_t n, int Hq, int Hkv, int64_t max_kv_len, const int32_t* row_kv_len, void* ws,
                                 int64_t ws_bytes) {
  AttentionShares a = {};
  a.max_shares = ws ? attention_key_shares(n, Hq, Hkv, max_kv_len, ws_bytes) : 1;
  if (a.max_shares <= 1) return a;
  a.n = (int)n;
  a.rows_per_tile = VR / (Hq / Hkv);
  a.tiles = (int)((n + a.rows_per_tile - 1) / a.rows_per_tile);
  a.slots = att_slots(Hkv);
  a.row_kv_len = row_kv_len;
  a.part_o = static_cast<float*>(ws);
  a.part_ml = a.part_o + (int64_t)a.max_shares * n * Hq * ATT_D;
  a.pieces = reinterpret_cast<int4*>(reinterpret_cast<char*>(a.part_ml) + ml_bytes(a.max_shares, n, Hq));
  a.tile_shares = reinterpret_cast<int32_t*>(a.pieces + a.slots);
  return a;
}

int launch_attention(const void* q, int64_t q_stride, const void* k_cache, const void* v_cache,
                     const int32_t* row_kv_start, const int32_t* row_kv_len, int64_t n, int Hq, int Hkv,
                     int D, float scale, void* out, int dtype, const AttentionShares* shares, hipStream_t st) {
  if (n <= 0) return VLC_OK;
  const int g = Hq / Hkv;
  if (dtype == VLC_BF16) {
    if (D != ATT_D) return fail(VLC_ERR_SHAPE, "attention(bf16): D=%d unsupported (128 only)", D);
    if (g > VR) return fail(VLC_ERR_SHAPE, "attention(bf16): Hq/Hkv=%d exceeds %d", g, VR);
    if (q_stride % 8) return fail(VLC_ERR_SHAPE, "attention(bf16): q row stride must be a multiple of 8");
    // 128 virtual rows per workgroup, two workgroups per CU
    const int rows_per_tile = VR / g;
    const int64_t tiles = (n + rows_per_tile - 1) / rows_per_tile;
    if (shares && shares->max_shares > 1) {
      hipLaunchKernelGGL((attention_bf16_kernel<true>), dim3((unsigned)(shares->slots * Hkv)), dim3(256), 0, st,
                         (const int4*)shares->pieces, row_kv_start, row_kv_len, (const uint16_t*)k_cache, (const uint16_t*)v_cache,
                         (int)n, Hkv, g, rows_per_tile, (const uint16_t*)q, q_stride, Hq, scale * 1.4426950408889634f,
                         (uint16_t*)out, shares->part_o, shares->part_ml);
      VLC_CHECK_LAUNCH("attention_bf16(split)");
      const int64_t threads = n * Hq * (ATT_D / 8);
      hipLaunchKernelGGL(attention_merge_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, shares->part_o,
                         shares->part_ml, (const int32_t*)shares->tile_shares, row_kv_len, n * Hq, rows_per_tile, Hq, (uint16_t*)out);
      VLC_CHECK_LAUNCH("attention_merge");
      return VLC_OK;
    }
    const dim3 grid((unsigned)att_grid((int)tiles, Hkv));
    hipLaunchKernelGGL((attention_bf16_kernel<false>), grid, dim3(256), 0, st, nullptr, row_kv_start, row_kv_len,
                       (const uint16_t*)k_cache, (const uint16_t*)v_cache, (int)n, Hkv, g, rows_per_tile, (const uint16_t*)q,
                       q_stride, Hq, scale * 1.4426950408889634f, (uint16_t*)out, nullptr, nullptr);
    VLC_CHECK_LAUNCH("attention_bf16");
    return VLC_OK;
  }
  if (dtype == VLC_F32) {
    if (n >= (int64_t)1 << 26 || Hq > 65535) return fail(VLC_ERR_SHAPE, "attention(f32): grid too large");
    if (D != 64 && D != 128) return fail(VLC_ERR_SHAPE, "attention(f32): D=%d unsupported", D);
    const int64_t pairs = n * g, tiles = (pairs + 15) / 16;   // of one kv head
    // at most 2^32 - 1 threads along a grid dimension
    const int64_t slices = (tiles + (1 << 22) - 1) >> 22;
    // workgroups per tile: those past the first, which come last in the grid, are for tiles of many requests only and bring the chip to
    // 2048 wavefronts
    const int f32_shares = tiles * Hkv <= 128 ? 4 : (tiles * Hkv <= 256 ? 2 : 1);
    const dim3 grid((unsigned)((tiles + slices - 1) / slices), (unsigned)Hkv, (unsigned)(f32_shares > 1 ? f32_shares : slices));
#define VLC_LAUNCH_F32_TILE(D_, W_)                                                                                 \
  hipLaunchKernelGGL((attention_f32_tile_kernel<D_, W_>), grid, dim3(64 * W_), 0, st, (const float*)q, row_kv_len,  \
                     row_kv_start, (const float*)k_cache, (const float*)v_cache, pairs, (int)q_stride, Hkv, g, scale, Hq, (float*)out, f32_shares)
#define VLC_LAUNCH_F32_PAIR(D_)                                                                                     \
  hipLaunchKernelGGL((attention_f32_pair_kernel<D_>), dim3((unsigned)n, (unsigned)Hq), dim3(1024), 0, st,           \
                     (const float*)q, row_kv_len, row_kv_start, (const float*)k_cache, (const float*)v_cache, (int)q_stride, \
                     Hkv, g, scale, Hq, (float*)out)
    if (n * Hq < kF32PairsPerTile) {
      if (D == 64) VLC_LAUNCH_F32_PAIR(64);
      else VLC_LAUNCH_F32_PAIR(128);
    } else if (n * Hq < kF32OneWavePairs) {
      if (D == 64) VLC_LAUNCH_F32_TILE(64, 4);
      else VLC_LAUNCH_F32_TILE(128, 4);
    } else {
      if (D == 64) VLC_LAUNCH_F32_TILE(64, 1);
      else VLC_LAUNCH_F32_TILE(128, 1);
    }
#undef VLC_LAUNCH_F32_TILE
#undef VLC_LAUNCH_F32_PAIR
    VLC_CHECK_LAUNCH("attention_f32");
    return VLC_OK;
  }
  return fail(VLC_ERR_DTYPE, "attention: dtype=%d", dtype);
}

}  // namespace vlc

extern "C" int vlc_probe_attention_shares(int64_t n, int Hq, int Hkv, int64_t max_kv_len) {
  if (n <= 0 || Hkv <= 0 || Hq <= 0 || Hq % Hkv || Hq / Hkv > vlc::VR) return 0;
  return vlc::attention_key_shares(n, Hq, Hkv, max_kv_len, vlc::attention_ws_bytes(n, Hq, Hkv, vlc::ATT_D, VLC_BF16));
}

extern "C" int vlc_sparse_q_attention(const void* q, const void* k_cache, const void* v_cache,
                                      const int32_t* row_kv_start, const int32_t* row_kv_len, int64_t n,
                                      int Hq, int Hkv, int D, float scale, void* out, int dtype,
                                      void* stream) {
  using vlc::fail;
  if (dtype != VLC_F32 && dtype != VLC_BF16) return fail(VLC_ERR_DTYPE, "vlc_sparse_q_attention: dtype=%d", dtype);
  if (n < 0 || Hq <= 0 || Hkv <= 0 || Hq % Hkv || (D != 64 && D != 128))
    return fail(VLC_ERR_SHAPE, "vlc_sparse_q_attention: n=%lld Hq=%d Hkv=%d D=%d", (long long)n, Hq, Hkv, D);
  if (n == 0) return VLC_OK;
  if (!q || !k_cache || !v_cache || !row_kv_start || !row_kv_len || !out)
    return fail(VLC_ERR_NULL, "vlc_sparse_q_attention: NULL pointer");
  if (((uintptr_t)q | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)out) & 15)
    return fail(VLC_ERR_SHAPE, "vlc_sparse_q_attention: pointers must be 16-byte aligned");
  return vlc::launch_attention(q, (int64_t)Hq * D, k_cache, v_cache, row_kv_start, row_kv_len, n, Hq, Hkv, D,
                               scale, out, dtype, nullptr, (hipStream_t)stream);
}
