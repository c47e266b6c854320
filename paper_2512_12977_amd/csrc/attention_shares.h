// Key shares of the bf16 attention: which keys of which row tile each of its workgroups takes.
#ifndef VLC_ATTENTION_SHARES_H_
#define VLC_ATTENTION_SHARES_H_

#include "vlc_internal.h"

namespace vlc {

constexpr int ATT_KB = 64;              // keys per block
constexpr int ATT_MAX_TILES = 512;      // row tiles of a launch with shares (fewer than 512 pairs)
constexpr int ATT_MAX_SHARES = 8;
constexpr int ATT_MIN_BLOCKS = 4;       // shorter shares cost more in partials and merging than they save

// largest value / sum over the wavefront, in every lane: within rows of 16 lanes by DPP, between them by register swaps
template <int CTRL>
__device__ __forceinline__ int max_dpp(int v) {
  return max(v, __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ int wave_max(int v) {
  v = max_dpp<0xb1>(v);     // quad_perm [1,0,3,2]
  v = max_dpp<0x4e>(v);     // quad_perm [2,3,0,1]
  v = max_dpp<0x141>(v);    // row_half_mirror
  v = max_dpp<0x140>(v);    // row_mirror
  const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = max((int)a[0], (int)a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return max((int)b[0], (int)b[1]);
}
template <int CTRL>
__device__ __forceinline__ int sum_dpp(int v) {
  return v + __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ int wave_sum(int v) {
  v = sum_dpp<0xb1>(v);
  v = sum_dpp<0x4e>(v);
  v = sum_dpp<0x141>(v);
  v = sum_dpp<0x140>(v);
  const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = (int)a[0] + (int)a[1];
  const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return (int)b[0] + (int)b[1];
}

__device__ __forceinline__ int ceil_div(int a, int b, float inv_b) {   // a below 2^25; inv_b = 1 / b
  int q = (int)((float)a * inv_b);
  q += q * b < a;
  q += q * b < a;
  q -= (q - 1) * b >= a;
  return q;
}

// Used when there are too few (row tile, kv head) pairs to occupy the chip and the key loop is the critical path.  Every kv
// head has `slots` workgroups.  A row tile that sees b key blocks is shared out over ceil(b / len) of them, in pieces of
// about equal length; len is the smallest share length with which the pieces of all tiles fit the slots - one round of
// workgroups, whatever the rows' layout.  They work about equally long where a tile's rows belong to one request; a tile that
// straddles r requests is planned by its longest row but walks its pieces once for each of them, so that with packed short
// questions the longest workgroups take up to r times what the plan gives them.  (Pieces of a common length cut from the whole
// batch's key range, as before, are many or few by the layout and take up to a second round.)  Attention per layer, before /
// after: 8 images and a text at the end (72B shape, 296 pairs) 206 / 167 us, four images between texts (7B, 212 pairs)
// 63 / 55, three images (8B, 112 pairs) 39 / 32, a question (7B, 24 pairs) 14.2 / 13.
// Found by one workgroup of 256 threads of the kernel in front of the attention (RoPE + scatter, at most 1 us longer for
// it); by every workgroup of the attention for itself it cost 4 us of a launch of 15.
// The code is kept short (loops, one place each): it runs cold, on one CU.
__device__ inline void plan_attention_shares(const AttentionShares& a) {
  __shared__ int blocks[ATT_MAX_TILES], count[ATT_MAX_TILES + 1];
  const int tid = threadIdx.x, lane = tid & 63;
#pragma unroll 1
  for (int t = tid; t < a.tiles; t += 256) blocks[t] = 0;
  __syncthreads();
#pragma unroll 1
  for (int i = tid; i < a.n; i += 256)
    atomicMax(&blocks[(uint32_t)i / (uint32_t)a.rows_per_tile], (a.row_kv_len[i] + ATT_KB - 1) / ATT_KB);
  __syncthreads();
  int sum = 0, most = 0;
#pragma unroll 1
  for (int t = lane; t < a.tiles; t += 64) {
    sum += blocks[t];
    most = max(most, blocks[t]);
  }
  sum = __builtin_amdgcn_readfirstlane(wave_sum(sum));
  most = __builtin_amdgcn_readfirstlane(wave_max(most));
  int lo = max(ATT_MIN_BLOCKS, max((most + a.max_shares - 1) / a.max_shares, (sum + a.slots - 1) / a.slots));
  int hi = max(lo, most), len = lo;            // tiles <= slots: one piece per tile always fits
#pragma unroll 1
  while (lo < hi) {                            // the smallest length first, then by halves
    const float inv = 1.0f / (float)len;
    int c = 0;
#pragma unroll 1
    for (int t = lane; t < a.tiles; t += 64) c += ceil_div(blocks[t], len, inv);
    if (__builtin_amdgcn_readfirstlane(wave_sum(c)) <= a.slots) hi = len;
    else lo = len + 1;
    len = (lo + hi) / 2;
  }
  const float inv = 1.0f / (float)hi;
#pragma unroll 1
  for (int t = tid; t < a.tiles; t += 256) count[t] = ceil_div(blocks[t], hi, inv);
  __syncthreads();
#pragma unroll 1
  for (int t = tid; t < a.tiles; t += 256) {
    int at = 0;                                // pieces of the tiles before this one
#pragma unroll 4
    for (int u = 0; u < t; ++u) at += count[u];
    const int c = count[t], bt = blocks[t];
    a.tile_shares[t] = c;
    const int q = (int)((float)bt * __builtin_amdgcn_rcpf((float)max(c, 1))), r = bt - q * c;   // up to c - 1 or c blocks over
    int first = 0;
#pragma unroll 1
    for (int z = 0; z < c; ++z) {
      const int end = z + 1 < c ? first + q + (z < r ? 1 : 0) : bt;
      a.pieces[at + z] = make_int4(t, z, first, end);
      first = end;
    }
    if (t + 1 == a.tiles) count[ATT_MAX_TILES] = at + c;
  }
  __syncthreads();
#pragma unroll 1
  for (int p = count[ATT_MAX_TILES] + tid; p < a.slots; p += 256) a.pieces[p] = make_int4(-1, 0, 0, 0);
}

}  // namespace vlc
#endif
