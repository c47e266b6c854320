// Mixture-of-experts MLP (the Qwen3-VL-30B-A3B-shaped layer of the paper's evaluation, Sec. 5.1):
// expert choice per recomputed row, grouping of the (row, expert) pairs by expert for the grouped
// GEMMs, and the weighted sum of the experts' outputs with the residual.
//
//   route   : per row, the top_k largest router scores (equal scores: lower expert index first),
//             weights exp(z_k - z_max) / sum over the chosen ones (the softmax denominator over
//             all experts cancels in the renormalised weights)
//   plan    : exclusive scan of the expert counts -> first pair of every expert, and the table of
//             row tiles (expert, first row, end row) the grouped GEMMs walk; pair position = first pair of its
//             expert + its rank there, and the inverse list position -> row (the order inside an expert
//             does not change any result: every pair is computed on its own)
//   combine : h_out[row] = h1[row] + sum_k w[row, k] * y[position(row, k)]   (float sum, one rounding)
#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>

#include "vlc_internal.h"

namespace vlc {
namespace {

constexpr int kMaxExperts = 256;   // four scores per lane
constexpr int kMaxTopK = 16;
constexpr int kMaxSplits = 8;      // the GEMM never splits the k range into more parts
// Up to here one workgroup groups the pairs, beyond it up to 64 that first count their slices.  Choice and grouping, 8 of 128
// experts per row, one / many workgroups: 4096 pairs 10.4 / 11.2 us, 6144 11.5 / 11.4, 8000 12.6 / 11.7, 16384 18.5 / 12.5,
// 56832 48.6 / 17.7, 528000 451 / 74.
constexpr int64_t kSmallPlanPairs = 6144;
constexpr int kPlanSlices = 64;

// A score and its expert as one number: larger score first, then lower index (scores are no NaNs; -0 counts as 0).
__device__ __forceinline__ uint64_t choice_key(float v, int e) {
  const uint32_t b = __float_as_uint(v + 0.0f);
  return ((uint64_t)(b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u)) << 32) | (uint32_t)(0x7fffffff - e);
}
__device__ __forceinline__ float choice_score(uint64_t k) {
  const uint32_t b = (uint32_t)(k >> 32);
  return __uint_as_float(b ^ ((b >> 31) ? 0x80000000u : 0xffffffffu));
}
__device__ __forceinline__ int choice_expert(uint64_t k) { return 0x7fffffff - (int)(uint32_t)k; }

template <int CTRL>
__device__ __forceinline__ uint64_t max_dpp(uint64_t k) {   // with the lane that the DPP control names (all are in range)
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)k, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(k >> 32), CTRL, 0xf, 0xf, true);
  const uint64_t o = ((uint64_t)hi << 32) | lo;
  return o > k ? o : k;
}
// largest key of the wavefront, in every lane: pairs, fours, eights and sixteens by DPP, then between the 16-lane rows by
// register swaps - no LDS round trips, of which a choice of 8 experts by shuffles has 48 in a row (10 -> 5 us at 97 rows)
__device__ __forceinline__ uint64_t wave_max(uint64_t k) {
  k = max_dpp<0xb1>(k);     // quad_perm [1,0,3,2]
  k = max_dpp<0x4e>(k);     // quad_perm [2,3,0,1]
  k = max_dpp<0x141>(k);    // row_half_mirror
  k = max_dpp<0x140>(k);    // row_mirror
  {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)k, (uint32_t)k, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
    const uint64_t a = ((uint64_t)hi[0] << 32) | lo[0], b = ((uint64_t)hi[1] << 32) | lo[1];
    k = a > b ? a : b;
  }
  {
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)k, (uint32_t)k, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
    const uint64_t a = ((uint64_t)hi[0] << 32) | lo[0], b = ((uint64_t)hi[1] << 32) | lo[1];
    k = a > b ? a : b;
  }
  return k;
}

// one wavefront per row
// logits: `splits` float partial matrices [n, E] (split_stride floats apart) whose sum are the scores
// (1: the scores themselves).
__global__ __launch_bounds__(256) void moe_route_kernel(const float* __restrict__ logits, int64_t split_stride,
                                                        int64_t n, int splits, int E, int K, int32_t* __restrict__ idx,
                                                        float* __restrict__ wts, float* __restrict__ sum_out) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  // all loads first (independent: one memory latency instead of one per partial matrix)
  float part[kMaxSplits][4];
#pragma unroll
  for (int s = 0; s < kMaxSplits; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      part[s][j] = 0.f;
      if (s < splits && lane + 64 * j < E) part[s][j] = logits[s * split_stride + row * E + lane + 64 * j];
    }
  uint64_t key[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = lane + 64 * j;
    float z = -INFINITY;
    if (e < E) {
      z = part[0][j];
#pragma unroll
      for (int s = 1; s < kMaxSplits; ++s)
        if (s < splits) z += part[s][j];                 // in split order
      if (sum_out) sum_out[row * E + e] = z;             // the scores the choice is taken from, for inspection
    }
    if (e < E && !(z >= -FLT_MAX)) z = -FLT_MAX;        // NaN or -inf scores rank last but stay selectable
    key[j] = e < E ? choice_key(z, e) : 0;              // 0: below every score
  }
  float my_v = 0.f, top_v = 0.f;
  int my_e = 0;
  for (int k = 0; k < K; ++k) {
    uint64_t best = key[0];
#pragma unroll
    for (int j = 1; j < 4; ++j) best = key[j] > best ? key[j] : best;
    best = wave_max(best);
    if (k == 0) top_v = choice_score(best);
    if (lane == k) {
      my_v = choice_score(best);
      my_e = choice_expert(best);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (key[j] == best) key[j] = 0;                    // taken
  }
  float ex = lane < K ? expf(my_v - top_v) : 0.f;
  float sum = ex;
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o);   // K <= 16: lanes 0..15
  if (lane < K) {
    const int e = my_e < E ? my_e : E - 1;
    idx[row * K + lane] = e;
    wts[row * K + lane] = ex / sum;
  }
}

// Pairs of slice [begin, end) per expert, by LDS atomics; eight experts per thread fetched together, so that the loads of
// a workgroup that walks many pairs overlap.  All 1024 threads call it with cnt[256] in LDS.
__device__ __forceinline__ void count_pairs(const int32_t* __restrict__ idx, int64_t begin, int64_t end, int* cnt) {
  const int t = threadIdx.x;
  if (t < 256) cnt[t] = 0;
  __syncthreads();
  for (int64_t i0 = begin + t; i0 < end; i0 += 8 * 1024) {
    int e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) e[u] = i0 + u * 1024 < end ? idx[i0 + u * 1024] : -1;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (e[u] >= 0) atomicAdd(&cnt[e[u]], 1);
  }
  __syncthreads();
}

// Thread t < 256 brings its expert's number of pairs c, of which `before` belong to earlier slices: cur[t] = position of the
// slice's first pair of that expert; the writer also leaves offsets and tile table.  All 1024 threads.
__device__ __forceinline__ void plan_experts(int c, int before, int E, int tile_rows, bool writer, int* sc, int* stl, int* cur,
                                             int32_t* __restrict__ offset, GroupTile* __restrict__ tiles,
                                             int32_t* __restrict__ n_tiles) {
  const int t = threadIdx.x;
  const int nt = (c + tile_rows - 1) / tile_rows;
  if (t < 256) {
    sc[t] = c;
    stl[t] = nt;
  }
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {      // inclusive scans over the 256 expert slots
    int a = 0, b = 0;
    if (t < 256 && t >= o) {
      a = sc[t - o];
      b = stl[t - o];
    }
    __syncthreads();
    if (t < 256) {
      sc[t] += a;
      stl[t] += b;
    }
    __syncthreads();
  }
  if (t < 256) {
    const int off = sc[t] - c, toff = stl[t] - nt;
    cur[t] = off + before;
    if (writer && t < E) {
      offset[t] = off;
      for (int k = 0; k < nt; ++k) {
        GroupTile g;
        g.expert = t;
        g.m0 = off + k * tile_rows;
        g.m_end = off + c;
        g.pad = 0;
        tiles[toff + k] = g;
      }
    }
    if (writer && t == 255) {
      offset[E] = sc[255];
      *n_tiles = stl[255];
    }
  }
  __syncthreads();
}

// Positions of the pairs of slice [begin, end) and the rows at these positions.
__device__ __forceinline__ void place_pairs(const int32_t* __restrict__ idx, int64_t begin, int64_t end, int K, int* cur,
                                            int32_t* __restrict__ pair_row, int32_t* __restrict__ pair_pos) {
  for (int64_t i0 = begin + threadIdx.x; i0 < end; i0 += 8 * 1024) {
    int e[8], pos[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) e[u] = i0 + u * 1024 < end ? idx[i0 + u * 1024] : -1;
#pragma unroll
    for (int u = 0; u < 8; ++u) pos[u] = e[u] >= 0 ? atomicAdd(&cur[e[u]], 1) : 0;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (e[u] >= 0) {
        const uint32_t i = (uint32_t)(i0 + u * 1024);
        pair_pos[i] = pos[u];
        pair_row[pos[u]] = (int32_t)(i / (uint32_t)K);
      }
  }
}

// Few pairs: counting, scan, tile table, positions and the inverse list in ONE workgroup.
__global__ __launch_bounds__(1024) void moe_plan_small_kernel(const int32_t* __restrict__ idx, int64_t pairs, int K,
                                                              int E, int tile_rows, int32_t* __restrict__ offset,
                                                              GroupTile* __restrict__ tiles,
                                                              int32_t* __restrict__ n_tiles,
                                                              int32_t* __restrict__ pair_row,
                                                              int32_t* __restrict__ pair_pos) {
  __shared__ int cnt[256], sc[256], stl[256], cur[256];
  count_pairs(idx, 0, pairs, cnt);
  plan_experts(threadIdx.x < 256 ? cnt[threadIdx.x] : 0, 0, E, tile_rows, true, sc, stl, cur, offset, tiles, n_tiles);
  place_pairs(idx, 0, pairs, K, cur, pair_row, pair_pos);
}

// Many pairs: one workgroup walking all of them is bound by its own LDS atomics (56832 pairs 39 us).  Every workgroup
// takes a slice: the first kernel leaves the slices' counts [slices][E], in the second every workgroup sums them up, scans,
// and places its slice behind the earlier ones.
__global__ __launch_bounds__(1024) void moe_count_kernel(const int32_t* __restrict__ idx, int64_t pairs, int64_t slice, int E,
                                                         int32_t* __restrict__ counts) {
  __shared__ int cnt[256];
  const int64_t begin = blockIdx.x * slice;
  count_pairs(idx, begin, min(pairs, begin + slice), cnt);
  if ((int)threadIdx.x < E) counts[(int64_t)blockIdx.x * E + threadIdx.x] = cnt[threadIdx.x];
}
__global__ __launch_bounds__(1024) void moe_place_kernel(const int32_t* __restrict__ idx, int64_t pairs, int64_t slice, int K,
                                                         int E, int tile_rows, const int32_t* __restrict__ counts,
                                                         int32_t* __restrict__ offset, GroupTile* __restrict__ tiles,
                                                         int32_t* __restrict__ n_tiles, int32_t* __restrict__ pair_row,
                                                         int32_t* __restrict__ pair_pos) {
  __shared__ int sc[256], stl[256], cur[256], part[2][4][256];
  const int t = threadIdx.x, e = t & 255, q = t >> 8;
  int all = 0, before = 0;                 // every fourth slice of expert e
  if (e < E) {
#pragma unroll
    for (int g = 0; g < kPlanSlices / 4; ++g) {
      const int s = 4 * g + q;
      const int v = s < (int)gridDim.x ? counts[(int64_t)s * E + e] : 0;
      all += v;
      before += s < (int)blockIdx.x ? v : 0;
    }
  }
  part[0][q][e] = all;
  part[1][q][e] = before;
  __syncthreads();
  if (t < 256) {
    all = part[0][0][t] + part[0][1][t] + part[0][2][t] + part[0][3][t];
    before = part[1][0][t] + part[1][1][t] + part[1][2][t] + part[1][3][t];
  }
  plan_experts(all, before, E, tile_rows, blockIdx.x == 0, sc, stl, cur, offset, tiles, n_tiles);
  const int64_t begin = blockIdx.x * slice;
  place_pairs(idx, begin, min(pairs, begin + slice), K, cur, pair_row, pair_pos);
}

__device__ __forceinline__ float ld_elem(const float* p) { return *p; }
__device__ __forceinline__ float ld_elem(const uint16_t* p) { return __uint_as_float(((uint32_t)*p) << 16); }
__device__ __forceinline__ void st_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_elem(uint16_t* p, float v) {
  uint32_t u = __float_as_uint(v);
  u += 0x7fffu + ((u >> 16) & 1u);
  *p = (uint16_t)(u >> 16);
}

// one workgroup per row; a thread owns 16-byte chunks of the row
template <typename T>
__global__ __launch_bounds__(256) void moe_combine_kernel(const T* __restrict__ h1, const T* __restrict__ y,
                                                          const float* __restrict__ wts,
                                                          const int32_t* __restrict__ pair_pos, int K, int H,
                                                          T* __restrict__ out) {
  constexpr int VEC = 16 / sizeof(T);
  const int64_t row = blockIdx.x;
  __shared__ float w[kMaxTopK];
  __shared__ int pos[kMaxTopK];
  if (threadIdx.x < K) {
    w[threadIdx.x] = wts[row * K + threadIdx.x];
    pos[threadIdx.x] = pair_pos[row * K + threadIdx.x];
  }
  __syncthreads();
  for (int c = threadIdx.x * VEC; c < H; c += 256 * VEC) {
    float acc[VEC];
    uint4 raw = *reinterpret_cast<const uint4*>(h1 + row * H + c);
    const T* hp = reinterpret_cast<const T*>(&raw);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    for (int k = 0; k < K; ++k) {
      const uint4 yr = *reinterpret_cast<const uint4*>(y + (int64_t)pos[k] * H + c);
      const T* yp = reinterpret_cast<const T*>(&yr);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = fmaf(w[k], ld_elem(yp + i), acc[i]);
    }
    uint4 o;
    T* op = reinterpret_cast<T*>(&o);
#pragma unroll
    for (int i = 0; i < VEC; ++i) st_elem(op + i, ld_elem(hp + i) + acc[i]);
    *reinterpret_cast<uint4*>(out + row * H + c) = o;
  }
}

// moe_combine_kernel followed by the RMSNorm of the row it has just written (the input norm of the layer below,
// weight nw): thread t owns chunks t, t + 256, ... as the stand-alone norm kernel does, and the sums are taken
// in the same order on the stored (rounded) values, so both routes give the same bits.  The normed row goes to
// yn[ymap ? ymap[row] : row]; a negative entry: no norm for this row.
template <typename T, int MAXC>
__global__ __launch_bounds__(256) void moe_combine_norm_kernel(const T* __restrict__ h1, const T* __restrict__ y,
                                                               const float* __restrict__ wts,
                                                               const int32_t* __restrict__ pair_pos,
                                                               const int32_t* __restrict__ ymap, const T* __restrict__ nw,
                                                               int K, int H, T* __restrict__ out, T* __restrict__ yn,
                                                               float inv_h, float eps) {
  constexpr int VEC = 16 / sizeof(T);
  const int64_t row = blockIdx.x;
  __shared__ float w[kMaxTopK];
  __shared__ int pos[kMaxTopK];
  __shared__ float red[4];
  if (threadIdx.x < K) {
    w[threadIdx.x] = wts[row * K + threadIdx.x];
    pos[threadIdx.x] = pair_pos[row * K + threadIdx.x];
  }
  __syncthreads();
  float v[MAXC][VEC];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < MAXC; ++j) {
    const int c = (threadIdx.x + j * 256) * VEC;
    if (c < H) {
      float acc[VEC];
      uint4 raw = *reinterpret_cast<const uint4*>(h1 + row * H + c);
      const T* hp = reinterpret_cast<const T*>(&raw);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
      for (int k = 0; k < K; ++k) {
        const uint4 yr = *reinterpret_cast<const uint4*>(y + (int64_t)pos[k] * H + c);
        const T* yp = reinterpret_cast<const T*>(&yr);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(w[k], ld_elem(yp + i), acc[i]);
      }
      uint4 o;
      T* op = reinterpret_cast<T*>(&o);
#pragma unroll
      for (int i = 0; i < VEC; ++i) st_elem(op + i, ld_elem(hp + i) + acc[i]);
      *reinterpret_cast<uint4*>(out + row * H + c) = o;
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        v[j][i] = ld_elem(op + i);
        ss += v[j][i] * v[j][i];
      }
    }
  }
  const int64_t yrow = ymap ? (int64_t)ymap[row] : row;
  if (yrow < 0) return;                    // the same for the whole workgroup
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) tot += red[i];
  const float r = 1.0f / sqrtf(tot * inv_h + eps);
#pragma unroll
  for (int j = 0; j < MAXC; ++j) {
    const int c = (threadIdx.x + j * 256) * VEC;
    if (c < H) {
      const uint4 wr = *reinterpret_cast<const uint4*>(nw + c);
      const T* wp = reinterpret_cast<const T*>(&wr);
      uint4 o;
      T* op = reinterpret_cast<T*>(&o);
#pragma unroll
      for (int i = 0; i < VEC; ++i) st_elem(op + i, v[j][i] * r * ld_elem(wp + i));
      *reinterpret_cast<uint4*>(yn + yrow * H + c) = o;
    }
  }
}

}  // namespace

int launch_moe_route(const float* logits, int splits, int64_t split_stride, float* sum_out, int64_t n,
                     int n_experts, int top_k, int tile_rows, const MoeScratch& s, hipStream_t st) {
  if (n <= 0) return VLC_OK;
  if (splits < 1 || splits > kMaxSplits) return fail(VLC_ERR_SHAPE, "moe: splits=%d", splits);
  if (n_experts < 1 || n_experts > kMaxExperts || top_k < 1 || top_k > kMaxTopK || top_k > n_experts)
    return fail(VLC_ERR_SHAPE, "moe: n_experts=%d (<= %d), top_k=%d (<= %d, <= n_experts)", n_experts, kMaxExperts,
                top_k, kMaxTopK);
  if (n * top_k > INT32_MAX) return fail(VLC_ERR_SHAPE, "moe: too many (row, expert) pairs");
  const int64_t pairs = n * top_k;
  hipLaunchKernelGGL(moe_route_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, logits, split_stride, n, splits,
                     n_experts, top_k, s.idx, s.wts, sum_out);
  VLC_CHECK_LAUNCH("moe_route");
  if (pairs <= kSmallPlanPairs) {
    hipLaunchKernelGGL(moe_plan_small_kernel, dim3(1), dim3(1024), 0, st, (const int32_t*)s.idx, pairs, top_k,
                       n_experts, tile_rows, s.offset, s.tiles, s.n_tiles, s.pair_row, s.pair_pos);
    VLC_CHECK_LAUNCH("moe_plan_small");
    return VLC_OK;
  }
  // at least 1024 pairs per slice: the slices' counts (at most 256 experts) fit the `pairs` integers of s.counts
  const int64_t want = pairs / 1024 < kPlanSlices ? pairs / 1024 : kPlanSlices;
  const int64_t slice = (pairs + want - 1) / want;
  const unsigned slices = (unsigned)((pairs + slice - 1) / slice);
  hipLaunchKernelGGL(moe_count_kernel, dim3(slices), dim3(1024), 0, st, (const int32_t*)s.idx, pairs, slice, n_experts,
                     s.counts);
  VLC_CHECK_LAUNCH("moe_count");
  hipLaunchKernelGGL(moe_place_kernel, dim3(slices), dim3(1024), 0, st, (const int32_t*)s.idx, pairs, slice, top_k,
                     n_experts, tile_rows, (const int32_t*)s.counts, s.offset, s.tiles, s.n_tiles, s.pair_row, s.pair_pos);
  VLC_CHECK_LAUNCH("moe_place");
  return VLC_OK;
}

int launch_moe_combine(const void* h1, const void* y, const float* wts, const int32_t* pair_pos, int64_t n,
                       int top_k, int H, void* out, int dtype, hipStream_t st) {
  if (n <= 0) return VLC_OK;
  if (top_k < 1 || top_k > kMaxTopK) return fail(VLC_ERR_SHAPE, "moe combine: top_k=%d", top_k);
  if (dtype == VLC_BF16) {
    if (H % 8) return fail(VLC_ERR_SHAPE, "moe combine: H=%d must be a multiple of 8", H);
    hipLaunchKernelGGL(moe_combine_kernel<uint16_t>, dim3((unsigned)n), dim3(256), 0, st, (const uint16_t*)h1,
                       (const uint16_t*)y, wts, pair_pos, top_k, H, (uint16_t*)out);
  } else if (dtype == VLC_F32) {
    if (H % 4) return fail(VLC_ERR_SHAPE, "moe combine: H=%d must be a multiple of 4", H);
    hipLaunchKernelGGL(moe_combine_kernel<float>, dim3((unsigned)n), dim3(256), 0, st, (const float*)h1,
                       (const float*)y, wts, pair_pos, top_k, H, (float*)out);
  } else {
    return fail(VLC_ERR_DTYPE, "moe combine: dtype=%d", dtype);
  }
  VLC_CHECK_LAUNCH("moe_combine");
  return VLC_OK;
}

int launch_moe_combine_norm(const void* h1, const void* y, const float* wts, const int32_t* pair_pos, int64_t n,
                            int top_k, int H, void* out, const void* norm_w, void* normed, const int32_t* ymap,
                            float eps, int dtype, hipStream_t st) {
  if (n <= 0) return VLC_OK;
  if (top_k < 1 || top_k > kMaxTopK) return fail(VLC_ERR_SHAPE, "moe combine: top_k=%d", top_k);
  if (dtype != VLC_BF16 && dtype != VLC_F32) return fail(VLC_ERR_DTYPE, "moe combine: dtype=%d", dtype);
  const int vec = dtype == VLC_BF16 ? 8 : 4;
  if (H % vec) return fail(VLC_ERR_SHAPE, "moe combine: H=%d must be a multiple of %d", H, vec);
  const int chunks = H / vec;
  const float inv_h = 1.0f / (float)H;
#define VLC_LAUNCH_MCN(T, MAXC)                                                                              \
  hipLaunchKernelGGL((moe_combine_norm_kernel<T, MAXC>), dim3((unsigned)n), dim3(256), 0, st, (const T*)h1,  \
                     (const T*)y, wts, pair_pos, ymap, (const T*)norm_w, top_k, H, (T*)out, (T*)normed, inv_h, eps)
  if (chunks <= 256 * 2) {
    if (dtype == VLC_BF16) VLC_LAUNCH_MCN(uint16_t, 2); else VLC_LAUNCH_MCN(float, 2);
  } else if (chunks <= 256 * 8) {
    if (dtype == VLC_BF16) VLC_LAUNCH_MCN(uint16_t, 8); else VLC_LAUNCH_MCN(float, 8);
  } else {   // very wide rows: the two kernels one after the other
    const int rc = launch_moe_combine(h1, y, wts, pair_pos, n, top_k, H, out, dtype, st);
    return rc ? rc : launch_rmsnorm(out, nullptr, norm_w, normed, n, H, eps, dtype, st, ymap);
  }
#undef VLC_LAUNCH_MCN
  VLC_CHECK_LAUNCH("moe_combine_norm");
  return VLC_OK;
}

}  // namespace vlc
