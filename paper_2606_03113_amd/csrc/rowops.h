// Block-level row reductions over a vocabulary-sized fp32 row (gfx950):
// statistics, fixed-order sums and inverse-CDF draws, used by the sampling
// and exit-policy kernels.
#pragma once

#include "device.h"

namespace lede {

// One block of SB threads per row.  Thread t owns the contiguous chunk
// [t C, (t+1) C) of the vocabulary (C = ceil(V / SB) rounded up to 4) and sums
// it in index order; the chunk sums are combined by one block scan in thread
// order.  Every sum therefore runs in one fixed order, and a row's statistics
// and draw depend on nothing but its inputs.  A wavefront reads its 64 chunks
// in batches of CB elements of each, four lanes to a chunk's 64 bytes, and
// passes them through LDS to the owning lanes: lanes that read their own
// chunks touch a cache line per lane and instruction, and what the L1 cannot
// hold of 16 wavefronts' lines is fetched again.  A draw from a row of 32000
// tokens takes 13.3 us, against 18.5 with own reads and a second pass for the
// sum.

constexpr int SB = 1024, SW = SB / 64, CB = 16;
constexpr int ROW_PITCH = CB + 4;                            // words between a batch's chunks in LDS
// Dynamic LDS of a kernel that reads rows: half of the batches at a time, so that
// a launch keeps to 64 KiB (asking for more takes the host 1 us a launch).
constexpr int ROW_LDS = SB / 2 * ROW_PITCH * (int)sizeof(float);
static_assert(ROW_LDS <= 48 * 1024, "and the kernels' own arrays, up to 13 KB");

__device__ __forceinline__ int chunk_len(int V) { return ((V + SB - 1) / SB + 3) / 4 * 4; }

// Elements [j0, j0 + CB) of this thread's chunk of row z into r, zero past the
// chunk's or the row's end; j0 is a multiple of CB.  Whole wavefronts call it.
__device__ __forceinline__ void load_chunks(const float* z, int V, int C, int j0, float (&r)[CB]) {
  extern __shared__ __align__(16) float row_lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* tb = row_lds + wave * 32 * ROW_PITCH;
  const bool vec = ((uintptr_t)z & 15) == 0;
  const int part = j0 + 4 * (lane & 3);
  float4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = 16 * i + (lane >> 2), e = (wave * 64 + c) * C + part;
    v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (part < C) {  // (C is a multiple of 4: a part is whole)
      if (vec && e + 4 <= V) {
        v[i] = *(const float4*)(z + e);
      } else {
        if (e < V) v[i].x = z[e];
        if (e + 1 < V) v[i].y = z[e + 1];
        if (e + 2 < V) v[i].z = z[e + 2];
        if (e + 3 < V) v[i].w = z[e + 3];
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // the first 32 lanes' chunks, then the others'
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i) *(float4*)&tb[(16 * i + (lane >> 2)) * ROW_PITCH + 4 * (lane & 3)] = v[2 * h + i];
    __builtin_amdgcn_wave_barrier();
    if (lane >> 5 == h)
#pragma unroll
      for (int i = 0; i < 4; ++i) *(float4*)&r[4 * i] = *(const float4*)&tb[(lane & 31) * ROW_PITCH + 4 * i];
    __builtin_amdgcn_wave_barrier();
  }
}
// Elements of the batch at j0 that belong to this thread's chunk and the row.
__device__ __forceinline__ int chunk_count(int V, int C, int j0) {
  return min(CB, min(C - j0, V - ((int)threadIdx.x * C + j0)));
}

// Elements [b, b + CB) of row z (zero from `end` on) into r, by one lane alone;
// b is a multiple of 4, so a 16-byte aligned row takes vector loads.
__device__ __forceinline__ void load_batch(const float* z, int end, int b, float (&r)[CB]) {
  if (((uintptr_t)z & 15) == 0 && b + CB <= end) {
#pragma unroll
    for (int j = 0; j < CB; j += 4) *(float4*)&r[j] = *(const float4*)(z + b + j);
  } else {
#pragma unroll
    for (int j = 0; j < CB; ++j) r[j] = b + j < end ? z[b + j] : 0.f;
  }
}

__device__ __forceinline__ float block_max_f(float v, float* red) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float m = red[0];
  for (int w = 1; w < SW; ++w) m = fmaxf(m, red[w]);
  return m;
}

__device__ __forceinline__ int block_max_i(int v, int* red) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  int m = red[0];
  for (int w = 1; w < SW; ++w) m = max(m, red[w]);
  return m;
}

// Exclusive prefix of v over the threads in index order, and the total.
__device__ __forceinline__ float block_excl_scan(float v, float* red, float& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const float y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  float ex = __shfl_up(x, 1);
  if (lane == 0) ex = 0.f;
  __syncthreads();
  if (lane == 63) red[wave] = x;
  __syncthreads();
  float base = 0.f;
  for (int w = 0; w < wave; ++w) base += red[w];
  total = base;
  for (int w = wave; w < SW; ++w) total += red[w];
  return base + ex;
}

// Sum of f(z1[v], z2[v]) over this thread's chunk, in index order.
template <typename F>
__device__ float chunk_sum(F f, const float* z1, const float* z2, int V) {
  const int C = chunk_len(V);
  float s = 0.f;
  for (int j0 = 0; j0 < C; j0 += CB) {
    float r1[CB], r2[CB];
    load_chunks(z1, V, C, j0, r1);
    if (z2) load_chunks(z2, V, C, j0, r2);
    const int n = chunk_count(V, C, j0);
#pragma unroll
    for (int j = 0; j < CB; ++j)
      if (j < n) s += f(r1[j], z2 ? r2[j] : 0.f);
  }
  return s;
}

// Inverse-CDF draw from the non-negative weights f(z1[v], z2[v]), of which this
// thread's chunk sums to s: the first index whose running sum exceeds
// u * total, else (rounding) the last index of positive weight in the owning
// chunk.  Returns -1 when every weight is 0; total receives the sum.
template <typename F>
__device__ int draw_chunk(F f, float s, const float* z1, const float* z2, int V, float u, float& total, float* red,
                          int* ired) {
  const float pre = block_excl_scan(s, red, total);
  const float thr = u * total;
  const int owner = block_max_i((s > 0.f && pre <= thr) ? (int)threadIdx.x : -1, ired);
  __shared__ int tok;
  if ((int)threadIdx.x == owner) {
    const int C = chunk_len(V), v0 = owner * C, v1 = min(V, v0 + C);
    float acc = pre;
    int hit = -1, last = -1;
    for (int b = v0; b < v1 && hit < 0; b += CB) {
      float r1[CB], r2[CB];
      load_batch(z1, v1, b, r1);
      if (z2) load_batch(z2, v1, b, r2);
      float w[CB];
#pragma unroll
      for (int j = 0; j < CB; ++j) w[j] = f(r1[j], z2 ? r2[j] : 0.f);
#pragma unroll
      for (int j = 0; j < CB; ++j)
        if (b + j < v1 && hit < 0) {
          if (w[j] > 0.f) last = b + j;
          acc += w[j];
          if (acc > thr) hit = b + j;
        }
    }
    tok = hit >= 0 ? hit : last;
  }
  if (threadIdx.x == 0 && owner < 0) tok = -1;
  __syncthreads();
  return tok;
}
// The same from the weights of chunks of at most 2 CB tokens, held by their
// threads.
__device__ inline int draw_held(const float (&w)[2][CB], float s, int V, float u, float& total, float* red, int* ired) {
  const float pre = block_excl_scan(s, red, total);
  const float thr = u * total;
  const int owner = block_max_i((s > 0.f && pre <= thr) ? (int)threadIdx.x : -1, ired);
  __shared__ int tok;
  if ((int)threadIdx.x == owner) {
    const int C = chunk_len(V), v0 = owner * C, n = min(C, V - v0);
    float acc = pre;
    int hit = -1, last = -1;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < CB; ++j)
        if (q * CB + j < n && hit < 0) {
          if (w[q][j] > 0.f) last = v0 + q * CB + j;
          acc += w[q][j];
          if (acc > thr) hit = v0 + q * CB + j;
        }
    tok = hit >= 0 ? hit : last;
  }
  if (threadIdx.x == 0 && owner < 0) tok = -1;
  __syncthreads();
  return tok;
}

template <typename F>
__device__ int block_draw(F f, const float* z1, const float* z2, int V, float u, float* red, int* ired) {
  float total;
  return draw_chunk(f, chunk_sum(f, z1, z2, V), z1, z2, V, u, total, red, ired);
}

// The row's maximum, and this thread's chunk sum of exp((z - max) * inv_t).
// Rows of up to 2 CB SB tokens (chunks of at most 2 CB) are read once, and r
// then holds the weights; rows of up to CB SB take one batch (a draw from 1000
// tokens 38.4 us with its read-back, 3 us more with the exponentials of an empty
// second batch).
__device__ inline float row_max_sum(const float* z, int V, float inv_t, float& s, float (&r)[2][CB], float* red) {
  const int C = chunk_len(V);
  float m = -INFINITY;
  s = 0.f;
  if (C <= 2 * CB) {
    const int n[2] = {chunk_count(V, C, 0), chunk_count(V, C, CB)};
    const int batches = C > CB ? 2 : 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == batches) break;
      load_chunks(z, V, C, q * CB, r[q]);
#pragma unroll
      for (int j = 0; j < CB; ++j)
        if (j < n[q]) m = fmaxf(m, r[q][j]);
    }
    m = block_max_f(m, red);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == batches) break;
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        r[q][j] = expf((r[q][j] - m) * inv_t);
        if (j < n[q]) s += r[q][j];
      }
    }
  } else {
    for (int j0 = 0; j0 < C; j0 += CB) {
      float r[CB];
      load_chunks(z, V, C, j0, r);
      const int n = chunk_count(V, C, j0);
#pragma unroll
      for (int j = 0; j < CB; ++j)
        if (j < n) m = fmaxf(m, r[j]);
    }
    m = block_max_f(m, red);
    s = chunk_sum([&](float x, float) { return expf((x - m) * inv_t); }, z, nullptr, V);
  }
  return m;
}

// (max, sum of exp((z - max) * inv_t)) of one row.
__device__ inline float2 row_stats(const float* z, int V, float inv_t, float* red) {
  float s, total, r[2][CB];
  const float m = row_max_sum(z, V, inv_t, s, r, red);
  (void)block_excl_scan(s, red, total);
  __syncthreads();
  return make_float2(m, total);
}

// ---- the same from per-group statistics --------------------------------------
// A row of V = 16 G tokens summarised by its groups' (max m_g, sum of
// exp((z - m_g) * inv_t)): thread t owns the contiguous groups
// [t D, (t+1) D) (D = ceil(G / SB)), and every sum runs in group order within
// a thread and in thread order across the block.

__device__ __forceinline__ int group_chunk(int G) { return (G + SB - 1) / SB; }

// Weight of group g relative to the row maximum mx: sum over its tokens of
// exp((z - mx) * inv_t).
__device__ __forceinline__ float group_weight(float2 st, float mx, float inv_t) {
  return st.x > -INFINITY ? st.y * expf((st.x - mx) * inv_t) : 0.f;
}

// A thread's groups of a row: in registers for rows of up to GH SB groups
// (131072 tokens), so that they are read once; past the end (-inf, 0), weight 0.
constexpr int GH = 8;
struct GroupChunk {
  const float2* gs;
  int g0, g1;
  float2 h[GH];
  __device__ __forceinline__ GroupChunk(const float2* gs_, int G) : gs(gs_) {
    const int D = group_chunk(G);
    g0 = threadIdx.x * D;
    g1 = min(G, g0 + D);
#pragma unroll
    for (int j = 0; j < GH; ++j) h[j] = gs[min(g0 + j, G - 1)];
#pragma unroll
    for (int j = 0; j < GH; ++j)
      if (g0 + j >= g1) h[j] = make_float2(-INFINITY, 0.f);
  }
  __device__ __forceinline__ float max() const {
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < GH; ++j) m = fmaxf(m, h[j].x);
    for (int g = g0 + GH; g < g1; ++g) m = fmaxf(m, gs[g].x);
    return m;
  }
  // the sum of the groups' weights, in group order
  __device__ __forceinline__ float sum(float mx, float inv_t) const {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < GH; ++j) s += group_weight(h[j], mx, inv_t);
    for (int g = g0 + GH; g < g1; ++g) s += group_weight(gs[g], mx, inv_t);
    return s;
  }
};

// (max, sum of exp((z - max) * inv_t)) of the row from its group statistics.
__device__ inline float2 group_row_stats(const float2* gs, int G, float inv_t, float* red) {
  const GroupChunk ch(gs, G);
  const float m = block_max_f(ch.max(), red);
  float total;
  (void)block_excl_scan(ch.sum(m, inv_t), red, total);
  __syncthreads();
  return make_float2(m, total);
}

// Inverse-CDF draw at temperature 1 / inv_t from the row z with group
// statistics gs and row maximum mx, of which this thread's groups weigh s: the
// group whose running weight crosses u * total, then the token within it whose
// running weight does (else, by rounding, the group's last token of positive
// weight).  -1 when the total weight is 0; total receives it.
__device__ inline int draw_group(const GroupChunk& ch, float s, const float* z, float mx, float inv_t, float u,
                                 float& total, float* red, int* ired) {
  const float pre = block_excl_scan(s, red, total);
  const float thr = u * total;
  const int owner = block_max_i((s > 0.f && pre <= thr) ? (int)threadIdx.x : -1, ired);
  __shared__ int tok;
  if ((int)threadIdx.x == owner) {
    float acc = pre;  // running weight before group g
    int gsel = -1, glast = -1;
    for (int g = ch.g0; g < ch.g1; ++g) {
      const float w = group_weight(ch.gs[g], mx, inv_t);
      if (w > 0.f) glast = g;
      if (w > 0.f && acc + w > thr) {
        gsel = g;
        break;
      }
      acc += w;
    }
    const int gg = gsel >= 0 ? gsel : glast;  // glast: rounding left the crossing past the chunk
    int hit = -1, last = -1;
    float w[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) w[j] = expf((z[gg * 16 + j] - mx) * inv_t);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (w[j] > 0.f) last = gg * 16 + j;
      acc += w[j];
      if (gsel >= 0 && hit < 0 && acc > thr) hit = gg * 16 + j;
    }
    tok = hit >= 0 ? hit : last;
  }
  if (threadIdx.x == 0 && owner < 0) tok = -1;
  __syncthreads();
  return tok;
}
__device__ inline int group_draw(const float2* gs, const float* z, int G, float mx, float inv_t, float u, float* red,
                                 int* ired) {
  const GroupChunk ch(gs, G);
  float total;
  return draw_group(ch, ch.sum(mx, inv_t), z, mx, inv_t, u, total, red, ired);
}

}  // namespace lede
