// Split-KV attention over the paged KV cache (gfx950).
#include "device.h"
#include "wide.h"

#include <float.h>

#include <type_traits>

namespace lede {

// ---- attention over the paged KV cache --------------------------------------

// Eight consecutive cache elements as fp32.
template <int DT>
__device__ __forceinline__ void load8(const void* base, size_t idx, float* o) {
  if (DT == 1) {
    const uint4 u = ld16((const uint16_t*)base + idx);
    o[0] = bf16lo(u.x); o[1] = bf16hi(u.x); o[2] = bf16lo(u.y); o[3] = bf16hi(u.y);
    o[4] = bf16lo(u.z); o[5] = bf16hi(u.z); o[6] = bf16lo(u.w); o[7] = bf16hi(u.w);
  } else {
    const float4 a = *(const float4*)((const float*)base + idx);
    const float4 b = *(const float4*)((const float*)base + idx + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
}

// One step of the page-ordered combine: fold a page's (max, sum, weighted
// value) into the running (mx, l, acc).
__device__ __forceinline__ void fold_step(float& mx, float& l, float& acc, float pm, float pl, float pa) {
  const float nm = fmaxf(mx, pm);
  const float so = (mx == -INFINITY) ? 0.f : __expf(mx - nm);
  const float sn = __expf(pm - nm);
  l = fmaf(pl, sn, l * so);  // (spelled out: the kernels that fold must round alike)
  acc = fmaf(pa, sn, acc * so);
  mx = nm;
}

// Attention output element (row m, column col of nq * hd).
template <int DT>
__device__ __forceinline__ void store_out(const AttnArgs& a, int m, int col, float v) {
  if (a.KT_tiled) Elem<DT>::store((uint8_t*)a.out + tiled_row_off<DT>(m, col, a.KT_tiled), 0, v);
  else Elem<DT>::store(a.out, (size_t)m * a.ldo + col, v);
}

// Partial attention of up to 16 query rows (row = (m, query head of the
// group)) against whole 64-token pages; pages are strided over the blocks of
// a split.  For every (row, page): running max, sum of exp and the
// exp-weighted value sum, stored for the combine kernel.  A row's partials
// do not depend on which other rows share the block.
// SHORT: one block takes every page and folds the partials itself, in page
// order as the combine kernel does up to 16 pages, and stores the result.
template <int DT, int HD, bool SHORT>
__device__ __forceinline__ void attn_partial(const AttnArgs& a) {
  constexpr int NPC = HD / 32;  // 8-element pieces per thread in the score phase
  constexpr int PV_DG = HD / 8, PV_TG = 256 / PV_DG, TPT = 64 / PV_TG;
  __shared__ float qs[16][HD];
  __shared__ float ss[16][64];
  __shared__ float st_m[16], st_l[16];
  __shared__ float red[4][16][HD];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int G = a.nq / a.nkv;
  const int R = a.M * G;
  const int n_rs = (R + a.rows_per_block - 1) / a.rows_per_block;
  const int kvh = blockIdx.x / n_rs, rs = blockIdx.x % n_rs;
  const int r0 = rs * a.rows_per_block;
  const int nr = min(a.rows_per_block, R - r0);
  const int pos0 = *a.seq_len + a.pos_off;
  const int pmax = pos0 + a.M - 1;
  const int n_chunks = pmax / 64 + 1;
  if ((int)blockIdx.y >= n_chunks) return;
  const float scale = rsqrtf((float)HD);
  // thread roles: scores (token t, part p covering dims p*8 + 32c + e);
  // values (dims dg*8.., tokens tg + PV_TG u)
  const int dg = tid % PV_DG, tg = tid / PV_DG;
  float vf[TPT][8], kf[NPC * 8];
  // Every token slot of an allocated page is readable, so the loads are
  // unconditional and tokens past the length are zeroed afterwards: guarded
  // loads compile to one branch and one wait per load.
  auto load_page = [&](int jj) {
    const int page = a.block_table[jj];
    const size_t base = (((size_t)a.layer * a.n_pages + page) * a.nkv + kvh) * 64 * HD;
    const int nvalid = min(64, pmax - jj * 64 + 1);
#pragma unroll
    for (int u = 0; u < TPT; ++u) load8<DT>(a.vcache, base + (size_t)(tg + PV_TG * u) * HD + dg * 8, vf[u]);
    const int t = tid >> 2, p = tid & 3;
#pragma unroll
    for (int c = 0; c < NPC; ++c) load8<DT>(a.kcache, base + (size_t)t * HD + p * 8 + 32 * c, kf + 8 * c);
#pragma unroll
    for (int u = 0; u < TPT; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) vf[u][e] = tg + PV_TG * u < nvalid ? vf[u][e] : 0.f;
#pragma unroll
    for (int e = 0; e < NPC * 8; ++e) kf[e] = t < nvalid ? kf[e] : 0.f;
  };
  load_page(blockIdx.y);  // the first page's keys and values are in flight with the query loads

  for (int idx = tid; idx < nr * (HD / 4); idx += 256) {
    const int r = idx / (HD / 4), i = 4 * (idx % (HD / 4));
    const int rr = r0 + r, m = rr / G, head = kvh * G + rr % G;
    const float4 v = *(const float4*)(a.q + (size_t)m * a.ldq + head * HD + i);
    qs[r][i] = v.x * scale;
    qs[r][i + 1] = v.y * scale;
    qs[r][i + 2] = v.z * scale;
    qs[r][i + 3] = v.w * scale;
  }
  __syncthreads();

  constexpr int NF = 16 * HD / 256;  // SHORT: elements (row, dim) of a thread
  float fm[NF], fl[NF], fa[NF];
#pragma unroll
  for (int k = 0; k < NF; ++k) fm[k] = -INFINITY, fl[k] = fa[k] = 0.f;
  for (int j = blockIdx.y; j < n_chunks; j += a.n_split) {
    const int tok0 = j * 64;
    {
      const int t = tid >> 2, p = tid & 3;
      for (int r = 0; r < nr; ++r) {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < NPC; ++c)
#pragma unroll
          for (int e = 0; e < 8; ++e) s = fmaf(qs[r][p * 8 + 32 * c + e], kf[8 * c + e], s);
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        const int m = (r0 + r) / G;
        if (p == 0) ss[r][t] = (tok0 + t <= pos0 + m) ? s : -INFINITY;
      }
    }
    __syncthreads();
    for (int r = wave; r < nr; r += 4) {  // softmax statistics, one lane per token
      const float v = ss[r][lane];
      const float mx = wave_max(v);
      const float e = (v == -INFINITY) ? 0.f : __expf(v - mx);
      const float l = wave_sum(e);
      ss[r][lane] = e;
      if (lane == 0) {
        st_m[r] = mx;
        st_l[r] = l;
      }
    }
    __syncthreads();
    {  // exp-weighted values: thread (dim group dg, token group tg)
      for (int r = 0; r < nr; ++r) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
        for (int u = 0; u < TPT; ++u) {
          const float w = ss[r][tg + PV_TG * u];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = fmaf(w, vf[u][e], o[e]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
          for (int off = PV_DG; off < 64; off <<= 1) o[e] += __shfl_xor(o[e], off);
        if (lane < PV_DG) {
#pragma unroll
          for (int e = 0; e < 8; ++e) red[wave][r][dg * 8 + e] = o[e];
        }
      }
    }
    __syncthreads();
    if (j + a.n_split < n_chunks) load_page(j + a.n_split);  // the next page of this block
    if (SHORT) {
#pragma unroll
      for (int k = 0; k < NF; ++k) {
        const int idx = tid + 256 * k, r = idx / HD, i = idx % HD;
        if (r < nr && j <= (pos0 + (r0 + r) / G) / 64)
          fold_step(fm[k], fl[k], fa[k], st_m[r], st_l[r], ((red[0][r][i] + red[1][r][i]) + red[2][r][i]) + red[3][r][i]);
      }
      __syncthreads();
      continue;
    }
    for (int idx = tid; idx < nr * HD; idx += 256) {
      const int r = idx / HD, i = idx % HD;
      const int rr = r0 + r, m = rr / G, head = kvh * G + rr % G;
      float* p = a.part + (((size_t)m * a.nq + head) * a.max_chunks + j) * (HD + 2);
      p[2 + i] = ((red[0][r][i] + red[1][r][i]) + red[2][r][i]) + red[3][r][i];
      if (i == 0) {
        p[0] = st_m[r];
        p[1] = st_l[r];
      }
    }
    __syncthreads();
  }
  if (SHORT) {
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int idx = tid + 256 * k, r = idx / HD, i = idx % HD, rr = r0 + r;
      if (r < nr) store_out<DT>(a, rr / G, (kvh * G + rr % G) * HD + i, fa[k] / fl[k]);
    }
  }
}
template <int DT, int HD>
__global__ __launch_bounds__(256) void k_attn_partial(AttnArgs a) {
  attn_partial<DT, HD, false>(a);
}
template <int DT, int HD>
__global__ __launch_bounds__(256) void k_attn_short(AttnArgs a) {
  attn_partial<DT, HD, true>(a);
}

// Combine the per-page partials of every (row, head): S = blockDim / HD
// groups of HD threads, group s folding pages 16 s .. 16 s + 15 (then
// 16 s + 16 S, ...) in page order, one thread per dim; the groups' running
// states are then folded in group order.  Up to 16 pages only group 0 has
// pages and the result is the plain page-ordered fold.  The loads are
// unconditional (a page index past the buffer is clamped to its last page,
// and pages past the row's position are loaded but not folded), so each
// group's 16 issue together, and before the sequence length arrives.
// GROUPS: the partials are the groups' own, already folded (max_chunks of them).
template <int DT, int HD, bool GROUPS = false>
__global__ __launch_bounds__(HD * COMBINE_GROUPS) void k_attn_combine(AttnArgs a) {
  constexpr int B = 16;
  __shared__ float st[COMBINE_GROUPS][3][HD];
  const int S = blockDim.x / HD;
  const int m = blockIdx.x / a.nq, head = blockIdx.x % a.nq;
  const int i = threadIdx.x % HD, sg = threadIdx.x / HD;
  const float* p = a.part + ((size_t)m * a.nq + head) * a.max_chunks * (HD + 2);
  float pm[B], pl[B], pa[B];
  auto load = [&](int j0) {
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const float* q = p + (size_t)min(j0 + u, a.max_chunks - 1) * (HD + 2);
      pm[u] = q[0];
      pl[u] = q[1];
      pa[u] = q[2 + i];
    }
  };
  if (!GROUPS) load(sg * B);
  const int pos = *a.seq_len + a.pos_off + m;
  const int nc = pos / 64 + 1;
  float mx = -INFINITY, l = 0.f, acc = 0.f;
  if (GROUPS && sg * B < nc) {
    const float* q = p + (size_t)sg * (HD + 2);
    mx = q[0];
    l = q[1];
    acc = q[2 + i];
  }
  for (int j0 = sg * B; !GROUPS && j0 < nc; j0 += S * B) {
    if (j0 > sg * B) load(j0);
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (j0 + u < nc) fold_step(mx, l, acc, pm[u], pl[u], pa[u]);
  }
  st[sg][0][i] = mx;
  st[sg][1][i] = l;
  st[sg][2][i] = acc;
  __syncthreads();
  if (sg == 0) {
    for (int q = 1; q < S && q * B < nc; ++q) fold_step(mx, l, acc, st[q][0][i], st[q][1][i], st[q][2][i]);
    store_out<DT>(a, m, head * HD + i, acc / l);
  }
}

// Eight fp32 values as bf16 high parts and the bf16 rounding of what is left,
// packed as two matrix-core fragments: x ~= hi + lo to about 16 bits.
__device__ __forceinline__ void split8(const float* x, uint4& hi, uint4& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = f32_to_bf16x2(x[2 * i], x[2 * i + 1]);
    l[i] = f32_to_bf16x2(x[2 * i] - bf16lo(h[i]), x[2 * i + 1] - bf16hi(h[i]));
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// Partial attention on the matrix cores (bf16 cache), the same partials as
// k_attn_partial for up to 16 query rows per block: per page, wavefront w
// scores the page's tokens 16w..16w+15 against all rows (S^T = K Q^T as
// 16x16x32 tiles, q split into bf16 high and low parts), the page's per-row
// max and sum combine the four wavefronts in order through LDS, and
// wavefront w forms its HD/4 output dims as V^T P^T (the weights split the
// same way; the wavefront's value columns are staged in LDS and read back
// transposed).  Every output element is a fixed-order function of its own
// row, so a row's partials do not depend on the rows sharing its block.
// SHORT: as in attn_partial.
template <int HD, bool SHORT>
__device__ __forceinline__ void attn_mfma(const AttnArgs& a) {
  constexpr int KS = HD / 32;          // k-steps of the scores
  constexpr int DW = HD / 4;           // output dims per wavefront
  constexpr int DT = DW / 16;          // 16-dim output tiles per wavefront
  constexpr int VS = DW + 4;           // LDS row stride (elements) of the staged values
  __shared__ float smax[4][16], ssum[4][16];
  __shared__ float ps[16][64 + 4];
  __shared__ uint16_t vs[4][64 * VS];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, lr = l & 15, lg = l >> 4;
  const int G = a.nq / a.nkv;
  const int R = a.M * G;
  const int n_rs = (R + a.rows_per_block - 1) / a.rows_per_block;
  const int kvh = blockIdx.x / n_rs, rs = blockIdx.x % n_rs;
  const int r0 = rs * a.rows_per_block;
  const int nr = min(a.rows_per_block, R - r0);
  const int pos0 = *a.seq_len + a.pos_off;
  const int pmax = pos0 + a.M - 1;
  const int n_chunks = pmax / 64 + 1;
  if ((int)blockIdx.y >= n_chunks) return;
  // this lane's query row as a matrix-core operand (rows past nr are zero)
  const bool row_ok = lr < nr;
  const int rr = r0 + lr, m_row = row_ok ? rr / G : 0, head = kvh * G + (row_ok ? rr % G : 0);
  const int row_pos = pos0 + m_row;
  uint4 qh[KS], ql[KS];
  {
    const float scale = rsqrtf((float)HD);
    const float* qp = a.q + (size_t)m_row * a.ldq + head * HD + lg * 8;
    // unconditional loads (a row past nr reads row 0's query, then zeroes it)
    float4 qu[KS], qv[KS];
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
      qu[s2] = *(const float4*)(qp + 32 * s2);
      qv[s2] = *(const float4*)(qp + 32 * s2 + 4);
    }
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
      const float4 u = qu[s2], v = qv[s2];
      float x[8];
      x[0] = row_ok ? u.x * scale : 0.f; x[1] = row_ok ? u.y * scale : 0.f;
      x[2] = row_ok ? u.z * scale : 0.f; x[3] = row_ok ? u.w * scale : 0.f;
      x[4] = row_ok ? v.x * scale : 0.f; x[5] = row_ok ? v.y * scale : 0.f;
      x[6] = row_ok ? v.z * scale : 0.f; x[7] = row_ok ? v.w * scale : 0.f;
      split8(x, qh[s2], ql[s2]);
    }
  }
  const uint16_t* kc = (const uint16_t*)a.kcache;
  const uint16_t* vc = (const uint16_t*)a.vcache;
  float fm[DT][4], fl[DT][4], fa[DT][4];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) fm[dt][i] = -INFINITY, fl[dt][i] = fa[dt][i] = 0.f;
  for (int j = blockIdx.y; j < n_chunks; j += a.n_split) {
    const int page = a.block_table[j];
    const size_t base = (((size_t)a.layer * a.n_pages + page) * a.nkv + kvh) * 64 * HD;
    const int nvalid = min(64, pmax - j * 64 + 1);
    // keys of tokens 16w + lr, dims 32 s + 8 lg; values of this wavefront's dims
    // (unconditional loads within the page, tokens past the length zeroed after)
    uint4 kf[KS];
    const int tk = 16 * w + lr;
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) kf[s2] = ld16(kc + base + (size_t)tk * HD + 32 * s2 + 8 * lg);
    constexpr int VC = 64 * DW / 8 / 64;   // 16-byte value chunks per lane
    uint4 vf[VC];
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      const int idx = l + 64 * c, t = idx / (DW / 8), d8 = idx % (DW / 8);
      vf[c] = ld16(vc + base + (size_t)t * HD + w * DW + 8 * d8);
    }
    // (masks, not selects of whole vectors: those select addresses and
    // put the arrays in scratch)
    const uint32_t km = tk < nvalid ? ~0u : 0u;
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
      kf[s2].x &= km; kf[s2].y &= km; kf[s2].z &= km; kf[s2].w &= km;
    }
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      const uint32_t vm = (l + 64 * c) / (DW / 8) < nvalid ? ~0u : 0u;
      vf[c].x &= vm; vf[c].y &= vm; vf[c].z &= vm; vf[c].w &= vm;
    }
    // S^T tile: lane holds tokens 16w + 4 lg + i of row lr
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
      sc = mfma_tile<1>(kf[s2], qh[s2], sc);
      sc = mfma_tile<1>(kf[s2], ql[s2], sc);
    }
    float sv[4], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = j * 64 + 16 * w + 4 * lg + i;
      sv[i] = (row_ok && t <= row_pos) ? sc[i] : -INFINITY;
      mx = fmaxf(mx, sv[i]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (lg == 0) smax[w][lr] = mx;
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      const int idx = l + 64 * c, t = idx / (DW / 8), d8 = idx % (DW / 8);
      uint16_t* dst = &vs[w][t * VS + 8 * d8];
      *(uint2*)dst = make_uint2(vf[c].x, vf[c].y);
      *(uint2*)(dst + 4) = make_uint2(vf[c].z, vf[c].w);
    }
    __syncthreads();
    const float pm = fmaxf(fmaxf(fmaxf(smax[0][lr], smax[1][lr]), smax[2][lr]), smax[3][lr]);
    float pv[4], sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pv[i] = sv[i] == -INFINITY ? 0.f : __expf(sv[i] - pm);
      sum += pv[i];
    }
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (lg == 0) ssum[w][lr] = sum;
    *(float4*)&ps[lr][16 * w + 4 * lg] = make_float4(pv[0], pv[1], pv[2], pv[3]);
    __syncthreads();
    // this wavefront's dims: D^T = V^T P^T over the page's 64 tokens
    f32x4 oc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      float px[8];
      const float4 u = *(const float4*)&ps[lr][32 * ks + 8 * lg], v = *(const float4*)&ps[lr][32 * ks + 8 * lg + 4];
      px[0] = u.x; px[1] = u.y; px[2] = u.z; px[3] = u.w; px[4] = v.x; px[5] = v.y; px[6] = v.z; px[7] = v.w;
      uint4 ph, pl;
      split8(px, ph, pl);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int d = 16 * dt + lr;
        uint32_t e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = 32 * ks + 8 * lg + 2 * i;
          e[i] = (uint32_t)vs[w][t * VS + d] | ((uint32_t)vs[w][(t + 1) * VS + d] << 16);
        }
        const uint4 vt = make_uint4(e[0], e[1], e[2], e[3]);
        oc[dt] = mfma_tile<1>(vt, ph, oc[dt]);
        oc[dt] = mfma_tile<1>(vt, pl, oc[dt]);
      }
    }
    // partials of row lr: dims w * DW + 16 dt + 4 lg + i
    if (SHORT) {
      const float pl = ((ssum[0][lr] + ssum[1][lr]) + ssum[2][lr]) + ssum[3][lr];
      if (j <= row_pos / 64)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 4; ++i) fold_step(fm[dt][i], fl[dt][i], fa[dt][i], pm, pl, oc[dt][i]);
    } else if (row_ok) {
      float* p = a.part + (((size_t)m_row * a.nq + head) * a.max_chunks + j) * (HD + 2);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int d0 = w * DW + 16 * dt + 4 * lg;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[2 + d0 + i] = oc[dt][i];
      }
      if (w == 0 && lg == 0) {
        p[0] = pm;
        p[1] = ((ssum[0][lr] + ssum[1][lr]) + ssum[2][lr]) + ssum[3][lr];
      }
    }
    __syncthreads();  // the next page rewrites the staging
  }
  if (SHORT && row_ok) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) store_out<1>(a, m_row, head * HD + w * DW + 16 * dt + 4 * lg + i, fa[dt][i] / fl[dt][i]);
  }
}
// Five waves per SIMD (at most 96 VGPRs, no spills) keeps five blocks per
// CU instead of four.
template <int HD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_attn_mfma(AttnArgs a) {
  attn_mfma<HD, false>(a);
}
template <int HD>
__global__ __launch_bounds__(256) void k_attn_mfma_short(AttnArgs a) {
  attn_mfma<HD, true>(a);
}

// The sum (or maximum) of the values of lanes l and l ^ X, X = 16 or 32, as
// vector instructions: a lane swap leaves the value of the lane without bit X
// in r[0] of both and that of the lane with it in r[1].
template <int X, bool MAX>
__device__ __forceinline__ float pair_lanes(float v) {
  const unsigned u = __float_as_uint(v);
  const auto r = X == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
  return MAX ? fmaxf(a, b) : a + b;
}

// Attention of a prefill pass's rows (bf16 cache): 8 wavefronts of 16 query
// rows walk a KV head's pages together, each page staged in LDS once for all
// of them -- keys as matrix-core tiles (direct global-to-LDS copies), values
// transposed -- while the next page is fetched.  A page's scores, maximum, sum
// and weighted values are computed as in k_attn_mfma, and folded at once in
// the order of k_attn_combine: pages in order within the runs of 16 that one
// of its thread groups folds, then the groups in order.  So a row has the bits
// of the two kernels at any row count, without their partials in memory.
// Bound by the chain within a page (products, maximum, exponentials, products:
// about 2.7 us with one or two wavefronts per SIMD, and the same with pages
// fetched two ahead): 2048 rows of the Llama-2-13B shape take 194 us a layer,
// against 2180 for the two kernels 16 rows at a time; 97 rows 13 against 74.
// SPLIT: few rows behind many pages leave CUs idle while the chain runs, so
// their pages go to several blocks and the partials (1: of each page, 2: of
// each group) through memory to k_attn_combine.  A pass of 97 tokens over two
// layers of the Llama-3-8B shape (head included) takes 627 us behind 1024
// positions, 668 unsplit; behind 2048 663 and 750, behind 8000 688 and 1194.
template <int HD, int SPLIT>
__global__ __launch_bounds__(512, 2) void k_attn_wide(AttnArgs a) {
  constexpr int KS = HD / 32, NT = HD / 16;  // k-steps of the scores, output tiles
  constexpr int NW = 8, KT = 4 * KS;         // wavefronts, key tiles of a page
  constexpr int VS = 36;                     // words between the dims of the transposed values (and rows of the weights)
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t* kb = smem;                                          // [2][KT][1 KiB]
  uint32_t* vb = (uint32_t*)(smem + 2 * KT * 1024);            // [2][HD][VS]: token pairs of a dim
  uint32_t* pb = vb + 2 * HD * VS;                             // [NW][2][16][VS]: weights of a row, high and low parts
  const int tid = threadIdx.x, l = tid & 63, lr = l & 15, lg = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.nq / a.nkv, R = a.M * G, n_rb = (R + 16 * NW - 1) / (16 * NW);
  int kvh, rb;
  attn_wide_block(blockIdx.x, a.nkv, n_rb, kvh, rb);
  const int pos0 = *a.seq_len + a.pos_off;
  const int r0 = rb * 16 * NW + 16 * w, rr = min(r0 + lr, R - 1);
  const bool row_ok = r0 + lr < R;
  const int m_row = rr / G, head = kvh * G + rr % G, row_pos = pos0 + m_row;
  const int nc_row = row_pos / 64 + 1;                                                // pages of this lane's row,
  const int last_wave = pos0 + min(r0 + 15, R - 1) / G;                               // (its wavefront's last position)
  const int nc_wave = r0 < R ? last_wave / 64 + 1 : 0;                                // of its wavefront's,
  const int nc_full = (pos0 + min(r0, R - 1) / G + 1) / 64;                            // those its first row sees whole,
  const int nc = (pos0 + min(rb * 16 * NW + 16 * NW - 1, R - 1) / G) / 64 + 1;        // of the block's
  const int S = min(COMBINE_GROUPS, (a.max_chunks + 15) / 16);  // groups of the combine kernel
  const int j_first = SPLIT == 0 ? 0 : blockIdx.y * (SPLIT == 1 ? a.pages_per_block : 16);
  if (SPLIT && j_first >= nc) return;
  uint4 qh[KS], ql[KS];
  {
    const float scale = rsqrtf((float)HD);
    const float* qp = a.q + (size_t)m_row * a.ldq + head * HD + lg * 8;
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
      const float4 u = *(const float4*)(qp + 32 * s2), v = *(const float4*)(qp + 32 * s2 + 4);
      float x[8];
      x[0] = row_ok ? u.x * scale : 0.f; x[1] = row_ok ? u.y * scale : 0.f;
      x[2] = row_ok ? u.z * scale : 0.f; x[3] = row_ok ? u.w * scale : 0.f;
      x[4] = row_ok ? v.x * scale : 0.f; x[5] = row_ok ? v.y * scale : 0.f;
      x[6] = row_ok ? v.z * scale : 0.f; x[7] = row_ok ? v.w * scale : 0.f;
      split8(x, qh[s2], ql[s2]);
    }
  }
  const uint8_t* kc = (const uint8_t*)a.kcache;
  const uint8_t* vc = (const uint8_t*)a.vcache;
  // this thread's values: tokens 2 tp, 2 tp + 1 of dims 8 dg ..
  const int tp = tid & 31, dg = tid >> 5;
  const bool v_on = dg < HD / 8;
  uint4 v0, v1;
  auto fetch = [&](int j, int buf) {
    const size_t base = (((size_t)a.layer * a.n_pages + a.block_table[j]) * a.nkv + kvh) * 64 * HD * 2;
#pragma unroll
    for (int i = 0; i < KT / NW; ++i) {
      const int u = w * (KT / NW) + i, tg = u / KS, s2 = u % KS;
      __builtin_amdgcn_global_load_lds((const void*)(kc + base + ((16 * tg + lr) * HD + 32 * s2 + 8 * lg) * 2),
                                       (__attribute__((address_space(3))) void*)(kb + (buf * KT + u) * 1024), 16, 0, 0);
    }
    const uint8_t* vp = vc + base + (2 * tp * HD + 8 * (v_on ? dg : 0)) * 2;
    v0 = ld16(vp);
    v1 = ld16(vp + HD * 2);
  };
  // the page after j in the combine's order (-1: none): runs of 16 pages,
  // group sg taking runs sg, sg + S, ...
  auto next = [&](int j) {
    if (SPLIT == 1) return j + 1 < min(nc, j_first + a.pages_per_block) ? j + 1 : -1;
    if ((j & 15) != 15 && j + 1 < nc) return j + 1;
    const int run = j >> 4;
    if ((run + S) * 16 < nc) return (run + S) * 16;
    if (SPLIT == 2) return -1;
    const int sg = run % S + 1;
    return sg < S && sg * 16 < nc ? sg * 16 : -1;
  };
  float gm = -INFINITY, gl = 0.f, tm = -INFINITY, tl = 0.f;  // the group's running maximum and sum, and the total's
  f32x4 ga[NT], ta[NT];
#pragma unroll
  for (int d = 0; d < NT; ++d) ga[d] = ta[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t* ph_s = pb + (w * 2) * 16 * VS;
  uint32_t* pl_s = ph_s + 16 * VS;
  float* part = SPLIT ? a.part + ((size_t)m_row * a.nq + head) * a.n_parts * (HD + 2) : nullptr;
  int buf = 0;
  fetch(j_first, 0);
  for (int j = j_first; j >= 0; buf ^= 1) {
    const int nj = next(j);
    if (v_on) {
      const uint32_t e0[4] = {v0.x, v0.y, v0.z, v0.w}, e1[4] = {v1.x, v1.y, v1.z, v1.w};
      uint32_t* dst = vb + (buf * HD + 8 * dg) * VS + tp;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dst[(2 * e) * VS] = __builtin_amdgcn_perm(e1[e], e0[e], 0x05040100u);
        dst[(2 * e + 1) * VS] = __builtin_amdgcn_perm(e1[e], e0[e], 0x07060302u);
      }
    }
    // page j is in LDS, and page j - 1 no longer read
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (nj >= 0) fetch(nj, buf ^ 1);
    if (j < nc_wave) {
      const bool ends = j >= nc_full;  // some row of the wavefront ends in or before this page
      // S^T tiles: lane holds tokens 16 tg + 4 lg + i of row lr
      // (products of different tiles side by side: one tile's are a chain)
      float pv[4][4], mx = -INFINITY;
      f32x4 sc4[4];
#pragma unroll
      for (int tg = 0; tg < 4; ++tg) sc4[tg] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2) {
        uint4 kf[4];
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) kf[tg] = lds_ld16(kb + (buf * KT + tg * KS + s2) * 1024 + l * 16);
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) sc4[tg] = mfma_tile<1>(kf[tg], qh[s2], sc4[tg]);
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) sc4[tg] = mfma_tile<1>(kf[tg], ql[s2], sc4[tg]);
      }
#pragma unroll
      for (int tg = 0; tg < 4; ++tg) {
        const f32x4 sc = sc4[tg];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = j * 64 + 16 * tg + 4 * lg + i;
          pv[tg][i] = sc[i];
          if (ends && t > row_pos) pv[tg][i] = -INFINITY;
          mx = fmaxf(mx, pv[tg][i]);
        }
      }
      mx = pair_lanes<32, true>(pair_lanes<16, true>(mx));
      // a row that ends before this page takes no part in it: weights of 0,
      // folded with factors that leave its state as it is (weights of 0 also
      // where every score overflowed to -infinity)
      const bool in = j < nc_row;
      const float ms = in ? fmaxf(mx, -FLT_MAX) : 0.f;
      float pl = 0.f;
#pragma unroll
      for (int tg = 0; tg < 4; ++tg) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pv[tg][i] = __expf(pv[tg][i] - ms);  // 0 where masked
          sum += pv[tg][i];
        }
        sum = pair_lanes<32, false>(pair_lanes<16, false>(sum));
        pl = tg ? pl + sum : sum;
        // the weights' high and low parts, for the lanes that need them
        // as the operand of the next product
        uint32_t hi[2], lo[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          hi[i] = f32_to_bf16x2(pv[tg][2 * i], pv[tg][2 * i + 1]);
          lo[i] = f32_to_bf16x2(pv[tg][2 * i] - bf16lo(hi[i]), pv[tg][2 * i + 1] - bf16hi(hi[i]));
        }
        *(uint2*)&ph_s[lr * VS + 8 * tg + 2 * lg] = make_uint2(hi[0], hi[1]);
        *(uint2*)&pl_s[lr * VS + 8 * tg + 2 * lg] = make_uint2(lo[0], lo[1]);
      }
      __builtin_amdgcn_wave_barrier();
      uint4 ph[2], po[2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        ph[ks] = *(const uint4*)&ph_s[lr * VS + 16 * ks + 4 * lg];
        po[ks] = *(const uint4*)&pl_s[lr * VS + 16 * ks + 4 * lg];
      }
      __builtin_amdgcn_wave_barrier();
      // fold: the scale of the running state and of this page
      const float nm = in ? fmaxf(gm, mx) : gm;
      const float so = !in ? 1.f : gm == -INFINITY ? 0.f : __expf(gm - nm), sn = in ? __expf(mx - nm) : 0.f;
      gl = fmaf(pl, sn, gl * so);
      gm = nm;
      auto weigh = [&](auto masked) {
        // slots past the wavefront's last position hold no value yet, or
        // another wavefront's, which a weight of 0 would not keep out if it
        // is infinite
        uint32_t vm[2][4];
        if (masked) {
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int t = j * 64 + 32 * ks + 8 * lg + 2 * i;
              vm[ks][i] = t < last_wave ? ~0u : t == last_wave ? 0xFFFFu : 0u;
            }
        }
#pragma unroll
        for (int d0 = 0; d0 < NT; d0 += 4) {
          f32x4 oc[4];
#pragma unroll
          for (int d = 0; d < 4; ++d) oc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            uint4 vt[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              vt[d] = lds_ld16((const uint8_t*)&vb[(buf * HD + 16 * (d0 + d) + lr) * VS + 16 * ks + 4 * lg]);
              if (masked) {
                vt[d].x &= vm[ks][0]; vt[d].y &= vm[ks][1]; vt[d].z &= vm[ks][2]; vt[d].w &= vm[ks][3];
              }
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) oc[d] = mfma_tile<1>(vt[d], ph[ks], oc[d]);
#pragma unroll
            for (int d = 0; d < 4; ++d) oc[d] = mfma_tile<1>(vt[d], po[ks], oc[d]);
          }
          if (SPLIT == 1) {
            if (row_ok && in) {
              float* q = part + (size_t)j * (HD + 2);
              if (d0 == 0 && lg == 0) *(float2*)q = make_float2(mx, pl);
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                float2* qd = (float2*)(q + 2 + 16 * (d0 + d) + 4 * lg);
                qd[0] = make_float2(oc[d][0], oc[d][1]);
                qd[1] = make_float2(oc[d][2], oc[d][3]);
              }
            }
            continue;
          }
#pragma unroll
          for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              // (weights of 0 make an infinite value that other rows see a NaN)
              const float o = masked && !in ? 0.f : oc[d][i];
              ga[d0 + d][i] = fmaf(o, sn, ga[d0 + d][i] * so);
            }
        }
      };
      if (ends) weigh(std::true_type{});
      else weigh(std::false_type{});
    }
    const int sg = (j >> 4) % S;
    if (SPLIT == 0 && (nj < 0 || (nj >> 4) % S != sg)) {  // the group ends: fold it into the total
      const bool in = 16 * sg < nc_row;
      const float nm = fmaxf(tm, gm);
      const float so = tm == -INFINITY ? 0.f : __expf(tm - nm), sn = __expf(gm - nm);
#pragma unroll
      for (int d = 0; d < NT; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float f = fmaf(ga[d][i], sn, ta[d][i] * so);
          ta[d][i] = sg == 0 ? ga[d][i] : in ? f : ta[d][i];
          ga[d][i] = 0.f;
        }
      const float fl = fmaf(gl, sn, tl * so);
      tl = sg == 0 ? gl : in ? fl : tl;
      tm = sg == 0 ? gm : in ? nm : tm;
      gm = -INFINITY;
      gl = 0.f;
    }
    j = nj;
  }
  if (SPLIT == 2 && row_ok && j_first < nc_row) {
    float* q = part + (size_t)blockIdx.y * (HD + 2);
    if (lg == 0) *(float2*)q = make_float2(gm, gl);
#pragma unroll
    for (int d = 0; d < NT; ++d) {
      float2* qd = (float2*)(q + 2 + 16 * d + 4 * lg);
      qd[0] = make_float2(ga[d][0], ga[d][1]);
      qd[1] = make_float2(ga[d][2], ga[d][3]);
    }
  }
  if (SPLIT == 0 && row_ok) {
#pragma unroll
    for (int d = 0; d < NT; ++d)
      store4<1>((uint8_t*)a.out + tiled_row_off<1>(m_row, head * HD + 16 * d + 4 * lg, a.KT_tiled), 0,
                make_float4(ta[d][0] / tl, ta[d][1] / tl, ta[d][2] / tl, ta[d][3] / tl));
  }
}

hipError_t launch_attention_wide(const AttnArgs& a, hipStream_t s) {
  const int rows = a.M * (a.nq / a.nkv), n_rb = (rows + 127) / 128;
  const dim3 grid(a.nkv * n_rb, a.wide_split ? a.n_split : 1);
  const int lds = 2 * (a.hd / 8) * 1024 + (2 * a.hd + 8 * 2 * 16) * 36 * 4;
  static const void* const kernels[2][3] = {
      {(const void*)k_attn_wide<64, 0>, (const void*)k_attn_wide<64, 1>, (const void*)k_attn_wide<64, 2>},
      {(const void*)k_attn_wide<128, 0>, (const void*)k_attn_wide<128, 1>, (const void*)k_attn_wide<128, 2>}};
  const void* f = kernels[a.hd == 128][a.wide_split];
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  void* args[] = {(void*)&a};
  e = hipLaunchKernel(f, grid, dim3(512), args, lds, s);
  if (e != hipSuccess || !a.wide_split) return e;
  // the combine's groups: those that have pages (page j belongs to group
  // j / 16 modulo the groups of max_ctx, so a group without pages may be left out)
  const int S = (a.max_chunks + 15) / 16 < COMBINE_GROUPS ? (a.max_chunks + 15) / 16 : COMBINE_GROUPS;
  AttnArgs b = a;
  b.max_chunks = a.n_parts;
  const int runs = a.wide_split == 1 ? (a.n_parts + 15) / 16 : a.n_parts, groups = runs < S ? runs : S;
  const dim3 cgrid(a.M * a.nq), cblock(a.hd * groups);
  if (a.wide_split == 1) {
    if (a.hd == 128) hipLaunchKernelGGL((k_attn_combine<1, 128>), cgrid, cblock, 0, s, b);
    else hipLaunchKernelGGL((k_attn_combine<1, 64>), cgrid, cblock, 0, s, b);
  } else {
    if (a.hd == 128) hipLaunchKernelGGL((k_attn_combine<1, 128, true>), cgrid, cblock, 0, s, b);
    else hipLaunchKernelGGL((k_attn_combine<1, 64, true>), cgrid, cblock, 0, s, b);
  }
  return hipGetLastError();
}

template <int DT, int HD>
static void launch_attention_t(const AttnArgs& a, hipStream_t s) {
  const int n_rs = (a.M * (a.nq / a.nkv) + a.rows_per_block - 1) / a.rows_per_block;
  const dim3 grid(a.nkv * n_rs, a.n_split);
  if (a.short_ctx) {
    if (DT == 1 && a.mfma) hipLaunchKernelGGL((k_attn_mfma_short<HD>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_attn_short<DT, HD>), grid, dim3(256), 0, s, a);
    return;
  }
  if (DT == 1 && a.mfma) hipLaunchKernelGGL((k_attn_mfma<HD>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_attn_partial<DT, HD>), grid, dim3(256), 0, s, a);
  const int groups = (a.max_chunks + 15) / 16 < COMBINE_GROUPS ? (a.max_chunks + 15) / 16 : COMBINE_GROUPS;
  hipLaunchKernelGGL((k_attn_combine<DT, HD>), dim3(a.M * a.nq), dim3(HD * groups), 0, s, a);
}

hipError_t launch_attention(int dtype, const AttnArgs& a, hipStream_t s) {
  if (dtype == 1) {
    if (a.hd == 128) launch_attention_t<1, 128>(a, s);
    else launch_attention_t<1, 64>(a, s);
  } else {
    if (a.hd == 128) launch_attention_t<0, 128>(a, s);
    else launch_attention_t<0, 64>(a, s);
  }
  return hipGetLastError();
}

}  // namespace lede
