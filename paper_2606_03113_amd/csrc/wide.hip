// Many-row linear kernels of the prefill path (gfx950): y = W x for up to
// thousands of rows, with the fused epilogues of the weight-streaming kernels.
//
// A row's result has the same bits as in a pass of the 16-row kernels
// (linear.hip), whatever the row count: those sum, for wavefront w = 0..7,
// the tiles w, w + 16, ... and w + 8, w + 24, ... of K in two matrix-core
// accumulators, add the two, and add the eight wavefronts' sums in order.
// So a prompt that is prefilled at once, in pieces, or replayed through
// verify passes leaves the same cache.
#include "device.h"
#include "wide.h"

namespace lede {

// ---- y = W x -----------------------------------------------------------------

// What a kernel does with a finished 16 x 16 output tile: lane (lr, lg) holds
// columns 4 lg + i of weight group g and row m.  Called by whole wavefronts.
template <int DT, int EPI>
__device__ __forceinline__ void finish(const WideArgs& a, int g, int m, float (&v)[4]) {
  typedef Tile<DT> TL;
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const bool row = m < a.M;
  const int mr = row ? m : 0;
  if (a.inv) {
    const float s = a.inv[mr];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] *= s;
  }
  if (EPI == EPI_RESID) {
    const int col = g * 16 + 4 * lg;
    float* hp = a.h + (size_t)mr * a.ldh + col;
    float gn[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) gn[i] = a.ss_out ? Elem<DT>::load(a.xg_gain, col + i) : 0.f;
    const float4 h4 = *(const float4*)hp;
    v[0] = h4.x + v[0]; v[1] = h4.y + v[1]; v[2] = h4.z + v[2]; v[3] = h4.w + v[3];
    if (row) *(float4*)hp = make_float4(v[0], v[1], v[2], v[3]);
    if (a.ss_out) {
      if (row)
        store4<DT>((uint8_t*)a.xg + tiled_row_off<DT>(m, col, a.KT_out), 0,
                   make_float4(v[0] * gn[0], v[1] * gn[1], v[2] * gn[2], v[3] * gn[3]));
      // the group's sum of squares in column order: the running sum passes
      // through the four lanes of a row
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q) s = __shfl(s, lr + 16 * (q - 1));
#pragma unroll
        for (int i = 0; i < 4; ++i) s = fmaf(v[i], v[i], s);
      }
      if (row && lg == 3) a.ss_out[(size_t)m * a.n_groups + g] = s;
    }
  } else if (EPI == EPI_SWIGLU) {
    // columns 0..7 are gate, 8..15 up: lanes lg and lg + 2 hold a pair
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float up = __shfl_xor(v[i], 32);
      const float gt = v[i];
      const float s = gt / (1.f + __expf(-gt));
      o[i] = s * up;
    }
    if (row && lg < 2)
      store4<DT>((uint8_t*)a.act + tiled_row_off<DT>(m, 8 * g + 4 * lg, a.KT_out), 0, make_float4(o[0], o[1], o[2], o[3]));
  } else {
    const int hd = a.hd, gph = hd / 16;
    const int qg = a.nq * gph, kg = a.nkv * gph;
    const int pos = *a.seq_len + a.pos_off + mr;
    if (g < qg + kg) {
      const bool isq = g < qg;
      const int gl = isq ? g : g - qg;
      const int head = gl / gph, i0 = 8 * (gl % gph) + 4 * (lg & 1);
      const float2* rp = a.rope + (size_t)pos * (hd / 2) + i0;
      float y[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 cs = rp[i];
        const float other = __shfl_xor(v[i], 32);
        const float x0 = lg < 2 ? v[i] : other, x1 = lg < 2 ? other : v[i];
        const float2 yy = rope_pair(x0, x1, cs);
        y[i] = lg < 2 ? yy.x : yy.y;
      }
      const int dim = i0 + (lg < 2 ? 0 : hd / 2);
      if (row) {
        if (isq) {
          *(float4*)(a.q + (size_t)m * a.ldq + head * hd + dim) = make_float4(y[0], y[1], y[2], y[3]);
        } else {
          const size_t base =
              ((((size_t)a.layer * a.n_pages + a.block_table[pos >> 6]) * a.nkv + head) * 64 + (pos & 63)) * hd + dim;
          store4<DT>((uint8_t*)a.kcache + base * TL::ES, 0, make_float4(y[0], y[1], y[2], y[3]));
        }
      }
    } else if (row) {
      const int dim = (g - qg - kg) * 16 + 4 * lg;
      const size_t base =
          ((((size_t)a.layer * a.n_pages + a.block_table[pos >> 6]) * a.nkv + dim / hd) * 64 + (pos & 63)) * hd + dim % hd;
      store4<DT>((uint8_t*)a.vcache + base * TL::ES, 0, make_float4(v[0], v[1], v[2], v[3]));
    }
  }
}

// The output tile of a block, from its place in the grid: blocks b, b + 8, ...
// run on one XCD, which takes every eighth column of tiles, in squares of sup_m
// row tiles, so that the tiles in flight on an XCD share their operands in its
// L2.  False past the end.
__device__ __forceinline__ bool block_tile(const WideArgs& a, int& nt, int& mt) {
  const int b = blockIdx.x, xcd = b & 7, j = b >> 3;
  const int per = a.sup_m * ((a.n_tiles + 7) / 8);  // tiles of one band of row tiles on one XCD
  const int band = j / per, jj = j - band * per;
  const int rows_here = min(a.sup_m, a.m_tiles - band * a.sup_m);
  mt = band * a.sup_m + jj % rows_here;
  nt = (jj / rows_here) * 8 + xcd;
  return nt < a.n_tiles && mt < a.m_tiles;
}

// One block computes TN x TM tiles of 16 x 16 outputs.  Wavefront w takes the
// K tiles w, w + 8, ... of every output tile, as the order above asks for, so
// the eight wavefronts share no operand and stream both from the L2 straight
// into registers, D steps ahead; the eight partial sums meet in LDS once at
// the end, and each wavefront finishes some of the tiles.
template <int DT, int TN, int TM, int D, int EPI>
__global__ __launch_bounds__(512) void k_wide(WideArgs a) {
  typedef Tile<DT> TL;
  constexpr int NW = LIN_WAVES;
  static_assert(D % 2 == 0, "even steps go to the first accumulator");
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  int nt, mt;
  if (!block_tile(a, nt, mt)) return;
  const int g0 = nt * TN, r0 = mt * TM;  // weight group, row group
  const int MG = (a.M + 15) >> 4;

  const int KT = a.KT;
  const uint8_t* wp[TN];
  const uint8_t* xp[TM];
#pragma unroll
  for (int i = 0; i < TN; ++i) wp[i] = a.w + (size_t)min(g0 + i, a.n_groups - 1) * KT * TILE_BYTES;
#pragma unroll
  for (int i = 0; i < TM; ++i) xp[i] = a.x + (size_t)min(r0 + i, MG - 1) * KT * TILE_BYTES;
  const uint32_t lo = lane * 16;

  f32x4 c0[TN][TM], c1[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int k = 0; k < TM; ++k) c0[i][k] = c1[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};

  uint4 wv[D][TN], xv[D][TM];
  auto load = [&](int u, int t) {  // unconditional: a step past the end re-reads the last tile
    const uint32_t o = (uint32_t)min(t, KT - 1) * TILE_BYTES + lo;
#pragma unroll
    for (int i = 0; i < TN; ++i) wv[u][i] = ld16(wp[i] + o);
#pragma unroll
    for (int i = 0; i < TM; ++i) xv[u][i] = ld16(xp[i] + o);
  };
#pragma unroll
  for (int u = 0; u < D; ++u) load(u, wave + NW * u);
  for (int t = wave; t < KT; t += NW * D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      if (t + NW * u < KT) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int k = 0; k < TM; ++k) {
            f32x4& c = (u & 1) ? c1[i][k] : c0[i][k];
            c = mfma_tile<DT>(wv[u][i], xv[u][k], c);
          }
      }
      load(u, t + NW * (u + D));
    }
  }

  float4* part = (float4*)smem;  // [NW][TN * TM][64]
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int k = 0; k < TM; ++k) {
      const f32x4 c = c0[i][k] + c1[i][k];
      part[(wave * TN * TM + i * TM + k) * 64 + lane] = make_float4(c[0], c[1], c[2], c[3]);
    }
  __syncthreads();

  // output tiles wave, wave + 8, ...: lane holds columns 4 lg + i of row lr
  for (int tt = wave; tt < TN * TM; tt += NW) {
    const int g = g0 + tt / TM, m = (r0 + tt % TM) * 16 + lr;
    if (g >= a.n_groups || (r0 + tt % TM) * 16 >= a.M) continue;  // uniform
    float4 v4 = part[tt * 64 + lane];
    float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
    for (int q = 1; q < NW; ++q) {
      const float4 p = part[(q * TN * TM + tt) * 64 + lane];
      v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
    }
    finish<DT, EPI>(a, g, m, v);
  }
}

// Both operands staged in LDS for WN x WM wavefronts of TN x TM tiles each:
// a block computes (WN TN 16) x (WM TM 16) outputs.  The K tiles are walked in
// the order the sum above asks for: class (w, 0) = tiles w, w + 16, ..., then
// (w, 1) = w + 8, w + 24, ..., w = 0..7; c accumulates a class, c0 keeps the
// even one, s the sum so far.  A stage is one K tile of every row group of the
// block (direct global-to-LDS copies of whole 1 KiB tiles, which are in
// operand order, so the reads have no bank conflicts); S stages are in flight.
template <int N>
__device__ __forceinline__ void stage_barrier() {  // this wavefront's copies but the last N, and its LDS reads; then all
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int DT, int TN, int TM, int WN, int WM, int S, int EPI>
__global__ __launch_bounds__(WN * WM * 64, 2) void k_wide_lds(WideArgs a) {
  constexpr int NWV = WN * WM, GN = WN * TN, GM = WM * TM, TILES = GN + GM;
  static_assert(TILES % NWV == 0, "every wavefront copies the same number of tiles");
  constexpr int PER = TILES / NWV;
  extern __shared__ __align__(16) uint8_t smem[];  // [S][TILES][1 KiB]
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int nt, mt;
  if (!block_tile(a, nt, mt)) return;
  const int g0 = nt * GN, r0 = mt * GM, MG = (a.M + 15) >> 4, KT = a.KT;
  const uint8_t* src[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = wave * PER + i;
    src[i] = (u < GN ? a.w + (size_t)min(g0 + u, a.n_groups - 1) * KT * TILE_BYTES
                     : a.x + (size_t)min(r0 + u - GN, MG - 1) * KT * TILE_BYTES) + lane * 16;
  }
  // the K walk: tile t of class base; next() steps it
  auto next = [&](int& t, int& base) {
    t += 16;
    if (t >= KT) {
      do base = base < 8 ? base + 8 : base - 7;
      while (base >= KT && base < 16);
      t = base;
    }
  };
  auto stage = [&](int slot, int t) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(src[i] + (size_t)t * TILE_BYTES),
                                       (__attribute__((address_space(3))) void*)(smem + (slot * TILES + wave * PER + i) * TILE_BYTES),
                                       16, 0, 0);
  };
  int lt = 0, lbase = 0;  // the walk of the copies, S - 1 tiles ahead
  for (int i = 0; i < S - 1; ++i)
    if (i < KT) {
      stage(i, lt);
      next(lt, lbase);
    }
  f32x4 c[TN][TM], c0[TN][TM], s[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int k = 0; k < TM; ++k) c[i][k] = c0[i][k] = s[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int wn = wave % WN, wm = wave / WN;
  const uint32_t la = wn * TN * TILE_BYTES + lane * 16, lb = (GN + wm * TM) * TILE_BYTES + lane * 16;
  int t = 0, base = 0, slot = 0;
  for (int st = 0; st < KT; ++st) {
    if (st + S - 1 <= KT) stage_barrier<(S - 2) * PER>();
    else stage_barrier<0>();
    if (st + S - 1 < KT) {
      stage(slot == 0 ? S - 1 : slot - 1, lt);
      next(lt, lbase);
    }
    const uint32_t o = slot * TILES * TILE_BYTES;
    uint4 wv[TN], xv[TM];
#pragma unroll
    for (int i = 0; i < TN; ++i) wv[i] = lds_ld16(smem + (o + la + i * TILE_BYTES));
#pragma unroll
    for (int i = 0; i < TM; ++i) xv[i] = lds_ld16(smem + (o + lb + i * TILE_BYTES));
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int k = 0; k < TM; ++k) c[i][k] = mfma_tile<DT>(wv[i], xv[k], c[i][k]);
    slot = slot == S - 1 ? 0 : slot + 1;
    if (t + 16 >= KT) {  // the class ends
      const bool odd = base >= 8;
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int k = 0; k < TM; ++k) {
          if (odd || KT - base <= 8) {  // (no tile w + 8 when K is that short)
            s[i][k] += c0[i][k] + c[i][k];
            c0[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
          } else {
            c0[i][k] = c[i][k];
          }
          c[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    next(t, base);
  }
#pragma unroll
  for (int k = 0; k < TM; ++k)
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int g = g0 + wn * TN + i, rg = r0 + wm * TM + k;
      if (g < a.n_groups && rg < MG) {
        float v[4] = {s[i][k][0], s[i][k][1], s[i][k][2], s[i][k][3]};
        finish<DT, EPI>(a, g, rg * 16 + lr, v);
      }
    }
}

// ---- the split norm's inverse RMS, and the head's rows -------------------------

// One half-wavefront per row, in the order of the 16-row kernels: thread j
// sums partials j, j + 32, ..., then the 32 sums are added in order.
__global__ __launch_bounds__(256) void k_row_inv(RowInvArgs a) {
  const int m = blockIdx.x * 8 + (threadIdx.x >> 5), j = threadIdx.x & 31;
  const int mm = min(m, a.M - 1);
  const float* row = a.ss + (size_t)mm * a.groups;
  float v[SS_MAX_GROUPS / 32];
#pragma unroll
  for (int i = 0; i < SS_MAX_GROUPS / 32; ++i) v[i] = j + 32 * i < a.groups ? row[j + 32 * i] : 0.f;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < SS_MAX_GROUPS / 32; ++i) s += v[i];
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i) t += __shfl(s, (threadIdx.x & 32) + i);
  if (j == 0 && m < a.M) a.inv[m] = rsqrtf(t / (float)a.K + a.eps);
}

template <int DT>
__global__ __launch_bounds__(256) void k_head_rows(HeadRowsArgs a) {
  typedef Tile<DT> TL;
  const int r = blockIdx.x;
  uint8_t* out = (uint8_t*)a.xn + (size_t)r * a.d * TL::ES;
  for (int c = threadIdx.x; c < a.d / TL::EPL; c += 256)
    *(uint4*)(out + c * 16) = ld16(a.x + tiled_row_off<DT>(a.r0 + r, c * TL::EPL, a.KT));
  for (int g = threadIdx.x; g < a.groups; g += 256) a.ss_out[(size_t)r * a.groups + g] = a.ss[(size_t)(a.r0 + r) * a.groups + g];
}

// ---- launchers ------------------------------------------------------------------

static hipError_t launch_tiles(const void* f, WideArgs& a, int gn, int gm, int threads, size_t lds, hipStream_t s) {
  a.n_tiles = (a.n_groups + gn - 1) / gn;
  a.m_tiles = ((a.M + 15) / 16 + gm - 1) / gm;
  a.sup_m = a.m_tiles < 8 ? a.m_tiles : 8;
  const int bands = (a.m_tiles + a.sup_m - 1) / a.sup_m;
  const int per = a.sup_m * ((a.n_tiles + 7) / 8);
  const dim3 grid((unsigned)(8 * bands * per));
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  void* args[] = {(void*)&a};
  return hipLaunchKernel(f, grid, dim3(threads), args, lds, s);
}

template <int DT, int TN, int TM, int D>
static hipError_t launch_shape(WideArgs& a, hipStream_t s) {
  const void* f = a.epi == EPI_QKV     ? (const void*)k_wide<DT, TN, TM, D, EPI_QKV>
                  : a.epi == EPI_RESID ? (const void*)k_wide<DT, TN, TM, D, EPI_RESID>
                                       : (const void*)k_wide<DT, TN, TM, D, EPI_SWIGLU>;
  return launch_tiles(f, a, TN, TM, LIN_WAVES * 64, (size_t)LIN_WAVES * TN * TM * 1024, s);
}

template <int DT, int TN, int TM, int WN, int WM, int S>
static hipError_t launch_staged(WideArgs& a, hipStream_t s) {
  const void* f = a.epi == EPI_QKV     ? (const void*)k_wide_lds<DT, TN, TM, WN, WM, S, EPI_QKV>
                  : a.epi == EPI_RESID ? (const void*)k_wide_lds<DT, TN, TM, WN, WM, S, EPI_RESID>
                                       : (const void*)k_wide_lds<DT, TN, TM, WN, WM, S, EPI_SWIGLU>;
  return launch_tiles(f, a, WN * TN, WM * TM, WN * WM * 64, (size_t)S * (WN * TN + WM * TM) * TILE_BYTES, s);
}

// Which kernel: the one with the least estimated time on 256 CUs, from the tile
// area per block and each kernel's rate when every CU is busy, measured on the
// Llama-2-7B layer at 2048 rows: 256 x 128 staged tiles 755 TFLOP/s, 128 x 128
// 640, 128 x 64 (two blocks per CU) 625, and 470 for the 32 x 64 tiles of
// k_wide.  Smaller tiles win where larger ones leave CUs idle: at 512 rows
// 128 x 64 takes 429 us a layer against 544 for 256 x 128 and 526 for 32 x 64,
// at 128 rows 283, 463 and 203.  A lone block of a kernel made for two per CU
// runs at about 0.65 of the CU's rate.
template <int DT>
static hipError_t launch_dt(WideArgs& a, hipStream_t s) {
  struct Shape { int n, m, resident; double rate; };
  static const Shape shapes[4] = {{32, 64, 2, 470.}, {128, 64, 2, 625.}, {128, 128, 1, 640.}, {256, 128, 1, 755.}};
  int best = 0;
  double best_t = 0.;
  for (int i = 0; i < 4; ++i) {
    const Shape& p = shapes[i];
    const int blocks = ((a.n_groups * 16 + p.n - 1) / p.n) * ((a.M + p.m - 1) / p.m), load = (blocks + 255) / 256;
    const double t = load * p.n * p.m / (p.rate * (load < p.resident ? 0.65 : 1.));
    if (i == 0 || t < best_t) {
      best = i;
      best_t = t;
    }
  }
  switch (best) {
    case 0: return launch_shape<DT, 2, 4, 2>(a, s);
    case 1: return launch_staged<DT, 4, 2, 2, 2, 5>(a, s);
    case 2: return launch_staged<DT, 4, 2, 2, 4, 6>(a, s);
    default: return launch_staged<DT, 4, 4, 4, 2, 6>(a, s);
  }
}

hipError_t launch_wide(int dtype, WideArgs a, hipStream_t s) { return dtype == 1 ? launch_dt<1>(a, s) : launch_dt<0>(a, s); }

hipError_t launch_row_inv(const RowInvArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_row_inv, dim3((a.M + 7) / 8), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_head_rows(int dtype, const HeadRowsArgs& a, hipStream_t s) {
  if (dtype == 1) hipLaunchKernelGGL(k_head_rows<1>, dim3(a.n), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_head_rows<0>, dim3(a.n), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace lede
