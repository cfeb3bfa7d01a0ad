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

// The operands of a finished 16 x 16 output tile's epilogue, loaded for all of
// a wavefront's tiles before the first is finished: a load behind another
// tile's store would wait for a round trip each.
template <int EPI> struct Extra {  // EPI_RESID: the residual and the next norm's gains
  float4 x, y;                     // EPI_QKV: the rotary pairs
  int page;                        // EPI_QKV: the row's cache page (keys and values)
  float inv;                       // the row's scale
};

// Lane (lr, lg) holds columns 4 lg + i of weight group g and row m.  Tiles past
// the matrix load some in-range operand.
template <int DT, int EPI>
__device__ __forceinline__ void finish_load(const WideArgs& a, int g, int m, Extra<EPI>& e) {
  const int lg = (threadIdx.x & 63) >> 4;
  const int mr = min(m, a.M - 1), gc = min(g, a.n_groups - 1);
  e.inv = a.inv ? a.inv[mr] : 1.f;
  if (EPI == EPI_RESID) {
    const int col = gc * 16 + 4 * lg;
    e.x = *(const float4*)(a.h + (size_t)mr * a.ldh + col);
    e.y = a.ss_out ? row_load4<DT>(nullptr, a.xg_gain, col) : make_float4(0.f, 0.f, 0.f, 0.f);
  } else if (EPI == EPI_QKV) {
    const int gph = a.hd / 16, qg = a.nq * gph, kg = a.nkv * gph;
    const int pos = *a.seq_len + a.pos_off + mr;
    e.page = gc >= qg ? a.block_table[pos >> 6] : 0;
    const int gl = gc < qg ? gc : gc < qg + kg ? gc - qg : 0;
    const float2* rp = a.rope + (size_t)pos * (a.hd / 2) + 8 * (gl % gph) + 4 * (lg & 1);
    e.x = *(const float4*)rp;
    e.y = *(const float4*)(rp + 2);
  }
}

// Called by whole wavefronts.
template <int DT, int EPI>
__device__ __forceinline__ void finish(const WideArgs& a, int g, int m, float (&v)[4], const Extra<EPI>& e) {
  typedef Tile<DT> TL;
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const bool row = m < a.M;
  if (a.inv) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] *= e.inv;
  }
  if (EPI == EPI_RESID) {
    const int col = g * 16 + 4 * lg;
    v[0] = e.x.x + v[0]; v[1] = e.x.y + v[1]; v[2] = e.x.z + v[2]; v[3] = e.x.w + v[3];
    if (row) *(float4*)(a.h + (size_t)m * a.ldh + col) = make_float4(v[0], v[1], v[2], v[3]);
    if (a.ss_out) {
      if (row)
        store4<DT>((uint8_t*)a.xg + tiled_row_off<DT>(m, col, a.KT_out), 0,
                   make_float4(v[0] * e.y.x, v[1] * e.y.y, v[2] * e.y.z, v[3] * e.y.w));
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
    const int pos = *a.seq_len + a.pos_off + m;
    const bool isq = g < qg, rot = g < qg + kg;
    float y[4];
    int head, dim;
    if (rot) {
      const int gl = isq ? g : g - qg;
      const float2 cs[4] = {make_float2(e.x.x, e.x.y), make_float2(e.x.z, e.x.w), make_float2(e.y.x, e.y.y),
                            make_float2(e.y.z, e.y.w)};
      head = gl / gph;
      dim = 8 * (gl % gph) + 4 * (lg & 1) + (lg < 2 ? 0 : hd / 2);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float other = __shfl_xor(v[i], 32);
        const float2 yy = rope_pair(lg < 2 ? v[i] : other, lg < 2 ? other : v[i], cs[i]);
        y[i] = lg < 2 ? yy.x : yy.y;
      }
    } else {
      head = (g - qg - kg) / gph;
      dim = 16 * ((g - qg - kg) % gph) + 4 * lg;
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = v[i];
    }
    if (row) {
      const float4 y4 = make_float4(y[0], y[1], y[2], y[3]);
      if (isq) {
        *(float4*)(a.q + (size_t)m * a.ldq + head * hd + dim) = y4;
      } else {
        const size_t at = ((((size_t)a.layer * a.n_pages + e.page) * a.nkv + head) * 64 + (pos & 63)) * hd + dim;
        store4<DT>((uint8_t*)(rot ? a.kcache : a.vcache) + at * TL::ES, 0, y4);
      }
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

  // the output tiles this wavefront finishes, wave, wave + 8, ...
  constexpr int FT = (TN * TM + NW - 1) / NW;
  Extra<EPI> e[FT];
#pragma unroll
  for (int f = 0; f < FT; ++f) {
    const int tt = min(wave + NW * f, TN * TM - 1);
    finish_load<DT, EPI>(a, g0 + tt / TM, (r0 + tt % TM) * 16 + lr, e[f]);
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

#pragma unroll
  for (int f = 0; f < FT; ++f) {
    const int tt = wave + NW * f, g = g0 + tt / TM, rg = r0 + tt % TM;
    if (tt >= TN * TM || g >= a.n_groups || rg >= MG) continue;  // uniform
    const float4 v4 = part[tt * 64 + lane];
    float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
    for (int q = 1; q < NW; ++q) {
      const float4 p = part[(q * TN * TM + tt) * 64 + lane];
      v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
    }
    finish<DT, EPI>(a, g, rg * 16 + lr, v, e[f]);
  }
}

// Both operands staged in LDS for WN x WM wavefronts of TN x TM tiles each:
// a block computes (WN TN 16) x (WM TM 16) outputs.  The K tiles are walked in
// the order the sum above asks for: class w = tiles w, w + 16, ... into one
// accumulator, class w + 8 into another, their sum onto the total, w = 0..7.
// The ring in LDS holds S K tiles of every row group of the block (direct
// global-to-LDS copies of whole 1 KiB tiles, which are in operand order, so the
// reads have no bank conflicts).  While a K tile is multiplied, the next one's
// operands are read into registers (all of them, or where three sets of
// accumulators leave no room PF of the TN weight tiles) and later ones are
// copied.  With two blocks of 128 x 128 outputs on every CU a K tile of both
// takes 487 ns and a launch 17 us besides (2048 rows, N = 4096: 79, 185 and 235
// us at K = 4096, 11008 and 14336), where the products alone would take 215 at
// the matrix cores' peak; the rest is copies, LDS reads and the barrier per tile.
template <int N>
__device__ __forceinline__ void stage_barrier() {  // this wavefront's copies but the last N, and its LDS reads; then all
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int DT, int TN, int TM, int WN, int WM, int S, int PF, int EPI>
__global__ __launch_bounds__(WN * WM * 64, 2) void k_wide_lds(WideArgs a) {
  constexpr int NWV = WN * WM, GN = WN * TN, GM = WM * TM, TILES = GN + GM;
  constexpr int D = PF == TN ? S : S - 1;  // copies run this many tiles ahead
  // every wavefront copies the same number of tiles (the last ones some twice),
  // so that one count of outstanding copies holds for all
  constexpr int PER = (TILES + NWV - 1) / NWV;
  extern __shared__ __align__(16) uint8_t smem[];  // [S][TILES][1 KiB]
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int nt, mt;
  if (!block_tile(a, nt, mt)) return;
  const int g0 = nt * GN, r0 = mt * GM, MG = (a.M + 15) >> 4, KT = a.KT;
  const uint8_t* src[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = min(wave * PER + i, TILES - 1);
    src[i] = (u < GN ? a.w + (size_t)min(g0 + u, a.n_groups - 1) * KT * TILE_BYTES
                     : a.x + (size_t)min(r0 + u - GN, MG - 1) * KT * TILE_BYTES) + lane * 16;
  }
  auto stage = [&](int slot, int t) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(src[i] + (size_t)t * TILE_BYTES),
                                       (__attribute__((address_space(3))) void*)(smem + (slot * TILES + min(wave * PER + i, TILES - 1)) * TILE_BYTES),
                                       16, 0, 0);
  };
  KWalk cw;  // the walk of the copies, D tiles ahead
  for (int i = 0; i < D; ++i)
    if (i < KT) {
      stage(i, cw.t);
      cw.next(KT);
    }
  const int wn = wave % WN, wm = wave / WN;
  const uint32_t la = wn * TN * TILE_BYTES + lane * 16, lb = (GN + wm * TM) * TILE_BYTES + lane * 16;
  // the operands of the next K tile (of the weights, PF tiles), and the rest
  uint4 wnext[PF], xnext[TM];
  auto read = [&](int slot) {
    const uint32_t o = slot * TILES * TILE_BYTES;
#pragma unroll
    for (int i = 0; i < PF; ++i) wnext[i] = lds_ld16(smem + (o + la + i * TILE_BYTES));
#pragma unroll
    for (int i = 0; i < TM; ++i) xnext[i] = lds_ld16(smem + (o + lb + i * TILE_BYTES));
  };
  int st = 0, slot = 0;
  // one K tile, whose operands have been read: a later tile's copy is started
  // and the next one's operands are read before the products
  auto step = [&](f32x4 (&c)[TN][TM], bool first) {
    if (st + D <= KT) stage_barrier<(D - 2) * PER>();
    else stage_barrier<0>();
    uint4 wv[TN], xv[TM];
#pragma unroll
    for (int i = 0; i < TN; ++i) wv[i] = i < PF ? wnext[i < PF ? i : 0] : lds_ld16(smem + (slot * TILES * TILE_BYTES + la + i * TILE_BYTES));
#pragma unroll
    for (int i = 0; i < TM; ++i) xv[i] = xnext[i];
    if (st + D < KT) {
      stage(PF == TN ? slot : slot == 0 ? S - 1 : slot - 1, cw.t);
      cw.next(KT);
    }
    slot = slot == S - 1 ? 0 : slot + 1;
    read(slot);
    ++st;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
#pragma unroll
      for (int k = 0; k < TM; ++k) c[i][k] = mfma_tile<DT>(wv[i], xv[k], first ? f32x4{0.f, 0.f, 0.f, 0.f} : c[i][k]);
      if (i == PF - 1) __builtin_amdgcn_sched_barrier(0);  // the products whose operands are here come first
    }
  };
  auto sum_class = [&](f32x4 (&c)[TN][TM], int base) {
    if (base < KT) {
      step(c, true);
      for (int t = base + 16; t < KT; t += 16) step(c, false);
    } else {
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int k = 0; k < TM; ++k) c[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  if (KT >= D) stage_barrier<(D - 1) * PER>();
  else stage_barrier<0>();
  read(0);
  f32x4 s[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int k = 0; k < TM; ++k) s[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int w = 0; w < LIN_WAVES; ++w) {
    f32x4 c0[TN][TM], c1[TN][TM];
    sum_class(c0, w);
    sum_class(c1, w + LIN_WAVES);
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int k = 0; k < TM; ++k) s[i][k] += c0[i][k] + c1[i][k];
  }
  Extra<EPI> e[TN][TM];
#pragma unroll
  for (int k = 0; k < TM; ++k)
#pragma unroll
    for (int i = 0; i < TN; ++i) finish_load<DT, EPI>(a, g0 + wn * TN + i, (r0 + wm * TM + k) * 16 + lr, e[i][k]);
#pragma unroll
  for (int k = 0; k < TM; ++k)
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int g = g0 + wn * TN + i, rg = r0 + wm * TM + k;
      if (g < a.n_groups && rg < MG) {
        float v[4] = {s[i][k][0], s[i][k][1], s[i][k][2], s[i][k][3]};
        finish<DT, EPI>(a, g, rg * 16 + lr, v, e[i][k]);
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

template <int DT, int TN, int TM, int WN, int WM, int S, int PF>
static hipError_t launch_staged(WideArgs& a, hipStream_t s) {
  const void* f = a.epi == EPI_QKV     ? (const void*)k_wide_lds<DT, TN, TM, WN, WM, S, PF, EPI_QKV>
                  : a.epi == EPI_RESID ? (const void*)k_wide_lds<DT, TN, TM, WN, WM, S, PF, EPI_RESID>
                                       : (const void*)k_wide_lds<DT, TN, TM, WN, WM, S, PF, EPI_SWIGLU>;
  return launch_tiles(f, a, WN * TN, WM * TM, WN * WM * 64, (size_t)S * (WN * TN + WM * TM) * TILE_BYTES, s);
}

template <int DT>
static hipError_t launch_dt(WideArgs& a, hipStream_t s) {
  const int shape = wide_shape(DT, a.n_groups, a.M);
  if (shape == 0) return launch_shape<DT, 2, 4, 2>(a, s);
  if (shape == 1) return launch_staged<DT, 4, 2, 2, 2, 5, 4>(a, s);
  if (DT == 1) {
    if (shape == 2) return launch_staged<1, 2, 2, 2, 2, 8, 2>(a, s);
    if (shape == 3) return launch_staged<1, 3, 4, 2, 2, 5, 3>(a, s);
  }
  return launch_staged<1, 4, 4, 2, 2, 5, 1>(a, s);
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
