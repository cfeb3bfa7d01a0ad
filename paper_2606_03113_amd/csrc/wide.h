// Interface of the many-row linear kernels (wide.hip): the prefill path for
// more rows than one pass of the weight-streaming kernels takes.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "linear.h"

namespace lede {

// Input rows of the many-row kernels are tiled like the weights: row group
// m / 16, tile k / TK, 1 KiB per tile in matrix-core operand order (lane
// (m & 15) + 16 ((k % TK) / EPL) holds EPL consecutive columns), so that a
// wave load of either operand is one contiguous KiB.  Byte offset of element
// (m, k) with KT tiles per row group:
template <int DT>
__host__ __device__ inline size_t tiled_row_off(int m, int k, int KT) {
  typedef Tile<DT> TL;
  return ((size_t)(m >> 4) * KT + k / TL::TK) * TILE_BYTES + (size_t)((m & 15) + 16 * ((k % TL::TK) / TL::EPL)) * 16 +
         (size_t)(k % TL::EPL) * TL::ES;
}

// The order in which the many-row kernels that stage their operands walk the
// K tiles: class 0, 8, 1, 9, ... 7, 15 (class c: tiles c, c + 16, ...; classes
// past the last tile are empty).  After the last tile t stays past the end:
// the walk stops at class 15, whatever classes are empty.
struct KWalk {
  int t = 0, base = 0;  // the tile, and its class
  __host__ __device__ inline void next(int KT) {
    t += 16;
    while (t >= KT && base != 15) t = base = base < 8 ? base + 8 : base - 7;
  }
};

constexpr int WIDE_ROW_PAD = 128;  // row buffers hold a multiple of this many rows
constexpr int WIDE_ROWS = 2048;    // rows of one prefill pass, at most
// Rows that a context's workspace holds, unless it is a smaller one.
inline int wide_rows(int max_ctx) {
  const int rows = (max_ctx + WIDE_ROW_PAD - 1) / WIDE_ROW_PAD * WIDE_ROW_PAD;
  return rows < WIDE_ROWS ? rows : WIDE_ROWS;
}

struct WideArgs {
  const uint8_t* w;    // tiled weights
  int n_groups;        // 16-row groups of the weights
  int KT, K;           // tiles along K, logical K
  int M;               // rows
  const uint8_t* x;    // tiled rows (KT tiles per row group)
  const float* inv;    // optional: scale of output row m (the split norm)
  int epi;             // EPI_QKV, EPI_RESID or EPI_SWIGLU
  // EPI_RESID
  float* h; int ldh;
  float* ss_out;       // optional, as in LinearArgs, with xg tiled (KT_out tiles per row group)
  const void* xg_gain; void* xg; int KT_out;
  // EPI_QKV
  float* q; int ldq;
  void* kcache; void* vcache;
  int layer, n_pages, nq, nkv, hd;
  const int32_t* block_table; const int32_t* seq_len; int pos_off;
  const float2* rope;
  // EPI_SWIGLU
  void* act;           // tiled, KT_out tiles per row group
  // grid geometry, filled by launch_wide
  int n_tiles, m_tiles, sup_m;
};

// The inverse RMS of M rows from their split-norm partial sums [M][groups].
struct RowInvArgs {
  const float* ss; int groups, M, K;
  float eps;
  float* inv;
};

// Rows r0 .. r0 + n - 1 (r0 a multiple of 16) of tiled rows and their partial
// sums, as the head's row-major input.
struct HeadRowsArgs {
  const uint8_t* x; int KT; int r0, n, d;
  void* xn;            // [n][d]
  const float* ss; float* ss_out; int groups;
};

// Which kernel a launch takes, by the columns and rows of a block's outputs:
// 32 x 64 (k_wide), or 128 x 64, 64 x 64, 96 x 128 or 128 x 128 (k_wide_lds).
// The one with the least estimated time on 256 CUs, from the tile
// area per block and each kernel's rate when every CU is busy (TFLOP/s measured
// at 2048 rows of the Llama-2-13B widths, 512 rows for the smaller tiles; two
// blocks of any of them fit a CU).  A lone block on a CU runs at about 0.65 of
// the CU's rate.  Smaller tiles win where larger ones leave CUs idle: at 512
// rows, N = K = 4096, 64 x 64 tiles take 39 us against 42 for 128 x 64, 51 for
// 96 x 128, 54 for 128 x 128 and 47 for the 32 x 64 tiles of k_wide; at
// N = 22016, 182, 143, 129, 120 and 211; at 97 rows, N = 28672, 77, 64, 78, 60
// and 85.  Over the four launches of a layer at the Llama-2-7B and 13B and
// Llama-3-8B widths with 33 to 2048 rows the choice is the best of the five or
// within 2 % of it in 86 of 120 cases and within 10 % in 104; the worst is
// 768 rows, N = 4096, K = 14336 (188 us, 146 with 128 x 128 tiles).  The fp32
// models are small: they take two of the shapes.
inline int wide_shape(int dtype, int n_groups, int M) {
  struct Shape { int n, m; double rate; };
  static const Shape shapes[5] = {{32, 64, 470.}, {128, 64, 720.}, {64, 64, 560.}, {96, 128, 840.}, {128, 128, 900.}};
  int best = 0;
  double best_t = 0.;
  for (int i = 0; i < (dtype == 1 ? 5 : 2); ++i) {
    const Shape& p = shapes[i];
    const int blocks = ((n_groups * 16 + p.n - 1) / p.n) * ((M + p.m - 1) / p.m), load = (blocks + 255) / 256;
    const double t = load * p.n * p.m / (p.rate * (load < 2 ? 0.65 : 1.));
    if (i == 0 || t < best_t) {
      best = i;
      best_t = t;
    }
  }
  return best;
}

// Prefill attention: the KV head and row block of block b of nkv * n_rb.  Blocks
// b, b + 8, ... run on one XCD.  Of each eight heads one runs on each XCD, whose
// L2 then holds its pages; what is left over eight is dealt to all XCDs in turn,
// so that 1, 2 or 4 heads have 8, 4 or 2 XCDs each.  A head's last rows, which
// see the most pages, come first.  2048 tokens behind 6000 over two layers: 1.38
// ms with one KV head (d_model 2048), 5.37 with one XCD per head; 1.39 and 2.99
// with two; 2.98 and 4.18 with four (d_model 4096); 1.28 both with twelve (1536).
__host__ __device__ inline void attn_wide_block(int b, int nkv, int n_rb, int& kvh, int& rb) {
  const int full = nkv & ~7, rem = nkv - full;
  if (b < full * n_rb) {
    kvh = (b >> 3) / n_rb * 8 + (b & 7);
    rb = n_rb - 1 - (b >> 3) % n_rb;
  } else {
    kvh = full + (b - full * n_rb) % rem;
    rb = n_rb - 1 - (b - full * n_rb) / rem;
  }
}

// At most this many thread groups in the attention's combine kernel (16 pages
// each per round of loads); a launch uses ceil(max_chunks / 16) of them.
constexpr int COMBINE_GROUPS = 8;

// How a prefill pass's pages are split, at n_pos positions in all: the pass's
// time is the chain of a block's pages, 2.7 us each, and, where they are split,
// 4 us for a second launch and the partials' way through memory at 4 TB/s.
// Partials of every page, split so that no CU gets two blocks, or of the
// combine's groups; part_bytes bounds them.  The estimate has to win by a
// tenth: at 64 to 200 cached positions (three to five pages) both ways take
// the same time within 0.5 %.
struct AttnPlan {
  int split = 0;                                  // 0 not split, 1 partials of pages, 2 of the combine's groups
  int n_blocks = 1, n_parts = 0, pages_per_block = 0;  // per row block; per row and head; of mode 1
};
inline AttnPlan plan_attention_wide(int M, int nq, int nkv, int hd, int max_chunks, int n_pos, size_t part_bytes) {
  const int rows = M * (nq / nkv), blocks = nkv * ((rows + 127) / 128);
  const int P = (n_pos + 63) / 64, S = (max_chunks + 15) / 16 < COMBINE_GROUPS ? (max_chunks + 15) / 16 : COMBINE_GROUPS;
  const int used = (P + 15) / 16 < S ? (P + 15) / 16 : S;  // groups that have pages
  const double part_mb = (double)M * nq * (hd + 2) * 4 * 1e-6;  // of one partial
  AttnPlan plan;
  double best = 2.7 * P * ((blocks + 255) / 256);
  auto consider = [&](int split, int n_blocks, int n_parts, int chain, int pages) {
    const double t = 1.1 * (2.7 * chain * ((blocks * n_blocks + 255) / 256) + 4 + 2 * part_mb * n_parts / 4);
    if (part_mb * 1e6 * n_parts > (double)part_bytes || t >= best) return;
    best = t;
    plan.split = split;
    plan.n_blocks = n_blocks;
    plan.n_parts = n_parts;
    plan.pages_per_block = pages;
  };
  const int per = 256 / blocks;  // blocks that a row block's pages may go to
  if (per >= 2) {
    const int pages = (P + per - 1) / per;
    consider(1, (P + pages - 1) / pages, P, pages, pages);
  }
  if (used >= 2) consider(2, used, used, ((P + 15) / 16 + S - 1) / S * 16, 0);
  return plan;
}

// Where the partials of a split pass lie: the largest region that holds nothing
// during attention -- the partials of 16-row passes, the normalised rows (read
// by the launch before, written by the next), or the activations' rows unless
// zeros past F in a last tile that is not full have to stay.
// (F = 1200, d = 448, two layers, 17 rows behind 3000 positions: 154 us, and 321
// when there was no other place than the activations' rows; 217 in 16-row passes.)
enum AttnPartAt : int { PART_ROWS16, PART_NORM, PART_ACT };
struct AttnRoom { int at; size_t bytes; };
inline AttnRoom attn_part_room(int rows, int max_chunks, int nq, int hd, int d, int F) {
  AttnRoom r{PART_ROWS16, (size_t)16 * nq * max_chunks * (hd + 2) * 4};
  const size_t norm = (size_t)rows * d * Tile<1>::ES, act = F % Tile<1>::TK ? 0 : (size_t)rows * F * Tile<1>::ES;
  if (norm > r.bytes) r = {PART_NORM, norm};
  if (act > r.bytes) r = {PART_ACT, act};
  return r;
}

hipError_t launch_wide(int dtype, WideArgs a, hipStream_t s);
hipError_t launch_row_inv(const RowInvArgs& a, hipStream_t s);
hipError_t launch_head_rows(int dtype, const HeadRowsArgs& a, hipStream_t s);

}  // namespace lede
