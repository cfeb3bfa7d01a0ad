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

hipError_t launch_wide(int dtype, WideArgs a, hipStream_t s);
hipError_t launch_row_inv(const RowInvArgs& a, hipStream_t s);
hipError_t launch_head_rows(int dtype, const HeadRowsArgs& a, hipStream_t s);

}  // namespace lede
