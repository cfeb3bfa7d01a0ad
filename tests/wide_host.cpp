// Host side of the many-row prefill kernels' interface (csrc/wide.h), for the
// tests: what the kernels and launchers compute from sizes alone.
#include "../paper_2606_03113_amd/csrc/wide.h"

extern "C" {

// The tiles of a K walk over KT tiles, in order, and the tile after the last.
void walk(int KT, int* tiles) {
  lede::KWalk w;
  for (int i = 0; i < KT; ++i, w.next(KT)) tiles[i] = w.t;
  tiles[KT] = w.t;
}

// (KV head, row block) of each of an attention launch's nkv * n_rb blocks.
void attn_blocks(int nkv, int n_rb, int* out) {
  for (int b = 0; b < nkv * n_rb; ++b) lede::attn_wide_block(b, nkv, n_rb, out[2 * b], out[2 * b + 1]);
}

// The kernel (index of its output tile) of a linear launch with M rows.
int linear_shape(int dtype, int n_groups, int M) { return lede::wide_shape(dtype, n_groups, M); }

// How an attention launch of M rows that ends at n_pos positions is split; the
// pages of a block in mode 1, and where the partials lie.
int attn_split(int nq, int nkv, int hd, int d, int F, int max_ctx, int M, int n_pos, int* pages, int* at) {
  const int chunks = (max_ctx + 63) / 64;
  const lede::AttnRoom room = lede::attn_part_room(lede::wide_rows(max_ctx), chunks, nq, hd, d, F);
  const lede::AttnPlan p = lede::plan_attention_wide(M, nq, nkv, hd, chunks, n_pos, room.bytes);
  *pages = p.pages_per_block;
  *at = room.at;
  return p.split;
}

}
