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

}
