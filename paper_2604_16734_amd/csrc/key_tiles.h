// Which of a workgroup's key tiles can be brought in through a descriptor that moves on from tile to tile (attention.hip).  No
// device code: the host tests run it, too.
#pragma once

#include "key_range.h"

namespace kvp {

// Work on tile t fetches K of tile t + 2 and V of tile t + 1, each of them one of `n_tiles` tiles of `size` keys: `cached` keys of the
// cache and the block's own rows behind them, `n_cand` keys together.  Behind the last tile the descriptors stay where they are, on
// the last tile, or on tile 0 where there is no tile 2 (K) or 1 (V).  Returns for how many tiles t from 0 on all that they fetch lies in the cache
// or in the block as a whole: not so do the tile in which the cache ends and the block begins, and one that ends past the last
// key.  Tile 0 may be either, but where it is fetched again.
KVP_HOST_DEVICE int fed_tiles(int cached, int n_cand, int size, int n_tiles) {
  const int first_new = (cached + size - 1) / size, part = n_cand / size;      // the first tile without cached keys; the one that is not full
  int n = n_tiles;
  const auto end_at = [&](int t) { n = n < t ? n : t > 0 ? t : 0; };
  if (cached % size != 0 && first_new - 1 < n_tiles && (first_new > 1 || n_tiles <= 2)) end_at(first_new - 3);
  if (part < n_tiles) end_at(part - 2);
  return n;
}

}  // namespace kvp
