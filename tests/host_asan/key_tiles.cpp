// fed_tiles(): the tiles that moving descriptors fetch, followed one by one as attention.hip moves them.
#include <cstdio>
#include <initializer_list>

#include "key_tiles.h"

int main() {
  for (int size : {64, 128})
    for (int cached = 0; cached <= 5 * size + 1; cached += cached % size < 2 || cached % size > size - 3 ? 1 : 7)
      for (int n_cand = cached + 1; n_cand <= cached + 6 * size; ++n_cand)
        for (int n_tiles = 1; n_tiles <= (n_cand + size - 1) / size; ++n_tiles) {
          auto whole = [&](int t) { return (t + 1) * size <= cached || (t * size >= cached && (t + 1) * size <= n_cand); };
          int k_tile = 2 < n_tiles ? 2 : 0, v_tile = 1 < n_tiles ? 1 : 0, fed = 0;
          for (; fed < n_tiles && whole(k_tile) && whole(v_tile); ++fed) {
            if (fed + 3 < n_tiles) k_tile = fed + 3;
            if (fed + 2 < n_tiles) v_tile = fed + 2;
          }
          const int said = kvp::fed_tiles(cached, n_cand, size, n_tiles);
          if (said != fed) {
            std::printf("tiles of %d: %d cached, %d keys, %d tiles: %d, not %d\n", size, cached, n_cand, n_tiles, said, fed);
            return 1;
          }
        }
  return 0;
}
