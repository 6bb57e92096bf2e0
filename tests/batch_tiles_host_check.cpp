// Host build of the tiles of the batched assembly: for every pair of orders
// in one launch "D other limbs highest size", the highest entry of LDS that
// a path of order D addresses beside one of order `other`, and the entries that
// the launch has.
#include "../paper_2301_12659_amd/csrc/batch_tiles.hpp"
#include <algorithm>
#include <cstdio>

using namespace mdk;

int main() {
  for (int D = 1; D <= 128; ++D)
    for (int other = 1; other <= 128; ++other)
      for (int L : {2, 4}) {
        int most = tile_doubles(tile_doubles(0, D), other), highest = 0;
        for (int l = 0; l < L; ++l)
          for (int s = 0; s < D; ++s)
            for (int row = 0; row < tile_rows(D); ++row) highest = std::max(highest, tile_index(D, l, s, row));
        printf("%d %d %d %d %d\n", D, other, L, highest, L * most);
      }
}
