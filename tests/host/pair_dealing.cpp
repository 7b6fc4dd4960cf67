// Host check of the dealing of work groups that take two 256-item blocks of the input transform: the map from
// slots to pairs is one-to-one, and all pairs of a unit have slots on one XCD (slot % 8).
#include <cstdio>
#include <vector>

#include "wino_kernels.hpp"

int main() {
  for (int frag = 0; frag < 2; ++frag)
    for (int N : {1, 7, 8, 9, 16, 17, 33, 250})
      for (int HW : {4, 8, 7, 12, 16})
        for (int C : {16, 80, 256, 272, 512, 768}) {
          wino::Geometry g0{};
          g0.N = N, g0.H = HW, g0.W = HW, g0.C = C, g0.K = 64, g0.m = 4, g0.frag = frag;
          g0.TH = (HW + 3) / 4, g0.TW = g0.TH, g0.T = N * g0.TH * g0.TW;
          const wino::Geometry g = wino::with_image_groups(g0, !frag && wino::whole_tiles(C, HW, HW), 2);
          const unsigned pairs = wino::input_pair_count(g0);
          std::vector<int> slot_of(pairs, -1);
          for (unsigned s = 0; s < pairs; ++s) {
            const unsigned p = wino::image_on_one_xcd(g, s);
            if (p >= pairs || slot_of[p] >= 0) return std::printf("slot %u -> %u of %u\n", s, p, pairs), 1;
            slot_of[p] = (int)s;
          }
          for (unsigned p = 0; g.img_blocks && p < (unsigned)g.img_blocks_end; ++p)
            if ((slot_of[p] ^ slot_of[p / g.img_blocks * g.img_blocks]) & 7)
              return std::printf("pair %u leaves its unit's XCD\n", p), 1;
        }
  std::printf("ok\n");
  return 0;
}
