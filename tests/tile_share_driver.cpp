// Deals lists of whole and short tiles to eight parts as the 256 x 256 contractions do; prints the first list of which a tile is
// dealt twice or not at all, or whose parts are uneven, and returns 1.
#include <cstdio>
#include <vector>

#include "../paper_2406_04984_amd/csrc/tile_share.h"

int main() {
  for (int tn : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 15, 16, 17, 64, 255, 256})
    for (int groups = 1; groups <= 7; ++groups) {
      for (int rows : {1, 128, 129, 256, 257, 1000, 2048, 2500}) {
        int whole = 0, shorts = 0;
        for (int g = 0; g < groups; ++g) {
          const int r = rows + 64 * g, f = (r + 127) / 256;
          whole += f * tn;
          shorts += r > 256 * f ? tn : 0;
        }
        std::vector<int> seen_f(whole, 0), seen_h(shorts, 0);
        int least = 1 << 30, most = 0, least_f = 1 << 30, most_f = 0;
        for (int x = 0; x < 8; ++x) {
          const int f0 = meft::tile_share_first(whole, x), f1 = meft::tile_share_first(whole, x + 1);
          const int h0 = meft::tile_share_first(shorts, 7 - x), h1 = meft::tile_share_first(shorts, 8 - x);
          for (int i = f0; i < f1; ++i) ++seen_f[i];
          for (int i = h0; i < h1; ++i) ++seen_h[i];
          const int f = f1 - f0, all = f + h1 - h0;
          least_f = f < least_f ? f : least_f; most_f = f > most_f ? f : most_f;
          least = all < least ? all : least; most = all > most ? all : most;
        }
        bool once = true;
        for (int n : seen_f) once = once && n == 1;
        for (int n : seen_h) once = once && n == 1;
        if (!once || most_f - least_f > 1 || most - least > 2)
          return std::printf("%d groups from %d rows, %d columns: once %d, parts of %d to %d\n", groups, rows, tn, once, least, most), 1;
      }
    }
  return 0;
}
