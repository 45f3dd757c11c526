// Checks tile_div against the division of the language; prints the first mismatch and returns 1.
#include <cstdio>
#include <initializer_list>

#include "../paper_2406_04984_amd/csrc/tile_div.h"

static int bad(long long w, long long m) {
  const int q = meft::tile_div((int)w, (int)m, meft::tile_div_inverse((uint32_t)m));
  if (q == w / m) return 0;
  std::printf("%lld / %lld: %d, not %lld\n", w, m, q, w / m);
  return 1;
}

int main() {
  const long long most = 0x7FFFFFFFll;
  uint32_t x = 12345u;
  for (long long m = 1; m < 300000; m = m < 3000 ? m + 1 : m + 7 + (x >> 24)) {
    for (long long nt = 1; nt <= 32; ++nt)                       // the ends of every n tile's m tiles
      for (long long w = nt * m - 3; w <= nt * m + 2; ++w)
        if (w >= 0 && w <= most && bad(w, m)) return 1;
    for (int i = 0; i < 20; ++i) {
      x = x * 1664525u + 1013904223u;
      if (bad((x >> 1), m)) return 1;
    }
    if (bad(most, m) || bad(most / m * m, m) || bad(most / m * m - 1, m)) return 1;
  }
  for (long long m : {65535ll, 65536ll, 65537ll, 65625ll, 120000ll, 1ll << 20, (1ll << 25) + 1, 1ll << 30, most}) {
    for (long long w = m - 2; w <= m + 2; ++w)
      if (w <= most && bad(w, m)) return 1;
    for (long long w = most; w > most - 1000; --w)
      if (bad(w, m)) return 1;
  }
  return 0;
}
