// Host-side check of pop::act_grid (csrc/launch.h): the grid of an acting launch covers all rows of all agents, takes no second
// piece where one does, and no dimension of it reaches 2^32 threads (the device would run what is left of the number).
#include <cstdio>
#include "launch.h"

int main() {
  int bad = 0;
  const int agents[] = {1, 2, 3, 80, 255, 256, 257, 4096, 65535, 65536};
  const int64_t rows[] = {1, 31, 32, 33, 1000, 65280 * 32, (1ll << 28) + 33, (1ll << 29) - 32, (1ll << 29) - 31, (1ll << 31) - 33, (1ll << 31) - 1};
  for (int64_t P : agents)
    for (int64_t n : rows) {
      if (P * n > 1ll << 36) continue;                 // more than memory holds: 4 bytes a row at the least
      const pop::ActGrid g = pop::act_grid((int)P, (int)n);
      const int64_t need = (n + 31) / 32, have = (int64_t)g.chunks * g.pieces;
      const bool one = P * need * 256 < 1ll << 32;
      if (g.chunks < 1 || have < need || have - need >= g.chunks || P * g.chunks * 256 >= 1ll << 32 || g.pieces > 65535 ||
          have > (1ll << 31) - 1 || (one && (g.pieces != 1 || g.chunks != need)))
        if (bad++ < 5) std::printf("P %lld rows %lld: %d chunks, %d pieces\n", (long long)P, (long long)n, g.chunks, g.pieces);
    }
  std::printf("bad %d\n", bad);
  return bad != 0;
}
