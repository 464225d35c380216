// Host-side check of pop::spread_of (csrc/launch.h): every workgroup of the launch it asks for gets a CU, and what it leaves out would not.
#include <cstdio>
#include "launch.h"

int main() {
  int bad = 0;
  pop::PopDev d{};
  d.B = 256;
  d.rows_t = d.rows_a = 16;
  d.rows_c = d.rows_c1 = 32;
  for (d.P = 1; d.P <= 40; ++d.P)
    for (bool forward : {false, true}) {
      const int s = pop::spread_of(d, forward), want = d.P <= 4 ? (forward ? 3 : 1) : d.P == 5 ? 1 : 0;
      const int blocks = d.P * (16 + 16) + (s & pop::kSpreadTargets ? 16 * d.P : 0) + (s & pop::kSpreadActor ? 16 * d.P : 0);
      if (s != want || (s && blocks > pop::kCUs)) { ++bad; std::printf("P %d: %d, %d workgroups\n", d.P, s, blocks); }
    }
  d.P = 2;
  for (int k = 0; k < 5; ++k) {                       // other rows, or the pass in the critics' workgroups
    pop::PopDev e = d;
    if (k == 0) e.rows_t = 32;
    if (k == 1) e.rows_c = e.rows_c1 = 64;
    if (k == 2) e.rows_c1 = 16;
    if (k == 3) e.rows_a = 32;
    if (k == 4) e.actor_ahead = 1;
    if (pop::spread_of(e, true)) { ++bad; std::printf("case %d\n", k); }
  }
  std::printf("bad %d\n", bad);
  return bad != 0;
}
