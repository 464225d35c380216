// Host-side check of pop::ActMap (csrc/chains.h): for every shape the library accepts, as many acting workgroups fit into a
// CU's LDS (two at most: their registers) as with the input tile, the head's weights staged beside it and no slabs.
#include <algorithm>
#include <cstdio>
#include "chains.h"

int main() {
  int bad = 0;
  for (int act = 1; act <= pop::kSacMaxAct; ++act)
    for (int obs = 1; obs + act <= pop::kSacMaxIn; ++obs)
      for (int outs : {act, 2 * act}) {
        const pop::ActMap m(obs);
        const size_t staged = pop::LdsMap<32, 8>(obs, 2 * (pop::kSacMaxAct / pop::kMaxAct)).bytes(pop::kH * outs + pop::kMaxHead);
        const size_t cu = pop::kLdsPerCU;
        if (m.bytes() > cu || (staged <= cu && std::min<size_t>(2, cu / m.bytes()) < std::min<size_t>(2, cu / staged))) {
          if (bad++ < 5) std::printf("obs %d outputs %d: %zu bytes, %zu\n", obs, outs, m.bytes(), staged);
        }
      }
  std::printf("bad %d\n", bad);
  return bad != 0;
}
