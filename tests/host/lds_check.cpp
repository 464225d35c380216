// Host-side check of pop::ActMap and pop::CriticMap (csrc/chains.h): for every shape the library accepts, as many acting
// workgroups fit into a CU's LDS (two at most: their registers) as with the input tile, the head's weights staged beside it and
// no slabs, and as many wide critic workgroups on four wavefronts as without slabs; those on eight, slabs beside the input tile, fit
// at all; no two regions of a wide critic's map overlap before the input tile is done with.
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
  for (int in = pop::kMaxIn + 1; in <= pop::kSacMaxIn; ++in) {
    const pop::CriticMap<pop::Rows32Deep<2, false>> m(in);
    const size_t without = pop::LdsMap<32, 8>(in).bytes(pop::vec_critic_floats), cu = pop::kLdsPerCU;
    const bool apart = m.buf + 32 * pop::kLda <= m.s0 && m.s0 + 32 * pop::kMaxAct <= m.s1 && m.s1 + 32 * pop::kMaxAct <= m.vec &&
                       m.vec + pop::vec_critic_floats <= m.input && m.input % 4 == 0 && m.stage == m.input &&
                       m.bytes() >= sizeof(float) * (m.input + std::max(32 * m.xld, pop::Rows32<1>::kStage));
    if (!apart || std::min<size_t>(2, cu / m.bytes()) < std::min<size_t>(2, cu / without)) {
      if (bad++ < 5) std::printf("critic, %d inputs: %zu bytes, %zu\n", in, m.bytes(), without);
    }
    const pop::CriticMap<pop::Rows32Wide> w(in);       // slabs beside the input tile
    const bool beside = w.input + 32 * w.xld <= w.buf && w.buf + 32 * pop::kLda <= w.s0 && w.s0 + 32 * pop::kMaxAct <= w.s1 &&
                        w.s1 + 32 * pop::kMaxAct <= w.vec && w.vec + pop::vec_critic_floats <= w.stage && w.stage % 4 == 0 &&
                        w.bytes() >= sizeof(float) * (w.stage + pop::Rows32Wide::kStage);
    if (!beside || w.bytes() > cu) {
      if (bad++ < 5) std::printf("critic on eight wavefronts, %d inputs: %zu bytes\n", in, w.bytes());
    }
  }
  std::printf("bad %d\n", bad);
  return bad != 0;
}
