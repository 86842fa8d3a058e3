// Host-side check (no GPU needed): every plan for 1 .. 512 tokens, over shapes, directions and workspace sizes, is one that
// launch_mid has a kernel for, and every such kernel has a plan.  Prints "OK <variants>" or the first that does not match.
#include <cstdio>
#include <random>
#include <set>

#include "launch.hpp"

using namespace qlora;

int main() {
  std::set<int> have, seen;                                  // 1000 bwd + 100 pack + 10 (KW == 8) + MF
  for (int mf = 2; mf <= 8; ++mf) have.insert(1100 + mf);
  for (int mf = 3; mf <= 8; ++mf) have.insert(100 + mf);
  have.insert({113, 114, 11, 12, 13});
  std::mt19937 rng(11);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  for (int M = 1; M <= kMidTokens; ++M)
    for (int it = 0; it < 60; ++it) {
      const bool bwd = it & 1;
      const int h = 64 * pick(1, it % 3 ? 64 : 344), o = 64 * pick(1, it % 3 ? 64 : 344), r = 16 * pick(0, 16);
      const MidPlan p = mid_plan(bwd, M, h, o, r, (size_t)h * o * 2 + ((size_t)pick(0, 64) << 20));
      if (!p.ok) continue;
      const int v = 1000 * bwd + 100 * p.pack + 10 * (p.KW == 8) + p.MF;
      if (!have.count(v) || (p.KW != 4 && p.KW != 8)) {
        std::printf("FAIL M %d h %d o %d bwd %d: KW %d MF %d pack %d has no kernel\n", M, h, o, bwd, p.KW, p.MF, p.pack);
        return 1;
      }
      seen.insert(v);
    }
  for (int v : have)
    if (!seen.count(v)) { std::printf("FAIL variant %d is never planned\n", v); return 1; }
  std::printf("OK %d\n", (int)seen.size());
  return 0;
}
