// Host-side check of the plan for tens to hundreds of tokens (no GPU needed): over random shapes, directions, ranks and
// workspace sizes the buffers fit the workspace, the ranges tile the line of units without an empty one, rho_of inverts
// start, every tile's contributors (brute force over the ranges) are those the kernels derive and fit the partial buffer.
// Prints "OK <plans>" or the first violation.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "launch.hpp"

using namespace qlora;

static int fail(const char* what, long a, long b, long c) {
  std::printf("FAIL %s (%ld, %ld, %ld)\n", what, a, b, c);
  return 1;
}
static size_t up(size_t b) { return (b + 255) / 256 * 256; }

int main() {
  std::mt19937 rng(7);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int plans = 0;
  for (int it = 0; it < 6000; ++it) {
    const bool bwd = rng() & 1;
    const int M = pick(1, kMidTokens), h = 64 * pick(1, it % 3 ? 24 : 344), o = 64 * pick(1, it % 3 ? 24 : 344), r = 16 * pick(0, 16);
    const size_t room = (size_t)h * o * 2 + (rng() & 1 ? 0 : (size_t)pick(0, 64) << 20);
    const MidPlan p = mid_plan(bwd, M, h, o, r, room);
    if (!p.ok) continue;
    ++plans;
    const int K = bwd ? o : h, N = bwd ? h : o;
    if (up(p.part_floats * 4) + up(p.lpart_floats * 4) + up(p.pack_elems * 2) > room) return fail("workspace", M, h, o);
    if (p.part_floats < (size_t)p.max_contrib * M * N || p.lpart_floats < (size_t)p.n_lparts * M * r) return fail("buffers", M, h, o);
    if (p.pack && p.pack_elems < (size_t)p.n_tg * p.MF * 16 * K) return fail("operand copy", M, h, o);
    if (p.n_tg * p.MF * 16 < M || p.n_slabs * 128 < N || p.n_slabs * 128 >= N + 128) return fail("tiles", M, h, o);
    if (r > 0 && ((long)p.chunk * p.n_lparts < K || p.chunk % 64 != 0)) return fail("chunks", p.chunk, p.n_lparts, K);
    if (p.steps * (bwd ? 64 : 32) != K || p.line.ups * p.KW < p.steps || (p.line.ups - 1) * p.KW >= p.steps) return fail("steps", p.steps, K, p.KW);
    const MidLine& L = p.line;
    if (L.units != p.n_tg * p.n_slabs * L.ups || L.wgs < 1 || L.wgs > 256) return fail("line", L.units, L.ups, L.wgs);
    if (L.start(0) != 0 || L.start(L.wgs) != L.units) return fail("ends", L.start(0), L.start(L.wgs), L.units);
    std::vector<int> first(p.n_tg * p.n_slabs, -1), last(p.n_tg * p.n_slabs, -1);
    for (int rho = 0; rho < L.wgs; ++rho) {
      const int a = L.start(rho), b = L.start(rho + 1);
      if (a >= b) return fail("empty range", rho, a, b);
      if (L.rho_of(a) != rho || L.rho_of(b - 1) != rho || L.rho_of((a + b) / 2) != rho) return fail("rho_of", rho, a, b);
      for (int t = a / L.ups; t <= (b - 1) / L.ups; ++t) { if (first[t] < 0) first[t] = rho; last[t] = rho; }
    }
    for (int t = 0; t < (int)first.size(); ++t)
      if (first[t] != L.rho_of(t * L.ups) || L.contributors(t) != last[t] - first[t] + 1 || L.contributors(t) > p.max_contrib)
        return fail("contributors", t, L.contributors(t), p.max_contrib);
  }
  std::printf("OK %d\n", plans);
  return 0;
}
