// Host-side check of which kernels a forward call takes (no GPU needed): over random shapes, weighted towards few outputs, the route and its
// plan are the same for every workspace from the reported size on; and with any accepted size, the plan's buffers lie in the workspace.
// Prints "OK <shapes> <of them with the shared decode>" or the first violation.
#include <cstdio>
#include <cstring>
#include <random>

#include "launch.hpp"
#include "../../include/qlora.h"

using namespace qlora;

static size_t up(size_t b) { return (b + 255) / 256 * 256; }
static size_t used(const FwdRoute& f) {
  if (f.wide.ok) return up(f.wide.lpart_floats * 4) + up(f.wide.pack_elems * 2);
  if (f.mid.ok) return up(f.mid.part_floats * 4) + up(f.mid.lpart_floats * 4) + up(f.mid.pack_elems * 2);
  return 0;
}
static bool same(const FwdRoute& a, const FwdRoute& b) {
  if (a.wide.ok != b.wide.ok || a.mid.ok != b.mid.ok) return false;
  if (a.wide.ok) return a.wide.MF == b.wide.MF && a.wide.BN == b.wide.BN && a.wide.chunk == b.wide.chunk && a.wide.n_lparts == b.wide.n_lparts;
  return !a.mid.ok || (a.mid.MF == b.mid.MF && a.mid.KW == b.mid.KW && a.mid.pack == b.mid.pack && a.mid.chunk == b.mid.chunk &&
                       a.mid.line.wgs == b.mid.line.wgs);
}

int main() {
  std::mt19937 rng(5);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int n = 0, wide = 0;
  for (int it = 0; it < 40000; ++it) {
    const bool few = it % 8 == 0;
    const long M = few ? pick(1, kFewTokens) : pick(1, it % 3 ? kWideTokens + 8 : kMidTokens);
    const long h = 64 * pick(1, 200), o = 64 * pick(1, it % 2 ? 24 : 200);
    const int r = 16 * pick(0, 16);
    size_t need = 0;
    if (qlora_linear_fwd_sizes(M, h, o, r, &need) != QLORA_OK) return 1;
    const bool dq = few || it % 16 < 12;                     // one size for weights with and without Double Quantization
    const FwdRoute a = fwd_route(M, h, o, r, few, dq, need);
    for (size_t more : {(size_t)256, (size_t)pick(1, 1 << 20) * 256, (size_t)1 << 40})
      if (!same(a, fwd_route(M, h, o, r, few, dq, need + more))) {
        std::printf("FAIL M %ld h %ld o %ld r %d: another route with %zu bytes more than reported\n", M, h, o, r, more);
        return 1;
      }
    if (!few) {                                              // down to the smallest accepted size: the dequantised weight's, the adapter's left out
      const size_t least = QLORA_WORKSPACE_HEADER_BYTES + up((size_t)(h + (r > 0 ? (r + 63) / 64 * 64 : 0)) * o * 2);
      for (int t = 0; t < 3; ++t) {
        const size_t ws = t == 0 || need <= least ? least : least + rng() % (need - least);
        if (used(fwd_route(M, h, o, r, few, dq, ws)) > ws - QLORA_WORKSPACE_HEADER_BYTES) {
          std::printf("FAIL M %ld h %ld o %ld r %d: buffers beyond %zu bytes\n", M, h, o, r, ws);
          return 1;
        }
      }
    }
    ++n;
    wide += a.wide.ok;
  }
  std::printf("OK %d %d\n", n, wide);
  return 0;
}
