// Host-side check of the choice between the product that decodes the weight itself and dequantise + GEMM (no GPU needed):
// calls measured clearly faster one way are sent that way.  Prints "OK <calls>" or the first that is not.
#include <algorithm>
#include <cstdio>

#include "launch.hpp"

using namespace qlora;

struct Call { bool bwd; int M, K, N, r; bool fix; double gemm_us, mid_us; };   // fix: under LoRA dropout
static const Call kCalls[] = {
    // the product that decodes the weight: the faster one
    {false, 40, 4096, 11008, 64, false, 83.5, 21.9},   {false, 256, 1024, 1024, 64, false, 23.1, 21.7},
    {false, 512, 4096, 4096, 64, false, 58.2, 44.2},   {true, 512, 4096, 4096, 64, false, 56.8, 47.5},
    {false, 256, 5120, 13824, 64, false, 89.1, 61.0},  {false, 320, 5120, 13824, 64, false, 96.0, 90.9},
    {false, 512, 8192, 1024, 256, false, 93.1, 60.8},  {true, 512, 22016, 8192, 256, false, 439.4, 272.5},
    {false, 256, 22016, 8192, 64, false, 421.0, 117.0}, {true, 256, 13824, 5120, 64, false, 154.1, 71.9},
    // short contractions, wide ranks: dequantise + GEMM
    {true, 384, 64, 16384, 0, false, 12.1, 43.5},      {false, 384, 64, 16384, 64, false, 18.6, 42.4},
    {true, 17, 64, 1024, 256, false, 15.4, 25.3},      {true, 128, 128, 4096, 256, false, 15.8, 31.3},
    {true, 512, 64, 4096, 256, false, 15.7, 36.5},     {true, 512, 1024, 8192, 256, false, 31.8, 65.6},
    {false, 512, 1024, 8192, 256, false, 31.9, 54.5},  {true, 512, 5120, 13824, 256, false, 100.0, 170.4},
    {true, 16, 192, 4096, 256, false, 15.7, 29.2},     {true, 384, 64, 16384, 256, true, 49.1, 70.3},
};

int main() {
  int n = 0;
  for (const Call& c : kCalls) {
    const long h = c.bwd ? c.N : c.K, o = c.bwd ? c.K : c.N;
    const MidPlan p = mid_plan(c.bwd, c.M, h, o, c.r, std::max((size_t)h * o * 2, (size_t)32 << 20));
    const bool mid = p.ok && mid_pays(p, c.bwd, c.M, h, o, c.r, c.fix);
    if (mid != (c.mid_us < c.gemm_us)) {
      std::printf("FAIL %s M %d K %d N %d r %d: %.1f us dequantised, %.1f decoded inside, takes the %s\n", c.bwd ? "bwd" : "fwd",
                  c.M, c.K, c.N, c.r, c.gemm_us, c.mid_us, mid ? "latter" : "former");
      return 1;
    }
    ++n;
  }
  std::printf("OK %d\n", n);
  return 0;
}
