// Host-side check of the choice between the product that decodes the weight itself and dequantise + GEMM (no GPU needed):
// calls measured clearly faster one way (three weights in turn, whole calls) are sent that way.  Prints "OK <calls>" or the first that is not.
#include <algorithm>
#include <cstdio>

#include "launch.hpp"

using namespace qlora;

struct Call { bool bwd; int M, K, N, r; bool fix; double gemm_us, mid_us; };   // fix: under LoRA dropout
static const Call kCalls[] = {
    // the product that decodes the weight: the faster one
    {false, 40, 4096, 11008, 64, false, 48.4, 21.7},   {false, 256, 1024, 1024, 64, false, 17.7, 15.1},
    {false, 512, 4096, 4096, 64, false, 44.9, 40.7},   {true, 256, 4096, 4096, 64, false, 44.2, 35.3},
    {false, 256, 5120, 13824, 64, false, 83.1, 62.6},  {false, 320, 5120, 13824, 64, false, 106.8, 89.2},
    {false, 512, 8192, 1024, 256, false, 65.5, 55.8},  {true, 512, 22016, 8192, 256, false, 358.6, 259.4},
    {false, 256, 22016, 8192, 64, false, 333.8, 111.8}, {true, 256, 13824, 5120, 64, false, 118.0, 66.3},
    {true, 384, 8192, 4096, 64, false, 65.2, 56.8},    {true, 128, 8192, 1024, 64, false, 60.4, 34.1},
    // the operand as it lies, above 48 tokens
    {false, 186, 2368, 384, 128, false, 28.4, 18.3},   {false, 65, 1664, 8768, 32, false, 29.3, 19.5},
    {false, 119, 6208, 128, 16, false, 44.0, 19.3},    {false, 72, 3776, 64, 256, false, 35.3, 26.1},
    // short contractions, wide ranks: dequantise + GEMM
    {true, 384, 64, 16384, 0, false, 10.4, 39.3},      {false, 384, 64, 16384, 64, false, 16.3, 39.8},
    {true, 17, 64, 1024, 256, false, 10.9, 24.4},      {true, 128, 128, 4096, 256, false, 13.0, 30.4},
    {true, 512, 64, 4096, 256, false, 13.1, 35.5},     {true, 512, 1024, 8192, 256, false, 28.8, 65.0},
    {false, 512, 1024, 8192, 256, false, 29.7, 57.6},  {true, 512, 5120, 13824, 256, false, 107.9, 163.9},
    {true, 16, 192, 4096, 256, false, 12.3, 28.9},     {true, 384, 64, 16384, 256, true, 50.6, 73.3},
    // the adapter's workgroups beside the product's, longer than those
    {false, 79, 256, 1088, 256, false, 13.5, 20.6},    {false, 114, 512, 448, 256, false, 15.7, 21.1},
    {false, 193, 192, 64, 256, false, 12.6, 18.8},     {false, 111, 256, 64, 256, false, 12.7, 20.4},
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
