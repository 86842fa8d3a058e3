// Host-side check of the plans of the path whose waves share a decode, and of the choice against the other two (no GPU needed).  Random plans: tiles,
// steps, chunks and buffers cover the call and fit the room, each is one that launch_wide has a kernel for, and every such kernel has a plan.
// Then calls measured clearly faster one way (three weights in turn, whole calls) are sent that way.  Prints "OK <calls> <plans>" or the first that is not.
#include <algorithm>
#include <cstdio>
#include <random>
#include <set>

#include "launch.hpp"

using namespace qlora;

struct Call { bool bwd; int M, K, N, r; bool fix; double other_us, wide_us; bool dq = true; };   // fix: under LoRA dropout; other: the path it takes otherwise
static const Call kCalls[] = {
    // the shared decode: the faster one; weights of less and of more than 2 M elements, operands larger than the dequantised weight
    {false, 1097, 1280, 832, 16, false, 22.8, 20.2},   {true, 572, 1344, 768, 16, true, 27.6, 18.2},
    {false, 744, 2944, 256, 16, false, 31.4, 28.0},    {true, 597, 1408, 896, 16, false, 21.5, 18.2},
    {false, 1252, 9984, 256, 64, false, 71.9, 61.5},   {false, 530, 7680, 512, 0, false, 51.5, 39.1},
    {false, 749, 8768, 384, 0, false, 55.3, 44.4},     {true, 562, 12544, 4096, 32, false, 100.1, 83.1},
    {false, 796, 11136, 2304, 16, false, 84.3, 73.9},  {true, 742, 2240, 1792, 128, true, 39.5, 34.9},
    {false, 701, 4736, 2112, 0, false, 38.4, 32.9},    {true, 731, 832, 9024, 64, true, 46.4, 40.5},
    {true, 291, 640, 576, 128, true, 27.4, 20.5},      {true, 47, 576, 8704, 32, false, 21.8, 13.6},
    {true, 85, 960, 1600, 32, true, 21.4, 14.9},       {true, 65, 1600, 12032, 64, false, 30.1, 20.8},
    // dequantise + GEMM; the last five where the packed copy of the operand is what costs
    {false, 921, 960, 1344, 128, false, 22.7, 26.8},   {false, 1390, 576, 1024, 0, false, 11.9, 13.4},
    {false, 738, 1088, 1024, 128, false, 22.2, 25.3},  {false, 910, 512, 4352, 64, false, 20.8, 24.7},
    {false, 1542, 6912, 704, 64, false, 56.0, 59.2},   {false, 1414, 3904, 128, 0, false, 26.8, 30.5},
    {false, 1995, 7744, 512, 32, false, 60.6, 67.7},   {false, 1752, 2624, 256, 0, false, 21.7, 25.6},
    {false, 1933, 5888, 1024, 32, false, 50.7, 60.3},
    // the form that splits the contraction
    {false, 179, 2304, 2624, 128, false, 21.2, 27.4},  {false, 31, 1024, 704, 32, false, 12.1, 15.0},
    {false, 488, 6208, 2688, 64, false, 41.5, 44.4},   {true, 37, 6592, 576, 256, false, 50.9, 61.1},
    // and with large ranks over a long contraction, where a tile's start sums eight partials for every 64 of them
    {false, 493, 9216, 384, 256, false, 51.1, 72.8},   {false, 444, 12864, 1088, 256, false, 67.7, 94.6},
    {true, 503, 14208, 768, 256, false, 81.0, 109.4},  {true, 425, 13568, 1152, 256, true, 83.0, 104.9},
    // without Double Quantization
    {false, 299, 3712, 2176, 64, false, 28.7, 32.1, false}, {false, 485, 5696, 1280, 128, false, 38.2, 45.6, false},
    {true, 1227, 9024, 3136, 0, false, 73.9, 86.9, false},  {true, 178, 2368, 1152, 64, false, 20.8, 16.6},
};

int main() {
  const std::set<int> have = {1128, 2128, 3128, 1064, 2064, 3064, 4064};      // 1000 MF + BN
  std::set<int> seen;
  std::mt19937 rng(13);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int plans = 0;
  for (int it = 0; it < 20000; ++it) {
    const bool bwd = it & 1;
    const long M = pick(1, kWideTokens + 8), h = 64 * pick(1, it % 3 ? 48 : 344), o = 64 * pick(1, it % 3 ? 48 : 344);
    const int r = 16 * pick(0, 16);
    const size_t room = (size_t)h * o * 2 + ((size_t)pick(0, 32) << 20);
    const WidePlan p = wide_plan(bwd, M, h, o, r, room);
    if (!p.ok) continue;
    ++plans;
    const long K = bwd ? o : h, N = bwd ? h : o;
    if (M > kWideTokens || (p.lpart_floats * 4 + 255) / 256 * 256 + p.pack_elems * 2 > room || !have.count(1000 * p.MF + p.BN) ||
        (long)p.n_tg * 64 * p.MF < M || (long)(p.n_tg - 1) * 64 * p.MF >= M || (long)p.n_slabs * p.BN < N || (long)(p.n_slabs - 1) * p.BN >= N ||
        (long)p.steps * (16384 / p.BN) != p.k_pad || p.k_pad < K || p.k_pad - K >= 16384 / p.BN ||
        p.pack_elems < (size_t)p.n_tg * 64 * p.MF * p.k_pad || p.lpart_floats < (size_t)p.n_lparts * M * r ||
        (r > 0 && ((long)p.n_lparts * p.chunk < K || p.chunk % 64 != 0 || p.n_lparts > 8))) {
      std::printf("FAIL plan bwd %d M %ld h %ld o %ld r %d: MF %d BN %d\n", bwd, M, h, o, r, p.MF, p.BN);
      return 1;
    }
    seen.insert(1000 * p.MF + p.BN);
  }
  if (seen != have) { std::printf("FAIL %d of %d variants planned\n", (int)seen.size(), (int)have.size()); return 1; }
  int n = 0;
  for (const Call& c : kCalls) {
    const long h = c.bwd ? c.N : c.K, o = c.bwd ? c.K : c.N;
    const size_t base = (size_t)(c.bwd ? h : h + (c.r + 63) / 64 * 64) * o * 2;
    const MidPlan m = mid_plan(c.bwd, c.M, h, o, c.r, std::max(base, (size_t)32 << 20));
    const bool mid = m.ok && mid_pays(m, c.bwd, c.M, h, o, c.r, c.fix);
    const WidePlan w = wide_plan(c.bwd, c.M, h, o, c.r, SIZE_MAX);
    const bool wide = w.ok && wide_pays(w, mid ? &m : nullptr, c.bwd, c.M, h, o, c.r, c.fix, c.dq);
    if (wide != (c.wide_us < c.other_us)) {
      std::printf("FAIL %s M %d K %d N %d r %d: %.1f us otherwise, %.1f with the shared decode, takes the %s\n", c.bwd ? "bwd" : "fwd", c.M, c.K, c.N,
                  c.r, c.other_us, c.wide_us, wide ? "latter" : "former");
      return 1;
    }
    ++n;
  }
  std::printf("OK %d %d\n", n, plans);
  return 0;
}
