// The 128-bit mean of exponent bins against the limb form, over random bins: few
// and many binades, sums near rounding ties, zeros, subnormals, quotients of fewer than 24 bits.
#define __host__
#define __device__
#include "dq_mean.hpp"

#include <cstdio>
#include <random>

int main() {
  std::mt19937_64 rng(20240607);
  long fast = 0;
  for (int it = 0; it < 400000; ++it) {
    unsigned long long lb[256] = {}, present[4] = {};
    const int kind = (int)(rng() % 6);
    const uint32_t n = kind == 0 ? 1u + (uint32_t)(rng() % 4) : kind == 1 ? 0xffffffffu - (uint32_t)(rng() % 5) : 1u + (uint32_t)(rng() % (1u << (1 + rng() % 31)));
    const int e0 = 1 + (int)(rng() % 254), span = kind == 2 ? 254 : (int)(rng() % 70);
    const int cnt = kind == 3 ? 1 : 1 + (int)(rng() % 24);
    for (int c = 0; c < cnt; ++c) {
      const int e = e0 + (span ? (int)(rng() % (span + 1)) : 0);
      if (e > 254) continue;
      unsigned long long v = rng() >> (8 + rng() % 56);      // below 2^56
      if (kind == 4) v = (unsigned long long)n << (rng() % 24);   // exact quotients and ties
      if (kind == 5 && (rng() & 1)) v = v / n * n + n / 2;
      lb[e] = v & ((1ull << 56) - 1);
    }
    for (int e = 0; e < 256; ++e)
      if (lb[e]) present[e >> 6] |= 1ull << (e & 63);
    const float a = qlora::mean_from_bins(lb, present, n), b = qlora::mean_from_bins_any(lb, present, n);
    uint32_t ua, ub;
    memcpy(&ua, &a, 4); memcpy(&ub, &b, 4);
    if (ua != ub) { printf("mismatch it=%d n=%u %08x %08x\n", it, n, ua, ub); return 1; }
    int lo = 256, hi = -1;
    for (int e = 0; e < 256; ++e) if (lb[e]) { if (lo == 256) lo = e; hi = e; }
    fast += hi >= 0 && hi - lo <= 60;
  }
  printf("ok %ld\n", fast);
  return 0;
}
