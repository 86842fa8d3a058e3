// The exact mean of the first-level constants from their exponent bins.  Integer code, the same on host and device.
#pragma once

#include <cstdint>
#include <cstring>

namespace qlora {

__host__ __device__ inline float dq_float(uint32_t bits) {
  float f;
  memcpy(&f, &bits, 4);
  return f;
}

// sum = SUM_e bins[e] * 2^(e-1) in units of 2^-149, as 12 x 32-bit limbs; mean = round_to_nearest_even_fp32(sum / n).
// Run by one lane; only the non-empty bins (bit e % 64 of present[e / 64]) and the non-zero limbs are visited, so the
// serial part is a few dozen operations.
__host__ __device__ inline float mean_from_bins_any(const unsigned long long* lb, const unsigned long long* present, uint32_t n) {
  constexpr int L = 12;
  uint32_t acc[L];
  for (int k = 0; k < L; ++k) acc[k] = 0;
  int top_limb = -1;
  for (int q = 0; q < 4; ++q) {
    unsigned long long mask = present[q];
    while (mask) {
      const int e = q * 64 + __builtin_ctzll(mask);
      mask &= mask - 1;
      if (e < 1 || e > 254) continue;                       // exponent 255 (inf/nan) never occurs: inputs are finite
      const unsigned long long b = lb[e];
      const int sh = e - 1, limb = sh >> 5, off = sh & 31;
      // b < 2^56; b << off spans at most three limbs
      const uint32_t p0 = (uint32_t)(b << off);
      const unsigned long long hi = off ? (b >> (32 - off)) : (b >> 32);
      const uint32_t parts[3] = {p0, (uint32_t)hi, (uint32_t)(hi >> 32)};
      unsigned long long carry = 0;
      for (int k = 0; k < L - limb; ++k) {
        const unsigned long long t = (unsigned long long)acc[limb + k] + (k < 3 ? parts[k] : 0u) + carry;
        acc[limb + k] = (uint32_t)t;
        carry = t >> 32;
        if (t && limb + k > top_limb) top_limb = limb + k;
        if (k >= 2 && carry == 0) break;
      }
    }
  }
  uint32_t q[L];
  for (int k = 0; k < L; ++k) q[k] = 0;
  unsigned long long rem = 0;
  for (int k = top_limb; k >= 0; --k) {                      // long division by n < 2^32
    const unsigned long long cur = (rem << 32) | acc[k];
    q[k] = (uint32_t)(cur / n);
    rem = cur % n;
  }
  int top = -1;
  for (int k = top_limb; k >= 0; --k)
    if (q[k]) { top = k * 32 + 31 - __builtin_clz(q[k]); break; }
  // keep the 24 leading bits of q (all of q if it is shorter), round on the rest and on rem/n
  const int drop = top >= 24 ? top - 23 : 0;
  auto bit = [&](int i) -> uint32_t { return (q[i >> 5] >> (i & 31)) & 1u; };
  uint32_t kept = 0;
  for (int i = top; i >= drop; --i) kept = (kept << 1) | bit(i);
  bool half, sticky;
  if (drop == 0) {
    half = 2 * rem >= n;
    sticky = 2 * rem > n;
  } else {
    half = bit(drop - 1) != 0;
    sticky = rem != 0;
    for (int i = drop - 2; i >= 0 && !sticky; --i) sticky = bit(i) != 0;
  }
  if (half && (sticky || (kept & 1u))) ++kept;              // kept <= 2^24
  // result = kept * 2^(drop - 149) with kept <= 2^24: with drop = 0 the integer is the bit pattern itself
  // (subnormals and the first binades); each further dropped bit raises the exponent field by one.
  return dq_float(kept + ((uint32_t)drop << 23));
}

// The same number when the non-empty bins lie within 60 binades and the quotient has at least 24 bits, as for any weight
// whose blocks are not mostly zeros: 128-bit arithmetic instead of limbs in indexed registers.  Every workgroup of the
// encode launch waits for one lane's answer: the general form took 5 us there.
__host__ __device__ inline float mean_from_bins(const unsigned long long* lb, const unsigned long long* present, uint32_t n) {
  int e_min = 256, e_max = -1;
  for (int q = 0; q < 4; ++q)
    if (present[q]) {
      const int lo = q * 64 + __builtin_ctzll(present[q]);
      e_max = q * 64 + 63 - __builtin_clzll(present[q]);
      e_min = lo < e_min ? lo : e_min;
    }
  if (e_max < 0 || e_min < 1 || e_max > 254 || e_max - e_min > 60) return mean_from_bins_any(lb, present, n);
  unsigned __int128 sum = 0;                                 // in units of 2^(e_min - 150); below 2^56 * 2^61
  for (int e = e_min; e <= e_max; ++e) sum += (unsigned __int128)lb[e] << (e - e_min);
  uint32_t quo[4];
  unsigned long long rem = 0;
#pragma unroll
  for (int k = 3; k >= 0; --k) {                             // long division by n < 2^32
    const unsigned long long cur = (rem << 32) | (uint32_t)(sum >> (32 * k));
    quo[k] = cur < n ? 0u : (uint32_t)(cur / n);
    rem = cur - (unsigned long long)quo[k] * n;
  }
  const unsigned long long hi = ((unsigned long long)quo[3] << 32) | quo[2], lo = ((unsigned long long)quo[1] << 32) | quo[0];
  const int top = hi ? 127 - __builtin_clzll(hi) : lo ? 63 - __builtin_clzll(lo) : -1;
  if (top < 23) return mean_from_bins_any(lb, present, n);
  const unsigned __int128 q = ((unsigned __int128)hi << 64) | lo;
  const int drop = top - 23;                                 // keep the 24 leading bits, round to nearest even on the rest
  uint32_t kept = (uint32_t)(q >> drop);
  bool half, sticky;
  if (drop == 0) {
    half = 2 * rem >= n;
    sticky = 2 * rem > n;
  } else {
    const unsigned __int128 low = q & (((unsigned __int128)1 << drop) - 1), h = (unsigned __int128)1 << (drop - 1);
    half = low >= h;
    sticky = rem != 0 || (low & (h - 1)) != 0;
  }
  if (half && (sticky || (kept & 1u))) ++kept;
  return dq_float(kept + ((uint32_t)(drop + e_min - 1) << 23));
}

}  // namespace qlora
