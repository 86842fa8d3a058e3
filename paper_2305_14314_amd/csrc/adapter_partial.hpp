// Partial sums of the adapter's inner product for the paths that decode the weight inside the product at tens to hundreds of
// tokens (midtok.hip, widetok.hip), and what both do with a T = X L1 that is not finite.
#pragma once

#include "common.hpp"

namespace qlora {

__device__ __forceinline__ u32x4 apply_mask(u32x4 v, uint32_t b) {
#pragma unroll
  for (int d = 0; d < 4; ++d)
    v[d] &= (((b >> (2 * d)) & 1u) ? 0x0000ffffu : 0u) | (((b >> (2 * d + 1)) & 1u) ? 0xffff0000u : 0u);
  return v;
}

// ---- adapter partials: lpart[chunk][m][j] = sum over the chunk of X[m][k] L1[k][j]  (dY[m][n] L2[j][n]) -----------------
// Args: MidArgs or WideArgs (X, M x K; L, r, mask, chunk, lpart).  One workgroup per 32 tokens and chunk; its KW waves take the chunk's
// 32-wide steps in turn, two steps of loads in flight each, and are summed through LDS.
constexpr int kAdTok = 32;
template <int KW, bool BWD, bool MASKED, typename Args>
__device__ __forceinline__ void adapter_partial(const Args& p, int item, float* red /* [KW][32][64] */) {
  constexpr int NT = KW * 64, D = 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int n_tt = (p.M + kAdTok - 1) / kAdTok;
  const int m0 = (item % n_tt) * kAdTok, q = item / n_tt;
  const int k_begin = q * p.chunk, k_end = k_begin + p.chunk < p.K ? k_begin + p.chunk : p.K;   // multiples of 64
  float* out = p.lpart + (int64_t)q * p.M * p.r;
  // Raw loads only, each a scalar base and a fixed 32-bit offset (64-bit addresses per lane and element cost more than the
  // loads).  Tokens >= M and rank columns >= r read any valid row and only reach sums that are never stored.
  struct St { u32x4 x[2]; uint32_t keep[2]; uint32_t l[16]; };
  uint32_t x_off[2];                                         // in 16-byte chunks of X, which are bytes of the mask
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int m = m0 + 16 * f + i;
    x_off[f] = (uint32_t)(m < p.M ? m : p.M - 1) * (uint32_t)(p.K >> 3) + (uint32_t)g;
  }
  for (int j0 = 0; j0 < p.r; j0 += 64) {
    const uint32_t l_off = (uint32_t)(2 * g * p.r + (j0 + 4 * i < p.r ? (j0 >> 2) + i : 0));    // forward: in 8-byte chunks
    const uint16_t* l_row[4];                                // backward: 4 rank columns
#pragma unroll
    for (int e = 0; e < 4; ++e) l_row[e] = p.L + (int64_t)(BWD && j0 + 4 * i + e < p.r ? j0 + 4 * i + e : 0) * p.K + 8 * g;
    auto load = [&](St& s, int kb) {
      const int kc = kb < k_end ? kb : k_begin;              // past the end: any valid step, never consumed
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        s.x[f] = ((const u32x4*)(p.X + kc))[x_off[f]];
        if (MASKED) s.keep[f] = (p.mask + (kc >> 3))[x_off[f]];
      }
      if (!BWD) {                                            // L1 is [k][j]: 8 rows x 4 columns
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint2 v = ((const uint2*)(p.L + (int64_t)(kc + j) * p.r))[l_off];
          s.l[2 * j] = v.x; s.l[2 * j + 1] = v.y;
        }
      } else {                                               // L2 is [j][n]: 8 columns of 4 rows
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const u32x4 v = *(const u32x4*)(l_row[e] + kc);
#pragma unroll
          for (int d = 0; d < 4; ++d) s.l[4 * e + d] = v[d];
        }
      }
    };
    f32x4 acc[2][4];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[f][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const St& s) {
      u32x4 x[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) x[f] = MASKED ? apply_mask(s.x[f], s.keep[f]) : s.x[f];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        u32x4 w;
        if (!BWD) {
          const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
          for (int jp = 0; jp < 4; ++jp) w[jp] = __builtin_amdgcn_perm(s.l[2 * (2 * jp + 1) + (e >> 1)], s.l[2 * (2 * jp) + (e >> 1)], sel);
        } else {
#pragma unroll
          for (int d = 0; d < 4; ++d) w[d] = s.l[4 * e + d];
        }
#pragma unroll
        for (int f = 0; f < 2; ++f)
          acc[f][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[f]), __builtin_bit_cast(bf16x8, w),
                                                             acc[f][e], 0, 0, 0);
      }
    };
    St ring[D];
    const int kb0 = k_begin + wave * 32, stride = KW * 32;
#pragma unroll
    for (int d = 0; d < D; ++d) load(ring[d], kb0 + d * stride);
    for (int kb = kb0; kb < k_end; kb += D * stride) {
      const bool more = kb + D * stride < k_end;             // uniform
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (kb + d * stride < k_end) compute(ring[d]);
        if (more) load(ring[d], kb + (d + D) * stride);
      }
    }
    __syncthreads();                                         // the previous rank columns' sums have been read
    float* my = red + wave * (kAdTok * 64);
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *(f32x4*)(my + (16 * f + 4 * g + v) * 64 + 4 * i) = f32x4{acc[f][0][v], acc[f][1][v], acc[f][2][v], acc[f][3][v]};
    __syncthreads();
    for (int idx = threadIdx.x; idx < kAdTok * 16; idx += NT) {
      const int ml = idx >> 4, c4 = (idx & 15) * 4;
      f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < KW; ++w) t += *(const f32x4*)(red + w * (kAdTok * 64) + ml * 64 + c4);
      if (m0 + ml < p.M && j0 + c4 < p.r) *(f32x4*)(out + (int64_t)(m0 + ml) * p.r + j0 + c4) = t;
    }
  }
}

// An infinite hi is the whole value: what is left of it is NaN (or, of a value that rounded up to infinity, -Inf).  Two bf16 per dword.
__device__ __forceinline__ uint32_t lo_of_finite(uint32_t hi, uint32_t lo) {
  const uint32_t m = ((hi & 0x7f807f80u) + 0x00800080u) & 0x80008000u;      // the exponent is all ones
  return lo & ~((m - (m >> 15)) | m);
}

}  // namespace qlora
