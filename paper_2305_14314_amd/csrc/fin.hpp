// The finalize step of the skinny products, as a device function: it runs in a launch of its own or as the first
// workgroups of a dequantise launch.
#pragma once

#include "common.hpp"
#include "launch.hpp"

namespace qlora {

constexpr int kFinThreads = 256;

// Sums the split partials of a job in a fixed order (deterministic); four neighbouring columns per thread (J, w0 and ld0
// are multiples of 4).
//   sum(i, j)  = sum over splits of part[s][i][j]
//   out0[i][j] = bf16(scale0 * sum) for j < J, zero for J <= j < w0                    (row stride ld0)
//   hl[i][j]   = bf16(sum),  hl[i][J + j] = bf16(sum - hl[i][j])                       (row stride 2 J)
//   acc[i][j] += scale0 * sum                                      (fp32, row stride J: gradient accumulation)
// A job with `src` instead copies: out0[i][j] = src[i][j] (bf16, row stride J) for j < J, zero for J <= j < w0.
template <int UNROLL = 8>
__device__ __forceinline__ void fin_job(const FinJob& p, int block, int blocks) {
  const int wq = ((p.out0 && p.w0 > p.J) ? p.w0 : p.J) >> 2;
  const int64_t total = (int64_t)p.I * wq, stride = (int64_t)blocks * kFinThreads;
  const int64_t plane = (int64_t)p.I * p.J;
  for (int64_t e = (int64_t)block * kFinThreads + threadIdx.x; e < total; e += stride) {
    const int i = (int)(e / wq), j = 4 * (int)(e - (int64_t)i * wq);
    const bool in = j < p.J;
    if (p.src) {
      *(uint2*)(p.out0 + (int64_t)i * p.ld0 + j) = in ? *(const uint2*)(p.src + (int64_t)i * p.J + j) : uint2{0u, 0u};
      continue;
    }
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
    if (in) {
      const float* src = p.part + (int64_t)i * p.J + j;
#pragma unroll UNROLL
      for (int sp = 0; sp < p.splits; ++sp) s += *(const f32x4*)(src + sp * plane);
    }
    if (p.out0 && j < p.w0) {
      uint2 o;
      o.x = pack_bf16x2(s[0] * p.scale0, s[1] * p.scale0);
      o.y = pack_bf16x2(s[2] * p.scale0, s[3] * p.scale0);
      *(uint2*)(p.out0 + (int64_t)i * p.ld0 + j) = o;
    }
    if (!in) continue;
    if (p.acc) {
      f32x4* a = (f32x4*)(p.acc + (int64_t)i * p.J + j);
      f32x4 t = *a;
#pragma unroll
      for (int v = 0; v < 4; ++v) t[v] += s[v] * p.scale0;
      *a = t;
    }
    if (p.hl) {
      uint2 hi, lo;
      hi.x = pack_bf16x2(s[0], s[1]);
      hi.y = pack_bf16x2(s[2], s[3]);
      lo.x = pack_bf16x2(s[0] - bf16_lo_to_f32(hi.x), s[1] - bf16_hi_to_f32(hi.x));
      lo.y = pack_bf16x2(s[2] - bf16_lo_to_f32(hi.y), s[3] - bf16_hi_to_f32(hi.y));
      *(uint2*)(p.hl + (int64_t)i * 2 * p.J + j) = hi;
      *(uint2*)(p.hl + (int64_t)i * 2 * p.J + p.J + j) = lo;
    }
  }
}

// The same for workgroup `block` of a list's.
template <int UNROLL = 8>
__device__ __forceinline__ void fin_block(const FinList& f, int block) {
  int q = 0;
  while (q + 1 < f.n && block >= f.first[q + 1]) ++q;
  fin_job<UNROLL>(f.j[q], block - f.first[q], f.first[q + 1] - f.first[q]);
}

}  // namespace qlora
