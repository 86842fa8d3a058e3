// Forward and input gradient of the QLoRA linear layer at tens to hundreds of tokens (arXiv 2305.14314, Eq. 5 / Eq. 6), second
// form: the eight waves of a workgroup share one decode of its part of the packed weight, through LDS, and the workgroup
// finishes its outputs itself.
//
// Against the first form (midtok.hip: every wave decodes what it multiplies, waves split the contraction): no partial sums of
// the product in memory, no cross-wave sum of whole tiles, no finalize launch, and with two waves per SIMD one wave's decode
// beside another's products; but a tile's contraction is not divided, so it takes as many workgroups as there are tiles.  Which of
// the two a call takes, or dequantise + GEMM, is wide_pays' choice.  Whole calls replayed, us, other path / this one: forward 333 tokens
// 5120 x 13824 88 / 70, 768 tokens 8192 x 8192 169 / 113, dX 512 tokens 4096 x 4096 41 / 33, 249 tokens 5568 x 1088 (no adapter) 21.4 / 14.2,
// 61 tokens 10752 x 768 rank 16 24.8 / 14.3.
//
// Two launches: `pre` puts the token operand into MFMA-fragment order and forms partials of the adapter's inner product
// T = X L1 (U = dY L2^T); `main` sums them, starts its accumulators with s T L2 (T as a [hi | lo] pair of bf16, 16 significant
// bits; under LoRA dropout masked, before the frozen product is added, so there is one rounding), multiplies and stores.
#include <algorithm>
#include <type_traits>

#include "adapter_partial.hpp"
#include "fewtok_common.hpp"

#define QL_INLINE __attribute__((always_inline))

namespace qlora {

namespace {

using few::kLutCopies;
using few::kLutBytes;
using few::init_pair_lut;
using few::pair_lookup_b;
using few::work_index;

// LDS map: the decode table, two buffers of decoded weights (32 KB each) -- where before the loop the adapter's operands lie: 64 ranks of
// its outer matrix, 16 KB, and of T, 16 KB per 64 tokens --, and what a wave keeps for itself
constexpr int kBufOff = kLutBytes, kBufBytes = 32 * 1024;
constexpr int kAdB = 16 * 1024;
constexpr int kWideUnit = kBufOff + kAdB + 64 * 1024;                         // float[256]
constexpr int kWideStrip = kWideUnit + 1024;                                  // float[8 waves][32]
constexpr int kWideRaw = kWideStrip + 8 * 128;                                // 1 KB per wave
constexpr int kWideSmem = kWideRaw + 8 * 1024;
static_assert(kBufOff + 2 * kBufBytes <= kWideUnit && kWideSmem <= 160 * 1024, "LDS map");

struct WideArgs {
  const uint16_t* X;                         // token operand as it lies: X (M x h) or dY (M x o)
  int M, K, N, h, o;                         // K: contraction length, N: outputs
  const char* Xf; uint32_t x_bytes;          // token operand in fragment order
  int tiles;                                 // its 16-token tiles
  const uint8_t* packed; const uint8_t* code; const float* c1; const float* mean;
  int dtype, dq; Table4 tab;
  int n_tg, steps;
  const uint16_t* L; int r;                  // adapter's inner matrix: L1 (h x r) or L2 (r x o)
  const uint8_t* mask;                       // keep-bits of X (forward), or NULL
  float* lpart; int n_lparts, chunk;         // [n_lparts][M][r]
  const uint16_t* B;                         // adapter's outer matrix: L2 (r x N) forward, L1 (N x r) backward
  float scale;
  const uint8_t* keep;                       // backward under LoRA dropout: keep-bits of the output elements, or NULL
  uint16_t* out; uint16_t* hl;
};

template <int N> using Int = std::integral_constant<int, N>;
// f(Int<B>), f(Int<B + 1>), .. f(Int<E - 1>)
template <int B, int E, typename F> __device__ __forceinline__ void each(F&& f) {
  if constexpr (B < E) {
    f(Int<B>{});
    each<B + 1, E>(f);
  }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t wide_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}

// ---- token operand in fragment order, and the adapter's partials --------------------------------------------------------
// Fragment of 16 tokens x 32 contraction elements = 1 KB: lane (i, g) at byte 16 (16 g + i) holds token i's elements
// 8g .. 8g+7; [32-wide step][token tile].  Tokens beyond M and elements beyond K are zeros.
constexpr int kPreK = 512;
template <bool BWD>
__global__ __launch_bounds__(512) void wide_pre_kernel(const WideArgs p, uint16_t* __restrict__ Xp, int items, int k_pad) {
  __shared__ __attribute__((aligned(16))) char smem[8 * kAdTok * 64 * 4];
  if ((int)blockIdx.x < items) {
    if (!BWD && p.mask) adapter_partial<8, BWD, !BWD>(p, blockIdx.x, (float*)smem);
    else adapter_partial<8, BWD, false>(p, blockIdx.x, (float*)smem);
    return;
  }
  const int n_kb = (k_pad + kPreK - 1) / kPreK, at = (int)blockIdx.x - items;
  const int tile = at / n_kb, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int k0 = (at - tile * n_kb) * kPreK + wave * 64, i = lane & 15, g = lane >> 4;
  if (k0 >= k_pad) return;
  const int m = 16 * tile + i;
  const bool ok = m < p.M && k0 < p.K;                       // K % 64 == 0
  const uint16_t* src = p.X + (int64_t)(m < p.M ? m : p.M - 1) * p.K + (k0 < p.K ? k0 : 0) + 8 * g;
  u32x4 v[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) v[t] = *(const u32x4*)(src + 32 * t);
#pragma unroll
  for (int t = 0; t < 2; ++t)
    *(u32x4*)(Xp + (((int64_t)(k0 >> 5) + t) * p.tiles + tile) * 512 + 8 * lane) = ok ? v[t] : u32x4{0u, 0u, 0u, 0u};
}

// ---- main ---------------------------------------------------------------------------------------------------------------
// Workgroup: 64 MF tokens x BN outputs, eight waves: wave = 4 kh + rw multiplies tokens 16 MF rw .. of the tile by half kh of
// every step's contraction elements.  A step is 16384 weights: 128 elements x 128 outputs or 256 x 64.  Decoded weights lie in
// LDS in MFMA-fragment order: [tile e of 16 outputs][32-wide substep][lane], two steps of them.
//
// What bounds it: the waves' issue and the waits around it.  A step of <3, 128> (192 tokens) takes 1.2 us on some compute units and
// 1.35 on all; its products alone 0.73, with the fragment reads, the barrier and the loads 0.9; lookups, factors and stores of the decode add about
// 0.1 each (timing builds with one of them taken out), the barrier 0.1.  Over the whole kernel of 333 tokens 5120 x 13824 the matrix pipes are
// 45 % busy, LDS 43 %, a wave waits for data or a barrier 33 % and for its turn 32 % of its time.  Slabs of 64 (half the outputs, twice the contraction a step) read the
// token operand twice as often, 64 bytes a clock per compute unit, and are for outputs that 128-wide slabs leave compute units idle
// with.  Tried and slower: four waves of twice the tokens with everything interleaved in one wave (1.64 at the same 192 tokens,
// 6.3 M multiply-adds a step in 2.4 us where this takes 2.4), the decode by the two halves in turn (spills), eight 2-byte loads per lane and step
// in the forward instead of 16 bytes and a transposing read (1.44), more requests in flight in `pre` (200 registers: 2 us a call); no
// difference: the barrier in the middle of a group, another order of the decode behind the products, a wave priority by half.
// The fixed part of a call is 8 us, and 3 - 5 us per 64 ranks: the launch of `pre`, and T's partials, 64 MF x 64 x 4 bytes each.
template <int BN> struct WideShape {
  static constexpr int NE = BN / 16, SUB = 512 / BN, WS = SUB / 2, KSTEP = 32 * SUB;
};

// A register of its own for what the next load overwrites: left to itself the compiler gives the load another one and moves that at
// the end of the loop, i.e. waits for it there.
template <typename T> __device__ __forceinline__ void keep_now(T& to, T from) { asm volatile("v_mov_b32 %0, %1" : "=v"(to) : "v"(from)); }

// raw loads of a lane's share of a step: 32 weights of a row, and a constant
struct WideW { u32x4 raw; uint32_t code; float c1; };

template <int MF, int BN, bool BWD>
__global__ __launch_bounds__(512) void wide_main_kernel(const WideArgs p) {
  using S = WideShape<BN>;
  constexpr int NE = S::NE, SUB = S::SUB, WS = S::WS, KSTEP = S::KSTEP, TT = 4 * MF;
  __shared__ __attribute__((aligned(256))) char smem[kWideSmem];
  f32x2* lut2 = (f32x2*)smem;
  float* unit = (float*)(smem + kWideUnit);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int rw = wave & 3, kh = wave >> 2, i = lane & 15, g = lane >> 4;
  const uint32_t lane_off = 8u * (uint32_t)(lane & (kLutCopies - 1));
  float* strip = (float*)(smem + kWideStrip) + wave * 32;
  const int work = work_index(), tg = work % p.n_tg, slab = work / p.n_tg;
  const int m0 = tg * 16 * TT, n0 = slab * BN;
  const float mean = p.dq ? *p.mean : 0.0f;
  const int bpr = p.o >> 6, rowb = p.o >> 1;

  // ---- loads: a resource over a tensor (or a step's rows), a fixed per-lane offset and a scalar one ----------------------
  const uint32_t n_blocks = (uint32_t)p.h * (uint32_t)bpr;
  const __amdgpu_buffer_rsrc_t code_rsrc = wide_rsrc(p.dq ? p.code : p.packed, n_blocks);
  const __amdgpu_buffer_rsrc_t c1_rsrc = wide_rsrc(p.c1, 4u * (p.dq ? (n_blocks + 255u) / 256u : n_blocks));
  const int c1_shift = p.dq ? 8 : 0, code_w = p.dq ? 1 : 0;
  const __amdgpu_buffer_rsrc_t x_rsrc = wide_rsrc(p.Xf, p.x_bytes);
  const uint32_t x_lane = (uint32_t)((tg * TT + rw * MF) * 1024 + lane * 16);
  auto load_x = [&](u32x4 (&x)[MF], int step, int sub) QL_INLINE {   // sub: 0 .. WS - 1 of this wave's half
    const int sc = step < p.steps ? step : p.steps - 1;
    const int so = (sc * SUB + kh * WS + sub) * p.tiles * 1024;
#pragma unroll
    for (int f = 0; f < MF; ++f) x[f] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, x_lane, so + f * 1024, 0);
  };
  // A wave decodes an eighth of a step.  Forward: 32 rows of one block of 64 columns; lane l loads half l / 32 of row l % 32.
  // Backward: lane (i, g) 32 elements of a row.
  const int ds = BN == 128 ? wave >> 1 : wave;               // forward: substep; its column block is wave % 2 of a slab of 128
  const int fblk = (n0 >> 6) + (BN == 128 ? wave & 1 : 0), fb = fblk < bpr ? fblk : bpr - 1;
  const int fw = (fb & ~3) + 4 <= bpr ? 4 : bpr - (fb & ~3);
  const uint32_t w_lane = (uint32_t)((lane & 31) * rowb) + 16u * (uint32_t)(lane >> 5);
  const int b_row = n0 + 16 * (BN == 128 ? wave : wave & 3) + i, bk = BN == 128 ? 0 : wave >> 2;
  const uint32_t brow = (uint32_t)(b_row < p.h ? b_row : p.h - 1);
  const int bdb = 2 * bk + (g >> 1);                         // backward: block of the step
  auto load_w = [&](WideW& s, int step) QL_INLINE {
    const int sc = step < p.steps ? step : p.steps - 1;
    if constexpr (!BWD) {
      const int k0 = sc * KSTEP + 32 * ds, kc = k0 < p.K ? k0 : 0;           // K % 64 == 0: a wave's rows are inside or outside together
      const __amdgpu_buffer_rsrc_t w_rsrc = wide_rsrc(p.packed + (int64_t)kc * rowb + fb * 32, 32u * (uint32_t)rowb);
      s.raw = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, 0, 0);
      s.code = __builtin_amdgcn_raw_buffer_load_b8(code_rsrc, (uint32_t)((lane & 31) * fw * code_w),
                                                   (4 * p.h * (fb >> 2) + (fb & 3) + kc * fw) * code_w, 0);
      const uint32_t idx = (uint32_t)kc * (uint32_t)bpr + (uint32_t)((lane & 31) * bpr + fb);
      s.c1 = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(c1_rsrc, (idx >> c1_shift) * 4u, 0, 0));
    } else {
      const __amdgpu_buffer_rsrc_t w_rsrc = wide_rsrc(p.packed + (int64_t)sc * (KSTEP / 2), (uint32_t)p.h * (uint32_t)rowb);
      const int b0 = sc * (KSTEP / 64), G = b0 >> 2, w = 4 * G + 4 <= bpr ? 4 : bpr - 4 * G;
      const bool ok = b0 + bdb < bpr;                        // past the last block: the step's first, times zero
      s.raw = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, brow * (uint32_t)rowb + (ok ? (uint32_t)(64 * bk + 16 * g) : 0u), 0, 0);
      s.code = __builtin_amdgcn_raw_buffer_load_b8(code_rsrc, (brow * (uint32_t)w + (uint32_t)((b0 & 3) + (ok ? bdb : 0))) * (uint32_t)code_w,
                                                   4 * p.h * G * code_w, 0);
      const uint32_t idx = brow * (uint32_t)bpr + (uint32_t)(b0 + (ok ? bdb : 0));
      s.c1 = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(c1_rsrc, (idx >> c1_shift) * 4u, 0, 0));
    }
  };

  WideW w0, w1, wb[2];                                       // steps 0 and 1; step s from 2 on is decoded from wb[s % 2]
  constexpr int XR = 4;                                      // substeps of the token operand in registers or on the way
  u32x4 xb[XR][MF];

  auto load_ahead = [&]() QL_INLINE {                         // in the order of the loop: its waits count the loads in flight
    load_w(wb[0], 2);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (BN == 128) {
      load_x(xb[0], 0, 0);
      load_x(xb[1], 0, 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    load_w(wb[1], 3);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = BN == 128 ? 2 : 0; q < XR; ++q) load_x(xb[q], q / WS, q % WS);
    __builtin_amdgcn_sched_barrier(0);
  };
  // ---- the adapter's term first: acc = s T B with T as a [hi | lo] pair, a half of the waves each ------------------------
  // In LDS both operands lie in fragment order with columns XORed by k group (and tile), so that what one instruction stores meets
  // at most twice in a bank (as they come, eight times: <3, 128> took 1.6 us a call more forward, 0.5 backward).
  f32x4 acc[MF][NE];
  char* adb = smem + kBufOff;                                // [tile e][RS substeps][lane]
  char* tf = smem + kBufOff + kAdB;                          // [hi, lo][RS substeps][token tile][lane]
  const int tok0 = m0 + 16 * MF * rw;                        // this wave's first token
  constexpr int RK = 64, RS = RK / 32, RQ = RK / 4;          // ranks at a time, substeps, quadruples
  constexpr int TR = 512 / RQ, QN = 64 * MF / TR;            // tokens per pass of the workgroup; quadruples of ranks per thread
  const __amdgpu_buffer_rsrc_t t_rsrc = wide_rsrc(p.lpart, (uint32_t)(p.n_lparts * p.M) * (uint32_t)p.r * 4u);
  const int tq = threadIdx.x & (RQ - 1), ml0 = threadIdx.x / RQ;
  // the outer matrix: forward 8 ranks x 4 outputs of L2 per lane, backward 8 ranks of a row of L1
  constexpr int kC4 = BN / 4, NB = BWD ? BN * RK / 4096 : 1;
  const int c4 = threadIdx.x % kC4, rgf = threadIdx.x / kC4;
  uint2 bf[BWD ? 1 : 8];
  u32x4 bb[NB];
  auto request_b = [&](int j0) QL_INLINE {
    if constexpr (!BWD) {
      const int n = n0 + 4 * c4;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int rr = j0 + 8 * rgf + j;
        bf[j] = *(const uint2*)(p.B + (int64_t)(rr < p.r ? rr : 0) * p.N + (n < p.N ? n : 0));
      }
    } else {
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        const int idx = threadIdx.x + 512 * x, rr = j0 + 8 * (idx & (RK / 8 - 1)), n = n0 + idx / (RK / 8);
        bb[x] = *(const u32x4*)(p.B + (int64_t)(n < p.N ? n : p.N - 1) * p.r + (rr < p.r ? rr : 0));
      }
    }
  };
  // partials s .. s + 3 of quadruples q0 .. q0 + QB - 1 of this thread
  auto request_t = [&](auto& v, auto Qb, int j0, int q0, int s) QL_INLINE {
    constexpr int QB = decltype(Qb)::value;
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int m = m0 + ml0 + TR * (q0 + q);
      const uint32_t off = ((uint32_t)(m < p.M ? m : p.M - 1) * (uint32_t)p.r + (uint32_t)(j0 + 4 * tq < p.r ? j0 + 4 * tq : 0)) * 4u;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(t_rsrc, off, (s + u < p.n_lparts ? s + u : s) * (p.M * p.r * 4), 0));
    }
  };
  auto take_t = [&](auto& v, auto Qb, int j0, int q0) QL_INLINE {
    constexpr int QB = decltype(Qb)::value;
    f32x4 t[QB];
#pragma unroll
    for (int q = 0; q < QB; ++q) t[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0;;) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < QB; ++q)
          if (s + u < p.n_lparts) t[q] += v[u][q];
      s += 4;
      if (s >= p.n_lparts) break;
      request_t(v, Qb, j0, q0, s);
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int ml = ml0 + TR * (q0 + q), m = m0 + ml;
      const bool ok = j0 + 4 * tq < p.r && m < p.M;          // r % 16 == 0
      uint2 hi, lo;
      few::split_hl(ok ? t[q] : f32x4{0.f, 0.f, 0.f, 0.f}, hi, lo);
      if (ok && p.hl && slab == 0) {
        *(uint2*)(p.hl + (int64_t)m * 2 * p.r + j0 + 4 * tq) = hi;
        *(uint2*)(p.hl + (int64_t)m * 2 * p.r + p.r + j0 + 4 * tq) = lo;
      }
      lo = uint2{lo_of_finite(hi.x, lo.x), lo_of_finite(hi.y, lo.y)};
      char* d = tf + ((tq >> 3) * TT + (ml >> 4)) * 1024 + (16 * ((tq >> 1) & 3) + ((ml & 15) ^ (4 * ((tq >> 1) & 3)))) * 16 + 8 * (tq & 1);
      *(uint2*)d = hi;
      *(uint2*)(d + RS * TT * 1024) = lo;
    }
  };
  auto multiply = [&](int j0) QL_INLINE {
    auto put_b = [&](int nl, int rg, u32x4 w) QL_INLINE {    // ranks 8 rg .. + 7 of output nl of the slab
      const int te = nl >> 4, ti = nl & 15;
      *(u32x4*)(adb + (te * RS + (rg >> 2)) * 1024 + (16 * (rg & 3) + (ti ^ (te & 3) ^ (4 * (rg & 3)))) * 16) = w;
    };
    if constexpr (!BWD) {
      if (threadIdx.x < RK / 8 * kC4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          u32x4 w;
          const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
          for (int jp = 0; jp < 4; ++jp)
            w[jp] = e < 2 ? __builtin_amdgcn_perm(bf[2 * jp + 1].x, bf[2 * jp].x, sel) : __builtin_amdgcn_perm(bf[2 * jp + 1].y, bf[2 * jp].y, sel);
          if (j0 + 8 * rgf >= p.r) w = u32x4{0u, 0u, 0u, 0u};  // r % 16 == 0: eight ranks are inside or outside together
          put_b(4 * c4 + e, rgf, w);
        }
      }
    } else {
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        const int idx = threadIdx.x + 512 * x, nl = idx / (RK / 8);
        put_b(nl, idx & (RK / 8 - 1), j0 + 8 * (idx & (RK / 8 - 1)) < p.r ? bb[x] : u32x4{0u, 0u, 0u, 0u});
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < RS; ++s) {
      bf16x8 a[MF];
#pragma unroll
      for (int f = 0; f < MF; ++f) a[f] = *(const bf16x8*)(tf + ((kh * RS + s) * TT + rw * MF + f) * 1024 + (lane ^ (4 * g)) * 16);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const bf16x8 b = *(const bf16x8*)(adb + (e * RS + s) * 1024 + (lane ^ (e & 3) ^ (4 * g)) * 16);
#pragma unroll
        for (int f = 0; f < MF; ++f) acc[f][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[f], b, acc[f][e], 0, 0, 0);
      }
    }
  };
  init_pair_lut<512>(lut2, unit, p.dtype, p.tab);            // as in midtok.hip before the first requests
  __builtin_amdgcn_sched_barrier(0);
  // quadruples of T whose partials are requested together: of the first ranks, and of later ones, with the accumulators live
  constexpr int QF = QN % 3 == 0 ? 3 : QN < 4 ? QN : 4, QL = 2;
  f32x4 tv[4][QF];
  load_w(w0, 0);
  load_w(w1, 1);
  if (p.r > 0) {                                             // uniform
    request_b(0);
    request_t(tv, Int<QF>{}, 0, 0, 0);
#pragma unroll
    for (int q0 = 0; q0 < QN; q0 += QF) {
      if (q0 > 0) request_t(tv, Int<QF>{}, 0, q0, 0);
      take_t(tv, Int<QF>{}, 0, q0);
    }
  }
  load_ahead();
#pragma unroll
  for (int f = 0; f < MF; ++f)
#pragma unroll
    for (int e = 0; e < NE; ++e) acc[f][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (p.r > 0) {                                             // uniform
    multiply(0);
    for (int j0 = RK; j0 < p.r; j0 += RK) {
      __syncthreads();                                       // the previous ranks have been read
      request_b(j0);
#pragma unroll
      for (int q0 = 0; q0 < QN; q0 += QL) {
        f32x4 v[4][QL];
        request_t(v, Int<QL>{}, j0, q0, 0);
        take_t(v, Int<QL>{}, j0, q0);
      }
      multiply(j0);
    }
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        uint32_t bits[NE / 2];                               // of outputs 32x .. 32x + 31
#pragma unroll
        for (int x = 0; x < NE / 2; ++x) bits[x] = 0xffffffffu;
        if (BWD && p.keep) {
          const int m = tok0 + 16 * f + 4 * g + v;
#pragma unroll
          for (int x = 0; x < NE / 4; ++x) {                 // N % 64 == 0: 64 outputs are inside or outside together
            const int n = n0 + 64 * x;
            uint2 b;                                         // the caller's bytes, at any address: one load all the same
            __builtin_memcpy(&b, p.keep + (((int64_t)(m < p.M ? m : 0) * p.N + (n < p.N ? n : 0)) >> 3), 8);
            bits[2 * x] = b.x; bits[2 * x + 1] = b.y;
          }
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[f][e][v] = ((bits[e >> 1] >> (16 * (e & 1) + i)) & 1u) ? p.scale * acc[f][e][v] : 0.0f;
      }
  }
  __syncthreads();                                           // the table stands; the adapter's operands have been read

  // ---- decoding ------------------------------------------------------------------------------------------------------------
  float c2[BWD ? 2 : 16];                                    // forward: of 16 rows; backward: of even and odd steps
  uint32_t pk[2][4];                                         // of even and odd steps
  f32x2 q[2][8];
  // Forward: the 32 x 64 codes of the wave pass through a kilobyte of its own and come back transposed: lane 16 (kb + 2 cb) + j of read t
  // gets elements 16 kb .. 16 kb + 15 of column 32 t + 16 cb + j.
  char* mine = smem + kWideRaw + wave * 1024;
  auto unpack = [&](const WideW& w, uint32_t (&o)[4]) QL_INLINE {
    if constexpr (!BWD) {
      *(u32x4*)(mine + lane * 16) = w.raw;
      typedef int i32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const i32x2 v = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr4_b64_v2i32(
            (i32x2 __attribute__((address_space(3)))*)(mine + t * 512 + ((g & 1) * 16 + i) * 16 + 8 * (g >> 1))));
        o[2 * t] = (uint32_t)v[0]; o[2 * t + 1] = (uint32_t)v[1];
      }
    } else {
#pragma unroll
      for (int d = 0; d < 4; ++d) keep_now(o[d], w.raw[d]);
    }
  };
  // The constants of a step, in three parts that lie apart: the lookup of the lane's code; its constant, kept (backward) or put where the
  // wave finds it (forward); forward: the lane's sixteen.
  float un, c1v;
  auto constant_a = [&](const WideW& w) QL_INLINE { un = unit[w.code]; keep_now(c1v, w.c1); };
  auto constant_b = [&](int par, int step) QL_INLINE {
    const int sc = step < p.steps ? step : p.steps - 1;
    const float d = __fadd_rn(__fmul_rn(un, c1v), mean);
    const float v = p.dq ? d : c1v;
    if constexpr (!BWD) strip[lane & 31] = sc * KSTEP + 32 * ds < p.K ? v : 0.0f;
    else c2[par] = sc * (KSTEP / 64) + bdb < bpr ? v : 0.0f;
  };
  auto constants = [&]() QL_INLINE {
    if constexpr (!BWD) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const f32x4 v = *(const f32x4*)&strip[16 * (g & 1) + 4 * x];
#pragma unroll
        for (int j = 0; j < 4; ++j) c2[4 * x + j] = v[j];
      }
    }
  };
  // A lane's 32 weights are four fragments of eight elements of one output: dword F of pk.  Two to a chunk of eight lookups.
  auto lookup = [&](const uint32_t (&k)[4], int ch, int l) QL_INLINE -> f32x2 { return pair_lookup_b(lut2, k[2 * ch + (l >> 2)], lane_off, l & 3); };
  // where the fragments of buffer 0 go: forward F = 2 t + d: tile 2 t + g / 2 (behind those of the block before), k group 2 (g % 2) + d
  char* wr;
  if constexpr (!BWD)
    wr = smem + kBufOff + ((BN == 128 ? 4 * (wave & 1) : 0) + (g >> 1)) * SUB * 1024 + ds * 1024 + (32 * (g & 1) + i) * 16;
  else
    wr = smem + kBufOff + (BN == 128 ? wave * SUB * 1024 + g * 1024 : (wave & 3) * SUB * 1024 + (4 * bk + g) * 1024) + i * 16;
  // Fragment F: four dwords of two factors and a rounding, and the store.
  u32x4 wf;
  float pr[2];
  constexpr int kItems = 13;
  auto item = [&](auto Fc, auto It, auto Par) QL_INLINE {
    constexpr int F = decltype(Fc)::value, ch = F >> 1, v = F & 1, it = decltype(It)::value, par = decltype(Par)::value;
    constexpr int sub = it % 3, d = it / 3 & 3;
    if constexpr (it == 12) *(u32x4*)(wr + par * kBufBytes + (BWD ? F * 256 : ch * 2 * SUB * 1024 + v * 256)) = wf;
    else if constexpr (sub == 2) wf[d] = pack_bf16x2(pr[0], pr[1]);
    else pr[sub] = __fmul_rn(q[ch & 1][4 * v + d][sub], c2[BWD ? par : 8 * v + 2 * d + sub]);
  };

  const char* rd = smem + kBufOff + kh * WS * 1024 + lane * 16;
  constexpr bool kPing = MF <= 2;                            // two sets of fragments, else each is replaced as it is used up
  bf16x8 fr[kPing ? 2 : 1][4];
  auto read_frag = [&](int par, int j, int x) QL_INLINE {    // fragment x of group j of the buffer of parity `par`
    const int e = BN == 128 ? 4 * (j & 1) + x : x, sub = BN == 128 ? j >> 1 : j;
    fr[kPing ? j & 1 : 0][x] = *(const bf16x8*)(rd + par * kBufBytes + (e * SUB + sub) * 1024);
  };
  // Group j (0 .. 3) of a step of parity par: 4 MF products.  While they run: the fragments of the next group; fragment F of the
  // weights of parity wpar into their buffer; four lookups of the chunk after the next.
  auto group = [&](auto Jc, auto Par) QL_INLINE {
    constexpr int J = decltype(Jc)::value, par = decltype(Par)::value;
    constexpr int NM = 4 * MF, next_par = J == 3 ? par ^ 1 : par, next = (J + 1) & 3;
    constexpr int slot = BN == 128 ? 2 * par + (J >> 1) : J;
    constexpr int F = (J + 1) & 3, wpar = J == 3 ? par : par ^ 1;          // J = 3: begins the step after the next
    constexpr int lch = (F >> 1) ^ 1, lpar = F >= 2 ? wpar ^ 1 : wpar;
    if constexpr (kPing) each<0, 4>([&](auto X) QL_INLINE { read_frag(next_par, next, decltype(X)::value); });
    each<0, NM>([&](auto Kc) QL_INLINE {
      constexpr int k = decltype(Kc)::value, x = k / MF, f = k % MF, e = BN == 128 ? 4 * (J & 1) + x : x;
      acc[f][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xb[slot][f]), fr[kPing ? J & 1 : 0][x], acc[f][e], 0, 0, 0);
      if constexpr (!kPing && f == MF - 1) read_frag(next_par, next, x);
      each<kItems * k / NM, kItems * (k + 1) / NM>([&](auto It) QL_INLINE { item(Int<F>{}, It, Int<wpar>{}); });
      each<4 * k / NM, 4 * (k + 1) / NM>([&](auto L) QL_INLINE {
        constexpr int l = 4 * (F & 1) + decltype(L)::value;
        q[lch & 1][l] = lookup(pk[lpar], lch, l);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto meet = [&]() QL_INLINE { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  // Step k: its products; step k + 1 is decoded meanwhile (fragments 1 .. 3), step k + 2 begun behind the barrier, in front of which
  // every wave has the step's last fragments in registers.
  auto step = [&](auto Par, int k) QL_INLINE {
    constexpr int PAR = decltype(Par)::value;
    auto refill = [&](auto Jc) QL_INLINE {                   // the token operand's slot that group j was the last to read
      constexpr int J = decltype(Jc)::value;
      if constexpr (BN == 64) load_x(xb[J], k + 1, J);
      else if constexpr (J & 1) load_x(xb[2 * PAR + (J >> 1)], k + 2, J >> 1);
    };
    each<0, 4>([&](auto Jc) QL_INLINE {
      constexpr int J = decltype(Jc)::value;
      if constexpr (J == 0) {
        constant_a(wb[PAR]);
        unpack(wb[PAR], pk[PAR]);
        load_w(wb[PAR], k + 4);
      }
      if constexpr (J == 2) constant_b(PAR, k + 2);
      if constexpr (J == 3) { constants(); meet(); }
      group(Jc, Par);
      refill(Jc);
    });
  };

  auto look8 = [&](const uint32_t (&w)[4], int ch) QL_INLINE {
#pragma unroll
    for (int l = 0; l < 8; ++l) q[ch][l] = lookup(w, ch, l);
  };
  auto fragment = [&](auto F, auto Par) QL_INLINE { each<0, kItems>([&](auto It) QL_INLINE { item(F, It, Par); }); };
  constant_a(w0);
  constant_b(0, 0);
  constants();
  unpack(w0, pk[0]);
  look8(pk[0], 0);
  look8(pk[0], 1);
  fragment(Int<0>{}, Int<0>{});
  fragment(Int<1>{}, Int<0>{});
  fragment(Int<2>{}, Int<0>{});
  fragment(Int<3>{}, Int<0>{});
  constant_a(w1);
  constant_b(1, 1);
  constants();
  unpack(w1, pk[1]);
  look8(pk[1], 0);
#pragma unroll
  for (int l = 0; l < 4; ++l) q[1][l] = lookup(pk[1], 1, l);
  fragment(Int<0>{}, Int<1>{});
  meet();
  each<0, 4>([&](auto X) QL_INLINE { read_frag(0, 0, decltype(X)::value); });
  int k = 0;
#pragma unroll 1
  for (; k + 1 < p.steps; k += 2) {
    step(Int<0>{}, k);
    step(Int<1>{}, k + 1);
  }
  if (k < p.steps) step(Int<0>{}, k);

  // ---- the two halves' sums, half of the tokens finished by each; rounded to bf16 they pass through LDS once more, so that a lane
  // stores 16 bytes of neighbouring outputs ---------------------------------------------------------------------------------
  __syncthreads();
  constexpr int NQ = NE / 4, kGive = MF * 2 * NQ * 1024, kTok = 8 * MF;       // kTok: tokens a wave finishes
  static_assert(8 * (kGive + kTok * NE * 32) <= kWideSmem, "LDS map");
  auto finish = [&](auto Kh) QL_INLINE {
    constexpr int KH = decltype(Kh)::value, V = 2 * KH, O = 2 - V;
    char* give = smem + wave * kGive + lane * 16;
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int x = 0; x < NQ; ++x)
          *(f32x4*)(give + ((f * 2 + v) * NQ + x) * 1024) = f32x4{acc[f][4 * x][O + v], acc[f][4 * x + 1][O + v],
                                                                 acc[f][4 * x + 2][O + v], acc[f][4 * x + 3][O + v]};
    __syncthreads();
    const char* take = smem + (wave ^ 4) * kGive + lane * 16;
    char* rows = smem + 8 * kGive + wave * (kTok * NE * 32);                  // [token][pair of tiles][i]: outputs 32x + i, 32x + 16 + i
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int x = 0; x < NQ; ++x) {
          const f32x4 other = *(const f32x4*)(take + ((f * 2 + v) * NQ + x) * 1024);
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = KH == 0 ? acc[f][4 * x + e][V + v] + other[e] : other[e] + acc[f][4 * x + e][V + v];
#pragma unroll
          for (int e = 0; e < 2; ++e)
            *(uint32_t*)(rows + (((f * 2 + v) * 4 + g) * (NE / 2) + ((2 * x + e) ^ (NE == 8 ? g : g >> 1))) * 64 + 4 * i) = pack_bf16x2(y[2 * e], y[2 * e + 1]);
        }
    // (token, pair of tiles, half) per lane: eight dwords, whose low halves and high halves are eight neighbouring outputs each
    constexpr int kTasks = kTok * NE;
#pragma unroll
    for (int t = 0; t < (kTasks + 63) / 64; ++t) {
      const int idx = t * 64 + lane, hf = idx & 1, x = (idx >> 1) % (NE / 2), tok = (idx >> 1) / (NE / 2);
      const u32x4* src = (const u32x4*)(rows + (tok * (NE / 2) + (x ^ (NE == 8 ? tok & 3 : (tok >> 1) & 1))) * 64 + hf * 32);
      const u32x4 a = src[0], b = src[1];
      const int m = tok0 + 16 * (tok >> 3) + 4 * (tok & 3) + V + ((tok >> 2) & 1), n = n0 + 32 * x + 8 * hf;
      if (idx < kTasks && m < p.M && n < p.N) {
        uint16_t* o = p.out + (int64_t)m * p.N + n;
        *(u32x4*)o = u32x4{__builtin_amdgcn_perm(a[1], a[0], 0x05040100u), __builtin_amdgcn_perm(a[3], a[2], 0x05040100u),
                           __builtin_amdgcn_perm(b[1], b[0], 0x05040100u), __builtin_amdgcn_perm(b[3], b[2], 0x05040100u)};
        *(u32x4*)(o + 16) = u32x4{__builtin_amdgcn_perm(a[1], a[0], 0x07060302u), __builtin_amdgcn_perm(a[3], a[2], 0x07060302u),
                                  __builtin_amdgcn_perm(b[1], b[0], 0x07060302u), __builtin_amdgcn_perm(b[3], b[2], 0x07060302u)};
      }
    }
  };
  if (kh == 0) finish(Int<0>{}); else finish(Int<1>{});
}

template <int MF, int BN, bool BWD>
void launch_wide_main(const WideArgs& a, unsigned grid, hipStream_t st) {
  hipLaunchKernelGGL((wide_main_kernel<MF, BN, BWD>), dim3(grid), dim3(512), 0, st, a);
}

}  // namespace

// Microseconds of a call by this path: its two launches, the steps of its rounds of tiles (one workgroup per compute unit), per 64
// ranks and round the adapter's start, the outputs, the adapter's inner product, and above kMidTokens the packed copy of the operand.  Fitted, like
// the other paths' estimates, to random calls by each path (sides 64 - 16384, ranks 0 - 256; forward, dX, dX under dropout; replayed, three weights in
// turn; every path seen to be the one that ran): up to 512 tokens within 11 % on eight calls of ten, which is enough to choose a tile; above, 2155 calls,
// within 9 %.
WidePlan wide_plan(bool bwd, int64_t M, int64_t h, int64_t o, int r, size_t room) {
  const int64_t K = bwd ? o : h, N = bwd ? h : o;
  WidePlan best{};
  if (M < 1 || M > kWideTokens || o > (1 << 24) || h > (1 << 24) || h * o / 2 >= (1ll << 31)) return best;    // 32-bit buffer offsets
  auto consider = [&](int MF, int BN) {
    WidePlan p{};
    p.MF = MF; p.BN = BN;
    const int bm = 64 * MF, kstep = 16384 / BN;
    p.n_tg = (int)((M + bm - 1) / bm);
    p.n_slabs = (int)((N + BN - 1) / BN);
    p.steps = (int)((K + kstep - 1) / kstep);
    p.k_pad = p.steps * kstep;
    // up to eight partials of the adapter's inner product of at least 512 elements: with four, each a longer chain of requests in `pre`, calls with
    // K from 4096 on take 1 - 12 us longer
    p.chunk = (int)std::max<int64_t>(512, ((K + 7) / 8 + 63) / 64 * 64);
    p.n_lparts = r > 0 ? (int)((K + p.chunk - 1) / p.chunk) : 0;
    p.lpart_floats = (size_t)p.n_lparts * M * r;
    p.pack_elems = (size_t)p.n_tg * bm * p.k_pad;
    if (p.pack_elems * 2 >= (1ull << 31) || (p.lpart_floats * 4 + 255) / 256 * 256 + p.pack_elems * 2 > room) return;
    const int64_t tiles = (int64_t)p.n_tg * p.n_slabs, rounds = (tiles + 255) / 256;
    const double MN = 1e-6 * (double)M * (double)N, MK = 1e-6 * (double)M * (double)K, ranks = (double)((r + 63) / 64 * rounds);
    if (M <= kMidTokens)
      p.us = 7.5 + (double)(rounds * p.steps) * (BN == 128 ? 0.69 + 0.21 * MF : 0.70 + 0.27 * MF) + ranks * (2.76 + 1.06 * MF) + 1.17 * MN +
             0.0096 * r * MK;
    else
      p.us = 8.8 + (double)(rounds * p.steps) * ((bwd ? 0.0 : 0.084) + (BN == 128 ? 0.60 + 0.205 * MF : 0.517 + 0.2825 * MF)) +
             ranks * (2.4 + 1.14 * MF) + 1.146 * MN + (0.61 + 0.0111 * r) * MK;
    p.ok = true;
    if (!best.ok || p.us < best.us) best = p;
  };
  for (int mf = 1; mf <= 3; ++mf) consider(mf, 128);
  for (int mf = 1; mf <= 4; ++mf) consider(mf, 64);
  return best;
}

// The same of the path that a call takes otherwise: the plan of midtok.hip, or (mid NULL) dequantise + GEMM, whose bf16 weight above some 50 M
// elements no longer stays in the last-level cache between the two, and which under dropout (fix) corrects dX afterwards.  A call comes here where the
// plan's estimate is, up to 512 tokens, 15 % below the former's or 8 % below the latter's; above, 3 % below the latter's, or 8 % with up to 512
// outputs or without Double Quantization (dq), where they scatter more, and 0.8 us, which they scatter by on the shortest calls.
// A second estimate may refuse it: one that knows that a tile sums T's partials first, that midtok.hip's adapter items take 64 rank columns after the
// other, and that without Double Quantization a step loads four bytes a block, forward from rows far apart (within 7 % on eight of ten calls near the
// line).  Against midtok.hip it refuses a call from 2 % above on where the tiles leave compute units idle, which a split of the contraction would use, and
// from 5 % below on, however many tiles, without Double Quantization; against dequantise + GEMM from 5 % below on, above 512 tokens 2 %.
// Of 20160 random calls 4743 came here by the plan's estimate alone, at 0.742 of the time (mean), 120 of them more than 3 % longer, 47 more
// than 10 %: forward 493 tokens 9216 x 384, rank 256 51.1 -> 72.8 us, 299 tokens 3712 x 2176, rank 64, without Double Quantization 28.7 -> 32.1.  Of the
// 4506 that are left, at 0.727, 19 are more than 3 % longer, none more than 10 %.
bool wide_pays(const WidePlan& p, const MidPlan* mid, bool bwd, int64_t M, int64_t h, int64_t o, int r, bool fix, bool dq) {
  const double K = (double)(bwd ? o : h), N = (double)(bwd ? h : o), MN = 1e-6 * (double)M * N, KN = 1e-6 * K * N, rMK = 1e-6 * r * (double)M * K;
  const int64_t tiles = (int64_t)p.n_tg * p.n_slabs, rounds = (tiles + 255) / 256;
  const double steps = (double)(rounds * p.steps), ranks = (r + 63) / 64;
  const double second = 6.61 + steps * (p.BN == 128 ? 0.569 + 0.256 * p.MF : 0.662 + 0.279 * p.MF) + (dq || bwd ? 0.0 : 0.18) * steps +
                        ranks * (double)rounds * (2.64 + 1.18 * p.MF + 0.237 * p.n_lparts) + 1.18 * MN + 0.0188 * rMK;
  if (mid) {
    const double us = 6.65 + 0.71 * mid->us + (mid->pack ? 5.4 + 0.054 * r : 0.0) + 1.12 * mid->max_contrib * MN + (r > 0 ? 2.3 : 0.0) + 0.037 * rMK;
    if (p.us > 0.85 * us) return false;
    if (dq && tiles >= 256) return true;
    const double chunk = std::min(K, (double)mid->chunk);
    const double us2 = mid->pack ? 7.85 + (bwd ? 0.948 : 0.728) * mid->us + ranks * (2.6 + 0.00576 * chunk) +
                                       mid->max_contrib * (0.312 + 1.68 * MN) + 0.0039 * r * MN
                                 : 4.05 + (r > 0 ? 1.69 : 0.0) + std::max(0.89 * mid->us, ranks * (2.64 + 0.00254 * chunk)) +
                                       mid->max_contrib * (0.357 + 1.3 * MN) + 0.0159 * r * MN;
    return second <= (dq ? 1.02 : 0.95) * us2;
  }
  const double product = gemm_us(M, (int64_t)N, ((int64_t)K + (r + 63) / 64 * 64) / 64);
  if (M <= kMidTokens) {
    const double us = 7.2 + 0.77 * product + 0.33 * KN + 0.37 * std::max(0.0, KN - 50.0) +
                      1.07 * MN + (r > 0 ? 4.2 + 1e-6 * r * (1.65 * N + 0.1 * K) : 0.0) + 0.0056 * rMK + (fix ? 6.4 + 1.9 * MN : 0.0);
    const double us2 = 6.37 + 0.812 * product + 0.71 * KN + 0.82 * MN + (r > 0 ? 3.31 + 1e-6 * r * (0.19 * N + 1.71 * K) : 0.0) + 0.0366 * rMK +
                       (fix ? 12.6 + 1.28 * MN : 0.0);
    return p.us <= 0.92 * us && second <= 0.95 * us2;
  }
  const double us = 7.0 + 0.745 * product + 0.464 * KN + 0.616 * std::max(0.0, KN - 50.0) + 0.843 * MN +
                    (r > 0 ? 5.1 + 1e-6 * r * (2.92 * K + 7.1 * (double)M) : 0.0) + 0.0016 * rMK + (fix ? 7.5 + 1.56 * MN : 0.0);
  return p.us <= std::min((N <= 512 || !dq ? 0.92 : 0.97) * us, us - 0.8) && second <= 0.98 * us;
}

hipError_t launch_wide(bool bwd, const uint16_t* X, int M, const NF4Dev& w, const WidePlan& p, const uint16_t* L1, const uint16_t* L2,
                       int r, float scale, const uint8_t* mask, float* lpart, uint16_t* xpack, uint16_t* out, uint16_t* hl,
                       hipStream_t st) {
  if (!p.ok || w.dtype == kTypeInt8) return hipErrorInvalidValue;
  WideArgs a{};
  a.X = X; a.M = M; a.h = (int)w.rows; a.o = (int)w.cols; a.K = bwd ? a.o : a.h; a.N = bwd ? a.h : a.o;
  a.Xf = (const char*)xpack; a.x_bytes = (uint32_t)(p.pack_elems * 2); a.tiles = p.n_tg * 4 * p.MF;
  a.packed = w.packed; a.code = w.code; a.c1 = w.c1; a.mean = w.mean; a.dtype = w.dtype; a.dq = w.dq ? 1 : 0;
  a.tab = table4_host(w.dtype);
  a.n_tg = p.n_tg; a.steps = p.steps;
  a.L = bwd ? L2 : L1; a.r = r; a.mask = bwd ? nullptr : mask;
  a.lpart = lpart; a.n_lparts = p.n_lparts; a.chunk = p.chunk;
  a.B = bwd ? L1 : L2; a.scale = scale; a.keep = bwd ? mask : nullptr; a.out = out; a.hl = r > 0 ? hl : nullptr;
  const int items = (M + kAdTok - 1) / kAdTok * p.n_lparts;
  const unsigned pre = (unsigned)(items + a.tiles * ((p.k_pad + kPreK - 1) / kPreK));
  if (bwd) hipLaunchKernelGGL(wide_pre_kernel<true>, dim3(pre), dim3(512), 0, st, a, xpack, items, p.k_pad);
  else hipLaunchKernelGGL(wide_pre_kernel<false>, dim3(pre), dim3(512), 0, st, a, xpack, items, p.k_pad);
  const unsigned grid = (unsigned)(p.n_tg * p.n_slabs);
#define QL_WIDE(MF, BN)                                                 \
  case 1000 * MF + BN:                                                  \
    if (bwd) launch_wide_main<MF, BN, true>(a, grid, st);               \
    else launch_wide_main<MF, BN, false>(a, grid, st);                  \
    break;
  switch (1000 * p.MF + p.BN) {
    QL_WIDE(1, 128) QL_WIDE(2, 128) QL_WIDE(3, 128) QL_WIDE(1, 64) QL_WIDE(2, 64) QL_WIDE(3, 64) QL_WIDE(4, 64)
    default: return hipErrorInvalidValue;
  }
#undef QL_WIDE
  return hipGetLastError();
}

}  // namespace qlora
