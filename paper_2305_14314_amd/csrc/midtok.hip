// Forward and input gradient of the QLoRA linear layer at tens to hundreds of tokens (arXiv 2305.14314, Eq. 5 / Eq. 6):
// the packed weight is read once per group of up to 128 tokens, decoded in registers to the bf16 values of the
// standalone doubleDequant and multiplied on the spot, so no bf16 copy of the weight is ever written.
//
// Why its own path: with 256 x 256 tiles a product of a few hundred tokens has 4 .. 100 tiles for 256 compute units, and
// the pass that dequantises the weight moves five times the bytes of the packed weight (2.5 against 0.5 per weight).
// Whole forward call, dequantise + GEMM against this: 4096 x 11008 at 40 tokens 108 -> 20 us.  With
// many tokens to a weight the form of widetok.hip, whose waves share the decode, is the faster one of the two (figures there).
//
// Two or three launches on the caller's stream:
//   pre       (where the plan finds it worth a launch) the token operand in MFMA-fragment order, so that the main kernel's operand
//             loads are whole contiguous kilobytes; beside it the partial sums of the adapter's inner product T = X L1 (U = dY L2^T)
//   main      the products of all tiles (16 MF tokens x 128 outputs) are one line of units (KW steps of the contraction),
//             cut into equal ranges, one per workgroup: whatever the shape, every compute unit multiplies the same
//             amount.  Within a tile a workgroup's waves take the steps in turn, each with the whole tile in
//             accumulators, and are summed through LDS into one fp32 partial tile.  No barrier in the loop.  Without a pre
//             launch the adapter's partial sums are extra workgroups here and the operand is read as it lies.
//   finalize  out = bf16( sum of a tile's partials + s * (sum of T's partials) * L2 ), in a fixed order, one rounding; T
//             as a [hi | lo] pair of bf16 operands (16 significant bits) on MFMA; writes T_save
//
// Lane layout of a step (MFMA 16x16x32, tokens = rows of A, weights = columns of B; lane = 16 g + i):
//   forward   32 weight rows x 128 columns: lane (i, g) holds packed dword i (columns 8i .. 8i+7) of rows 8g .. 8g+7;
//             phase e (0 .. 7) multiplies columns 8i + e
//   backward  128 weight rows x 64 columns: lane (i, g) holds columns 16g .. 16g+15 of rows 8i .. 8i+7; phase (t, u)
//             multiplies dword t of row 8i + u: columns 16g + 8t .. +7
// Either way accumulator column e (u) of lane (i, g) is output 8i + e, so a lane ends with eight neighbouring outputs.
#include <algorithm>
#include <type_traits>

#include "adapter_partial.hpp"
#include "fewtok_common.hpp"

namespace qlora {

namespace {

using few::kLutCopies;
using few::kLutBytes;
using few::init_pair_lut;
using few::pair_lookup_b;
using few::work_index;

constexpr int kSlab = 128;                   // outputs per workgroup
// LDS map: the decode table stays for all segments of a workgroup; beside it the cross-wave sums
constexpr int kRedMid = 64 * 1024, kMRed = kLutBytes;
constexpr int kMUnit = kMRed + kRedMid;      // float[256]
constexpr int kMStrip = kMUnit + 1024;       // float[8 waves][128]
constexpr int kMidSmem = kMStrip + 4 * 1024;
static_assert(kMidSmem <= 160 * 1024, "LDS map");

struct MidArgs {
  const uint16_t* X;                         // token operand as it lies: X (M x h) or dY (M x o)
  const char* Xf;                            // what the main loop reads: X, or its copy in fragment order
  uint32_t x_bytes;                          // of Xf
  int x_step;                                // bytes between two 32-wide (forward) / 64-wide (backward) steps of Xf
  int x_sub;                                 // backward: bytes between the two phases t of a step
  int M, h, o, K, N;                         // K: contraction length, N: outputs
  const uint8_t* packed; const uint8_t* code; const float* c1; const float* mean;
  int dtype, dq; Table4 tab;
  float* part;                               // [contributor][M][N]
  int n_tg, n_slabs, steps;
  MidLine line;
  const uint16_t* L; int r;                  // adapter's inner matrix: L1 (h x r) or L2 (r x o)
  const uint8_t* mask;                       // keep-bits of X (forward), or NULL
  float* lpart;                              // [n_lparts][M][r]
  int n_lparts, chunk, n_items;              // adapter items this launch computes (32 tokens x chunk), first in the work list
};

// ---- token operand in fragment order, and the adapter's partials --------------------------------------------------------
// Fragment of 16 tokens x 32 contraction elements = 1 KB: lane (i, g) at byte 16 (16 g + i) holds token i's eight elements
// of k group g.  Forward: [32-wide step][token tile].  Backward: [64-wide step][phase t][token tile], group g of phase t
// being columns 16g + 8t .. +7.  Tokens beyond M are zeros.
// A workgroup of 8 waves packs 16 tokens x 512 contraction elements, a wave 64 of them: two fragments, no index arithmetic
// beyond one division per workgroup (with a 64-bit division per
// 16 bytes and adapter partials by 64-bit addresses the launch took 9.8 us for 512 x 4096 at rank 64, 8.0 now; 333 x 5120 8.3 -> 6.1).
constexpr int kPreK = 512;
template <bool BWD>
__global__ __launch_bounds__(512) void mid_pre_kernel(const MidArgs p, uint16_t* __restrict__ Xp, int tiles, int items) {
  __shared__ __attribute__((aligned(16))) char smem[8 * kAdTok * 64 * 4];
  if ((int)blockIdx.x < items) {
    if (!BWD && p.mask) adapter_partial<8, BWD, !BWD>(p, blockIdx.x, (float*)smem);
    else adapter_partial<8, BWD, false>(p, blockIdx.x, (float*)smem);
    return;
  }
  const int n_kb = (p.K + kPreK - 1) / kPreK, at = (int)blockIdx.x - items;
  const int tile = at / n_kb, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int k0 = (at - tile * n_kb) * kPreK + wave * 64, i = lane & 15, g = lane >> 4;
  if (k0 >= p.K) return;
  const int m = 16 * tile + i;
  const uint16_t* src = p.X + (int64_t)(m < p.M ? m : p.M - 1) * p.K + k0 + (BWD ? 16 : 8) * g;
  u32x4 v[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) v[t] = *(const u32x4*)(src + (BWD ? 8 : 32) * t);
#pragma unroll
  for (int t = 0; t < 2; ++t)
    *(u32x4*)(Xp + (((int64_t)(k0 >> 5) + t) * tiles + tile) * 512 + 8 * lane) = m < p.M ? v[t] : u32x4{0u, 0u, 0u, 0u};
}

// ---- main ---------------------------------------------------------------------------------------------------------------
// A raw buffer resource over `bytes` bytes at `base` (loads beyond them return zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t mid_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}

template <int N> using Int = std::integral_constant<int, N>;

template <bool BWD> struct MidW;               // raw loads of a step
template <> struct MidW<false> { uint32_t pk[8]; uint32_t code; float c1; };
template <> struct MidW<true> { uint32_t pk[8][2]; uint32_t code[2]; float c1[2]; };

// What bounds it: with one wave per SIMD (KW = 4) the wave's instruction issue.  An MFMA 16x16x32 occupies the matrix pipe
// for 16 cycles and comes with 3.2 other instructions (2.1 vector-ALU: address permute, two products and a rounding per
// pair of weights and eight MFMAs; 0.56 lookups; 0.28 loads), measured 1.0 us per 64 of them (8 token tiles; the plain GEMM,
// with 0.9 others, takes 0.6).  Without the lookups the kernel is 5 % faster, with its operands in L2 not at all.  The
// fixed part of a call is 12 us: launch, first loads, the ends of segments (16 MB of partials).  Two waves per SIMD with
// tiles of 64 tokens (KW = 8) take 1.37 us for the same work -- every weight is decoded twice as often -- but 7 us of fixed
// part.  Flat-address loads (a third of the loop's instructions) cost 5 - 10 %, a wait per lookup instead of one per group
// the same, idle cycles behind every accumulator's statement instead of once 2.7 us per segment.
//
// PACK: the token operand is in fragment order, zero-padded to whole tiles (always so in the backward direction).
template <int MF, int KW, bool BWD, bool PACK>
__global__ __launch_bounds__(KW * 64) void mid_main_kernel(const MidArgs p) {
  constexpr int NT = KW * 64;
  static_assert(PACK || !BWD, "the backward operand is always packed");
  __shared__ __attribute__((aligned(256))) char smem[kMidSmem];
  const int work = work_index();
  if constexpr (!PACK) {
    if (work < p.n_items) {
      if (!BWD && p.mask) adapter_partial<KW, BWD, !BWD>(p, work, (float*)smem);
      else adapter_partial<KW, BWD, false>(p, work, (float*)smem);
      return;
    }
  }
  f32x2* lut2 = (f32x2*)smem;
  float* unit = (float*)(smem + kMUnit);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const uint32_t lane_off = 8u * (uint32_t)(lane & (kLutCopies - 1));
  float* strip = (float*)(smem + kMStrip) + wave * 128;
  const int rho = work - p.n_items;
  const float mean = p.dq ? *p.mean : 0.0f;
  const int bpr = p.o >> 6;
  const int rowb = p.o >> 1;                                 // bytes per packed row
  // without Double Quantization c1 holds one constant per block, and the code (any valid byte) is not used
  const __amdgpu_buffer_rsrc_t code_rsrc = mid_rsrc(p.dq ? p.code : p.packed, (uint32_t)p.h * (uint32_t)bpr);
  const uint32_t n_blocks = (uint32_t)p.h * (uint32_t)bpr;
  const __amdgpu_buffer_rsrc_t c1_rsrc = mid_rsrc(p.c1, 4u * (p.dq ? (n_blocks + 255u) / 256u : n_blocks));
  const int c1_shift = p.dq ? 8 : 0, code_w = p.dq ? 1 : 0;

  // The table comes before the first loads: behind them it would wait until the queues of the memory pipe have room for all
  // of their requests, i.e. for the first data (ready 5 - 7 us into the kernel that way, 1.2 so).
  init_pair_lut<NT>(lut2, unit, p.dtype, p.tab);
  const int u_end = p.line.start(rho + 1);
  for (int u = p.line.start(rho); u < u_end;) {
  // ---- one segment: a run of units of one tile ---------------------------------------------------------------------
  const int tile = u / p.line.ups, u0 = u - tile * p.line.ups;
  const int u1 = u0 + (u_end - u) < p.line.ups ? u0 + (u_end - u) : p.line.ups;
  u += u1 - u0;
  const int tg = tile % p.n_tg, slab = tile / p.n_tg;
  const int s_begin = u0 * KW, s_end = u1 * KW < p.steps ? u1 * KW : p.steps;
  const int m0 = tg * 16 * MF, n0 = slab * kSlab;

  // All loads of the loop are raw buffer loads: a resource over the whole tensor, a per-lane offset that does not change in
  // a segment and a scalar offset that the step moves, so that a load costs one vector-memory and at most one scalar
  // instruction (with flat addresses the address arithmetic was a third of the loop's instructions).
  // token operand, per 16-token tile; packed: tiles are 1 KB apart
  const __amdgpu_buffer_rsrc_t x_rsrc = mid_rsrc(p.Xf, p.x_bytes);
  uint32_t x_off[PACK ? 1 : MF];
  if constexpr (PACK) x_off[0] = (uint32_t)((m0 >> 4) * 1024 + lane * 16);
  else {
#pragma unroll
    for (int f = 0; f < MF; ++f) {
      const int m = m0 + 16 * f + i;
      x_off[f] = (uint32_t)(m < p.M ? m : p.M - 1) * (uint32_t)(2 * p.K) + 16u * (uint32_t)g;
    }
  }
  auto load_x = [&](u32x4 (&x)[MF], int st, int t) {
    const int sc = st < s_end ? st : s_end - 1;
    const int so = sc * p.x_step + (BWD ? t * p.x_sub : 0);
#pragma unroll
    for (int f = 0; f < MF; ++f)
      x[f] = PACK ? __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, x_off[0] + (f & 3) * 1024, so + (f >> 2) * 4096, 0)
                  : __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, x_off[PACK ? 0 : f], so, 0);
  };

  // Weights and constants.
  // forward: this lane's dword of a row, and the constant it decodes: row lane / 2, block lane % 2 of the slab (both blocks
  // of a slab lie in one group of the column-group-major order)
  // backward: weight rows 8i .. 8i+7 of the slab (h % 64 == 0: inside or outside together; outside: the slab's first
  // rows), and the constants of rows lane and lane + 64
  const bool col_ok = n0 + 8 * i < p.o, row_ok = n0 + 8 * i < p.h;
  const uint32_t w_lane = BWD ? (uint32_t)(row_ok ? 8 * i : 0) * (uint32_t)rowb + 8u * (uint32_t)g
                              : (uint32_t)(8 * g * rowb + (col_ok ? 4 * i : 0));
  // the packed weight moves through the resource's base: a step's rows (32, or 128 of the slab) lie within w_span bytes of it
  const uint8_t* w_slab = p.packed + (BWD ? (int64_t)n0 * rowb : n0 >> 1);
  const uint32_t w_span = (BWD ? 128u : 32u) * (uint32_t)rowb;
  const int fblk = n0 >> 6, fb = fblk + (lane & 1) < bpr ? (lane & 1) : 0;
  const int fw = (fblk & ~3) + 4 <= bpr ? 4 : bpr - (fblk & ~3);
  const uint32_t code_lane = (uint32_t)(((lane >> 1) * fw + (fblk & 3) + fb) * code_w);
  const uint32_t c1_lane = (uint32_t)((lane >> 1) * bpr + fblk + fb);
  const int code_slab = 4 * p.h * (fblk >> 2) * code_w;
  const int half2 = n0 + 64 < p.h ? 64 : 0;                  // backward: the slab's second 64 rows, if they exist
  auto load_w = [&](MidW<BWD>& s, int st) {
    const int sc = st < s_end ? st : s_end - 1;
    const __amdgpu_buffer_rsrc_t w_rsrc = mid_rsrc(w_slab + (int64_t)sc * (BWD ? 32 : 32 * rowb), w_span);
    if constexpr (!BWD) {
#pragma unroll
      for (int j = 0; j < 8; ++j) s.pk[j] = __builtin_amdgcn_raw_buffer_load_b32(w_rsrc, w_lane, j * rowb, 0);
      const uint32_t idx = (uint32_t)(sc * 32) * (uint32_t)bpr + c1_lane;
      s.code = __builtin_amdgcn_raw_buffer_load_b8(code_rsrc, code_lane, code_slab + sc * 32 * (fw * code_w), 0);
      s.c1 = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(c1_rsrc, (idx >> c1_shift) * 4u, 0, 0));
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(w_rsrc, w_lane, q * rowb, 0));
        s.pk[q][0] = v[0]; s.pk[q][1] = v[1];
      }
      const int G = sc >> 2, w = 4 * G + 4 <= bpr ? 4 : bpr - 4 * G;               // block sc of a row
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int row0 = n0 + (c ? half2 : 0);
        const uint32_t idx = (uint32_t)row0 * (uint32_t)bpr + (uint32_t)sc + (uint32_t)(lane * bpr);
        s.code[c] = __builtin_amdgcn_raw_buffer_load_b8(code_rsrc, (uint32_t)(lane * w * code_w),
                                                        (4 * p.h * G + row0 * w + (sc & 3)) * code_w, 0);
        s.c1[c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(c1_rsrc, (idx >> c1_shift) * 4u, 0, 0));
      }
    }
  };

  f32x4 acc[MF][8];
#pragma unroll
  for (int f = 0; f < MF; ++f)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[f][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (KW == 4) {                                   // see QL_MID_MFMA: zeroing well ahead of the first product
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int e = 0; e < 8; ++e) asm volatile("" : "+a"(acc[f][e]));
    asm volatile("s_nop 3");                                 // volatile statements keep their order: zeroing, wait, first product
  }
  // One wave per SIMD (KW = 4): MFMAs as volatile asm on accumulators pinned to AGPRs (left to itself the compiler copies
  // a third of them between the register files every step).  Asm MFMAs are invisible to the hazard recogniser: an operand
  // written by the vector ALU needs two wait states, so a group's fragments are complete two MFMAs before it begins.
#define QL_MID_MFMA(x_, w_, f_, e_)                                                                                    \
  if constexpr (KW == 4) {                                                                                             \
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[f_][e_]) : "v"(x_), "v"(w_));                    \
  } else {                                                                                                             \
    acc[f_][e_] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x_), __builtin_bit_cast(bf16x8, w_), \
                                                         acc[f_][e_], 0, 0, 0);                                        \
  }

  // A step is kGroups groups of two weight fragments (eight table lookups per lane).  While group G is multiplied, group
  // G + 1 is decoded and the lookups of group G + 2 are issued, a few instructions behind every MFMA, across step
  // boundaries: the matrix pipe never waits for a burst of vector work.  Three steps of weights and three fragment sets of
  // the token operand are in registers: a load has two steps (fragment sets) to arrive.
  constexpr int kGroups = BWD ? 8 : 4, kPhases = BWD ? 2 : 1, R = KW == 8 && MF >= 3 ? 2 : 3;
  MidW<BWD> wb[R];
  u32x4 xb[R][MF];
  const int st0 = s_begin + wave;
#pragma unroll
  for (int d = 0; d < R; ++d) {                              // in the order of the loop: its waits count outstanding loads
    load_w(wb[d], st0 + d * KW);
    __builtin_amdgcn_sched_barrier(0);
    load_x(xb[d], st0 + (d / kPhases) * KW, d % kPhases);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();

  float c2[R][8];                                            // constants of the step being decoded / of the next
  f32x2 q[2][8];                                             // looked-up pairs: of the group being decoded / landing
  u32x4 wf[2][2];                                            // fragments being multiplied / being decoded
  // the constants of a step: decoded once per row and block (two separately rounded fp32 steps), exchanged through a
  // wave-private strip; c2[.][j] belongs to this lane's row j
  auto constant = [&](uint32_t cd, float c1) {
    const float v = __fadd_rn(__fmul_rn(unit[cd], c1), mean);
    return p.dq ? v : c1;
  };
  auto constants = [&](const MidW<BWD>& s, float (&o)[8]) {
    const f32x4* sp;
    if constexpr (!BWD) {
      strip[(lane & 1) * 32 + (lane >> 1)] = constant(s.code, s.c1);
      sp = (const f32x4*)&strip[(i >> 3) * 32 + 8 * g];
    } else {
#pragma unroll
      for (int c = 0; c < 2; ++c) strip[c * 64 + lane] = constant(s.code[c], s.c1[c]);
      sp = (const f32x4*)&strip[8 * i];
    }
    const f32x4 ca = sp[0], cb = sp[1];
#pragma unroll
    for (int j = 0; j < 4; ++j) { o[j] = ca[j]; o[4 + j] = cb[j]; }
  };
  auto lookup = [&](const MidW<BWD>& s, int G, int l) -> f32x2 {
    if constexpr (!BWD) return pair_lookup_b(lut2, s.pk[l], lane_off, G);
    else return pair_lookup_b(lut2, s.pk[2 * (G & 3) + (l >> 2)][G >> 2], lane_off, l & 3);
  };
  // factor `half` (0, 1) of dword d % 4 of fragment d / 4 of group G
  auto product = [&](const f32x2 (&qq)[8], const float (&c)[8], int G, int d, int half) -> float {
    if constexpr (!BWD) {
      const int j = 2 * (d & 3) + half;
      return __fmul_rn(qq[j][d >> 2], c[j]);
    } else {
      return __fmul_rn(qq[d][half], c[2 * (G & 3) + (d >> 2)]);
    }
  };
  // Group G (0 .. kGroups - 1) of step number S of the unrolled loop (compile-time): multiplies the fragments in wf[G & 1].
  auto group = [&](auto Sc, auto Gc, const int st) {
    constexpr int S = decltype(Sc)::value, G = decltype(Gc)::value;
    constexpr int G1 = (G + 1) % kGroups, S1 = G + 1 < kGroups ? S : S + 1;      // decoded meanwhile
    constexpr int G2 = (G + 2) % kGroups, S2 = G + 2 < kGroups ? S : S + 1;      // looked up meanwhile
    constexpr int ph = S * kPhases + (BWD ? G >> 2 : 0);     // phase of the unrolled loop: fragment set ph % R
    if (G == kGroups - 2) constants(wb[(S + 1) % R], c2[(S + 1) % R]);
    else if (2 * MF >= 12) __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): one wait for the eight lookups of the group before
    // Behind MFMA k: one of the eight lookups (early, so that all have landed when the next group waits once for them) and
    // the share of the eight dwords of the next fragments, one third (a product or the rounding) at a time.
    float pr[2];
    int done = 0;
#pragma unroll
    for (int k = 0; k < 2 * MF; ++k) {
      const int v = k / MF, f = k % MF;
      QL_MID_MFMA(xb[ph % R][f], wf[G & 1][v], f, BWD ? 2 * (G & 3) + v : 2 * G + v)
      constexpr int kPerMfma = 2 * MF >= 12 ? 1 : (8 + 2 * MF - 1) / (2 * MF);   // lookups behind an MFMA
#pragma unroll
      for (int l = k * kPerMfma; l < (k + 1) * kPerMfma && l < 8; ++l) q[G & 1][l] = lookup(wb[S2 % R], G2, l);
      constexpr int kSlots = 2 * MF - 2 > 0 ? 2 * MF - 2 : 1;   // the last two MFMAs are the wait states before the next group
      const int upto = (24 * (k + 1)) / kSlots < 24 ? (24 * (k + 1)) / kSlots : 24;
#pragma unroll
      for (int it = 0; it < 24; ++it) {
        if (it < done || it >= upto) continue;
        const int d = it / 3;
        if (it % 3 < 2) pr[it % 3] = product(q[(G + 1) & 1], c2[S1 % R], G1, d, it % 3);
        else wf[(G + 1) & 1][d >> 2][d & 3] = pack_bf16x2(pr[0], pr[1]);
      }
      done = upto;
      __builtin_amdgcn_sched_barrier(0);
    }
    if (G == kGroups - 3) load_w(wb[S % R], st + R * KW);    // its last lookups have been issued
    if ((G & 3) == 3) {                                      // the phase's fragment set is free: the set R phases ahead
      constexpr int pn = ph % kPhases + R;
      load_x(xb[ph % R], st + (pn / kPhases) * KW, pn % kPhases);
    }
  };
  auto step = [&](auto S, const int st) {
    group(S, Int<0>{}, st); group(S, Int<1>{}, st); group(S, Int<2>{}, st); group(S, Int<3>{}, st);
    if constexpr (BWD) {
      group(S, Int<4>{}, st); group(S, Int<5>{}, st); group(S, Int<6>{}, st); group(S, Int<7>{}, st);
    }
  };

  // Two waves per SIMD (KW = 8): the other wave fills the gaps; only the lookups run a group ahead.
  auto step8 = [&](auto Sc, const int st) {
    constexpr int S = decltype(Sc)::value;
    constants(wb[S], c2[0]);
    f32x2 qn[8];
#pragma unroll
    for (int l = 0; l < 8; ++l) qn[l] = lookup(wb[S], 0, l);
#pragma unroll
    for (int G = 0; G < kGroups; ++G) {
      f32x2 qc[8];
#pragma unroll
      for (int l = 0; l < 8; ++l) qc[l] = qn[l];
      if (G + 1 < kGroups) {
#pragma unroll
        for (int l = 0; l < 8; ++l) qn[l] = lookup(wb[S], G + 1, l);
      }
      __builtin_amdgcn_sched_barrier(0);
      u32x4 w[2];
#pragma unroll
      for (int d = 0; d < 8; ++d) w[d >> 2][d & 3] = pack_bf16x2(product(qc, c2[0], G, d, 0), product(qc, c2[0], G, d, 1));
      const int ph = S * kPhases + (BWD ? G >> 2 : 0);
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int f = 0; f < MF; ++f)
          acc[f][BWD ? 2 * (G & 3) + v : 2 * G + v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, xb[ph % R][f]), __builtin_bit_cast(bf16x8, w[v]), acc[f][BWD ? 2 * (G & 3) + v : 2 * G + v], 0, 0, 0);
      if ((G & 3) == 3) load_x(xb[ph % R], st + (ph % kPhases + R) / kPhases * KW, (ph % kPhases + R) % kPhases);
    }
    load_w(wb[S], st + R * KW);
  };
  if constexpr (KW == 8) {
    int st = st0;
#pragma unroll 1
    for (; st + (R - 1) * KW < s_end; st += R * KW) {
      step8(Int<0>{}, st);
      step8(Int<1>{}, st + KW);
      if constexpr (R == 3) step8(Int<2>{}, st + 2 * KW);
    }
    if (st < s_end) step8(Int<0>{}, st);
    if constexpr (R == 3)
      if (st + KW < s_end) step8(Int<1>{}, st + KW);
  } else {
  if (st0 < s_end) {
    constants(wb[0], c2[0]);
#pragma unroll
    for (int l = 0; l < 8; ++l) q[0][l] = lookup(wb[0], 0, l);
#pragma unroll
    for (int l = 0; l < 8; ++l) q[1][l] = lookup(wb[0], 1, l);
#pragma unroll
    for (int d = 0; d < 8; ++d)
      wf[0][d >> 2][d & 3] = pack_bf16x2(product(q[0], c2[0], 0, d, 0), product(q[0], c2[0], 0, d, 1));
    if constexpr (KW == 4) asm volatile("s_nop 3" : "+v"(wf[0][0]), "+v"(wf[0][1]));   // wait states, as between the groups
  }
  int st = st0;
#pragma unroll 1
  for (; st + (R - 1) * KW < s_end; st += R * KW) {
    step(Int<0>{}, st);
    step(Int<1>{}, st + KW);
    if constexpr (R == 3) step(Int<2>{}, st + 2 * KW);
  }
  if (st < s_end) step(Int<0>{}, st);
  if constexpr (R == 3)
    if (st + KW < s_end) step(Int<1>{}, st + KW);
  }
  if constexpr (KW == 4) {                                   // an MFMA's result may be read by the vector ALU 18 wait states later
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3");
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int e = 0; e < 8; ++e) asm volatile("" : "+a"(acc[f][e]));   // every read of an accumulator comes after its statement
  }
#undef QL_MID_MFMA

  // ---- sum over the waves, PH token tiles at a time; thread -> (token, four neighbouring outputs) -------------------
  constexpr int PH = kRedMid / (KW * 8192);                  // 8 KB per wave and token tile
  float* out = p.part + (int64_t)(rho - p.line.rho_of(tile * p.line.ups)) * p.M * p.N;
#pragma unroll
  for (int f0 = 0; f0 < MF; f0 += PH) {
    __syncthreads();                                         // the previous tiles (the previous segment) are done with
    float* my = (float*)(smem + kMRed) + wave * (PH * 2048);
#pragma unroll
    for (int f = f0; f < f0 + PH && f < MF; ++f)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int eh = 0; eh < 2; ++eh)
          *(f32x4*)(my + ((((f - f0) * 4 + v) * 2 + eh) * 64 + lane) * 4) =
              f32x4{acc[f][4 * eh][v], acc[f][4 * eh + 1][v], acc[f][4 * eh + 2][v], acc[f][4 * eh + 3][v]};
    __syncthreads();
    const int n_idx = (MF - f0 < PH ? MF - f0 : PH) * 512;
    for (int idx = threadIdx.x; idx < n_idx; idx += NT) {
      const int eh = idx & 1, ln = (idx >> 1) & 63, fv = idx >> 7;
      const float* src = (const float*)(smem + kMRed) + ((fv * 2 + eh) * 64 + ln) * 4;
      f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < KW; ++w) t += *(const f32x4*)(src + w * (PH * 2048));
      const int m = m0 + 16 * (f0 + (fv >> 2)) + 4 * (ln >> 4) + (fv & 3), n = n0 + 8 * (ln & 15) + 4 * eh;
      if (m < p.M && n < p.N) *(f32x4*)(out + (int64_t)m * p.N + n) = t;
    }
  }
  }                                                          // segment
}

// ---- finalize -------------------------------------------------------------------------------------------------------------
// Workgroup: 16 TF tokens x 256 outputs, a wave 64 of them; lane (i, g) owns outputs 4i .. 4i+3 of tokens 4g + v.
// Up to kLeanBlocks workgroups everything a workgroup needs is requested at once (see below); with more, occupancy hides the
// round trips and the registers for that cost more than they save (LEAN).  Whole calls, us, all at once / lean: 4096 x 11008
// forward at 40 tokens (129 workgroups) 20.5 / 21.5, 4096 x 4096 at 128 (128) 23.6 / 24.2; dX 4096 x 4096 at 512 (512)
// 41.8 / 40.9, forward 5120 x 13824 at 333 (1134) 87.4 / 84.6.
constexpr unsigned kLeanBlocks = 256;
struct MidFinArgs {
  const float* part; int M, N;
  MidLine line; int MF, n_tg;                // which contributors a tile has
  const float* lpart; int n_lparts, r;
  const uint16_t* B;                         // adapter's outer matrix: L2 (r x N) forward, L1 (N x r) backward
  float scale;
  uint16_t* out; uint16_t* hl;
  const uint8_t* mask;                       // backward under LoRA dropout: keep-bits of the output elements, or NULL
};

// Quadruples of ranks of a token, as a shift, and how many of them a thread of a finalize workgroup sums together: one by one up
// to rank 64 and at few tokens, else all of its two or up to four.  (A batch of requests for each, one after the other, found by
// divisions, and the tokens past M summed too: forward calls of 2 tokens 256 x 1344 at rank 256 19.1 us, 47 tokens 256 x 7296 at
// rank 256 22.4, 25 tokens 512 x 2048 at rank 128 13.3, 39 tokens 2944 x 1280 at rank 128 17.6; now 17.2, 20.4, 12.2, 17.1 -- the last 17.8
// with four quadruples per thread where there are two.)
__host__ __device__ inline int mid_quad_shift(int r) { return r <= 32 ? 3 : r <= 64 ? 4 : r <= 128 ? 5 : 6; }
inline int mid_quads(int M, int r) {
  const int n = std::min(M, 16) << mid_quad_shift(r);
  return n <= 256 ? 1 : n <= 512 ? 2 : 4;
}

// TERMS: bf16 terms of T.  Two carry 16 significant bits; at few tokens, where the streaming kernels multiply the fp32 value, three
// hold it whole (3 x 8 bits).
// TI: quadruples of T per thread that are summed together (mid_quads).
template <int TF, bool BWD, bool LEAN, int TERMS, int TI>
__global__ __launch_bounds__(256) void mid_finalize_kernel(const MidFinArgs p) {
  static_assert(LEAN || TF == 1, "two token tiles only where there are many workgroups");
  constexpr int kPitch = 256 + 8;
  __shared__ __attribute__((aligned(16))) uint16_t Tp[TERMS][16 * TF * kPitch];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.y * 16 * TF;
  const int nb = blockIdx.x * 256 + wave * 64;
  const bool n_ok = nb < p.N;                                // N % 64 == 0: a wave's outputs are inside or outside together
  const int n = (n_ok ? nb : 0) + 4 * i;

  // What a workgroup waits for is memory round trips: the partials of T, the first fragments of the outer matrix and the
  // first two partials of the tile are requested together, without branches between them (clamped addresses).
  // T in quadruples of ranks: number idx is quadruple idx % 2^qs of token idx / 2^qs (past the rank zeros; rows of tokens >= M stay
  // as they are and only reach outputs that are not stored).  LB / TI partials of TI quadruples per round trip.
  const int r4 = p.r >> 2, qs = mid_quad_shift(p.r), n_idx = (p.M - m0 < 16 * TF ? p.M - m0 : 16 * TF) << qs;
  constexpr int LB = LEAN ? 4 : 8, TQ = LB / TI;             // partials of T in flight
  f32x4 lp[LB];
  uint32_t off[TI];
  auto t_load = [&](int idx, int q0) {
#pragma unroll
    for (int k = 0; k < TI; ++k) {
      const int at = TI == 1 || idx + 256 * k < n_idx ? idx + 256 * k : 0, c = at & ((1 << qs) - 1);
      off[k] = (uint32_t)((m0 + (at >> qs)) * p.r + (c < r4 ? 4 * c : 0));
    }
#pragma unroll
    for (int k = 0; k < LB; ++k) {
      const int q = q0 + k % TQ;
      lp[k] = *(const f32x4*)(p.lpart + (int64_t)(q < p.n_lparts ? q : p.n_lparts - 1) * (p.M * p.r) + off[k / TQ]);
    }
  };
  constexpr int RB = LEAN ? 1 : 2;                           // steps of 32 ranks in flight
  struct OutFrag { u32x4 w[4]; };                            // forward: 8 rows x 4 columns as loaded; backward: [e], ranks of output 4i + e
  OutFrag bf[RB];
  auto b_load = [&](OutFrag& o, int t0) {
    if (!BWD) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = t0 + 8 * g + j;
        const uint2 v = *(const uint2*)(p.B + (int64_t)(t < p.r ? t : 0) * p.N + n);
        o.w[j >> 1][2 * (j & 1)] = t < p.r ? v.x : 0u;
        o.w[j >> 1][2 * (j & 1) + 1] = t < p.r ? v.y : 0u;
      }
    } else {
      const bool ok = t0 + 8 * g < p.r;                      // r % 16 == 0: a lane's 8 ranks are inside or outside together
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const u32x4 v = *(const u32x4*)(p.B + (int64_t)(n + e) * p.r + (ok ? t0 + 8 * g : 0));
        o.w[e] = ok ? v : u32x4{0u, 0u, 0u, 0u};
      }
    }
  };
  if (p.r > 0) {                                             // uniform
    t_load((int)threadIdx.x < n_idx ? threadIdx.x : 0, 0);
#pragma unroll
    for (int k = 0; k < RB; ++k) b_load(bf[k], 32 * k);
  }
  // a wave's outputs lie in one slab, the workgroup's tokens in one token group (per 16-token tile)
  int contrib[TF];
#pragma unroll
  for (int f = 0; f < TF; ++f) {
    const int tt = (m0 >> 4) + f, tile = ((n_ok ? nb : 0) / kSlab) * p.n_tg + (tt * 16 < p.M ? tt / p.MF : 0);
    contrib[f] = p.line.contributors(tile);
  }
  const int most = TF == 2 ? max(contrib[0], contrib[TF - 1]) : contrib[0];
  constexpr int CB = LEAN ? 1 : 2;                           // partials of the tile in flight
  f32x4 sum[TF][4], x[CB][TF][4];
#pragma unroll
  for (int f = 0; f < TF; ++f)
#pragma unroll
    for (int v = 0; v < 4; ++v) sum[f][v] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto x_load = [&](int s0) {
#pragma unroll
    for (int k = 0; k < CB; ++k) {
      const float* ps = p.part + (int64_t)(s0 + k < most ? s0 + k : most - 1) * p.M * p.N + n;
#pragma unroll
      for (int f = 0; f < TF; ++f)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int m = m0 + 16 * f + 4 * g + v;
          x[k][f][v] = *(const f32x4*)(ps + (int64_t)(m < p.M ? m : p.M - 1) * p.N);
        }
    }
  };
  x_load(0);
  __builtin_amdgcn_sched_barrier(0);
  f32x4 lora[TF][4];                                         // [tile][e]: tokens 4g .. 4g+3 of output 4i + e
#pragma unroll
  for (int f = 0; f < TF; ++f)
#pragma unroll
    for (int e = 0; e < 4; ++e) lora[f][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (p.r > 0) {
    auto store = [&](int idx, f32x4 t) {
      const int ml = idx >> qs, c = idx & ((1 << qs) - 1), m = m0 + ml;
      const bool ok = c < r4;
      if (!ok) t = f32x4{0.f, 0.f, 0.f, 0.f};
      uint2 hi, lo;
      few::split_hl(t, hi, lo);
      uint2 term[TERMS];
      if constexpr (TERMS == 3) few::split3(t, term);
      else {
        term[0] = hi;
        term[1] = uint2{lo_of_finite(hi.x, lo.x), lo_of_finite(hi.y, lo.y)};
      }
#pragma unroll
      for (int k = 0; k < TERMS; ++k) *(uint2*)(Tp[k] + ml * kPitch + 4 * c) = term[k];
      if (ok && p.hl && blockIdx.x == 0) {
        *(uint2*)(p.hl + (int64_t)m * 2 * p.r + 4 * c) = hi;
        *(uint2*)(p.hl + (int64_t)m * 2 * p.r + p.r + 4 * c) = lo;
      }
    };
    for (int idx = threadIdx.x; idx < n_idx; idx += 256 * TI) {
      if (idx >= 256 * TI) t_load(idx, 0);
      f32x4 t[TI];
#pragma unroll
      for (int k = 0; k < TI; ++k) t[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int q0 = 0;;) {
#pragma unroll
        for (int k = 0; k < LB; ++k)
          if (q0 + k % TQ < p.n_lparts) t[k / TQ] += lp[k];
        q0 += TQ;
        if (q0 >= p.n_lparts) break;
        t_load(idx, q0);
      }
#pragma unroll
      for (int k = 0; k < TI; ++k)
        if (idx + 256 * k < n_idx) store(idx + 256 * k, t[k]);
    }
    __syncthreads();
    for (int tb = 0; tb < p.r; tb += 32 * RB) {
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        const int t0 = tb + 32 * k;
        if (t0 >= p.r) break;
        u32x4 w[4];                                          // [e]: ranks t0 + 8g .. +7 of output 4i + e
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (BWD) { w[e] = bf[k].w[e]; continue; }
          const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
          for (int jp = 0; jp < 4; ++jp) w[e][jp] = __builtin_amdgcn_perm(bf[k].w[jp][2 + (e >> 1)], bf[k].w[jp][e >> 1], sel);
        }
        if (t0 + 32 * RB < p.r) b_load(bf[k], t0 + 32 * RB);
#pragma unroll
        for (int f = 0; f < TF; ++f) {
          bf16x8 tt[TERMS];
#pragma unroll
          for (int k2 = 0; k2 < TERMS; ++k2) tt[k2] = *(const bf16x8*)(Tp[k2] + (16 * f + i) * kPitch + t0 + 8 * g);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k2 = 0; k2 < TERMS; ++k2)
              lora[f][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tt[k2], __builtin_bit_cast(bf16x8, w[e]), lora[f][e], 0, 0, 0);
        }
      }
    }
  }
  for (int s0 = 0;;) {                                       // the partials in their fixed order
#pragma unroll
    for (int k = 0; k < CB; ++k)
#pragma unroll
      for (int f = 0; f < TF; ++f)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (s0 + k < contrib[f]) sum[f][v] += x[k][f][v];
    s0 += CB;
    if (s0 >= most) break;
    x_load(s0);
  }
  if (!n_ok) return;
#pragma unroll
  for (int f = 0; f < TF; ++f)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = m0 + 16 * f + 4 * g + v;
      if (m >= p.M) continue;
      const int64_t at = (int64_t)m * p.N + n;
      uint32_t keep = 0xfu;
      if (BWD && p.mask) keep = (uint32_t)p.mask[at >> 3] >> (at & 4);
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = sum[f][v][e] + (((keep >> e) & 1u) ? p.scale * lora[f][e][v] : 0.0f);
      uint2 q;
      q.x = pack_bf16x2(y[0], y[1]);
      q.y = pack_bf16x2(y[2], y[3]);
      *(uint2*)(p.out + at) = q;
    }
}

template <int MF, int KW, bool BWD, bool PACK>
void launch_main(const MidArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((mid_main_kernel<MF, KW, BWD, PACK>), dim3((unsigned)(a.n_items + a.line.wgs)), dim3(KW * 64), 0, st, a);
}

}  // namespace

namespace {
// Forward, the token operand as it lies or packed by a launch of its own: kPackLaunch us for that launch, kScattered us per step
// of a wave for the loads of 64-byte row pieces (backward operands are always packed).  Whole calls, us, as it lies / packed: 64 tokens
// 1024 x 1024 12.1 / 18.6, 4096 x 4096 17.8 / 22.5, 8192 x 2048 19.2 / 27.5; 128 tokens 4096 x 4096 21.4 / 24.2; 256 tokens 1024 x 1024
// 14.8 / 19.8; but 64 tokens 4096 x 11008 28.3 / 26.6, 80 tokens 8192 x 8192 40 / 34, 256 tokens 4096 x 4096 34 / 29.  Up to
// kMidPackFrom tokens, one group of three tiles, packing never won (40 tokens 8192 x 8192 25.5 / 28.1).
constexpr double kScattered = 0.24, kPackLaunch = 4.8;
// One of the launch shapes: kw = 4, one wave per SIMD with tiles of up to `group` = 128 or 64 tokens, or kw = 8, two waves
// per SIMD with tiles of up to 64.  Per unit of work tiles of 128 tokens are fastest (a decoded fragment meets twice the
// tokens); tiles of 64 have the cheaper fixed part and give a small layer twice the workgroups (dX of
// 1024 x 1024 at 256 tokens: main kernel 16.5 -> 12.7 us with 128 workgroups instead of 64; 4096 x 4096 at 128 tokens, the
// three kernels together: 37.1 -> 33.8; 4096 x 4096 at 512 tokens, where both fill the chip: 48.3, and 51.5 with 64).
MidPlan plan_shape(bool bwd, int kw, int group, bool pack, int64_t M, int64_t K, int64_t N, int r, size_t room, double* us) {
  MidPlan p{};
  const int n_tg = (int)((M + group - 1) / group);
  p.KW = kw;
  p.MF = (int)((M + 16 * n_tg - 1) / (16 * n_tg));
  if (kw == 4 && p.MF < 2) p.MF = 2;                         // the software pipeline of that shape needs two token tiles
  p.n_tg = (int)((M + 16 * p.MF - 1) / (16 * p.MF));
  p.n_slabs = (int)((N + kSlab - 1) / kSlab);
  p.steps = (int)(bwd ? K / 64 : K / 32);
  p.pack = pack;
  // about ten partials of the adapter's inner product, of at least 512 contraction elements each
  p.chunk = (int)std::max<int64_t>(512, ((K + 9) / 10 + 63) / 64 * 64);
  p.n_lparts = r > 0 ? (int)((K + p.chunk - 1) / p.chunk) : 0;
  p.lpart_floats = (size_t)p.n_lparts * M * r;
  p.pack_elems = p.pack ? (size_t)p.n_tg * p.MF * 16 * K : 0;
  auto bytes = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t fixed = bytes(p.lpart_floats * 4) + bytes(p.pack_elems * 2);
  const int64_t tiles = (int64_t)p.n_tg * p.n_slabs;
  const int ups = (p.steps + p.KW - 1) / p.KW;
  if (tiles * ups >= (1ll << 30)) return p;
  const int items = p.pack ? 0 : (int)((M + kAdTok - 1) / kAdTok) * p.n_lparts;
  // The number of workgroups (at most one per compute unit, and what the workspace has room for): the smallest estimated
  // time in microseconds of the longest workgroup -- its units, and the ends of its segments -- plus the partials' way
  // through memory.  Measured (main kernel, r = 64): kw = 4 with 8 token tiles 28.5 at 16 steps a wave, 56.4 at 43;
  // (4 token tiles 31.8 at 32); kw = 8 with 4 tiles 29.5 at 16, 66.8 at 43; a workgroup whose range crosses into a second tile pays a second end
  // (4096 x 11008 at 40 tokens: 21.3 with ranges that cross, 17.4 with every tile in two equal parts).  All in closed form:
  // a call plans on the host every time.
  const double step = (bwd ? 2.0 : 1.0) * ((kw == 4 ? 0.38 + 0.0775 * p.MF : 0.55 + 0.20 * p.MF) + (pack ? 0.0 : kScattered));
  const double seg_end = 2.0 + 0.75 * p.MF, tile_us = p.MF * 16 * kSlab * 4 / 4.0e6;
  const int64_t units = tiles * ups, most = std::min<int64_t>(256 - std::min(items, 128), units);
  const size_t one = (size_t)M * N * 4;
  auto consider = [&](int64_t wgs, int64_t segments, int64_t contrib) {
    const double t = (double)((units + wgs - 1) / wgs) * step + (double)segments * seg_end + (double)(tiles + wgs) * tile_us;
    if ((p.ok && t >= *us) || fixed + bytes((size_t)contrib * one) > room) return;
    *us = t; p.line = MidLine{(int)units, ups, (int)wgs}; p.max_contrib = (int)contrib; p.ok = true;
  };
  for (int64_t k = 1; tiles * k <= most && k <= ups; ++k) consider(tiles * k, 1, k);        // every tile in k equal parts
  const int64_t len = units / most;                          // ranges of len or len + 1 units wherever they fall
  consider(most, (len - 1) / ups + 2, (ups - 1 + len - 1) / len + 1);
  p.part_floats = (size_t)p.max_contrib * M * N;
  return p;
}
}  // namespace

MidPlan mid_plan(bool bwd, int64_t M, int64_t h, int64_t o, int r, size_t room, bool packed) {
  const int64_t K = bwd ? o : h, N = bwd ? h : o;
  if (M < 1 || M > kMidTokens || o > (1 << 24) || h > (1 << 24) || (M + 127) * K * 2 >= (1ll << 31) || h * o / 2 >= (1ll << 31))
    return MidPlan{};                                        // 32-bit buffer offsets
  // the least estimated time, with the launch that packs the operand; of equal ones the first
  MidPlan best{};
  double best_us = 0;
  auto consider = [&](int kw, int group, bool pack) {
    double us = 0;
    const MidPlan p = plan_shape(bwd, kw, group, pack, M, K, N, r, room, &us);
    const double all = us + (pack ? kPackLaunch : 0.0);
    if (p.ok && (!best.ok || all < best_us)) { best = p; best.us = us; best_us = all; }
  };
  if (!bwd && !(packed && M > kMidPackFrom)) consider(8, 48, false);
  if (bwd || M > kMidPackFrom) {
    if (!bwd) consider(8, 64, true);
    consider(4, 128, true);
    if (M > 64) consider(4, 64, true);                       // below, tiles of 128 hold all tokens anyway
  }
  return best;
}

// Both sides from their parts, in microseconds, fitted to 1645 calls of either path (1 .. 512 tokens, contractions of 64 ..
// 22016, 64 .. 65536 outputs, ranks 0 .. 256; each estimate within 20 % on nine calls of ten).  Decoding inside the product
// loses where the contraction is short (its partials are then as large as the product: dX with K = 64, N = 16384 at 384 tokens
// 43 us against 12) or the rank large (K = 1024, N = 8192, rank 256 at 512 tokens 66 against 32); it wins where the weight is
// what counts (K = 22016, N = 8192, rank 64 at 256 tokens 117 against 421; 112 against 334 now).  A call goes to the other path where that
// is estimated faster by a fifth.  The fit is older than the 128 x 128 tiles, with which the other path's estimate has become
// some 17 % high, and the line has not been moved since: of 947 random calls that it decides 285 are now more than 3 % from the
// faster path and 131 more than 20 %, all of these decoded here, the worst 1.9 x (under dropout 30 tokens 256 x 64 at rank 256 23.6 us
// here, 12.6 dequantised; dX 2752 x 3136, rank 144, 511 tokens 53.8 and 35.1).  They take no longer here than they did before those tiles.
bool mid_pays(const MidPlan& p, bool bwd, int64_t M, int64_t h, int64_t o, int r, bool fix) {
  const double K = (double)(bwd ? o : h), N = (double)(bwd ? h : o), MN = 1e-6 * (double)M * N;
  const double mid = 6.5 + 0.88 * p.us + (p.pack ? 4.3 + 0.053 * r : 0.027 * r) + 0.35 * p.max_contrib * MN + 0.0034 * r * MN +
                     3.3e-8 * (double)M * K * r;
  const double gemm = 9.7 + 0.7 * gemm_rounds_us(M, (int64_t)N, ((int64_t)K + (r + 63) / 64 * 64) / 64) + 0.62e-6 * K * N +
                      0.6 * MN + (r > 0 ? 3.6 + 1e-6 * r * (0.2 * N + 3.8 * K) : 0.0) + (fix ? 5.5 + 2.2 * MN : 0.0);
  if (!p.pack && M > kMidPackFrom) {
    // The adapter's workgroups run beside the product's, 64 rank columns after the other: a launch takes as long as the longer of
    // the two.  (The sum above is fitted to calls that pack the operand or have up to 48 tokens.  By it 127 of 556 random such calls
    // came here that take up to 1.86 x as long as the other path, 62 of them longer than when every operand of that size was packed:
    // under dropout 111 tokens 256 x 64 at rank 256 24.6 us against 13.2, 114 tokens 512 x 448 25.6 against 16.2.  By this one 22 of them are
    // more than 3 % from the faster path, the worst 13 %, none longer than then.  The other side's estimate is some 17 % high.)
    const double chain = (1.8 + 2.7 / 512 * std::min(K, 512.0)) * ((r + 63) / 64);
    const double beside = 5.8 + (r > 0 ? 2.4 : 0.0) + std::max(0.88 * p.us, chain) + (0.35 * p.max_contrib + 0.0034 * r) * MN;
    return beside <= 0.95 * gemm;
  }
  return mid <= 1.2 * gemm;
}

// Up to 16 tokens the streaming kernel reads the weight once and ends in an output stage of its own; two launches here, but a
// decode that all tokens share and an output stage on many workgroups.  Forward calls, us, streamed / here (rank 64 but where
// stated): 1024 x 1024 rank 16 at 3, 8, 16 tokens 10.7 / 10.0, 12.1 / 10.1, 14.5 / 10.3; 2048 x 2048 rank 16 at 6, 11, 16
// 11.6 / 10.9, 12.8 / 11.0, 14.5 / 11.1; 4096 x 4096 at 8, 11, 16 14.0 / 14.4, 14.5 / 14.4, 16.2 / 14.8; 4096 x 11008 at 14, 16
// 18.4 / 16.3, 19.2 / 16.5; 1024 x 16384 at 8, 11, 16 13.6 / 13.3, 14.5 / 13.5, 16.0 / 13.7; 8192 x 8192 at 12 19.9 / 20.0.  A
// contraction longer than the outputs are wide has too few strips (3072 x 1536 at 4, 11 11.6 / 12.7, 13.2 / 13.4), and a large rank
// makes the adapter's launch the longer part (2048 x 2048 rank 256 at 4, 11 22.7 / 23.9, 24.8 / 24.9).  And two launches cost the host
// 12.5 us a call against 9.2: called one by one, 1024 x 2624 rank 32 at 5 tokens takes 11.5 streamed and 12.6 here, 2048 x 2048 at
// 8, 11, 14 12.6 / 12.6, 13.4 / 12.8, 14.5 / 12.7, 1024 x 1024 at 16 15.0 / 12.8.  So: from 12 tokens, above sqrt(4 weights / 2^20),
// contraction no longer than the outputs, rank up to 128, and a contraction that streams for as long as the host takes over two
// launches.  One by one at 12, 16 tokens on 4096 outputs: rank 64, K = 64 9.9 / 11.4, 10.8 / 11.4, 256 11.2 / 11.9, 12.3 / 11.9,
// 512 12.9 / 12.1, 13.8 / 12.2, 1024 13.1 / 12.1, 14.0 / 12.0; rank 128, K = 64 11.2 / 11.2, 12.0 / 11.3, 256 12.4 / 12.3, 13.3 / 12.5;
// no adapter, K = 256 8.8 / 11.6, 8.9 / 11.8, 1024 10.2 / 11.8, 10.6 / 11.9, 2048 11.0 / 11.9, 11.8 / 11.8, 2752 11.4 / 11.0,
// 12.3 / 10.9, 4096 12.1 / 11.7, 12.9 / 11.8 (2048 x 2048 at 16 11.5 / 11.9).  Replayed from a graph most of what that last condition leaves
// to the streaming kernel would be faster here (rank 64, 256 x 4096 at 16 12.8 / 10.6; no adapter, 1024 x 4096 11.2 / 9.4).
bool mid_beats_few(int64_t M, int64_t h, int64_t o, int r) {
  const bool long_enough = r > 64 ? h >= 256 : r > 0 ? h >= 512 : M * h > 32768;
  return M >= 12 && long_enough && h <= o && r <= 128 && (double)(M * M) > 4. * (double)h * (double)o / (1 << 20);
}

hipError_t launch_mid(bool bwd, const uint16_t* X, int M, const NF4Dev& w, const MidPlan& p, const uint16_t* L1,
                      const uint16_t* L2, int r, float scale, const uint8_t* mask, float* part, float* lpart, uint16_t* xpack,
                      uint16_t* out, uint16_t* hl, hipStream_t st) {
  if (!p.ok || w.dtype == kTypeInt8) return hipErrorInvalidValue;
  MidArgs a{};
  a.X = X; a.M = M; a.h = (int)w.rows; a.o = (int)w.cols;
  a.K = bwd ? a.o : a.h; a.N = bwd ? a.h : a.o;
  a.packed = w.packed; a.code = w.code; a.c1 = w.c1; a.mean = w.mean; a.dtype = w.dtype; a.dq = w.dq ? 1 : 0;
  a.tab = table4_host(w.dtype);
  a.part = part; a.n_tg = p.n_tg; a.n_slabs = p.n_slabs; a.steps = p.steps; a.line = p.line;
  a.L = bwd ? L2 : L1; a.r = r; a.mask = bwd ? nullptr : mask;
  a.lpart = lpart; a.n_lparts = r > 0 ? p.n_lparts : 0; a.chunk = p.chunk;
  const int tiles = p.n_tg * p.MF, items = (M + kAdTok - 1) / kAdTok * a.n_lparts;
  if (p.pack) {
    a.Xf = (const char*)xpack;
    a.x_step = tiles * 1024 * (bwd ? 2 : 1);
    a.x_bytes = (uint32_t)(p.pack_elems * 2);
    a.x_sub = tiles * 1024;
    const unsigned grid = (unsigned)(items + tiles * ((a.K + kPreK - 1) / kPreK));
    if (bwd) hipLaunchKernelGGL(mid_pre_kernel<true>, dim3(grid), dim3(512), 0, st, a, xpack, tiles, items);
    else hipLaunchKernelGGL(mid_pre_kernel<false>, dim3(grid), dim3(512), 0, st, a, xpack, tiles, items);
  } else {
    a.Xf = (const char*)X;
    a.x_step = 64;
    a.x_bytes = (uint32_t)((int64_t)M * a.K * 2);
    a.n_items = items;
  }
  // what mid_plan makes of 1 .. 512 tokens; packed forward operands have three token tiles at least
#define QL_MID_BWD(MF) case 40 + MF: launch_main<MF, 4, true, true>(a, st); break;
#define QL_MID_FWD(MF) case 40 + MF: launch_main<MF, 4, false, true>(a, st); break;
  if (bwd) {
    switch (10 * p.KW + p.MF) {
      QL_MID_BWD(2) QL_MID_BWD(3) QL_MID_BWD(4) QL_MID_BWD(5) QL_MID_BWD(6) QL_MID_BWD(7) QL_MID_BWD(8)
      default: return hipErrorInvalidValue;
    }
  } else if (p.pack) {
    switch (10 * p.KW + p.MF) {
      case 83: launch_main<3, 8, false, true>(a, st); break;
      case 84: launch_main<4, 8, false, true>(a, st); break;
      QL_MID_FWD(3) QL_MID_FWD(4) QL_MID_FWD(5) QL_MID_FWD(6) QL_MID_FWD(7) QL_MID_FWD(8)
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (10 * p.KW + p.MF) {
      case 81: launch_main<1, 8, false, false>(a, st); break;
      case 82: launch_main<2, 8, false, false>(a, st); break;
      case 83: launch_main<3, 8, false, false>(a, st); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef QL_MID_FWD
#undef QL_MID_BWD
  if (hipError_t e = hipGetLastError()) return e;
  MidFinArgs f{};
  f.part = part; f.line = p.line; f.MF = p.MF; f.n_tg = p.n_tg; f.M = M; f.N = a.N; f.lpart = lpart; f.n_lparts = a.n_lparts; f.r = r;
  f.B = bwd ? L1 : L2; f.scale = scale; f.out = out; f.hl = r > 0 ? hl : nullptr; f.mask = bwd ? mask : nullptr;
  const unsigned gx = (unsigned)((a.N + 255) / 256);
  static_assert(kLeanBlocks < 1024, "two token tiles: lean");
  const bool two = (int64_t)gx * ((M + 31) / 32) >= 1024;
  const dim3 grid(gx, (unsigned)(two ? (M + 31) / 32 : (M + 15) / 16));
  const bool lean = grid.x * grid.y > kLeanBlocks;
  auto launch = [&](auto T, auto D, auto L, auto terms, auto quads) {
    hipLaunchKernelGGL((mid_finalize_kernel<T.value, D.value, L.value, terms.value, quads.value>), grid, dim3(256), 0, st, f);
  };
  auto pick = [&](auto D, auto terms) {                      // one tile of tokens
    if (lean) launch(Int<1>{}, D, std::true_type{}, terms, Int<1>{});
    else if (mid_quads(M, r) == 1) launch(Int<1>{}, D, std::false_type{}, terms, Int<1>{});
    else if (mid_quads(M, r) == 2) launch(Int<1>{}, D, std::false_type{}, terms, Int<2>{});
    else launch(Int<1>{}, D, std::false_type{}, terms, Int<4>{});
  };
  if (!bwd && M <= 16) pick(std::false_type{}, Int<3>{});
  else if (two && bwd) launch(Int<2>{}, std::true_type{}, std::true_type{}, Int<2>{}, Int<1>{});      // 1024 workgroups and more
  else if (two) launch(Int<2>{}, std::false_type{}, std::true_type{}, Int<2>{}, Int<1>{});
  else if (bwd) pick(std::true_type{}, Int<2>{});
  else pick(std::false_type{}, Int<2>{});
  return hipGetLastError();
}

}  // namespace qlora
