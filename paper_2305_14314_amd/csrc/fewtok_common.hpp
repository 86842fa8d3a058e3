// Building blocks shared by the few-token (M <= 16) streaming kernels of the QLoRA linear layer
// (arXiv 2305.14314, Eq. 5 / Eq. 6 at generation-time batch sizes): the replicated byte -> (value, value)
// decode table in LDS, the per-layer argument block, the workgroup -> die map and the adapter's inner
// products T = X L1 and U = dY L2^T on MFMA 16x16x32.
#pragma once

#include "common.hpp"
#include "launch.hpp"

namespace qlora {
namespace few {

constexpr int kFewThreads = 1024;            // 16 waves share one replicated decode table (8 where 256 VGPRs are needed)
constexpr int kWaves = kFewThreads / 64;
constexpr int kLutCopies = 32;
constexpr int kBwdDepth = 2;
constexpr int kLoraDepth = 2;
constexpr int kLoraK = 1024;                 // forward: rows of L1 per adapter workgroup (short: they must not arrive last)
constexpr int kLoraN = 1024;                 // backward: columns of L2 per adapter workgroup

// LDS map of a main workgroup.  The decode table is dead once the main loop is over, so the cross-wave
// sums reuse the space from offset 0.
constexpr int kLutBytes = 256 * kLutCopies * 8;              // 64 KB
constexpr int kRedBytes = kWaves * 16 * 128 * 4;             // 128 KB: one 16 x 128 fp32 tile per wave
constexpr int kUnitOff = kRedBytes;                          // float[256]
constexpr int kStripOff = kUnitOff + 1024;                   // float[kWaves][2][32]
constexpr int kSmemBytes = kStripOff + kWaves * 256;
static_assert(kLutBytes <= kRedBytes && kSmemBytes <= 160 * 1024, "LDS map");

// Entry e = 32 b + copy of the table belongs to byte b = e / 32; thread t writes the pairs of copies t, t + NT, ... (16 bytes
// each): byte t / 16 + NT / 16 k, whose low nibble is the same for all of them and whose high nibble is the same for 256
// threads and advances by NT / 256.  So the low value is picked once per thread from the 16 values in scalar registers (NF4's,
// or another data type's from the arguments: Section 4) and the high ones are scalar: no memory round trip (a lane-indexed read
// of a constant array is one), no barrier of its own.  The caller's barrier makes the table visible.
template <int NT>
__device__ __forceinline__ void init_pair_lut(f32x2* lut2 /* [256][32] */, float* unit /* [256] */, int dtype, const Table4& tab) {
  static_assert(NT % 256 == 0 && 4096 % NT == 0, "whole high nibbles per pass");
  constexpr float t[16] = {QLORA_NF4_VALUES};
  constexpr int H = NT / 256;
  const int hi_first = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), lo_nibble = (threadIdx.x >> 4) & 15;
  float v[16], lo = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    v[i] = t[i];
    if (dtype != 0) v[i] = tab.v[i];                         // uniform
    lo = lo_nibble == i ? v[i] : lo;
  }
#pragma unroll
  for (int k = 0; k < 16 / H; ++k) {
    float hi = v[H * k];
#pragma unroll
    for (int q = 1; q < H; ++q) hi = hi_first == q ? v[H * k + q] : hi;
    *(f32x4*)(lut2 + 2 * (threadIdx.x + NT * k)) = f32x4{lo, hi, lo, hi};
  }
  for (int i = threadIdx.x; i < 256; i += NT) unit[i] = e4m3_unit(i);
}
// (value[lo nibble], value[hi nibble]) of byte B (0..3) of packed dword `pk`, from this lane's copy of the table.
// Entry e of copy c sits at byte offset 256 e + 8 c: the offset is assembled by one byte permute
// (byte 1 = the weight byte, byte 0 = 8 * copy), instead of shift, mask and add.
template <int B>
__device__ __forceinline__ f32x2 pair_lookup(const f32x2* lut2, uint32_t pk, uint32_t lane_off /* 8 * (lane % 32) */) {
  const uint32_t off = __builtin_amdgcn_perm(pk, lane_off, 0x0c0c0400u + ((uint32_t)B << 8));
  return *(const f32x2*)((const char*)lut2 + off);
}

// the same with the byte number as a (constant-folded) argument
__device__ __forceinline__ f32x2 pair_lookup_b(const f32x2* lut2, uint32_t pk, uint32_t lane_off, int b) {
  switch (b) {
    case 0: return pair_lookup<0>(lut2, pk, lane_off);
    case 1: return pair_lookup<1>(lut2, pk, lane_off);
    case 2: return pair_lookup<2>(lut2, pk, lane_off);
    default: return pair_lookup<3>(lut2, pk, lane_off);
  }
}

struct FewArgs {
  const uint16_t* X; int M;                  // tokens x contraction dim (X for forward, dY for backward)
  const uint8_t* packed; const uint8_t* code; const float* c1; const float* mean;
  int dtype; Table4 tab;                     // data type of the weight (0 = NF4) and, for the others, its 16 values
  int h, o;
  float* part;                               // [splits][M][N]
  int per_split;                             // contraction elements per split
  int n_slabs, splits;
  // adapter inner product, handled by the first n_lparts workgroups in work_index() order
  const uint16_t* L; int r;                  // forward: L1 (h x r); backward: L2 (r x o)
  float* lpart;                              // [n_lparts][M][r]
  int n_lparts;
  // output stage, run by the last workgroup to arrive at a slab
  unsigned* ctr;                             // arrival counters (split arrivals, adapter handshakes, adapter count); zero on entry and exit
  const uint16_t* Bmat;                      // forward: L2 (r x o); backward: L1 (h x r)
  float scale;
  uint16_t* out;                             // M x N bf16
  uint16_t* hl;                              // M x 2r: T (resp. U) as a [hi | lo] bf16 pair, or NULL
  int lora_chunk;                            // contraction elements per adapter workgroup (kLoraK / kLoraN in the one-layer kernels)
  // work-list kernels only
  unsigned* hdr;                             // start of the counter header (status word)
  unsigned nonce;                            // this call's tag, in bits 31:24 of every arrival word it touches
  int spin_limit;                            // polls of a slab's last contributor for the adapter's partials
};

// Workgroup b runs on die (XCD) b % 8, and each die has its own L2.  The work list -- adapter partials first,
// then (split, slab) pairs in split-major order -- is cut into 8 contiguous pieces, one per die, so that the
// workgroups of one split sit together: they read the same rows of the token operand and, in the forward, the
// same 128-byte lines of the 8-bit constants (a line holds one row's constants of 32 slabs).  With the plain
// b -> (b % n_slabs, b / n_slabs) map every die pulled every constant line: 1.5x the algorithmic HBM bytes.
__device__ __forceinline__ int work_index() {
  const int grid = gridDim.x, b = blockIdx.x;
  const int x = b & 7, q = b >> 3;
  return x * (grid >> 3) + (x < (grid & 7) ? x : (grid & 7)) + q;
}

// ---- between the workgroups of a launch --------------------------------------------------------------
// Partials travel past the L2 of a die (agent scope: sc1): they are stored so, every wave waits for its stores to be
// acknowledged before the workgroup is counted in, and they are read so; no fence is needed -- an agent-scope release is
// a write-back of the die's whole L2, an acquire an invalidation.
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr int kAgent = 16;                   // cache policy of the buffer instructions: sc1
__device__ __forceinline__ Rsrc agent_rsrc(const float* p) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 0x7fffffff, 0x00020000);
}
//   four floats at element `at`: the partials of a layer are far below 2 GiB
__device__ __forceinline__ void agent_store(Rsrc r, uint32_t at, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, at * 4u, 0, kAgent);
}
__device__ __forceinline__ f32x4 agent_load(Rsrc r, uint32_t at) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at * 4u, 0, kAgent));
}
__device__ __forceinline__ void agent_zero(unsigned* p) { __hip_atomic_store(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned agent_word(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// every store of this workgroup has reached the point where all dies see it
__device__ __forceinline__ void all_stored() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// ---- adapter partials -----------------------------------------------------------------------------
// Both run on MFMA 16x16x32 with the tokens as one 16-wide dimension and 16 rank columns as the other,
// kLoraDepth steps of loads in flight, and a cross-wave sum through LDS; one partial slot per workgroup.
// A call waits for them, so they are short: tokens >= M and rank columns >= r read any valid row and only reach sums that
// are never stored (no masks), a load is a scalar base and a fixed 32-bit offset, and none is issued past the end (a load
// in flight holds its registers, and whoever needs them next waits for it).  With 64-bit addresses and masks per element
// and two steps of loads past the end a partial was stored 11.4 us into a call at 8192 x 8192 (and 9.3 us into one at
// 4096 x 4096, where the output waited for it); now 5.7 and 4.1.
//
// forward: lpart[wg][m][j] = sum over k in [chunk * wg, +chunk) of X[m][k] * L1[k][j]
// L1 is [h][r] (rank contiguous), so a fragment of 8 consecutive k for one rank column is gathered from
// 8 rows: lane (i, g) loads columns 4i .. 4i+3 of rows kb + 8g + j and splits them with byte permutes.
struct LFwdStep { uint2 l[8]; u32x4 x; };

// The waves' sums: acc[e][v] of lane (i, g) belongs to token 4g + v and rank column j0 + col(i, e).
template <int NT, bool BWD>
__device__ __forceinline__ void lora_store(const FewArgs& p, int wg, int j0, const f32x4 (&acc)[4], float* red) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const Rsrc lpart = agent_rsrc(p.lpart);
  __syncthreads();                                           // previous chunk's sums have been read
  float* my = red + wave * (16 * 64);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (4 * g + v >= p.M) continue;
    if (BWD) {
#pragma unroll
      for (int e = 0; e < 4; ++e) my[(4 * g + v) * 64 + 16 * e + i] = acc[e][v];
    } else {
      *(f32x4*)(my + (4 * g + v) * 64 + 4 * i) = f32x4{acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < p.M * 16; idx += NT) {
    const int m = idx >> 4, c = (idx & 15) * 4;
    f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += *(const f32x4*)(red + w * 16 * 64 + m * 64 + c);
    if (j0 + c < p.r) agent_store(lpart, (uint32_t)((wg * p.M + m) * p.r + j0 + c), t);   // r % 16 == 0
  }
}

template <int NT>
__device__ void lora_fwd_partial(const FewArgs& p, int wg, float* red /* [NT / 64][16][64] */) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave index is uniform
  const int i = lane & 15, g = lane >> 4;
  const int k_begin = wg * p.lora_chunk;
  const int k_end = (k_begin + p.lora_chunk < p.h) ? k_begin + p.lora_chunk : p.h;              // multiples of 64
  const int stride = (NT / 64) * 32, kb0 = k_begin + wave * 32; // the waves interleave 32-row steps
  const uint32_t x_off = (uint32_t)(i < p.M ? i : 0) * (uint32_t)(p.h >> 3) + (uint32_t)g;      // in 16-byte chunks
  for (int j0 = 0; j0 < p.r; j0 += 64) {
    const uint32_t l_off = (uint32_t)(2 * g * p.r + (j0 + 4 * i < p.r ? (j0 >> 2) + i : 0));    // in 8-byte chunks; r % 16 == 0: 4 columns are in or out together
    auto load_step = [&](LFwdStep& s, int kb) {
      s.x = ((const u32x4*)(p.X + kb))[x_off];
#pragma unroll
      for (int j = 0; j < 8; ++j) s.l[j] = ((const uint2*)(p.L + (int64_t)(kb + j) * p.r))[l_off];
    };
    f32x4 acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    LFwdStep buf[kLoraDepth];
#pragma unroll
    for (int d = 0; d < kLoraDepth; ++d) load_step(buf[d], kb0 + d * stride < k_end ? kb0 + d * stride : k_begin);
    for (int kb = kb0; kb < k_end; kb += kLoraDepth * stride) {
#pragma unroll
      for (int d = 0; d < kLoraDepth; ++d) {
        if (kb + d * stride < k_end) {
          const bf16x8 xa = __builtin_bit_cast(bf16x8, buf[d].x);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            u32x4 w;
#pragma unroll
            for (int jp = 0; jp < 4; ++jp)
              w[jp] = e >> 1 ? __builtin_amdgcn_perm(buf[d].l[2 * jp + 1].y, buf[d].l[2 * jp].y, sel)
                             : __builtin_amdgcn_perm(buf[d].l[2 * jp + 1].x, buf[d].l[2 * jp].x, sel);
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, __builtin_bit_cast(bf16x8, w), acc[e], 0, 0, 0);
          }
          if (kb + (d + kLoraDepth) * stride < k_end) load_step(buf[d], kb + (d + kLoraDepth) * stride);
        }
      }
    }
    lora_store<NT, false>(p, wg, j0, acc, red);
  }
}

// backward: lpart[wg][m][j] = sum over n in [chunk * wg, +chunk) of dY[m][n] * L2[j][n]
// Both operands are contiguous along n: fragments are plain 16-byte loads.
struct LBwdStep { u32x4 l[4]; u32x4 y; };

template <int NT>
__device__ void lora_bwd_partial(const FewArgs& p, int wg, float* red /* [NT / 64][16][64] */) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave index is uniform
  const int i = lane & 15, g = lane >> 4;
  const int n_begin = wg * p.lora_chunk;
  const int n_end = (n_begin + p.lora_chunk < p.o) ? n_begin + p.lora_chunk : p.o;              // multiples of 64
  const int stride = (NT / 64) * 32, nb0 = n_begin + wave * 32; // the waves interleave 32-column steps
  const uint16_t* y_row = p.X + (int64_t)(i < p.M ? i : 0) * p.o + 8 * g;
  for (int j0 = 0; j0 < p.r; j0 += 64) {
    const uint16_t* l_row[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) l_row[e] = p.L + (int64_t)(j0 + 16 * e + i < p.r ? j0 + 16 * e + i : 0) * p.o + 8 * g;
    auto load_step = [&](LBwdStep& s, int nb) {
      s.y = *(const u32x4*)(y_row + nb);
#pragma unroll
      for (int e = 0; e < 4; ++e) s.l[e] = *(const u32x4*)(l_row[e] + nb);
    };
    f32x4 acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    LBwdStep buf[kLoraDepth];
#pragma unroll
    for (int d = 0; d < kLoraDepth; ++d) load_step(buf[d], nb0 + d * stride < n_end ? nb0 + d * stride : n_begin);
    for (int nb = nb0; nb < n_end; nb += kLoraDepth * stride) {
#pragma unroll
      for (int d = 0; d < kLoraDepth; ++d) {
        if (nb + d * stride < n_end) {
          const bf16x8 ya = __builtin_bit_cast(bf16x8, buf[d].y);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya, __builtin_bit_cast(bf16x8, buf[d].l[e]), acc[e], 0, 0, 0);
          if (nb + (d + kLoraDepth) * stride < n_end) load_step(buf[d], nb + (d + kLoraDepth) * stride);
        }
      }
    }
    lora_store<NT, true>(p, wg, j0, acc, red);
  }
}

// Four fp32 values as three bf16 terms each whose sum they are (3 x 8 bits hold fp32's 24), cut off rather than rounded: every
// term has its value's sign, and none overflows where the value does not.  What has nothing left to hold takes 2^-40 of the
// value instead of zero, far below fp32's last bit: an infinite value, or an infinite factor, then gives the infinity that
// the product with the fp32 value gives, where Inf - Inf and 0 * Inf gave NaN.
__device__ __forceinline__ void split3(f32x4 t, uint2 (&term)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const u32x4 b = __builtin_bit_cast(u32x4, t);
    term[k].x = __builtin_amdgcn_perm(b[1], b[0], 0x07060302u);
    term[k].y = __builtin_amdgcn_perm(b[3], b[2], 0x07060302u);
    if (k < 2) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float rest = t[d] - __builtin_bit_cast(float, b[d] & 0xffff0000u);
        t[d] = __builtin_fabsf(rest) > 0.0f ? rest : t[d] * 0x1p-40f;   // no rest: zero, or Inf - Inf
      }
    }
  }
}
// Four fp32 values as [hi | lo] bf16 pairs, both rounded (16 significant bits): what is saved of T.
__device__ __forceinline__ void split_hl(f32x4 t, uint2& hi, uint2& lo) {
  hi.x = pack_bf16x2(t[0], t[1]);
  hi.y = pack_bf16x2(t[2], t[3]);
  lo.x = pack_bf16x2(t[0] - bf16_lo_to_f32(hi.x), t[1] - bf16_hi_to_f32(hi.x));
  lo.y = pack_bf16x2(t[2] - bf16_lo_to_f32(hi.y), t[3] - bf16_hi_to_f32(hi.y));
}

// ---- output stage ---------------------------------------------------------------------------------
// An arrival's outcome: others are still to come (0); the last one; ... and the adapter's partials are all there.
constexpr int kLast = 1, kReady = 2;

// out[m][n] = bf16( sum_s part_s[m][n] + scale * sum_j T[m][j] * B(j, n) ),  T = sum_p lpart[p], for the 256
// outputs n of one slab; forward: B(j, n) = L2[j][n]; backward: B(j, n) = L1[n][j].  Run by all NT threads of one
// workgroup; slab 0 also stores T as a [hi | lo] bf16 pair.  part: the slab's first output of partial 0, token 0; the n_part
// partials lie ld_part floats apart, tokens ld_tok.
// What it costs is round trips to memory, so everything is requested at once, in the order in which it is needed: the
// partials of T, the split partials, the first tile of the adapter's outer matrix -- and by as few lanes as there are
// values, a wave per token: a 16-byte request per lane occupies the address unit for 16 cycles, and with every wave asking
// for its share of the outputs in MFMA layout (4 of 64 lanes with a value at one token) the requests alone took 1.7 us.
// `meet`: the adapter's workgroups are not known to be done; `met` waits for them, and what was read of T before is read
// again (false: they come later and finish the slab).  The adapter's product runs on MFMA 16x16x32, a wave 16 (NT = 512: 32)
// outputs: T travels as three bf16 terms that hold all of it (split3), so its products with the bf16 matrix are
// those of the fp32 value, summed in fp32.  Weight side first: lane (i, g) ends with the four neighbouring outputs 4g .. 4g+3
// of token i.
constexpr int kTileRanks = 64;               // ranks staged at a time
constexpr int kTPitch = 256 + 8, kTPlane = 16 * kTPitch, kSumPitch = 256 + 4;
constexpr int kOutStageBytes = (3 * kTPlane + kTileRanks * kTPitch) * 2;   // the product's sums reuse the front
static_assert(16 * kSumPitch * 4 <= kOutStageBytes, "sums over the terms of T");
// this thread's share of a tile of the adapter's outer matrix.  Forward: rows j0 + e / 32 of L2, columns 8 (e % 32) .. +7 of
// the slab, staged in LDS; backward: MFMA fragments, ranks j0 + 32 t + 8g .. +7 of row 16 (wave + W c) + i of the slab of L1.
template <bool BWD, int NT> struct OutTile { u32x4 v[2048 / NT]; };
template <bool BWD, int NT>
__device__ __forceinline__ void tile_load(OutTile<BWD, NT>& t, const FewArgs& p, int slab, int j0) {
  const uint16_t* src = p.r > 0 ? p.Bmat : p.X;              // without an adapter: any valid bytes
#pragma unroll
  for (int it = 0; it < 2048 / NT; ++it) {
    bool ok;
    int64_t off;
    if (!BWD) {
      const int e = it * NT + threadIdx.x, j = j0 + (e >> 5), n = slab * 256 + 8 * (e & 31);
      ok = j < p.r && n < p.o;
      off = (int64_t)j * p.o + n;
    } else {
      const int lane = threadIdx.x & 63, c = it >> 1;
      const int n = slab * 256 + 16 * ((int)(threadIdx.x >> 6) + NT / 64 * c) + (lane & 15), j = j0 + 32 * (it & 1) + 8 * (lane >> 4);
      ok = j < p.r && n < p.h;
      off = (int64_t)n * p.r + j;
    }
    const u32x4 v = *(const u32x4*)(src + (ok ? off : 0));
    t.v[it] = ok ? v : u32x4{0u, 0u, 0u, 0u};
  }
}
//   PB, LB: split partials and partials of T in flight per token and wave
//   EXACT: nothing is requested for an adapter that is not there, and two partials instead of a batch where there are no more: at
//   16 tokens a batch that nobody needs is 0.85 us of the address unit.  (8 tokens, three layers of 384 x 512 without an adapter
//   10.4 -> 9.4 us, 14 tokens, three of 576 x 1344 12.7 -> 11.0.)  The backward kernels with an adapter have no registers for
//   the branches: 8192 x 8192 at one token 22.4 -> 23.7 with both, at 16 30.2 -> 30.6 with the first.
template <bool BWD, int NT, int PB, int LB, bool EXACT, class Met>
__device__ __forceinline__ void output_stage(const FewArgs& p, int slab, const float* part0, int n_part, int ld_part, int ld_tok,
                                             char* smem /* kOutStageBytes */, bool meet, Met&& met) {
  constexpr int RC = kTileRanks;
  constexpr int W = NT / 64, PW = 16 / W;                    // waves; tokens, and groups of 16 outputs, of a wave
  constexpr int IT = 2048 / NT;
  static_assert(PB >= 2, "the first two partials are always requested");
  uint16_t* Tp = (uint16_t*)smem;                            // [3][16][kTPitch]: the terms of T[m][j]
  uint16_t* Bs = Tp + 3 * kTPlane;                           // forward: [RC][kTPitch]
  float* sum = (float*)smem;                                 // [16][kSumPitch]: the adapter's product, once the terms are done with
  const int N = BWD ? p.h : p.o;
  const int n0 = slab * 256;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int rp = (p.r + 31) & ~31;                           // ranks in whole MFMA steps: zeros beyond r on both sides
  const Rsrc part = agent_rsrc(part0), lpart = agent_rsrc(p.lpart);

  // A wave takes tokens wave, wave + W; a lane four outputs of the split partials and four ranks of T's.  Past the end of a
  // batch requests repeat the last: with a branch around each the compiler waits for all before the first is used.
  const int n = n0 + 4 * lane;                               // N % 64 == 0: four outputs are inside or outside together
  const bool n_ok = n < N, t_lane = 4 * lane < p.r;
  f32x4 acc[PW], v[PW][PB], lp[PW][LB];
  auto part_load = [&](int u, int s0) {
    const uint32_t at = (uint32_t)((wave + W * u) * ld_tok + (n_ok ? 4 * lane : 0));
    auto one = [&](int q) { v[u][q] = agent_load(part, at + (uint32_t)((s0 + q < n_part ? s0 + q : n_part - 1) * ld_part)); };
    one(0);
    one(1);
    if (!EXACT || n_part - s0 > 2) {
#pragma unroll
      for (int q = 2; q < PB; ++q) one(q);
    }
  };
  auto t_load = [&](int u, int q0) {
#pragma unroll
    for (int q = 0; q < LB; ++q) {
      const int qc = q0 + q < p.n_lparts ? q0 + q : (p.n_lparts > 0 ? p.n_lparts - 1 : 0);
      lp[u][q] = agent_load(lpart, (uint32_t)((qc * p.M + wave + W * u) * p.r + (t_lane ? 4 * lane : 0)));
    }
  };
  OutTile<BWD, NT> tile;
#pragma unroll
  for (int u = 0; u < PW; ++u)
    if (wave + W * u < p.M) {                                // uniform
      if (!EXACT || p.r > 0) t_load(u, 0);
      part_load(u, 0);
    }
  if (!EXACT || p.r > 0) tile_load(tile, p, slab, 0);
  if (p.r > 0) {
    if (meet && !met()) return;                              // the adapter came after the bounded wait: the slab is its
#pragma unroll
    for (int u = 0; u < PW; ++u) {
      const int m = wave + W * u;
      if (m >= p.M) continue;
      if (meet) t_load(u, 0);
      f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int q0 = 0;;) {
#pragma unroll
        for (int q = 0; q < LB; ++q)
          if (q0 + q < p.n_lparts) t += lp[u][q];
        q0 += LB;
        if (q0 >= p.n_lparts) break;
        t_load(u, q0);
      }
      if (!t_lane) t = f32x4{0.f, 0.f, 0.f, 0.f};
      uint2 term[3];
      split3(t, term);
      if (4 * lane < rp) {
#pragma unroll
        for (int k = 0; k < 3; ++k) *(uint2*)(Tp + k * kTPlane + m * kTPitch + 4 * lane) = term[k];
      }
      if (p.hl && slab == 0 && t_lane) {
        uint2 hi, lo;
        split_hl(t, hi, lo);
        *(uint2*)(p.hl + (int64_t)m * 2 * p.r + 4 * lane) = hi;
        *(uint2*)(p.hl + (int64_t)m * 2 * p.r + p.r + 4 * lane) = lo;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < PW; ++u) {                             // the splits in their fixed order
    acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave + W * u >= p.M) continue;
    for (int s0 = 0;;) {
#pragma unroll
      for (int q = 0; q < PB; ++q)
        if (s0 + q < n_part) acc[u] += v[u][q];
      s0 += PB;
      if (s0 >= n_part) break;
      part_load(u, s0);
    }
  }
  if (p.r > 0) {
    f32x4 lora[PW];
#pragma unroll
    for (int c = 0; c < PW; ++c) lora[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < p.r; j0 += RC) {
      OutTile<BWD, NT> cur = tile;
      if (!BWD) {
        if (j0 > 0) __syncthreads();                         // previous tile consumed
#pragma unroll
        for (int it = 0; it < IT; ++it) {
          const int e = it * NT + threadIdx.x;
          *(u32x4*)(Bs + (e >> 5) * kTPitch + 8 * (e & 31)) = tile.v[it];
        }
      }
      if (j0 + RC < p.r) tile_load(tile, p, slab, j0 + RC);
      if (!BWD || j0 == 0) __syncthreads();                  // T, and the tile, visible
#pragma unroll
      for (int t0 = 0; t0 < RC; t0 += 32) {
        if (j0 + t0 >= rp) break;
        bf16x8 tt[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) tt[k] = *(const bf16x8*)(Tp + k * kTPlane + i * kTPitch + j0 + t0 + 8 * g);
#pragma unroll
        for (int c = 0; c < PW; ++c) {
          u32x4 w;                                           // ranks t0 + 8g .. +7 of output 16 (wave + W c) + i
          if (!BWD) {
            const uint16_t* src = Bs + (t0 + 8 * g) * kTPitch + 16 * (wave + W * c) + i;
#pragma unroll
            for (int d = 0; d < 4; ++d)
              w[d] = (uint32_t)src[2 * d * kTPitch] | (uint32_t)src[(2 * d + 1) * kTPitch] << 16;
          } else {
            w = cur.v[2 * c + t0 / 32];
          }
#pragma unroll
          for (int k = 0; k < 3; ++k)
            lora[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), tt[k], lora[c], 0, 0, 0);
        }
      }
    }
    __syncthreads();                                         // everybody is done with the terms of T
#pragma unroll
    for (int c = 0; c < PW; ++c) *(f32x4*)(sum + i * kSumPitch + 16 * (wave + W * c) + 4 * g) = lora[c];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PW; ++u)
      if (wave + W * u < p.M) {
        const f32x4 l = *(const f32x4*)(sum + (wave + W * u) * kSumPitch + 4 * lane);
#pragma unroll
        for (int d = 0; d < 4; ++d) acc[u][d] += p.scale * l[d];
      }
  }
  if (!n_ok) return;
#pragma unroll
  for (int u = 0; u < PW; ++u)
    if (wave + W * u < p.M) {
      uint2 q;
      q.x = pack_bf16x2(acc[u][0], acc[u][1]);
      q.y = pack_bf16x2(acc[u][2], acc[u][3]);
      *(uint2*)(p.out + (int64_t)(wave + W * u) * N + n) = q;
    }
}

}  // namespace few
}  // namespace qlora
