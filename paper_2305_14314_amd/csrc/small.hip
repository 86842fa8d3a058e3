// Skinny bf16 MFMA GEMMs of the LoRA branch (arXiv 2305.14314, Eq. 3 / Eq. 5 and the adapter
// gradients): T = X L1, U = dY L2^T, dL1 = s X^T U, dL2 = s T^T dY.  One dimension is the adapter
// rank (<= 256), so these are bound by streaming X or dY from HBM, not by MFMA.
//
//   part[split][I x J] (fp32) = sum over this split's K range of A(i,k) * B(k,j)
//   finalize (fin.hpp): out = bf16(scale * sum over splits) and/or the sum as a [hi | lo] pair of bf16 matrices; dL1 and
//   dL2 do it in the product's own epilogue where small_groups says so: their splits are then groups of four waves in one
//   workgroup, whose sums meet in LDS.  What that saves is the finalize launch (4 - 6 us) and the partials' way through
//   memory; the loop is the same.  dL1 and dL2 of 4096 x 4096, rank 64, 512 tokens under dropout, kernels' times: 9.0 + 4.6 ->
//   10.1 us; of stacked q, k, v of 5120 x 5120 at 2000 tokens 40.4 + 6.3 -> 43.5
//
// Up to eight such products (of one or more layers) share a launch, and so do their finalize steps, which may also ride in
// a dequantise launch.  A stacked q / k / v forward + backward at 2000 tokens (5120 x 5120, rank 64) spent 204 of 770 us in
// 28 launches of 5 - 12 us here; it takes 95 us in 5 now, and a launch streams X or dY at 2.6 - 3.1 TB/s.
//
// Such a pair carries 16 significant bits of an intermediate (T or U) into the adapter gradients.  Where it is
// an operand (HL = 1: A, HL = 2: B) the kernel loads both halves' tiles and issues two MFMAs per fragment of
// the other operand into the same accumulators, so X (resp. dY) is streamed once.
//
// MASK: LoRA dropout on the adapter's input (hyperparameter appendix): operand A is X, and an element of X enters as
// zero where its bit in the caller's keep-mask (bit e % 8 of byte e / 8 for the flat element index e = token * h + k)
// is clear; the 1/(1-p) of the kept elements is folded into the scale of the finalize step.
//
// Operand layouts are template flags: TA = false means A is stored [i][k] (K-contiguous),
// TA = true means A is stored [k][i] (the contraction index is the row index, as for X^T);
// likewise TB for B ([j][k] or [k][j]).  K-contiguous tiles are kept in LDS XOR-swizzled in 16-byte
// chunks and read with ds_read_b128; row-index-contracted tiles are kept as loaded ([k][64 rows], pitch 72)
// and their MFMA fragments come from the transposing LDS read of gfx950 (ds_read_b64_tr_b16): within a group
// of 16 lanes, lane c supplies the address of an 8-byte chunk and lane i receives element i % 4 of the chunks
// i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12 -- so with lane c pointing at (k0 + c / 4, rows R0 + 4 (c % 4) .. +3),
// lane i ends up with row R0 + i at k0 .. k0 + 3, which is half an MFMA fragment (8 gathers of 16 bits before).
#include <algorithm>

#include "common.hpp"
#include "fin.hpp"
#include "launch.hpp"

namespace qlora {

constexpr int ST = 64;                       // tile edge in I, J and K
constexpr int kSmallThreads = 256;
constexpr int kTPitch = 72;                  // elements per k-row of a row-index-contracted tile: 4 consecutive k-rows hit distinct banks
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;

typedef __attribute__((address_space(3))) char lds_char;

// fetch one 16-byte chunk of an operand tile (zero outside the matrix)
template <bool T>
__device__ __forceinline__ u32x4 fetch_chunk(const uint16_t* __restrict__ src, int64_t ld, int r0, int R, int k0,
                                             int k_end, int c) {
  const u32x4 z = {0u, 0u, 0u, 0u};
  if constexpr (!T) {                         // src[row][k]: chunk = (row, 8 consecutive k)
    const int row = r0 + (c >> 3), k = k0 + (c & 7) * 8;
    if (row < R && k < k_end) return *(const u32x4*)(src + (int64_t)row * ld + k);
    return z;
  } else {                                    // src[k][row]: chunk = (k, 8 consecutive rows)
    const int k = k0 + (c >> 3), row = r0 + (c & 7) * 8;
    if (k < k_end && row < R) return *(const u32x4*)(src + (int64_t)k * ld + row);
    return z;
  }
}

// the same for operand A under a keep-mask: a chunk is 8 consecutive elements of storage, i.e. one mask byte
template <bool T>
__device__ __forceinline__ u32x4 fetch_chunk_masked(const uint16_t* __restrict__ src, const uint8_t* __restrict__ mask,
                                                    int64_t ld, int r0, int R, int k0, int k_end, int c) {
  u32x4 v = {0u, 0u, 0u, 0u};
  int64_t off;
  bool ok;
  if constexpr (!T) {
    const int row = r0 + (c >> 3), k = k0 + (c & 7) * 8;
    ok = row < R && k < k_end;
    off = (int64_t)row * ld + k;
  } else {
    const int k = k0 + (c >> 3), row = r0 + (c & 7) * 8;
    ok = k < k_end && row < R;
    off = (int64_t)k * ld + row;
  }
  if (ok) {
    v = *(const u32x4*)(src + off);
    const uint32_t b = mask[off >> 3];                       // ld and the chunk start are multiples of 8
#pragma unroll
    for (int d = 0; d < 4; ++d)
      v[d] &= (((b >> (2 * d)) & 1u) ? 0x0000ffffu : 0u) | (((b >> (2 * d + 1)) & 1u) ? 0xffff0000u : 0u);
  }
  return v;
}

template <bool T>
__device__ __forceinline__ void stash_chunk(lds_char* tile, int c, u32x4 v) {
  if constexpr (!T) {
    const int row = c >> 3, kc = c & 7;
    *(u32x4 __attribute__((address_space(3)))*)(tile + row * 128 + ((kc ^ (row & 7)) * 16)) = v;
  } else {
    *(u32x4 __attribute__((address_space(3)))*)(tile + (c >> 3) * (kTPitch * 2) + (c & 7) * 16) = v;   // [k][64 rows], as loaded
  }
}

// MFMA 32x32x16 fragment: lane holds row (lane % 32) of the 32-row sub-tile, 8 consecutive k
template <bool T>
__device__ __forceinline__ bf16x8 small_frag(const lds_char* tile, int row, int kk, int half) {
  if constexpr (!T) {
    const int chunk = (2 * kk + half) ^ (row & 7);
    return *(const bf16x8 __attribute__((address_space(3)))*)(tile + row * 128 + chunk * 16);
  } else {
    // lane l = 32 half + row32: 16-lane group g = l / 16 covers rows R0 = 16 (g % 2) .. +15 of the sub-tile
    const int lane = threadIdx.x & 63, c = lane & 15;
    const int r0 = (row & ~31) + (lane & 16);               // first row of this group's 16 rows
    const int k0 = kk * 16 + half * 8;
    const lds_char* src = tile + ((k0 + (c >> 2)) * kTPitch + r0 + 4 * (c & 3)) * 2;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)src);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(src + 4 * kTPitch * 2));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
    const s16x8 f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, f);
  }
}

// What the loop over K reads of a job, held in scalar registers.  A job is read through an index into the kernel's arguments,
// and the compiler would rather read it again in front of every predicated load than keep it: eight scalar loads and their
// waits per two K-steps (U of 4096 tokens by 16384 outputs at rank 128, under the profiler: 51 us so, 43 with them held).
struct SmallOperands { const uint16_t *A, *B; const uint8_t* amask; int64_t lda, ldb, hl_off; int I, J, K, k_per_split; };
template <typename T> __device__ __forceinline__ T* pin(T* q) {
  uint64_t u = (uint64_t)q;
  asm volatile("" : "+s"(u));
  return (T*)(__attribute__((address_space(1))) T*)u;        // still known to be global memory
}
__device__ __forceinline__ SmallOperands pin_operands(const SmallJob& j) {
  SmallOperands p{pin(j.A), pin(j.B), pin(j.amask), j.lda, j.ldb, j.hl_off, j.I, j.J, j.K, j.k_per_split};
  asm volatile("" : "+s"(p.lda), "+s"(p.ldb), "+s"(p.hl_off), "+s"(p.I), "+s"(p.J), "+s"(p.K), "+s"(p.k_per_split));
  return p;
}

constexpr int kSmallTile = ST * kTPitch * 2;  // bytes of one operand tile in LDS
// G > 1: a tile's K ranges are summed by G groups of four waves in one workgroup, each with operand tiles of its own
// (27 KB: one workgroup of four groups to a CU, two of two).
template <bool TA, bool TB, int HL, bool MASK, int G>
__device__ __forceinline__ void small_gemm_body(const SmallJob& job, int local, char* smem0) {
  const SmallOperands p = pin_operands(job);
  static_assert(HL == 0 || (HL == 1 && TA) || (HL == 2 && TB), "a [hi | lo] operand is stored token-major");
  static_assert(!MASK || HL != 1, "the masked operand is X itself");
  const int group = G > 1 ? (int)threadIdx.x / kSmallThreads : 0;
  constexpr int kGroupLds = (HL != 0 ? 3 : 2) * kSmallTile;
  char* smem = smem0 + group * kGroupLds;
  lds_char* sA = (lds_char*)smem;
  lds_char* sB = (lds_char*)(smem + kSmallTile);
  lds_char* sC = (lds_char*)(smem + 2 * kSmallTile);
  const int gi = (p.I + ST - 1) / ST, gj = (p.J + ST - 1) / ST;
  const int bi = local % gi, bj = local / gi % gj, split = G > 1 ? group : local / (gi * gj);

  const int tid = G > 1 ? (int)threadIdx.x % kSmallThreads : threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i0 = bi * ST, j0 = bj * ST;
  const int k_begin = split * p.k_per_split;
  const int k_end = (k_begin + p.k_per_split < p.K) ? k_begin + p.k_per_split : p.K;
  const int wi = wave >> 1, wj = wave & 1;
  const int a_row = wi * 32 + (lane & 31), b_row = wj * 32 + (lane & 31), half = lane >> 5;
  const uint16_t* lo_src = (HL == 1) ? p.A + p.hl_off : p.B + p.hl_off;
  const int64_t lo_ld = (HL == 1) ? p.lda : p.ldb;
  const int lo_r0 = (HL == 1) ? i0 : j0, lo_R = (HL == 1) ? p.I : p.J;

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

  // Two steps of operand tiles are kept in flight in registers (sets 0 and 1 alternate): with two or three
  // workgroups per CU one step ahead is too little to cover the HBM latency.
  struct Regs { u32x4 a[2], b[2], c[2]; };
  auto fetch = [&](Regs& R, int k0) {                       // k0 >= k_end loads nothing and yields zeros
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if constexpr (MASK) R.a[u] = fetch_chunk_masked<TA>(p.A, p.amask, p.lda, i0, p.I, k0, k_end, tid + 256 * u);
      else R.a[u] = fetch_chunk<TA>(p.A, p.lda, i0, p.I, k0, k_end, tid + 256 * u);
      R.b[u] = fetch_chunk<TB>(p.B, p.ldb, j0, p.J, k0, k_end, tid + 256 * u);
      if constexpr (HL != 0) R.c[u] = fetch_chunk<true>(lo_src, lo_ld, lo_r0, lo_R, k0, k_end, tid + 256 * u);
    }
  };
  auto step = [&](Regs& R, int k_next) {
    __syncthreads();                                        // previous step's fragment reads are done
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      stash_chunk<TA>(sA, tid + 256 * u, R.a[u]);
      stash_chunk<TB>(sB, tid + 256 * u, R.b[u]);
      if constexpr (HL != 0) stash_chunk<true>(sC, tid + 256 * u, R.c[u]);
    }
    __syncthreads();
    fetch(R, k_next);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const bf16x8 a = small_frag<TA>(sA, a_row, kk, half);
      const bf16x8 b = small_frag<TB>(sB, b_row, kk, half);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
      if constexpr (HL == 1) {
        const bf16x8 a2 = small_frag<true>(sC, a_row, kk, half);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b, acc, 0, 0, 0);
      }
      if constexpr (HL == 2) {
        const bf16x8 b2 = small_frag<true>(sC, b_row, kk, half);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b2, acc, 0, 0, 0);
      }
    }
  };
  Regs R0, R1;
  fetch(R0, k_begin);
  fetch(R1, k_begin + ST);
  const int k_last = G > 1 ? k_begin + p.k_per_split : k_end;   // every group takes part in every barrier: past k_end it adds zeros
  for (int k0 = k_begin; k0 < k_last; k0 += 2 * ST) {
    step(R0, k0 + 2 * ST);
    if (k0 + ST < k_last) step(R1, k0 + 3 * ST);
  }

  const int j = j0 + wj * 32 + (lane & 31);
  if constexpr (G > 1) {                                     // the finalize step's sum, in its order; a group takes 1/G of the tile
    static_assert(HL != 0 && kGroupLds >= 16 * kSmallThreads * 4, "a group's tiles make room for its sums");
    __syncthreads();
    float* mine = (float*)smem + tid;
#pragma unroll
    for (int v = 0; v < 16; ++v) mine[v * kSmallThreads] = acc[v];
    __syncthreads();
    if (j >= p.J) return;
#pragma unroll
    for (int q = 0; q < 16 / G; ++q) {
      const int v = group * (16 / G) + q, i = i0 + wi * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
      if (i >= p.I) continue;
      float sum = 0.0f;
#pragma unroll
      for (int g = 0; g < G; ++g) sum += ((const float*)(smem0 + g * kGroupLds))[v * kSmallThreads + tid];
      if (job.fin.out0) job.fin.out0[(int64_t)i * job.fin.ld0 + j] = bf16_bits(sum * job.fin.scale0);
      if (job.fin.acc) job.fin.acc[(int64_t)i * p.J + j] += sum * job.fin.scale0;
    }
    return;
  }
  if (j >= p.J) return;
  if (HL != 0 && job.direct) {                               // one split: what the finalize step would do, right here
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = i0 + wi * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
      if (i >= p.I) continue;
      if (job.fin.out0) job.fin.out0[(int64_t)i * job.fin.ld0 + j] = bf16_bits(acc[v] * job.fin.scale0);
      if (job.fin.acc) job.fin.acc[(int64_t)i * p.J + j] += acc[v] * job.fin.scale0;
    }
    return;
  }
  float* out = const_cast<float*>(job.fin.part) + (int64_t)split * p.I * p.J;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = i0 + wi * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
    if (i < p.I) out[(int64_t)i * p.J + j] = acc[v];
  }
}

template <int KIND, bool MASK, int G = 1>
__device__ __forceinline__ void small_gemm_kind(const SmallJob& p, int local, char* smem) {
  if constexpr (KIND == kSmallT) small_gemm_body<false, true, 0, MASK, 1>(p, local, smem);
  if constexpr (KIND == kSmallU) small_gemm_body<false, false, 0, false, 1>(p, local, smem);
  if constexpr (KIND == kSmallDL1) small_gemm_body<true, true, 2, MASK, G>(p, local, smem);
  if constexpr (KIND == kSmallDL2) small_gemm_body<true, true, 1, false, G>(p, local, smem);
}
constexpr int small_lds(int kinds) { return ((kinds & 12) ? 3 : 2) * kSmallTile; }

// One product: its job alone is the argument (a list is 1.4 KB to hand over and three dependent reads to find the job in:
// 0.4 us a launch).
template <int KIND, bool MASK>
__global__ __launch_bounds__(kSmallThreads) void small_job_kernel(const SmallJob job) {
  __shared__ __attribute__((aligned(16))) char smem[small_lds(1 << KIND)];
  small_gemm_kind<KIND, MASK>(job, blockIdx.x, smem);
}

// Several products in one launch: workgroup b belongs to the last job whose first workgroup is <= b.  KINDS: the kinds that
// occur (1 << kind), so that a launch carries no code it cannot reach.
template <int KINDS, bool MASK, int G = 1>
__global__ __launch_bounds__(kSmallThreads * G) void small_jobs_kernel(const SmallJobs jobs) {
  static_assert(G == 1 || !(KINDS & 3), "groups finish dL1 and dL2 only");
  __shared__ __attribute__((aligned(16))) char smem[G * small_lds(KINDS)];
  int q = 0;
  while (q + 1 < jobs.n && (int)blockIdx.x >= jobs.first[q + 1]) ++q;
  const SmallJob& p = jobs.j[q];
  const int local = blockIdx.x - jobs.first[q];
  if ((KINDS & 1) && p.kind == kSmallT) small_gemm_kind<kSmallT, MASK>(p, local, smem);
  if ((KINDS & 2) && p.kind == kSmallU) small_gemm_kind<kSmallU, MASK>(p, local, smem);
  if ((KINDS & 4) && p.kind == kSmallDL1) small_gemm_kind<kSmallDL1, MASK, G>(p, local, smem);
  if ((KINDS & 8) && p.kind == kSmallDL2) small_gemm_kind<kSmallDL2, MASK, G>(p, local, smem);
}

__global__ __launch_bounds__(kFinThreads) void fin_job_kernel(const FinJob job) { fin_job(job, blockIdx.x, gridDim.x); }
__global__ __launch_bounds__(kFinThreads) void fin_kernel(const FinList f) { fin_block(f, blockIdx.x); }

// ~2 workgroups per CU over all jobs of a launch: every further split adds an fp32 partial tile to write and read back,
// and past this point that traffic costs more than the extra loads in flight gain (measured: 256 -> +30 %, 1024 -> +8 %
// time).  `floor`: the job's own workgroups are not fewer than that.  Without it the small one of two unlike gradients is
// left with a few long chains that outlast the launch: dL1 and dL2 of 16384 x 64 at rank 128 and 4096 tokens (512 and 2
// tiles, one split each) 115 us, with dL2 in 64 splits 78; 8192 x 2048, rank 256 98 -> 89; 5120 x 13824, rank 16 66 -> 62.
int small_job_splits(int I, int J, int K, int other_tiles, int floor) {
  const int ksteps = (K + ST - 1) / ST, own = small_tiles(I, J), tiles = own + other_tiles;
  return std::max(1, std::min(std::min(std::max((512 + tiles - 1) / tiles, (floor + own - 1) / own), 64), ksteps));
}
int small_tiles(int I, int J) { return ((I + ST - 1) / ST) * ((J + ST - 1) / ST); }

// Whole backward calls, us, with partials and a finalize launch -> finished in the products' launch.
// - Up to four K-steps (256 tokens) one group reads them in a chain that is no longer than a finalize launch; while there is
//   a CU to every tile, as many groups as K-steps shorten it: 4096 x 4096, rank 64, 256 tokens, one -> four groups 64.4 -> 63.1.
//   With more tiles the wide workgroups queue up: 5120 x 13824, rank 64 (296 tiles) 130.8 -> 132.9.
// - Five to eight K-steps: four groups while there is a CU to every tile, 4096 x 4096, rank 64, 512 tokens 85.1 -> 80.3; two up to 512
//   tiles, where four take a second round (257 - 352 tiles, 119 calls: by four as long as with partials on average, by two 3.6 us shorter: 262 tokens 3072 x 14080,
//   rank 16, dropout 22.0, by four 24.9, by two 21.2); 688 tiles and more lose (4096 x 11008, rank 256, 330 tokens 200 -> 205), see below.
// - Longer chains: four groups to a tile leave the CUs without a tile idle, so up to one tile per CU it takes enough of them
//   for the length: 1024 tokens (16 K-steps), 64 tiles +0.5, 80 tiles 74.9 -> 71.7, 256 tiles 320 -> 316; 1400 tokens, 112 and
//   144 tiles +0.7, 2048 tokens, 160 tiles 226.8 -> 225.2; 3000 tokens, 256 tiles 239 -> 236.
// - More tiles than CUs have two splits, i.e. two groups, which do not spread as well as split workgroups if the tiles are
//   few: 600 tokens, 288 tiles 327 -> 322, but 4096 tokens, 288 tiles +5 and 320 tiles 188 -> 194; 472 tiles at 1024 tokens
//   867 -> 860, at 4096 and stacked q, k, v of 2000 tokens (480 tiles) even.  Where `floor` gives a product of few tiles more splits than
//   that, it keeps them.
// - From 512 tiles on a tile has one split, which needs no sum: 4096 x 11008, rank 256 (944 tiles), 512 tokens 236 -> 225;
//   11008 x 4096 at 4096 tokens 757 -> 751.
int small_groups(int K, int tiles, int least) {
  const int ksteps = (K + ST - 1) / ST;
  if (ksteps <= 4) return tiles > 256 || ksteps == 1 ? 1 : ksteps == 2 ? 2 : 4;
  if (ksteps <= 8 && tiles <= 512) return tiles <= 256 ? 4 : 2;
  if (tiles <= 256) return tiles >= 5 * ksteps && (ksteps <= 16 || tiles >= 150) ? 4 : 0;
  if (tiles < 512) return least >= 128 && (ksteps <= 16 || tiles >= 400) ? 2 : 0;
  return least >= 256 ? 1 : 0;
}

hipError_t launch_small_jobs(SmallJobs& jobs, hipStream_t st) {
  if (jobs.n == 0) return hipSuccess;
  if (jobs.groups != 1 && jobs.groups != 2 && jobs.groups != 4) return hipErrorInvalidValue;
  int kinds = 0, wgs = 0;
  bool mask = false;
  for (int q = 0; q < jobs.n; ++q) {
    SmallJob& p = jobs.j[q];
    const int ksteps = (p.K + ST - 1) / ST;
    const int splits = p.direct ? jobs.groups : p.fin.splits;
    p.k_per_split = (ksteps + splits - 1) / splits * ST;
    p.fin.I = p.I; p.fin.J = p.J;
    if (p.direct ? (p.kind != kSmallDL1 && p.kind != kSmallDL2) || p.fin.splits != 1 || p.fin.hl || (p.fin.out0 && p.fin.w0 != p.J)
                 : jobs.groups != 1)
      return hipErrorInvalidValue;
    if (p.amask && (p.lda % 8 != 0 || (p.kind != kSmallT && p.kind != kSmallDL1))) return hipErrorInvalidValue;
    kinds |= 1 << p.kind;
    mask |= p.amask != nullptr;
    jobs.first[q] = wgs;
    wgs += small_tiles(p.I, p.J) * p.fin.splits;
  }
  if (mask)                                                  // one mask for a launch: every T and dL1 job brings it
    for (int q = 0; q < jobs.n; ++q)
      if ((jobs.j[q].kind == kSmallT || jobs.j[q].kind == kSmallDL1) && !jobs.j[q].amask) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs), block(kSmallThreads * jobs.groups);
#define QL_SMALL_G(KINDS, MASK, G)                                                                                   \
  case (2 * KINDS + MASK) * 8 + G: hipLaunchKernelGGL((small_jobs_kernel<KINDS, MASK, G>), grid, block, 0, st, jobs); break;
  if (jobs.groups > 1) {
    switch ((2 * kinds + mask) * 8 + jobs.groups) {
      QL_SMALL_G(4, 0, 2) QL_SMALL_G(4, 1, 2) QL_SMALL_G(8, 0, 2) QL_SMALL_G(12, 0, 2) QL_SMALL_G(12, 1, 2)
      QL_SMALL_G(4, 0, 4) QL_SMALL_G(4, 1, 4) QL_SMALL_G(8, 0, 4) QL_SMALL_G(12, 0, 4) QL_SMALL_G(12, 1, 4)
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
#undef QL_SMALL_G
#define QL_SMALL_ONE(KIND, MASK)                                                                                     \
  case 2 * (1 << KIND) + MASK: hipLaunchKernelGGL((small_job_kernel<KIND, MASK>), grid, block, 0, st, jobs.j[0]); break;
#define QL_SMALL(KINDS, MASK)                                                                                        \
  case 2 * KINDS + MASK: hipLaunchKernelGGL((small_jobs_kernel<KINDS, MASK>), grid, block, 0, st, jobs); break;
  if (jobs.n == 1) {
    switch (2 * kinds + mask) {
      QL_SMALL_ONE(kSmallT, 0) QL_SMALL_ONE(kSmallT, 1) QL_SMALL_ONE(kSmallU, 0) QL_SMALL_ONE(kSmallDL1, 0)
      QL_SMALL_ONE(kSmallDL1, 1) QL_SMALL_ONE(kSmallDL2, 0)
      default: return hipErrorInvalidValue;
    }
  } else {                                                   // a layer's T with dL1, dL1 with dL2; the same of stacked layers (no mask)
    switch (2 * kinds + mask) {
      QL_SMALL(1, 0) QL_SMALL(2, 0) QL_SMALL(3, 0) QL_SMALL(4, 0) QL_SMALL(5, 0) QL_SMALL(5, 1) QL_SMALL(8, 0) QL_SMALL(12, 0)
      QL_SMALL(12, 1)
      default: return hipErrorInvalidValue;
    }
  }
#undef QL_SMALL_ONE
#undef QL_SMALL
  return hipGetLastError();
}

int FinList::add(const FinJob& job) {
  j[n] = job;
  const int64_t quads = (int64_t)job.I * std::max(job.out0 ? job.w0 : 0, job.J) / 4;
  const int blocks = (int)std::min<int64_t>((quads + kFinThreads - 1) / kFinThreads, 1024);
  first[n + 1] = first[n] + blocks;
  return ++n;
}

hipError_t launch_fin(const FinList& f, hipStream_t st) {
  if (f.n == 0) return hipSuccess;
  const dim3 grid((unsigned)f.blocks()), block(kFinThreads);
  if (f.n == 1) hipLaunchKernelGGL(fin_job_kernel, grid, block, 0, st, f.j[0]);
  else hipLaunchKernelGGL(fin_kernel, grid, block, 0, st, f);
  return hipGetLastError();
}

// LoRA dropout, input gradient: the main GEMM has written dX = dY What^T + Us L1^T with Us = bf16(s/(1-p) dY L2^T),
// which is right wherever the adapter saw the input element; a dropped element gets no gradient through the
// adapter, so its adapter term -- recomputed here from the same bf16 operands -- is taken off again (one more
// rounding for those elements).  A workgroup takes 256 mask bytes (2048 consecutive elements), lists the dropped
// ones in LDS (a few per cent) and spreads them over its threads, eight lanes to a dot product of length r: with
// one thread per mask byte nearly every wave would walk all eight bit positions for two or three useful lanes.
__global__ __launch_bounds__(256) void dropout_dx_fix_kernel(uint16_t* __restrict__ dX, int64_t n_bytes, int h,
                                                             const uint8_t* __restrict__ mask,
                                                             const uint16_t* __restrict__ Us, int ld_us,
                                                             const uint16_t* __restrict__ L1, int r) {
  __shared__ uint16_t list[2048];
  __shared__ int wave_cnt[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t q = (int64_t)blockIdx.x * 256 + tid;
  const uint32_t drop = q < n_bytes ? (~(uint32_t)mask[q]) & 0xffu : 0u;
  const int cnt = __builtin_popcount(drop);
  // exclusive prefix sum of cnt over the workgroup: within the wave by shuffles, across the 4 waves through LDS
  int incl = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane == 63) wave_cnt[wave] = incl;
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int c = wave_cnt[w];
    if (w < wave) base += c;
    total += c;
  }
  int pos = base + incl - cnt;
  for (uint32_t d = drop; d != 0; d &= d - 1) list[pos++] = (uint16_t)(tid * 8 + (__builtin_ctz(d)));
  __syncthreads();
  // eight lanes per dropped element, 16 bytes of both rows per lane and step, summed by shuffles; two elements per
  // lane group and iteration, so that the loads of the second are in flight while the first is summed
  const int64_t e_base = (int64_t)blockIdx.x * 2048;
  const int sub = tid & 7;
  for (int idx0 = 0; idx0 < total; idx0 += 64) {             // uniform trip count: the shuffles below need every lane
    int64_t e[2];
    bool live[2];
    float dot[2], old[2];
    u32x4 a[2], w[2];
    const uint16_t* us[2];
    const uint16_t* l1[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const int idx = idx0 + 32 * z + (tid >> 3);
      live[z] = idx < total;
      e[z] = e_base + list[live[z] ? idx : 0];               // flat element index token * h + k
      const int m = (int)(e[z] / h), k = (int)(e[z] - (int64_t)m * h);
      us[z] = Us + (int64_t)m * ld_us;
      l1[z] = L1 + (int64_t)k * r;
      const bool in = 8 * sub < r;                           // r % 16 == 0: a lane's chunk is inside the row or not at all
      a[z] = *(const u32x4*)(us[z] + (in ? 8 * sub : 0));
      w[z] = *(const u32x4*)(l1[z] + (in ? 8 * sub : 0));
      old[z] = bf16_lo_to_f32(dX[e[z]]);
      dot[z] = 0.0f;
      if (!in) { a[z] = u32x4{0u, 0u, 0u, 0u}; }
    }
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      for (int t = 8 * sub;;) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          dot[z] = __builtin_fmaf(bf16_lo_to_f32(a[z][d]), bf16_lo_to_f32(w[z][d]), dot[z]);
          dot[z] = __builtin_fmaf(bf16_lo_to_f32(a[z][d] >> 16), bf16_lo_to_f32(w[z][d] >> 16), dot[z]);
        }
        t += 64;
        if (t >= r) break;
        a[z] = *(const u32x4*)(us[z] + t);
        w[z] = *(const u32x4*)(l1[z] + t);
      }
      dot[z] += __shfl_xor(dot[z], 1, 64);
      dot[z] += __shfl_xor(dot[z], 2, 64);
      dot[z] += __shfl_xor(dot[z], 4, 64);
      if (live[z] && sub == 0) dX[e[z]] = bf16_bits(old[z] - dot[z]);
    }
  }
}

hipError_t launch_dropout_dx_fix(uint16_t* dX, int M, int h, const uint8_t* mask, const uint16_t* Us, int ld_us,
                                 const uint16_t* L1, int r, hipStream_t st) {
  const int64_t n = (int64_t)M * h / 8;
  hipLaunchKernelGGL(dropout_dx_fix_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, dX, n, h, mask, Us,
                     ld_us, L1, r);
  return hipGetLastError();
}

}  // namespace qlora
