// Blockwise NF4 quantisation with Double Quantization (arXiv 2305.14314, Eq. 1 and Section 3).
//
// Three launches on the caller's stream, no host synchronisation:
//   zero_bins      clears the 256 exponent bins used for the exact mean
//   quantize_nf4   per 64-block: absmax (DPP row reduce), reciprocal, nearest NF4 index (32-bucket table
//                  in LDS plus one comparison), nibble pack;
//                  writes the fp32 constant c2 to scratch and adds it to the exponent bins
//   dq_encode      exact sum of all c2 from the bins, divided by n, rounded once to fp32 (every workgroup for itself: the
//                  2 KB of bins and a few dozen operations, against 5.5 us for a launch of its own; the two
//                  steps together took 11.4 us at 11008 x 4096 and take 7.1); then per run of
//                  256 constants: c2 - mean, absmax -> c1, E4M3 codes
//
// The mean is exact and independent of summation order: every fp32 constant is
// mantissa * 2^(exponent), the mantissas are summed per exponent in 64-bit integers
// (integer atomics commute), and the bins are combined in multi-word integer arithmetic.
#include <algorithm>
#include <mutex>

#include "common.hpp"
#include "dq_mean.hpp"
#include "launch.hpp"

namespace qlora {

// Loads in flight: kQUnroll float4 per lane, kQWgsPerCu workgroups per CU (grid-stride beyond that).  What counts is few
// workgroups with many loads each: every workgroup pays the decision table, and with many of them the last round over a
// matrix is uneven.  Whole call, us, on 4096 x 11008 / 5120 x 5120 / 8192 x 8192 / 8192 x 22016 read cold, unroll x
// workgroups: 2 x 6 (the earlier choice) 65 / 48 / 90 / 193; 4 x 4: 60 / 45 / 88 / 200; 6 x 3: 60 / 41 / 89 / 196; 8 x 2:
// 58 / 39 / 89 / 193, with non-temporal loads (the weights are read once) 59 / 39 / 89 / 190; 8 x 3: 60 / 40 / 86 / 199;
// 10 x 2: 58 / 38 / 87 / 202; 12 x 2: 61 / 40 / 91 / 209; 16 x 1: 72 / 47 / 106 / 237.  Matrices of 2 M weights or fewer
// take 25 - 26 us with any of them.
constexpr int kQUnroll = 8, kQWgsPerCu = 2;
constexpr int kQThreads = 256;
typedef __attribute__((ext_vector_type(4))) float q_f32x4;

__global__ void zero_bins_kernel(unsigned long long* bins) { bins[threadIdx.x] = 0ull; }

// One float4 per lane per step; 16 consecutive lanes hold one 64-block.
// MODE 0: NF4.  1: one of the other 4-bit data types (Section 4); its decision thresholds arrive as an argument.
// 2: 8-bit integers, Eq. 1 as printed: q = round_to_nearest_even(fl32(127 / absmax) * x), one signed byte per weight.
template <int MODE>
__global__ __launch_bounds__(kQThreads) void quantize_nf4_kernel(
    const float4* __restrict__ W, int64_t n_vec4,          // n_vec4 = elements / 4
    void* __restrict__ packed,                             // one store per lane: 4 nibbles (16 bit) or 4 bytes
    float* __restrict__ c2_out, unsigned long long* __restrict__ bins, const Thresholds4 thr) {
  constexpr bool OTHER = MODE == 1;
  __shared__ unsigned long long lbins[256];
  __shared__ __attribute__((aligned(256))) Nf4Bucket buckets[32];
  __shared__ float th[16];
  lbins[threadIdx.x] = 0ull;
  nf4_bucket_table_init(buckets, threadIdx.x);
  if (OTHER && threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < 15; ++j) th[j] = thr.t[j];
  }
  __syncthreads();

  // kQUnroll independent float4 loads are issued before any is used.
  const int64_t stride = (int64_t)gridDim.x * kQThreads;
  for (int64_t v0 = (int64_t)blockIdx.x * kQThreads + threadIdx.x; v0 < n_vec4; v0 += kQUnroll * stride) {
    q_f32x4 wv[kQUnroll];
#pragma unroll
    for (int u = 0; u < kQUnroll; ++u) {
      const int64_t v = v0 + u * stride;
      wv[u] = __builtin_nontemporal_load((const q_f32x4*)W + (v < n_vec4 ? v : v0));   // clamped: no branch around the load
    }
#pragma unroll
    for (int u = 0; u < kQUnroll; ++u) {
      const int64_t v = v0 + u * stride;
      if (v >= n_vec4) break;                                 // whole 16-lane rows drop out together
      const q_f32x4 w = wv[u];
      float amax = __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(w.x), __builtin_fabsf(w.y)),
                                   __builtin_fmaxf(__builtin_fabsf(w.z), __builtin_fabsf(w.w)));
      amax = row16_max(amax);                                 // c2 of this lane's block
      // Eq. 1: the constant is range/absmax (range 1); elements are multiplied by it.
      float rc = (amax < __FLT_MIN__) ? 0.0f : __fdiv_rn(MODE == 2 ? 127.0f : 1.0f, amax);
      if constexpr (MODE == 2) {
        if (__builtin_isinf(rc)) rc = 0.0f;                   // 127 / absmax beyond fp32: the block quantises to zeros
        auto q8 = [&](float x) -> uint32_t {                  // the product lies in [-127, 127] up to rounding: clamp anyway
          const float t = __builtin_fminf(__builtin_fmaxf(__builtin_rintf(__fmul_rn(x, rc)), -127.0f), 127.0f);
          return (uint32_t)(int)t & 0xffu;
        };
        ((uint32_t*)packed)[v] = q8(w.x) | (q8(w.y) << 8) | (q8(w.z) << 16) | (q8(w.w) << 24);
      }
      uint32_t i0 = 0, i1 = 0, i2 = 0, i3 = 0;
      if constexpr (MODE == 2) {
      } else if constexpr (OTHER) {
        i0 = index_search4(__fmul_rn(w.x, rc), th);
        i1 = index_search4(__fmul_rn(w.y, rc), th);
        i2 = index_search4(__fmul_rn(w.z, rc), th);
        i3 = index_search4(__fmul_rn(w.w, rc), th);
      } else {
        i0 = nf4_index(__fmul_rn(w.x, rc), buckets);
        i1 = nf4_index(__fmul_rn(w.y, rc), buckets);
        i2 = nf4_index(__fmul_rn(w.z, rc), buckets);
        i3 = nf4_index(__fmul_rn(w.w, rc), buckets);
      }
      if constexpr (MODE != 2) ((uint16_t*)packed)[v] = (uint16_t)(i0 | (i1 << 4) | (i2 << 8) | (i3 << 12));
      if ((threadIdx.x & 15) == 0) {
        c2_out[v >> 4] = amax;
        const uint32_t u32 = __builtin_bit_cast(uint32_t, amax);
        uint32_t e = u32 >> 23, m = u32 & 0x7fffffu;
        if (e == 0) e = 1; else m |= 0x800000u;               // value = m * 2^(e - 150)
        atomicAdd(&lbins[e], (unsigned long long)m);
      }
    }
  }
  __syncthreads();
  const unsigned long long mine = lbins[threadIdx.x];
  if (mine) atomicAdd(&bins[threadIdx.x], mine);
}

// A run of 256 first-level constants at a time; the constants of a workgroup's first run are in flight while it works out
// the mean.
constexpr int kEncWgs = 1024;
__global__ __launch_bounds__(kDqBlock) void dq_encode_kernel(const float* __restrict__ c2, int64_t n,
                                                             const unsigned long long* __restrict__ bins,
                                                             float* __restrict__ mean_out, uint8_t* __restrict__ code,
                                                             float* __restrict__ c1, uint32_t rows, uint32_t bpr) {
  __shared__ float wmax[2][kDqBlock / 64];
  __shared__ unsigned long long lb[256], present[4];
  __shared__ float mean_s;
  static_assert(kDqBlock == 256, "one bin per thread");
  const int64_t runs = (n + kDqBlock - 1) / kDqBlock;
  auto load = [&](int64_t run) {
    const int64_t b = run * kDqBlock + threadIdx.x;
    return c2[b < n ? b : 0];
  };
  float next = load(blockIdx.x);
  const unsigned long long v = bins[threadIdx.x];
  lb[threadIdx.x] = v;
  const unsigned long long some = __ballot(v != 0ull);
  if ((threadIdx.x & 63) == 0) present[threadIdx.x >> 6] = some;
  __syncthreads();
  if (threadIdx.x == 0) {
    mean_s = mean_from_bins(lb, present, (uint32_t)n);
    if (blockIdx.x == 0) *mean_out = mean_s;
  }
  __syncthreads();
  const float mean = mean_s;
  int par = 0;
  for (int64_t run = blockIdx.x; run < runs; run += gridDim.x, par ^= 1) {
    const float c = next;
    const int64_t b = run * kDqBlock + threadIdx.x;
    if (run + gridDim.x < runs) next = load(run + gridDim.x);
    const float d = (b < n) ? __fsub_rn(c, mean) : 0.0f;    // centred constant
    const float m = wave_max(__builtin_fabsf(d));
    if ((threadIdx.x & 63) == 0) wmax[par][threadIdx.x >> 6] = m;
    __syncthreads();                                         // two sets in turn: one barrier per run is enough
    const float amax = __builtin_fmaxf(__builtin_fmaxf(wmax[par][0], wmax[par][1]), __builtin_fmaxf(wmax[par][2], wmax[par][3]));
    float rc1 = (amax < __FLT_MIN__) ? 0.0f : __fdiv_rn(kF8Max, amax);
    if (__builtin_isinf(rc1)) rc1 = 0.0f;
    if (b < n) {                                             // runs follow the flattened order, storage is column-group-major
      const uint32_t row = (uint32_t)b / bpr, blk = (uint32_t)b - row * bpr;
      code[code_pos(rows, (int)bpr, row, (int)blk)] = (uint8_t)e4m3_encode(__fmul_rn(d, rc1));
    }
    if (threadIdx.x == 0) c1[run] = amax;
  }
}

hipError_t launch_quantize(const float* W, int64_t rows, int64_t cols, uint8_t* packed, uint8_t* code, float* c1,
                           float* mean, void* scratch, hipStream_t st, int dtype, bool dq) {
  if (dtype < 0 || dtype >= kNumTypes) return hipErrorInvalidValue;
  const Thresholds4 thr = thresholds4_host(table4_host(dtype));
  const int64_t elems = rows * cols;
  const int64_t n = elems / kBlock;
  unsigned long long* bins = (unsigned long long*)scratch;           // 256 x u64
  // without Double Quantization the first-level constants are the result and go straight to the caller's buffer
  float* c2 = dq ? (float*)((char*)scratch + 256 * sizeof(unsigned long long)) : c1;
  const int64_t n_vec4 = elems / 4;
  int64_t blocks = (n_vec4 + kQThreads - 1) / kQThreads;
  const int64_t cap = 256 * kQWgsPerCu;
  if (blocks > cap) blocks = cap;
  hipLaunchKernelGGL(zero_bins_kernel, dim3(1), dim3(256), 0, st, bins);
  if (dtype == 0)
    hipLaunchKernelGGL(quantize_nf4_kernel<0>, dim3((unsigned)blocks), dim3(kQThreads), 0, st, (const float4*)W,
                       n_vec4, (void*)packed, c2, bins, thr);
  else if (dtype == kTypeInt8)
    hipLaunchKernelGGL(quantize_nf4_kernel<2>, dim3((unsigned)blocks), dim3(kQThreads), 0, st, (const float4*)W,
                       n_vec4, (void*)packed, c2, bins, thr);
  else
    hipLaunchKernelGGL(quantize_nf4_kernel<1>, dim3((unsigned)blocks), dim3(kQThreads), 0, st, (const float4*)W,
                       n_vec4, (void*)packed, c2, bins, thr);
  if (!dq) return hipGetLastError();
  const int64_t n1 = std::min<int64_t>((n + kDqBlock - 1) / kDqBlock, kEncWgs);
  hipLaunchKernelGGL(dq_encode_kernel, dim3((unsigned)n1), dim3(kDqBlock), 0, st, c2, n, bins, mean, code, c1,
                     (uint32_t)rows, (uint32_t)(cols / kBlock));
  return hipGetLastError();
}

// ---- the variant for callers that cannot allocate ---------------------------------------------------------------
// Its scratch (the exponent bins and the fp32 constants c2 of up to kStaticQuantBlocks blocks) is this array; every
// device the library runs on holds its own copy at its own address, found once per device.
static __device__ __align__(256) unsigned char scratch[kQuantBinsBytes + kStaticQuantBlocks * sizeof(float)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t quantize_static_scratch(void** ptr) {
  int dev = -1;
  if (hipError_t e = hipGetDevice(&dev)) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_quantize_static(const float* W, int64_t rows, int64_t cols, uint8_t* packed, uint8_t* code,
                                  float* c1, float* mean, hipStream_t st, int dtype, bool dq) {
  if (rows * cols / kBlock > (int64_t)kStaticQuantBlocks) return hipErrorInvalidValue;
  void* ptr = nullptr;
  if (hipError_t e = quantize_static_scratch(&ptr)) return e;
  return launch_quantize(W, rows, cols, packed, code, c1, mean, ptr, st, dtype, dq);
}

}  // namespace qlora
