// norms.hip - Frobenius norms of attention-state outputs (gfx950).
//
// For listed slots j: || OUT_j - REF ||_2 over all (b, r, h, d), REF optional.
// These feed the error model of the selection planner: the scale ratio
// alpha(i) = ||AS(i)|| / ||AS(i_loc)|| (Sec. 4.1.2, Eq. scale_ratio) and the
// local-state drift ||AS_t(i_loc) - AS_tc(i_loc)|| that the age penalty
// extrapolates (Eq. error_extrapolation).  Bound by HBM: every listed slot is
// read once (and REF once per four slots).  The sums of squares are reduced in
// a fixed order (per workgroup, then one workgroup per slot over the
// partials), so the result is bitwise reproducible.
#include "internal.h"

namespace ditango {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

// 16 bytes of a state (8 bf16 or 4 float32 elements), loaded in the state
// type and squared as float
template <typename T> struct Unit;
template <> struct Unit<__bf16> {
  typedef bf16x8 type;
  typedef f32x8 wide;
  static constexpr int N = 8;
};
template <> struct Unit<float> {
  typedef f32x4 type;
  typedef f32x4 wide;
  static constexpr int N = 4;
};

// the workgroup's sum of x in every thread, in a fixed order: a butterfly
// over the wave, then the waves in order
__device__ __forceinline__ float block_sum(float x, float* red) {
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) x += __shfl_xor(x, k, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < kNormThreads / 64; ++w) sum += red[w];
  return sum;
}

// Each workgroup sums the squares of a fixed range of elements of NS listed
// slots (NS = 1, or up to 4 that share the reference) into
// partial[slot][block].  grid: (blocks per slot, groups of NS slots).
//
// Bound by HBM.  The slots of a call that subtracts a reference are read
// together, so that the reference is read once and not once per slot: four
// snapshots of 9,450 rows x 40 heads at D=128 in bf16 125.8 -> 77.1 us (484 MB
// instead of 774, 6.3 TB/s; the final sums included, one workgroup per slot
// instead of one for all); without a reference 8 slots 136 -> 119 us, 3
// float32 slots 104 -> 88 us (consecutive 16-byte loads).
template <typename T, int NS, bool REF>
__global__ __launch_bounds__(kNormThreads) void norms_partial_kernel(const NormArgs a, int slot0) {
  __shared__ float red[NS][kNormThreads / 64];
  using U = Unit<T>;
  const int tid = threadIdx.x;
  const int s0 = slot0 + blockIdx.y * NS;
  const int64_t units = a.elems / U::N;
  constexpr int kPer = kNormChunksPerBlock * 8 / U::N / kNormThreads;   // units per thread and slot
  const int64_t u0 = (int64_t)blockIdx.x * kPer * kNormThreads + tid;
  const T* src[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) src[j] = (const T*)a.states + (int64_t)a.slots[s0 + j] * a.elems;
  const T* ref = (const T*)a.ref;
  // batches of units: every load of a batch (states and reference) is issued
  // before the first is used, and unconditionally (a unit past the end reads
  // the last unit and is then replaced by zeros, which leave the sum's bits
  // alone): a load under a per-lane condition is waited for inside its branch.
  constexpr int kBatch = NS == 1 ? 8 : 4;
  static_assert(kPer % kBatch == 0, "batches");
  float sum[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) sum[j] = 0.f;
#pragma unroll 1
  for (int i0 = 0; i0 < kPer; i0 += kBatch) {
    typename U::type x[NS][kBatch], y[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int64_t u = u0 + (int64_t)(i0 + i) * kNormThreads;
      const int64_t at = (u < units ? u : units - 1) * U::N;
      if constexpr (REF) y[i] = __builtin_nontemporal_load((const typename U::type*)(ref + at));
#pragma unroll
      for (int j = 0; j < NS; ++j) x[j][i] = __builtin_nontemporal_load((const typename U::type*)(src[j] + at));
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const bool ok = u0 + (int64_t)(i0 + i) * kNormThreads < units;
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        typename U::wide v = __builtin_convertvector(x[j][i], typename U::wide);
        if constexpr (REF) v -= __builtin_convertvector(y[i], typename U::wide);
#pragma unroll
        for (int e = 0; e < U::N; ++e) {
          const float d = ok ? v[e] : 0.f;
          sum[j] = __builtin_fmaf(d, d, sum[j]);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const float t = block_sum(sum[j], red[j]);
    if (tid == 0) a.partial[(int64_t)(s0 + j) * a.blocks + blockIdx.x] = t;
  }
}

// one workgroup per listed slot
__global__ __launch_bounds__(kNormThreads) void norms_final_kernel(const NormArgs a) {
  __shared__ float red[kNormThreads / 64];
  const int si = blockIdx.x;
  float sum = 0.f;
  for (int b = threadIdx.x; b < a.blocks; b += kNormThreads) sum += a.partial[(int64_t)si * a.blocks + b];
  const float t = block_sum(sum, red);
  if (threadIdx.x == 0) a.norms[si] = __builtin_sqrtf(t);
}

template <typename T, int NS, bool REF>
hipError_t launch_slots(const NormArgs& a, int slot0, int groups, hipStream_t s) {
  const dim3 grid((unsigned)a.blocks, (unsigned)groups);
  hipLaunchKernelGGL((norms_partial_kernel<T, NS, REF>), grid, dim3(kNormThreads), 0, s, a, slot0);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_norms_t(const NormArgs& a, hipStream_t s) {
  if (a.ref == nullptr) return launch_slots<T, 1, false>(a, 0, a.n, s);
  hipError_t e = hipSuccess;
  if (a.n >= 4) e = launch_slots<T, 4, true>(a, 0, a.n / 4, s);
  if (e != hipSuccess) return e;
  const int s0 = a.n / 4 * 4;
  switch (a.n - s0) {
    case 1: return launch_slots<T, 1, true>(a, s0, 1, s);
    case 2: return launch_slots<T, 2, true>(a, s0, 1, s);
    case 3: return launch_slots<T, 3, true>(a, s0, 1, s);
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_norms(const NormArgs& a, ditango_dtype dt, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  const hipError_t e = dt == DITANGO_BF16 ? launch_norms_t<__bf16>(a, s) : launch_norms_t<float>(a, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(norms_final_kernel, dim3(a.n), dim3(kNormThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace ditango
