// merge.hip - composition of attention states and contribution weights (gfx950).
//
// merge: the n-ary state composition of Sec. 2.2.4 (Eq. composition),
//   M = max_j LSE_j, LSE = M + log sum_j e^{LSE_j - M}, OUT = sum_j e^{LSE_j - LSE} OUT_j,
// over a list of cached/fresh state slots.  Pure streaming: every OUT slot is
// read once and the output written once, so the kernel is bound by HBM
// bandwidth.  A row's LSE loads are issued first, then its state loads; the
// weights are formed while the states are in flight.
//
// contrib: per-row weights W_j = e^{LSE_j - LSE} (w_i of Sec. 4.1.1; the
// anchor weights of Eq. lse_weight) and their mean over all rows per
// partition, reduced in a fixed order (per workgroup, then one workgroup per
// partition over the partial sums) so results are bitwise reproducible.
#include <string.h>

#include <mutex>

#include "internal.h"

namespace ditango {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// A lane's 8 elements of a state row: loaded in the state type (bf16 chunks
// stay 4 registers until they are weighted), used as float.  `first(ch)` and
// `second(ch)` are the places of their two halves in the row of D elements.
//
// bf16 states: 8 consecutive elements, one 16-byte load.  float32 states: two
// groups of 4, half a row apart, so that the lanes of a row read consecutive
// 16-byte pieces in each of the two loads (8 consecutive floats per lane put
// every load at a 32-byte stride: half of each line per instruction, read
// past the caches; 9,450 rows x 40 heads x 5 float32 slots at D=128, 265 us,
// 4.05 TB/s).
template <typename T, int D> struct Chunk8;
template <int D> struct Chunk8<__bf16, D> {
  typedef bf16x8 type;
  static __device__ __forceinline__ int first(int ch) { return ch * 8; }
  static __device__ __forceinline__ int second(int ch) { return ch * 8 + 4; }
  static __device__ __forceinline__ type load(const __bf16* row, int ch) {
    return __builtin_nontemporal_load((const bf16x8*)(row + ch * 8));
  }
  static __device__ __forceinline__ f32x8 f32(const type& x) { return __builtin_convertvector(x, f32x8); }
};
template <int D> struct Chunk8<float, D> {
  typedef f32x8 type;
  static __device__ __forceinline__ int first(int ch) { return ch * 4; }
  static __device__ __forceinline__ int second(int ch) { return D / 2 + ch * 4; }
  static __device__ __forceinline__ type load(const float* row, int ch) {
    const f32x4 a = __builtin_nontemporal_load((const f32x4*)(row + first(ch)));
    const f32x4 b = __builtin_nontemporal_load((const f32x4*)(row + second(ch)));
    return f32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  }
  static __device__ __forceinline__ f32x8 f32(const type& x) { return x; }
};
// the lane's 8 output elements, at the places its state elements came from
template <typename CK>
__device__ __forceinline__ void store8(__bf16* row, int ch, const f32x8& v) {
  const bf16x8 x = __builtin_convertvector(v, bf16x8);
  if constexpr (sizeof(typename CK::type) == 16) {
    __builtin_nontemporal_store(x, (bf16x8*)(row + CK::first(ch)));
  } else {
    __builtin_nontemporal_store(__builtin_shufflevector(x, x, 0, 1, 2, 3), (bf16x4*)(row + CK::first(ch)));
    __builtin_nontemporal_store(__builtin_shufflevector(x, x, 4, 5, 6, 7), (bf16x4*)(row + CK::second(ch)));
  }
}
template <typename CK>
__device__ __forceinline__ void store8(float* row, int ch, const f32x8& v) {
  __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, (f32x4*)(row + CK::first(ch)));
  __builtin_nontemporal_store(f32x4{v[4], v[5], v[6], v[7]}, (f32x4*)(row + CK::second(ch)));
}

constexpr int kMergeThreads = 64;      // small workgroups keep every CU evenly fed
constexpr int kMergeBatch = 8;         // slots whose loads are in flight together

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) x += __shfl_xor(x, k, 64);
  return x;
}

// Composed log-sum-exp of a row's NMAX values (-inf past the list), which are
// replaced by e^{LSE_j - M}; *sum is their sum.
template <int NMAX>
__device__ __forceinline__ float row_lse(float (&lv)[NMAX], float* sum) {
  float mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < NMAX; ++j) mx = fmaxf(mx, lv[j]);
  float tot = 0.f;
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    lv[j] = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((lv[j] - mx) * kLog2e);
    tot += lv[j];
  }
  *sum = tot;
  return tot > 0.f ? mx + __builtin_amdgcn_logf(tot) * kLn2 : -INFINITY;
}

// e^{LSE_j - LSE}, 0 where either is -inf
__device__ __forceinline__ float weight_of(float lj, float lo) {
  return lo != -INFINITY && lj != -INFINITY ? __builtin_amdgcn_exp2f((lj - lo) * kLog2e) : 0.f;
}

// Row blocks of the mean weights: the sums over one block, and over the
// blocks, are formed in the same order by the weight workgroups of a
// composition and by the weight kernels on their own, so that both give the
// same bits.
constexpr int kContribThreads = 256;
constexpr int kContribRowsPerThread = 2;
constexpr int kContribRowsPerBlock = kContribThreads * kContribRowsPerThread;
constexpr int kContribWaves = kContribThreads / 64;

// One weight workgroup (one wave) of a composition with weights.  The wave
// composes its rows' log-sum-exps itself (the composed ones are being written
// by other workgroups) and forms the sums of w_iters units - a unit is what
// one of the kContribWaves waves of a contrib_partial_kernel workgroup takes.
// contrib_final_kernel, launched after the composition, adds them up.  (The
// last of these waves to finish could do that itself and spare the launch,
// but only by a counter that has to be zero when the call begins: memory that
// was never written, a call that was interrupted, or two calls that overlap on
// a workspace then leave every later call without weights.)
template <int NMAX>
__device__ void weights_block(const MergeArgs& a) {
  constexpr int R = kContribRowsPerThread;
  const int lane = threadIdx.x;
  const int n = a.n;
  const int64_t n_rows = a.rows;
  const int units = a.w_blocks * kContribWaves;
  const int u1 = min(((int)blockIdx.x + 1) * a.w_iters, units);
  for (int u = blockIdx.x * a.w_iters; u < u1; ++u) {
    const int64_t base = (int64_t)(u / kContribWaves) * kContribRowsPerBlock + (u % kContribWaves) * 64 + lane;
    float lv[R][NMAX];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int64_t r = base + i * kContribThreads;
      const int64_t rc = r < n_rows ? r : n_rows - 1;
#pragma unroll
      for (int j = 0; j < NMAX; ++j) {
        lv[i][j] = -INFINITY;
        if (j < n) lv[i][j] = a.lse[(int64_t)a.slots[j] * n_rows + rc];
      }
    }
    float acc[NMAX];
#pragma unroll
    for (int j = 0; j < NMAX; ++j) acc[j] = 0.f;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const bool ok = base + i * kContribThreads < n_rows;
      float e[NMAX], tot;
#pragma unroll
      for (int j = 0; j < NMAX; ++j) e[j] = lv[i][j];
      const float lo = row_lse<NMAX>(e, &tot);
#pragma unroll
      for (int j = 0; j < NMAX; ++j)
        if (j < n) acc[j] += ok ? weight_of(lv[i][j], lo) : 0.f;
    }
    float mine = 0.f;                    // lane j: the sum of slot j
#pragma unroll
    for (int j = 0; j < NMAX; ++j)
      if (j < n) {
        const float t = wave_sum(acc[j]);
        mine = lane == j ? t : mine;
      }
    if (lane < n) a.w_partial[(int64_t)u * n + lane] = mine;
  }
}

// Each thread owns 8 elements of one row (row = (b*q_len + r)*H + h,
// rows contiguous in every slot), so the CPR = D/8 lanes of a row are
// consecutive lanes of one wave.  The thread first issues the loads of the
// row's LSEs (the row's lanes share the addresses, so each load instruction
// touches one line per row), then the state loads of the first batch of
// slots; it forms the row's maximum, log-sum-exp and weights itself (no
// cross-lane exchange, no LDS, no barrier) while the states are in flight,
// and weights each chunk as it lands: OUT = sum_j w_j OUT_j in float32.
// Issuing the LSE loads first makes the weights ready before the first chunk
// arrives, so no chunk waits in registers for them (measured at the
// video-DiT shape: 148.7 / 156.6 us warm / cold against 152.6 / 159.5 us
// with the state loads first).
// NMAX bounds the slot count n (read from the arguments): every loop is
// unrolled over NMAX with wave-uniform guards, so the weights stay in
// registers and small counts (group composition: 2 slots; a composed step:
// a handful) use a small, high-occupancy instantiation.  IDX32: row and LSE
// indices in 32-bit arithmetic (a 64-bit division by a run-time value is a
// long instruction sequence in front of the LSE loads).
// W: with weight workgroups, in instances of their own: a composition without
// weights keeps its registers and waves (bf16 states, D=128, 4 / 8 / 16 / 64
// slots: 38 / 58 / 68 / 142 registers, with weights 36 / 57 / 79 / 195; one
// instance for both, with the final sums in it, took 60 / 100 / 101 / 196.
// 3,000 rows x 12 heads x 20 slots 43.4 -> 36.9 us, 4,095 x 12 x 5 14.9 ->
// 13.4; 9,450 x 40 x 8 138.0 -> 139.0: a launch that HBM alone bounds gains
// nothing from more waves).
template <typename TS, typename TO, int D, int NMAX, bool IDX32, bool W>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(const MergeArgs a) {
  constexpr int CPR = D / 8;                      // chunks (lanes) per row
  using CK = Chunk8<TS, D>;
  int block = (int)blockIdx.x;
  if constexpr (W) {
    block -= a.n_wblocks;
    if (block < 0) {
      weights_block<NMAX>(a);
      return;
    }
  }
  const int n = a.n;
  const int64_t c = (int64_t)block * kMergeThreads + threadIdx.x;
  const bool live = c < a.rows * CPR;
  const int64_t row = live ? c / CPR : 0;
  const int ch = (int)(c % CPR);
  const int64_t slot_elems = a.rows * D;
  const int64_t lse_slot = (int64_t)a.B * a.H * a.q_len;
  const TS* __restrict__ st = (const TS*)a.states + row * D;

  // LSE index of the row: (b*H + h)*q_len + r for row = (b*q_len + r)*H + h
  int64_t li;
  if constexpr (IDX32) {
    const uint32_t r32 = (uint32_t)row, H = (uint32_t)a.H, L = (uint32_t)a.q_len;
    const uint32_t br = r32 / H;
    const uint32_t b = br / L;
    li = (int64_t)((b * H + (r32 - br * H)) * L + (br - b * L));
  } else {
    const int h = (int)(row % a.H);
    const int64_t br = row / a.H;
    li = ((br / a.q_len) * a.H + h) * a.q_len + br % a.q_len;
  }
  // No load is under a per-lane condition (a lane past the last row reads row
  // 0): such a load is issued inside a branch and waited for before the
  // branch ends, which serialises the slots' loads of a thread.  A position
  // past the list is skipped by a branch of the whole wave, which costs
  // nothing; reading its first slot again instead took 60 % more requests at
  // 5 slots of an 8-slot instance (9,450 rows x 40 heads, D=128: bf16 103 ->
  // 92 us, float32 198 -> 167 us; 2 of 4: 58 -> 48 us; 11 of 16 at 8,192 x 24:
  // 117 -> 102 us).
  int sl[NMAX];
#pragma unroll
  for (int j = 0; j < NMAX; ++j) sl[j] = a.slots[j];
  float lv[NMAX];
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    lv[j] = -INFINITY;
    if (j < n) lv[j] = a.lse[(int64_t)sl[j] * lse_slot + li];
  }
  typename CK::type x[kMergeBatch];
#pragma unroll
  for (int u = 0; u < kMergeBatch && u < NMAX; ++u) {
    x[u] = typename CK::type{};
    if (u < n) x[u] = CK::load(st + (int64_t)sl[u] * slot_elems, ch);
  }

  float tot;
  const float lse = row_lse<NMAX>(lv, &tot);
  const float inv = tot > 0.f ? 1.0f / tot : 0.f;
  auto weight = [&](int j) { return lv[j] * inv; };
  f32x8 acc = f32x8{};
#pragma unroll
  for (int u = 0; u < kMergeBatch && u < NMAX; ++u)
    if (u < n) acc += weight(u) * CK::f32(x[u]);
  // later batches: fully unrolled over the largest slot count so that every
  // weight index is a compile-time constant (the weights stay in registers)
#pragma unroll
  for (int j0 = kMergeBatch; j0 < NMAX; j0 += kMergeBatch) {
    if (j0 < n) {
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u)
        if (j0 + u < n) x[u] = CK::load(st + (int64_t)sl[j0 + u] * slot_elems, ch);
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u)
        if (j0 + u < n) acc += weight(j0 + u) * CK::f32(x[u]);
    }
  }
  if (live) {
    store8<CK>((TO*)a.out + row * D, ch, acc);
    if (a.lse_out != nullptr && ch == 0) a.lse_out[li] = lse;
  }
}

template <typename TS, typename TO, int D, bool IDX32, bool W>
void launch_merge_n(const MergeArgs& a, dim3 g, dim3 t, hipStream_t s) {
  if (a.n <= 4)
    hipLaunchKernelGGL((merge_kernel<TS, TO, D, 4, IDX32, W>), g, t, 0, s, a);
  else if (a.n <= 8)
    hipLaunchKernelGGL((merge_kernel<TS, TO, D, 8, IDX32, W>), g, t, 0, s, a);
  else if (a.n <= 16)
    hipLaunchKernelGGL((merge_kernel<TS, TO, D, 16, IDX32, W>), g, t, 0, s, a);
  else
    hipLaunchKernelGGL((merge_kernel<TS, TO, D, kMaxParts, IDX32, W>), g, t, 0, s, a);
}

template <typename TS, typename TO, int D>
hipError_t launch_merge_t(const MergeArgs& a, hipStream_t s) {
  const int64_t blocks = (a.rows * (D / 8) + kMergeThreads - 1) / kMergeThreads;
  if (blocks == 0) return hipSuccess;
  if (blocks + a.n_wblocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  const dim3 g((unsigned)(blocks + a.n_wblocks)), t(kMergeThreads);
  const bool idx32 = a.rows < 0x7fffffffLL;
  if (a.n_wblocks > 0) {
    if (idx32)
      launch_merge_n<TS, TO, D, true, true>(a, g, t, s);
    else
      launch_merge_n<TS, TO, D, false, true>(a, g, t, s);
  } else {
    if (idx32)
      launch_merge_n<TS, TO, D, true, false>(a, g, t, s);
    else
      launch_merge_n<TS, TO, D, false, false>(a, g, t, s);
  }
  return hipGetLastError();
}

template <typename TS, typename TO>
hipError_t launch_merge_d(const MergeArgs& a, int D, hipStream_t s) {
  if (D == 128) return launch_merge_t<TS, TO, 128>(a, s);
  if (D == 64) return launch_merge_t<TS, TO, 64>(a, s);
  return hipErrorInvalidValue;
}

// ---- contribution weights: per-workgroup partial sums, fixed order
//
// Every thread forms the weights of its rows for all listed partitions at
// once (P accumulators in registers), then each partition's sum is reduced
// with a butterfly over the wave (lane l adds lane l^k's value, so every lane
// holds the same bits) and the waves' sums are added in wave order: one
// barrier for all partitions, and bitwise the same result on every run.

// Per-row weights are written through LDS, 16 partitions at a time: a wave's
// 64 rows x P floats are consecutive in memory, and its lanes write them in
// that order (each lane writing its own row put the 64 lanes of a store 4 * P
// bytes apart).  24 heads x 8,192 rows x 16 partitions, both kernels: 31.0 ->
// 15.8 us with the rows (26 MB), 18.1 -> 13.1 us without: the final sums take
// one workgroup per partition instead of one for all.  The weights stay in
// registers until they are staged: 207 of them in the 64-partition instance
// (145 when each lane wrote its row), two waves per SIMD instead of three,
// and still faster (3,000 rows x 12 heads x 40: 45.3 -> 31.1 us with the rows,
// 40.2 -> 23.1 without).
constexpr int kRowsStage = 16;

template <int PMAX>
__global__ __launch_bounds__(kContribThreads) void contrib_partial_kernel(const ContribArgs a) {
  constexpr int R = kContribRowsPerThread;
  __shared__ float red[kContribWaves][PMAX];
  __shared__ float stage[kContribWaves][64 * (kRowsStage + 1)];
  const int tid = threadIdx.x;
  const int P = a.P;
  const int64_t n = a.n_rows;
  const float* __restrict__ lse = a.lse;
  const float* __restrict__ lse_out = a.lse_out;
  float* __restrict__ w_rows = a.w_rows;
  const int64_t base = (int64_t)blockIdx.x * kContribRowsPerBlock;
  // every load of the thread's rows first, then the weights: the loads are
  // all in flight at once.  None is under a per-lane condition (a row past
  // the end reads the last row and is masked afterwards): such a load is
  // waited for inside its branch, one after another; partitions past P are
  // skipped by the whole wave.
  float lo[R], lj[R][PMAX];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int64_t r = base + i * kContribThreads + tid;
    const int64_t rc = r < n ? r : n - 1;
    lo[i] = lse_out[rc];
#pragma unroll
    for (int j = 0; j < PMAX; ++j) {
      lj[i][j] = -INFINITY;
      if (j < P) lj[i][j] = lse[(int64_t)j * n + rc];
    }
  }
  float acc[PMAX];
#pragma unroll
  for (int j = 0; j < PMAX; ++j) acc[j] = 0.f;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const bool ok = base + i * kContribThreads + tid < n;
#pragma unroll
    for (int j = 0; j < PMAX; ++j) {
      if (j < P) {
        const float w = ok ? weight_of(lj[i][j], lo[i]) : 0.f;
        acc[j] += w;
        lj[i][j] = w;
      }
    }
  }
  if (w_rows != nullptr) {
    const int lane = tid & 63;
    float* st = stage[tid >> 6];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int64_t r0 = base + i * kContribThreads + (tid & ~63);     // the wave's first row
      const int rows = (int)min((int64_t)64, n - r0);
#pragma unroll
      for (int j0 = 0; j0 < PMAX; j0 += kRowsStage) {
        if (j0 < P) {
          const int cnt = min(kRowsStage, P - j0);
          // LDS operations of a wave run in order: no barrier
#pragma unroll
          for (int j = 0; j < kRowsStage && j0 + j < PMAX; ++j) st[lane * (kRowsStage + 1) + j] = lj[i][j0 + j];
          __builtin_amdgcn_wave_barrier();
          int row = lane / cnt, col = lane % cnt;
          const int dr = 64 / cnt, dc = 64 % cnt;
          for (int k = 0; k < cnt; ++k) {
            if (row < rows) w_rows[(r0 + row) * P + j0 + col] = st[row * (kRowsStage + 1) + col];
            row += dr;
            col += dc;
            if (col >= cnt) {
              col -= cnt;
              ++row;
            }
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < PMAX; ++j)
    if (j < P) acc[j] = wave_sum(acc[j]);
  if ((tid & 63) == 0) {
#pragma unroll
    for (int j = 0; j < PMAX; ++j)
      if (j < P) red[tid >> 6][j] = acc[j];
  }
  __syncthreads();
  if (tid < P) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kContribWaves; ++w) sum += red[w][tid];
    a.partial[(int64_t)blockIdx.x * P + tid] = sum;
  }
}

// The row blocks' sums added in a fixed order, one workgroup per partition
// (thread t takes blocks t, t + kContribThreads, ...).  A block's sum is one
// partial, or (UNITS > 1) that many, added in order.
template <int UNITS>
__global__ __launch_bounds__(kContribThreads) void contrib_final_kernel(const ContribArgs a) {
  __shared__ float red[kContribWaves];
  const int tid = threadIdx.x;
  const int P = a.P, j = blockIdx.x;
  float acc = 0.f;
  for (int blk = tid; blk < a.n_blocks; blk += kContribThreads) {
    const float* p = a.partial + (int64_t)blk * UNITS * P + j;
    float x[UNITS], block = 0.f;
#pragma unroll
    for (int v = 0; v < UNITS; ++v) x[v] = p[v * P];
#pragma unroll
    for (int v = 0; v < UNITS; ++v) block += x[v];
    acc += block;
  }
  acc = wave_sum(acc);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kContribWaves; ++w) sum += red[w];
    a.w_part[j] = a.n_rows > 0 ? sum / (float)a.n_rows : 0.f;
  }
}

template <int PMAX>
hipError_t launch_contrib_t(const ContribArgs& a, hipStream_t s) {
  if (a.n_blocks > 0) {
    hipLaunchKernelGGL(contrib_partial_kernel<PMAX>, dim3(a.n_blocks), dim3(kContribThreads), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(contrib_final_kernel<1>, dim3(a.P), dim3(kContribThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_merge(const MergeArgs& a, ditango_dtype sdt, ditango_dtype odt, int D, hipStream_t s) {
  if (sdt == DITANGO_BF16 && odt == DITANGO_BF16) return launch_merge_d<__bf16, __bf16>(a, D, s);
  if (sdt == DITANGO_BF16 && odt == DITANGO_F32) return launch_merge_d<__bf16, float>(a, D, s);
  if (sdt == DITANGO_F32 && odt == DITANGO_F32) return launch_merge_d<float, float>(a, D, s);
  if (sdt == DITANGO_F32 && odt == DITANGO_BF16) return launch_merge_d<float, __bf16>(a, D, s);
  return hipErrorInvalidValue;
}

hipError_t launch_compose(const MergeArgs& a, ditango_dtype sdt, ditango_dtype odt, int D, hipStream_t s) {
  const hipError_t e = launch_merge(a, sdt, odt, D, s);
  if (e != hipSuccess) return e;
  ContribArgs c;
  memset(&c, 0, sizeof(c));
  c.w_part = a.w_part;
  c.partial = a.w_partial;
  c.n_rows = a.rows;
  c.P = a.n;
  c.n_blocks = a.w_blocks;
  hipLaunchKernelGGL(contrib_final_kernel<kContribWaves>, dim3(c.P), dim3(kContribThreads), 0, s, c);
  return hipGetLastError();
}

// Up to 256 weight workgroups, each taking as many units as that needs.  They
// come first in the grid and run beside the composition; fewer take longer
// than the composition, more hold up its first workgroups (9,450 rows x 40
// heads x 8 slots at D=128: composition alone 140 us, with weights 145 / 142 /
// 143 / 145 us with up to 128 / 256 / 512 / 1,024 of them, 150 with the two
// weight kernels after it; 14,850 x 48 x 8 at D=64: 148 alone, 205 / 156 / 153
// / 154, 161; 2,048 x 12 x 8 at D=64: 6.0 alone, 11.2 / 8.4 / 8.4 / 8.4, 12.8;
// 3,000 x 12 x 20 at D=128: 43.3 alone, 49.5 / 45.7 / 45.9 / 45.8, 59.1).
constexpr int kComposeBlocks = 256;
int compose_wblocks(int64_t n_rows, int* iters) {
  const int64_t units = contrib_blocks(n_rows) * kContribWaves;
  const int64_t it = (units + kComposeBlocks - 1) / kComposeBlocks;
  *iters = (int)it;
  return (int)((units + it - 1) / it);
}

size_t compose_ws_bytes(int64_t n_rows, int n) {
  return kComposeHeadBytes + (size_t)contrib_blocks(n_rows) * kContribWaves * n * sizeof(float);
}

int64_t contrib_blocks(int64_t n_rows) { return (n_rows + kContribRowsPerBlock - 1) / kContribRowsPerBlock; }

hipError_t launch_contrib(const ContribArgs& a, hipStream_t s) {
  if (a.P <= 8) return launch_contrib_t<8>(a, s);
  if (a.P <= 16) return launch_contrib_t<16>(a, s);
  return launch_contrib_t<kMaxParts>(a, s);
}

// ---- scratch of the allocation-free contrib entry point
//
// The per-workgroup partial sums live in a file-scope device array: one copy
// per GPU, held until the process ends.  In host code `scratch` names a
// host-side stand-in, not device memory, so its device address is looked up
// once per device (with that device current) and only that address is
// passed to kernels.
static __device__ __align__(256) float scratch[kContribScratchBytes / sizeof(float)];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};
}  // namespace

hipError_t contrib_scratch(float** ptr) {
  *ptr = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = (float*)g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace ditango
