// attn_f32.hip - fresh attention states of selected key/value partitions,
// float32 inputs and states (gfx950).
//
// Same computation as the bf16 kernel (the blocked attention state of Sec.
// 2.2.4, Eq. attention_state, by online softmax over key tiles), in float32
// precision.  Scores are computed transposed, S^T = K Q^T, so that each lane
// holds one query's scores; the output is accumulated as O^T = V^T P^T.
//
// Products
//   The float32 MFMA runs at a sixteenth of the bf16 one.  Every float32
//   operand x is split into three bf16 planes, x = x1 + x2 + x3 (each the
//   rounding of what the planes before it leave: 3 x 8 bits, exact), and a
//   product is the sum of six bf16 MFMAs with float32 accumulation,
//     x3 y1 + x2 y2 + x1 y3 + x2 y1 + x1 y2 + x1 y1,
//   6/16 of the float32 MFMA's time.  The three products left out come to at
//   most 2^-24 |x y| (two of 2^-8 x 2^-17; the rounding of one float32
//   product) and to 2^-27 ... 2^-26.5 as a root mean square, and there are
//   fewer accumulations: against 64 bits, OUT is off by
//   2e-7 ... 7e-7 (norm ratio, 1,000 ... 2,000 keys) where the float32 MFMA's
//   was off by 5e-7 ... 9e-7; LSE is the same.  The scores' five small terms
//   have an accumulator of their own.
//   What the planes cannot hold goes through the float32 MFMA: a workgroup
//   runs its task again with it
//    - where some row's sum or output ends up not finite.  A value that is not
//      finite, or rounds to infinity in bf16, gives NaN in the planes and in
//      every row it enters; the float32 MFMA treats infinities as float32
//      arithmetic does;
//    - where nonzero values below 2^-110 matter.  Their third plane falls
//      under bf16's smallest subnormal (2^-133), so such a value is off by up
//      to 2^-134.  Its queries are looked at as they are split: one of these
//      values, or one so large (2^100 after scaling) that what a key of this
//      kind is off by would show in the scores (below it: 2^-27 at most).  In
//      V the error is under 2^-34 of an output of 2^-100 or more, so V is
//      looked through only where some output is smaller or zero (a column of
//      zeros in V: 7,750 keys in the 128-row form 670 -> 753 us; 2,000 keys
//      and 24 heads in the 256-row form 890 -> 938).
//   Probabilities under 2^-110 are off by 2^-134 too: OUT by 2^-134 max|v|.
//
// Work decomposition
//   A workgroup has RW x KW waves and 32 * RW query rows of one (partition,
//   batch, head).  RW waves share 32-key tiles: together they load a tile's
//   float32 rows, split them once and write the planes to LDS, double
//   buffered.  With KW > 1 the waves split the partition's keys instead
//   (RW = 1): each wave stages its own tiles in its own LDS, without
//   barriers, and the KW partial states are composed through LDS at the end.
//
// What bounds it: at D=128 the MFMAs (96 per wave and tile, busy 69 % of the
// cycles at 1.84 GHz); at D=64 MFMAs and vector work alike (48 MFMAs, busy
// 53-58 %, beside about 280 vector instructions: the planes of the staged
// tile and of the probabilities take 11 per pair of values).
#include <type_traits>

#include "attn_tile.h"
#include "internal.h"

namespace ditango {
namespace {

__device__ __forceinline__ f32x16 mfma32f(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// three bf16 planes of 8 floats
struct Planes {
  bf16x8 p[3];
};
// Pairs of values: one conversion instruction packs a pair's plane, and the
// values it stands for are read back out of the packed word (the empty asm
// hides from the compiler that they are conversions, which it would repeat
// value by value).
__device__ __forceinline__ Planes split8(f32x8 x) {
  u32x4 w[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
      if (j < 2) {
        asm("" : "+v"(p));
        a -= __builtin_bit_cast(float, p << 16);
        b -= __builtin_bit_cast(float, p & 0xffff0000u);
      }
      w[j][i] = p;
    }
  }
  Planes r;
#pragma unroll
  for (int j = 0; j < 3; ++j) r.p[j] = __builtin_bit_cast(bf16x8, w[j]);
  return r;
}

// 2^-110: nonzero values below it are not exact in the planes
constexpr uint32_t kPlanesMin = 0x08800000u;
__device__ __forceinline__ bool below_planes(float x) {
  return (__float_as_uint(x) & 0x7fffffffu) - 1u < kPlanesMin - 1u;
}

// the six plane products, smallest first
constexpr int kTerms = 6;
constexpr int kTermA[kTerms] = {2, 1, 0, 1, 0, 0};
constexpr int kTermB[kTerms] = {0, 1, 2, 0, 1, 0};

template <int D_, int RW_, int KW_, int WPE_, bool PIPED_>
struct CfgF {
  static constexpr int D = D_, RW = RW_, KW = KW_, WPE = WPE_;
  static constexpr bool PIPED = PIPED_;
  static constexpr int BN = 32;                   // keys per tile
  static constexpr int NT = RW * KW * 64;
  static constexpr int BM = RW * 32;              // query rows per workgroup
  static constexpr int KS = D / 16;               // bf16 MFMA k-steps over the head dim
  static constexpr int DB = D / 32;
  static constexpr int UNITS = D / 8;             // 8-element units per row
  static constexpr int ROWB = D * 2;              // bytes per plane row
  static constexpr int PLANE = BN * ROWB;
  static constexpr int TILE = 3 * PLANE;          // one operand's tile
  static constexpr int KST = D + 1;               // float rows of the float32 form
  static constexpr int VST = D + 8;
  // K and V take turns in one buffer when a wave has it to itself
  static constexpr int GROUP = RW == 1 ? TILE : 4 * TILE;
  static constexpr int UT = BN * UNITS / (RW * 64);   // units per thread and tile
  static constexpr int LDS = KW * GROUP + KW * 64 * 4 + 16;
  static_assert(RW == 1 || KW == 1, "waves share a tile or split the keys");
  static_assert(BN * VST * 4 <= TILE, "float rows fit the planes' space");
  static_assert(BN * UNITS % (RW * 64) == 0, "units divide over the threads");
  static_assert(BM * D * 4 <= TILE || KW == 1, "partial output fits the wave's space");
  static_assert(LDS <= 163840, "LDS of one compute unit");
};

// One pass over this wave's (KW > 1) or workgroup's (KW = 1) key tiles
// [t0, t1): unnormalised O^T, row maximum m (base 2, scaled) and the lane's
// half of the row sum.  SPLIT: bf16 planes, otherwise the float32 MFMA.
// `ask`: the lanes whose query values need the latter.
template <class C, bool SPLIT>
__device__ __forceinline__ void key_loop(const float* __restrict__ qrow, bool row_ok, const float* __restrict__ kg,
                                         const float* __restrict__ vg, int64_t HD, int kv_len, int t0, int t1,
                                         float sl2, unsigned char* buf, int gt, f32x16 (&o)[C::DB],
                                         float& m, float& l, uint64_t& ask) {
  constexpr int D = C::D;
  const int lane = threadIdx.x & 63;
  const int lr = lane & 31;
  const int g = lane >> 5;
#pragma unroll
  for (int db = 0; db < C::DB; ++db) o[db] = f32x16{};
  m = -INFINITY;
  l = 0.f;
  if (t0 >= t1) return;

  Planes qp[SPLIT ? C::KS : 1];
  float qf[SPLIT ? 1 : D / 2];
  if constexpr (SPLIT) {
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      const f32x4 x0 = *(const f32x4*)(qrow + 16 * s + 8 * g), x1 = *(const f32x4*)(qrow + 16 * s + 8 * g + 4);
      f32x8 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = row_ok ? x0[e] : 0.f;
        x[4 + e] = row_ok ? x1[e] : 0.f;
      }
      // smallest nonzero and largest magnitude (as bits; 0 - 1 is the largest)
      uint32_t lo = ~0u, hi = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t u = __float_as_uint(x[e]) & 0x7fffffffu;
        lo = min(lo, u - 1u);
        hi = max(hi, u);
      }
      ask |= __builtin_amdgcn_ballot_w64(lo < kPlanesMin - 1u || __uint_as_float(hi) * sl2 >= 0x1p100f);
      qp[s] = split8(x);
    }
  } else {
#pragma unroll
    for (int s = 0; s < D / 2; ++s) qf[s] = row_ok ? qrow[2 * s + g] : 0.f;
  }

  // this thread's units of a tile: unit u = gt + i * RW * 64, key u / UNITS.
  // Rows past the end read the last key: their scores are masked, and in the
  // float32 form (whose operands may be infinite) they are staged as zeros.
  // A lane's byte offset from the tile's first row is the same for every
  // tile but for that clamp; the tile's base is wave-uniform.
  struct Stage {
    f32x4 x[C::UT][2];
  };
  const uint32_t row_bytes = (uint32_t)HD * 4;
  const int last_tile = (kv_len - 1) / C::BN;
  uint32_t off_key[C::UT];
#pragma unroll
  for (int i = 0; i < C::UT; ++i) off_key[i] = (uint32_t)((gt + i * C::RW * 64) / C::UNITS) * row_bytes;
  auto load = [&](Stage& st, const float* src, int tile) {
    const int tb = min(tile, last_tile);
    const char* base = (const char*)(src + (int64_t)tb * C::BN * HD);
    const uint32_t lim = (uint32_t)min(kv_len - 1 - tb * C::BN, C::BN - 1) * row_bytes;
#pragma unroll
    for (int i = 0; i < C::UT; ++i) {
      const char* p = base + (min(off_key[i], lim) + (uint32_t)((gt + i * C::RW * 64) % C::UNITS) * 32);
      st.x[i][0] = *(const f32x4*)p;
      st.x[i][1] = *(const f32x4*)(p + 16);
    }
  };
  auto store = [&](const Stage& st, unsigned char* buf, int tile, bool is_k) {
#pragma unroll
    for (int i = 0; i < C::UT; ++i) {
      const int u = gt + i * C::RW * 64;
      const int key = u / C::UNITS, c = u % C::UNITS;
      f32x8 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = st.x[i][0][e];
        x[4 + e] = st.x[i][1][e];
      }
      if constexpr (SPLIT) {
        const Planes pl = split8(x);
        unsigned char* p = buf + key * C::ROWB + (c ^ (is_k ? swz_k<D>(key) : swz_v<D>(key))) * 16;
#pragma unroll
        for (int j = 0; j < 3; ++j) *(bf16x8*)(p + j * C::PLANE) = pl.p[j];
      } else {
        float* p = (float*)buf + key * (is_k ? C::KST : C::VST) + c * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = tile * C::BN + key < kv_len ? x[e] : 0.f;
      }
    }
  };

  // V^T fragments by transpose reads, as in the bf16 kernel: source lane r of
  // a 16-lane group points at row 4g + r/4 (+ 16s + 8) and dims
  // 32db + 16*(group%2) + 4*(r%4)
  const int vrow = 4 * g + ((lane & 15) >> 2);
  const int vdim = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  uint32_t voff[C::DB];
#pragma unroll
  for (int db = 0; db < C::DB; ++db) {
    const int dim = 32 * db + vdim;
    voff[db] = vrow * C::ROWB + ((dim >> 3) ^ swz_v<D>(vrow)) * 16 + (dim & 7) * 2;
  }
  auto v_frag = [&](const unsigned char* vb, int plane, int s, int db) {
    const unsigned char* p = vb + plane * C::PLANE + 16 * s * C::ROWB + voff[db];
    const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p)));
    const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + 8 * C::ROWB)));
    return __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
  };

  // S^T = K Q^T of the tile in kb
  auto qk = [&](const unsigned char* kb, f32x16& sc) {
    sc = f32x16{};
    if constexpr (SPLIT) {
      f32x16 sm = f32x16{};
#pragma unroll
      for (int s = 0; s < C::KS; ++s) {
        bf16x8 ka[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
          ka[j] = *(const bf16x8*)(kb + j * C::PLANE + lr * C::ROWB + ((2 * s + g) ^ swz_k<D>(lr)) * 16);
#pragma unroll
        for (int i = 0; i < kTerms - 1; ++i) sm = mfma32(ka[kTermA[i]], qp[s].p[kTermB[i]], sm);
        sc = mfma32(ka[0], qp[s].p[0], sc);
      }
      sc += sm;
    } else {
#pragma unroll
      for (int s = 0; s < D / 2; ++s) sc = mfma32f(((const float*)kb)[lr * C::KST + 2 * s + g], qf[s], sc);
    }
  };
  // the running maximum raised to the scores' (masked past the last key)
  auto raise = [&](f32x16& sc, int t) {
    if ((t + 1) * C::BN > kv_len) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (t * C::BN + 8 * (r >> 2) + 4 * g + (r & 3) >= kv_len) sc[r] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    const float mnew = fmaxf(m, pair_max(mx) * sl2);
    // the outputs are rescaled only when some row's maximum rose
    if (__builtin_amdgcn_ballot_w64(!(mnew == m)) != 0) {
      const float alpha = mnew == m ? 1.f : fast_exp2(m - mnew);
      m = mnew;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < C::DB; ++db) o[db] *= alpha;
    }
  };
  // scores -> probabilities against the running maximum (left in sc, and as
  // planes), row sums
  auto probs = [&](f32x16& sc, Planes (&pp)[2]) {
    // a row without a finite score so far (infinite operands) adds nothing
    const float mm = !SPLIT && m == -INFINITY ? 0.f : m;
    float ls = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = fast_exp2(__builtin_fmaf(sc[r], sl2, -mm));
      ls += sc[r];
    }
    l += ls;
    if constexpr (SPLIT) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        f32x8 x;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = sc[8 * s + e];
        pp[s] = split8(x);
      }
    }
  };
  // O^T += V^T P^T of the tile in vb
  auto pv = [&](const unsigned char* vb, const Planes (&pp)[2], const f32x16& sc) {
    if constexpr (SPLIT) {
      constexpr int DP = 2;                          // dim blocks in flight together
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int d0 = 0; d0 < C::DB; d0 += DP) {
          bf16x8 va[DP][3];
#pragma unroll
          for (int d = 0; d < DP; ++d)
#pragma unroll
            for (int j = 0; j < 3; ++j) va[d][j] = v_frag(vb, j, s, d0 + d);
#pragma unroll
          for (int i = 0; i < kTerms; ++i)
#pragma unroll
            for (int d = 0; d < DP; ++d) o[d0 + d] = mfma32(va[d][kTermA[i]], pp[s].p[kTermB[i]], o[d0 + d]);
        }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
          o[db] = mfma32f(((const float*)vb)[(8 * (r >> 2) + 4 * g + (r & 3)) * C::VST + db * 32 + lr], sc[r], o[db]);
    }
  };

  if constexpr (C::RW > 1) {
    // Two K and two V buffers: later tiles are split and written beside the
    // MFMAs of this one, those after them are on their way to registers; one
    // barrier per tile.
    unsigned char* vbuf = buf + 2 * C::TILE;
    Stage sk, sv;
    load(sk, kg, t0);
    load(sv, vg, t0);
    store(sk, buf, t0, true);
    store(sv, vbuf, t0, false);
    load(sk, kg, t0 + 1);
    load(sv, vg, t0 + 1);
    __syncthreads();
    if constexpr (C::PIPED) {
      // The scores of tile t+1 are computed beside the probabilities of tile
      // t, so that a wave's own vector work runs under its MFMAs.  K_{t+2}
      // replaces K_t, last read before the previous barrier.
      f32x16 s0, s1;
      qk(buf, s0);
      store(sk, buf + C::TILE, t0 + 1, true);
      load(sk, kg, t0 + 2);
      __syncthreads();
      auto iteration = [&](int t, f32x16& scur, f32x16& snxt, auto ph) {
        constexpr int cur = decltype(ph)::value * C::TILE, nxt = C::TILE - cur;
        raise(scur, t);
        Planes pp[2];
        qk(buf + nxt, snxt);
        probs(scur, pp);
        if constexpr (SPLIT) {
          // one MFMA, six vector instructions, an LDS read every other time
          __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
          for (int i = 0; i < kTerms * C::KS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
            if (i % 2) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
        }
        store(sv, vbuf + nxt, t + 1, false);
        load(sv, vg, t + 2);
        pv(vbuf + cur, pp, scur);
        store(sk, buf + cur, t + 2, true);
        load(sk, kg, t + 3);
        __syncthreads();
      };
      for (int t = t0; t < t1; t += 2) {
        iteration(t, s0, s1, std::integral_constant<int, 0>{});
        if (t + 1 < t1) iteration(t + 1, s1, s0, std::integral_constant<int, 1>{});
      }
    } else {
      for (int t = t0; t < t1; ++t) {
        const int cur = ((t - t0) & 1) * C::TILE, nxt = C::TILE - cur;
        store(sk, buf + nxt, t + 1, true);
        load(sk, kg, t + 2);
        f32x16 sc;
        Planes pp[2];
        qk(buf + cur, sc);
        raise(sc, t);
        probs(sc, pp);
        store(sv, vbuf + nxt, t + 1, false);
        load(sv, vg, t + 2);
        pv(vbuf + cur, pp, sc);
        __syncthreads();
      }
    }
  } else {
    // The wave's own buffer holds K_t, then V_t: LDS operations of a wave run
    // in order, so no barrier is needed.
    Stage sk, sv;
    load(sk, kg, t0);
    for (int t = t0; t < t1; ++t) {
      store(sk, buf, t, true);
      load(sv, vg, t);
      f32x16 sc;
      Planes pp[2];
      qk(buf, sc);
      raise(sc, t);
      probs(sc, pp);
      store(sv, buf, t, false);
      load(sk, kg, t + 1);
      pv(buf, pp, sc);
    }
  }
}

template <class C>
__global__ __launch_bounds__(C::NT, C::WPE) void attn_f32_kernel(const AttnArgs a) {
  constexpr int D = C::D;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int task = xcd_remap(blockIdx.x, gridDim.x);
  const int qt = task % a.q_tiles;
  int t = task / a.q_tiles;
  const int h = t % a.H;
  t /= a.H;
  const int b = t % a.B;
  const int sel = t / a.B;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31;
  const int g = lane >> 5;

  const int64_t HD = (int64_t)a.H * D;
  const int kv_len = a.kv_len[sel];
  const int64_t kv0 = a.kv_begin[sel];
  const int slot = a.slot[sel];
  const float* kg = (const float*)a.k + ((int64_t)b * a.S + kv0) * HD + (int64_t)h * D;
  const float* vg = (const float*)a.v + ((int64_t)b * a.S + kv0) * HD + (int64_t)h * D;
  const int rl = (C::KW == 1 ? wave * 32 : 0) + lr;          // row within the workgroup's tile
  const int64_t row = (int64_t)qt * C::BM + rl;
  const bool row_ok = row < a.q_len;
  const float* qrow = (const float*)a.q + (int64_t)b * a.q_stride + (row_ok ? row : 0) * HD + (int64_t)h * D;

  // this wave's key tiles, and its tile space in LDS
  const int tiles = (kv_len + C::BN - 1) / C::BN;
  const int per = (tiles + C::KW - 1) / C::KW;
  const int kw = C::KW == 1 ? 0 : wave;
  const int t0 = min(kw * per, tiles), t1 = min(t0 + per, tiles);
  unsigned char* kb = smem + kw * C::GROUP;
  const int gt = C::KW == 1 ? tid : lane;
  float* part_m = (float*)(smem + C::KW * C::GROUP);         // [KW][32] maximum, then [KW][32] row sum
  float* part_l = part_m + C::KW * 32;
  // run the task again; look through V; V asks for it (a word each: a wave may
  // still be reading one when another writes the next)
  int* redo = (int*)(part_l + C::KW * 32);

  f32x16 o[C::DB];
  float m, l;
  if (tid < 3) redo[tid] = 0;
  uint64_t ask = 0;
  key_loop<C, true>(qrow, row_ok, kg, vg, HD, kv_len, t0, t1, a.scale_log2, kb, gt, o, m, l, ask);
  // sum of 0 * x: NaN where a value is not finite
  float bad = l * 0.f, low = INFINITY;
#pragma unroll
  for (int db = 0; db < C::DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      bad = __builtin_fmaf(o[db][r], 0.f, bad);
      low = fminf(low, fabsf(o[db][r]));
    }
  const float below = pair_sum(l) * 0x1p-100f;
  const bool small = row_ok && low < below;
  __syncthreads();
  if ((__builtin_amdgcn_ballot_w64(!(bad == 0.f)) | ask) != 0 && lane == 0) redo[0] = 1;
  if (__builtin_amdgcn_ballot_w64(small) != 0 && lane == 0) redo[1] = 1;
  __syncthreads();
  bool again = __builtin_amdgcn_readfirstlane(redo[0]) != 0;
  if (!again && __builtin_amdgcn_readfirstlane(redo[1]) != 0) {
    constexpr int kBatch = 8;                                // loads in flight
    const int64_t units = (int64_t)kv_len * (D / 4);
    bool found = false;
    for (int64_t i0 = tid; i0 < units; i0 += kBatch * C::NT) {
      f32x4 x[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int64_t u = min(i0 + i * C::NT, units - 1);
        x[i] = *(const f32x4*)(vg + u / (D / 4) * HD + u % (D / 4) * 4);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) found |= below_planes(x[i][e]);
    }
    if (__builtin_amdgcn_ballot_w64(found) != 0 && lane == 0) redo[2] = 1;
    __syncthreads();
    again = __builtin_amdgcn_readfirstlane(redo[2]) != 0;
  }
  if (again) {
    key_loop<C, false>(qrow, row_ok, kg, vg, HD, kv_len, t0, t1, a.scale_log2, kb, gt, o, m, l, ask);
    __syncthreads();
  }

  const float lt = pair_sum(l);
  const int64_t slot_elems = (int64_t)a.B * a.q_len * HD;
  float* outg = (float*)a.out_states + (int64_t)slot * slot_elems + (int64_t)b * a.q_len * HD + (int64_t)h * D;
  float* lseg = a.lse_states + (((int64_t)slot * a.B + b) * a.H + h) * a.q_len;
  if constexpr (C::KW == 1) {
    if (row_ok) {
      const float inv = lt > 0.f ? 1.0f / lt : 0.f;
      float* dst = outg + row * HD + 4 * g;
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          f32x4 x;
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = o[db][4 * r4 + e] * inv;
          *(f32x4*)(dst + db * 32 + 8 * r4) = x;
        }
      if (g == 0) lseg[row] = lt > 0.f ? (m + __builtin_amdgcn_logf(lt)) * kLn2 : -INFINITY;
    }
  } else {
    // partial states through LDS: O rows of 16-byte units, swizzled by row
    float* po = (float*)kb;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = o[db][4 * r4 + e];
        *(f32x4*)(po + lr * D + (((8 * db + 2 * r4 + g) ^ (lr & 15)) * 4)) = x;
      }
    if (g == 0) {
      part_m[kw * 32 + lr] = m;
      part_l[kw * 32 + lr] = lt;
    }
    __syncthreads();
    constexpr int CH = 32 * D / 4;
    static_assert(CH % C::NT == 0, "chunks divide over the threads");
#pragma unroll
    for (int i = 0; i < CH / C::NT; ++i) {
      const int c = tid + i * C::NT;
      const int r = c / (D / 4), u = c % (D / 4);
      if ((int64_t)qt * C::BM + r >= a.q_len) continue;
      float mk[C::KW], M = -INFINITY;
#pragma unroll
      for (int k = 0; k < C::KW; ++k) {
        mk[k] = part_m[k * 32 + r];
        M = fmaxf(M, mk[k]);
      }
      float tot = 0.f;
      f32x4 acc = f32x4{};
#pragma unroll
      for (int k = 0; k < C::KW; ++k) {
        // a range without keys has m = -inf, sum 0 and output 0
        const float w = mk[k] == -INFINITY && part_l[k * 32 + r] == 0.f ? 0.f : fast_exp2(mk[k] - M);
        tot = __builtin_fmaf(w, part_l[k * 32 + r], tot);
        acc += w * *(const f32x4*)((const float*)(smem + k * C::GROUP) + r * D + ((u ^ (r & 15)) * 4));
      }
      const float inv = tot > 0.f ? 1.0f / tot : 0.f;
      *(f32x4*)(outg + ((int64_t)qt * C::BM + r) * HD + u * 4) = acc * inv;
      if (u == 0) lseg[(int64_t)qt * C::BM + r] = tot > 0.f ? (M + __builtin_amdgcn_logf(tot)) * kLn2 : -INFINITY;
    }
  }
}

template <class C>
hipError_t launch_cfg_f(const AttnArgs& a0, int dev, hipStream_t s) {
  static OncePerDevice once;
  const hipError_t attr = once.run(dev, [] {
    return hipFuncSetAttribute((const void*)attn_f32_kernel<C>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
  });
  if (attr != hipSuccess) return attr;
  AttnArgs a = a0;
  a.q_tiles = (int)((a.q_len + C::BM - 1) / C::BM);
  const int64_t nblk = (int64_t)a.q_tiles * a.H * a.B * a.n_sel;
  if (nblk <= 0) return hipSuccess;
  if (nblk > 0x7fffffff) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((attn_f32_kernel<C>), dim3((unsigned)nblk), dim3(C::NT), C::LDS, s, a);
  return hipGetLastError();
}

// Which form a launch runs, by how its workgroups fill the compute units
// (times on one card, float32 MFMA kernel before / the forms of this one):
//  - Split, 32 rows and all the waves on one tile of rows, up to two rounds.
//    It splits every key tile per 32 rows and is bound by that vector work,
//    but fills the chip with the fewest rows: 1,024 rows x 2 heads x 4
//    partitions of 1,024 keys at D=64 24 us (93; Shared 52), 1,024 rows x 4
//    heads x 2 partitions at D=128 45 us (161; Shared 114).  At three rounds
//    Mid and Shared are as fast.
//  - Mid, 128 rows, while every workgroup has a compute unit to itself: one
//    wave per SIMD (D=128; 7,750 rows x 4 heads x 7,750 keys 654 us, Shared
//    815, Split 1,062).  At D=64 two workgroups share a compute unit and
//    Mid is Shared.
//  - Shared otherwise: 256 rows at D=128, two waves per SIMD (2,000 rows x 24
//    heads x 4 partitions of 2,000 keys: 0.88 ms, 224 TFLOP/s, MFMAs busy
//    69 %, against 1.87 ms and 105 TFLOP/s; Mid 1.13 ms); 128 rows at D=64
//    (the same: 0.51 ms, 194 TFLOP/s, against 0.93 ms and 106 TFLOP/s; with
//    the scores not pipelined 0.55 ms).
template <class Shared, class Mid, class Split>
hipError_t launch_f32(const AttnArgs& a, hipStream_t s) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int64_t tiles = (int64_t)a.H * a.B * a.n_sel;
  if ((a.q_len + Split::BM - 1) / Split::BM * tiles <= 2 * (int64_t)cus) return launch_cfg_f<Split>(a, dev, s);
  if ((a.q_len + Mid::BM - 1) / Mid::BM * tiles <= cus) return launch_cfg_f<Mid>(a, dev, s);
  return launch_cfg_f<Shared>(a, dev, s);
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, int D, hipStream_t s) {
  if (D == 128)
    return launch_f32<CfgF<128, 8, 1, 2, false>, CfgF<128, 4, 1, 1, true>, CfgF<128, 1, 4, 1, false>>(a, s);
  if (D == 64) return launch_f32<CfgF<64, 4, 1, 2, true>, CfgF<64, 4, 1, 2, true>, CfgF<64, 1, 8, 2, false>>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace ditango
