// Device-side helpers shared by the decoding kernels (gfx950, 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rb {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kMaxBeam = 16;
constexpr int kCtxMax = 8;          // tokens of history kept per hypothesis (LM order <= 9, stateless ctx <= 4)
constexpr uint64_t kHashBase = 1000003ull;
constexpr uint64_t kHashMod = 2147483647ull;  // 2^31 - 1

// One 32x32x2 fp32 matrix-core step: acc[i][j] += sum_{k<2} A[i][k] B[k][j].
// Lane l supplies A[i = l % 32][k = l / 32] and B[k = l / 32][j = l % 32]; it
// receives acc[i = 8 * (r / 4) + 4 * (l / 32) + r % 4][j = l % 32] in register r.
__device__ __forceinline__ floatx16 mfma32(float a, float b, floatx16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
}

// float32 -> bfloat16 (round to nearest even) -> float32
__device__ __forceinline__ float bf16_round(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return x;
  u += 0x7fffu + ((u >> 16) & 1u);
  u &= 0xffff0000u;
  return __uint_as_float(u);
}

__device__ __forceinline__ float4 bf16_round4(float4 v) {
  return make_float4(bf16_round(v.x), bf16_round(v.y), bf16_round(v.z), bf16_round(v.w));
}

// ---- bfloat16 operands of the bf16 matrix instructions
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4_t __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2_t __attribute__((ext_vector_type(2)));

// two float32 -> two bfloat16 in one word (low half first), round to nearest even: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  const floatx2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// One 32x32x16 bf16 matrix-core step fed from float32 registers: the lane's 8 k-values are the 4 + 4 floats it holds
// for two consecutive 8-k rounds of the float32 scheme (see mfma32), rounded to bf16 here.  Both operands use the
// same lane -> k assignment, so every k of the 16 meets its partner exactly once.
__device__ __forceinline__ floatx16 mfma32_bf16_from_f32(float4 a0, float4 a1, float4 b0, float4 b1, floatx16 acc) {
  const uintx4_t pa = {pack_bf16_rne(a0.x, a0.y), pack_bf16_rne(a0.z, a0.w), pack_bf16_rne(a1.x, a1.y),
                       pack_bf16_rne(a1.z, a1.w)};
  const uintx4_t pb = {pack_bf16_rne(b0.x, b0.y), pack_bf16_rne(b0.z, b0.w), pack_bf16_rne(b1.x, b1.y),
                       pack_bf16_rne(b1.z, b1.w)};
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pa), __builtin_bit_cast(bf16x8_t, pb), acc, 0,
                                                 0, 0);
}

// ---- float32 products on the 16-bit matrix cores
// A float32 x as hi + lo, hi = x rounded to float16, lo = the rest rounded to float16 and kept 2^11 times as large, so that neither is a
// subnormal number for x down to 2^-28 of the largest that shares its scale: x to 2^-23 of itself (a unit in the last place of float32,
// for a quarter of all x; the others exactly).  Smaller ones are right to 2^-50 of the largest.  A product is then hi hi + (hi lo + lo hi)
// 2^-11, to which decoders less than 640 wide add lo lo 2^-22 (see kSplitLoLo).  Three or four float16 matrix instructions replace eight
// float32 ones of twice the cycles each.  (Unscaled, lo is a subnormal number below 2^-15 of the largest: with one weight of a row 2^24 times the others the
// error of their products was 1.3e-5.  The scale takes a multiplication per pair of values, less than 1 % of a decode.)
// How the instructions add up (measured): acc + the eight products of one lane in one rounding, the lanes of a row or column
// one after the other in the order of their k.  Which of the shapes 32x32x16, 16x16x32 and 16x16x16 takes the k does not matter.
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
constexpr float kHidScale = 32768.f;  // of hidden states, whose values lie in [-1, 1]
// Of values whose size is not known ahead (the joint's activations): m, the largest of a hypothesis in a slice of the k, goes to
// [2^14, 2^15) (from 2^-84 on).  inv takes the scale off the slice's sum again, and kActUnscale more, for the largest sums of the largest
// values to stay finite, which the scale of the weights' rows gives back.
constexpr float kActUnscale = 1.f / (1 << 25);
__device__ __forceinline__ float split_scale(float m, float &inv) {
  uint32_t e = __float_as_uint(m) & 0x7f800000u;
  e = e > 43u << 23 ? e : 43u << 23;
  inv = __uint_as_float(e - (39u << 23));
  return __uint_as_float((268u << 23) - e);
}
constexpr float kLoScale = 2048.f;
// acc + the sum of the products with a lo in them
template <class V>
__device__ __forceinline__ V split_join(V acc, V cor) { return acc + cor * (1.f / kLoScale); }
// Whether and how a decoder's weights are split.  kSplitLoLo: with the products of two lo, up to 2^-22 of a product, which the sums of
// 640 make up for and those of 320 do not: error of scores with large logits against 64 bits, split over float32 (plus or minus 0.02),
// 320 wide 1.04 without them and 1.01 with them, 384 0.99 / 0.96, 512 0.99 / 0.97, 640 0.91 / 0.90.  320 wide they cost 1 % of a decode;
// 640 wide, where they take registers that there are not, 7 %.
constexpr int kNotSplit = 0, kSplit = 1, kSplitLoLo = 2;
// lo words without their scale
template <class V>
__device__ __forceinline__ V unscaled_lo(V lo) {
  constexpr int N = sizeof(V) / 2;
  typedef _Float16 Halves __attribute__((ext_vector_type(N)));
  return __builtin_bit_cast(V, __builtin_bit_cast(Halves, lo) * (_Float16)(1.f / kLoScale));
}
// two values -> their two hi and their two lo, each pair in one word
__device__ __forceinline__ void split_f16(float a, float b, uint32_t &hi, uint32_t &lo) {
  const floatx2_t v = {a, b};
  const f16x2_t h = __builtin_convertvector(v, f16x2_t);
  const floatx2_t r = {(a - (float)h[0]) * kLoScale, (b - (float)h[1]) * kLoScale};
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2_t));
}
// one value -> hi | lo << 16
__device__ __forceinline__ uint32_t split_f16(float a) {
  const _Float16 h = (_Float16)a, l = (_Float16)((a - (float)h) * kLoScale);
  return (uint32_t)__builtin_bit_cast(uint16_t, h) | (uint32_t)__builtin_bit_cast(uint16_t, l) << 16;
}
__device__ __forceinline__ floatx16 mfma32_f16(uintx4_t a, uintx4_t b, floatx16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), acc, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma16_f16(uintx4_t a, uintx4_t b, floatx4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), acc, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma16_f16(uintx2_t a, uintx2_t b, floatx4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4_t, a), __builtin_bit_cast(f16x4_t, b), acc, 0, 0, 0);
}
// 32x32x16 steps of a split product on N (two or four) consecutive 8-k rounds of the float32 scheme (see mfma32): weights come
// split and scaled (k_split_rows), activations are scaled and split here.  The order in `cor` is that of the 16x16x32 instructions of the
// resident loop, which take four rounds at a time.
template <int N, bool LOLO>
__device__ __forceinline__ void mfma32_split(const float4 (&a)[N], const float4 (&b)[N], float scale, floatx16 &acc, floatx16 &cor) {
  uintx4_t wh[N / 2], wl[N / 2], xh[N / 2], xl[N / 2];
#pragma unroll
  for (int i = 0; i < N; i += 2) {
    const uintx4_t w0 = __builtin_bit_cast(uintx4_t, a[i]), w1 = __builtin_bit_cast(uintx4_t, a[i + 1]);
    wh[i / 2] = uintx4_t{w0[0], w0[1], w1[0], w1[1]};
    wl[i / 2] = uintx4_t{w0[2], w0[3], w1[2], w1[3]};
    uint32_t h[4], l[4];
    split_f16(b[i].x * scale, b[i].y * scale, h[0], l[0]);
    split_f16(b[i].z * scale, b[i].w * scale, h[1], l[1]);
    split_f16(b[i + 1].x * scale, b[i + 1].y * scale, h[2], l[2]);
    split_f16(b[i + 1].z * scale, b[i + 1].w * scale, h[3], l[3]);
    xh[i / 2] = uintx4_t{h[0], h[1], h[2], h[3]};
    xl[i / 2] = uintx4_t{l[0], l[1], l[2], l[3]};
  }
#pragma unroll
  for (int i = 0; i < N / 2; ++i) acc = mfma32_f16(wh[i], xh[i], acc);
#pragma unroll
  for (int i = 0; i < N / 2; ++i) cor = mfma32_f16(wh[i], xl[i], cor);
#pragma unroll
  for (int i = 0; i < N / 2; ++i) cor = mfma32_f16(wl[i], xh[i], cor);
  if constexpr (LOLO) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) cor = mfma32_f16(wl[i], unscaled_lo(xl[i]), cor);
  }
}
// the same on ITERS rounds
template <int ITERS, bool LOLO>
__device__ __forceinline__ void mfma32_split_rounds(const float4 (&a)[ITERS], const float4 (&b)[ITERS], float scale, floatx16 &acc, floatx16 &cor) {
  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < ITERS; i += 4) {
    if (ITERS - i > 2) {
      const bool four = i + 3 < ITERS;
      const int i3 = four ? i + 3 : i;
      const float4 w[4] = {a[i], a[i + 1 < ITERS ? i + 1 : i], a[i + 2 < ITERS ? i + 2 : i], four ? a[i3] : zero4};
      const float4 x[4] = {b[i], b[i + 1 < ITERS ? i + 1 : i], b[i + 2 < ITERS ? i + 2 : i], four ? b[i3] : zero4};
      mfma32_split<4, LOLO>(w, x, scale, acc, cor);
    } else {
      const bool two = i + 1 < ITERS;
      const int i1 = two ? i + 1 : i;
      const float4 w[2] = {a[i], two ? a[i1] : zero4}, x[2] = {b[i], two ? b[i1] : zero4};
      mfma32_split<2, LOLO>(w, x, scale, acc, cor);
    }
  }
}

__device__ __forceinline__ double logaddexp_d(double a, double b) {
  if (a == -INFINITY) return b;
  if (b == -INFINITY) return a;
  double m = a > b ? a : b;
  return m + log(exp(a - m) + exp(b - m));
}

// Stores and loads that are coherent across the whole device on their own (they bypass the caches
// that are private to a group of compute units), for the few words that one block hands to another
// inside a kernel.  A device-wide release / acquire fence would write back and invalidate the whole
// L2 instead, which costs microseconds.
template <typename T>
__device__ __forceinline__ void store_agent(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_agent(const T *p) {
  return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Blocks the calling wave until every global load and store it has issued has completed; a write-through
// store completes when the memory side has acknowledged it.  (gfx9 counts stores in vmcnt.)
__device__ __forceinline__ void wait_stores_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Results that only a LATER launch reads.  A plain store leaves its line dirty in the XCD's L2, and the end of
// every kernel waits until all dirty lines have been written back (the L2s of the XCDs are not coherent with each
// other, so that is how one launch's output becomes visible to the next).  Writing through at once takes that
// wait off the chain of dependent launches: 20.0 -> 19.5 ms per decode at 2 061 launches.
template <typename T>
__device__ __forceinline__ void store_through(T *p, T v) {
  store_agent(p, v);
}

// 16 bytes written through (one instruction; the atomic store above exists for 4 and 8 bytes only)
__device__ __forceinline__ void store16_through(float *p, floatx4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory");
}

// Candidate order used everywhere a "best" is chosen: larger value first, then
// smaller index.  Returns true if (v1, i1) comes before (v2, i2).
template <typename V, typename I>
__device__ __forceinline__ bool comes_before(V v1, I i1, V v2, I i2) {
  return v1 > v2 || (v1 == v2 && i1 < i2);
}
// the same without short circuits, for unrolled runs of comparisons (the compiler turns the form above into a branch
// per comparison when the values are doubles, which costs more than the compares themselves)
template <typename V, typename I>
__device__ __forceinline__ int comes_before_count(V v1, I i1, V v2, I i2) {
  return (int)(v1 > v2) | ((int)(v1 == v2) & (int)(i1 < i2));
}

// ---- cross-lane exchange without the LDS crossbar --------------------------
// __shfl_* compiles to ds_bpermute (LDS latency, ~100+ cycles per exchange); a
// data-parallel-primitive move costs one VALU instruction.  The four patterns
// below are butterflies inside a row of 16 lanes: lane ^ 1, lane ^ 2, then the
// mirror of each half row (pairs quads) and the mirror of the row (pairs halves).
constexpr int kDppXor1 = 0xB1;        // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141; // row_half_mirror
constexpr int kDppMirror = 0x140;     // row_mirror

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_i<CTRL>((int)(b & 0xffffffffll)), hi = dpp_i<CTRL>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float readlane_f(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double readlane_d(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// all-reduce over aligned groups of LANES (4, 8 or 16) lanes
template <int LANES>
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp_f<kDppXor1>(v));
  v = fmaxf(v, dpp_f<kDppXor2>(v));
  if constexpr (LANES >= 8) v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  if constexpr (LANES >= 16) v = fmaxf(v, dpp_f<kDppMirror>(v));
  return v;
}
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp_f<kDppXor1>(v);
  v += dpp_f<kDppXor2>(v);
  if constexpr (LANES >= 8) v += dpp_f<kDppHalfMirror>(v);
  if constexpr (LANES >= 16) v += dpp_f<kDppMirror>(v);
  return v;
}
template <int CTRL, typename V>
__device__ __forceinline__ void best_step(V &v, int &i) {
  V v2;
  if constexpr (sizeof(V) == 8) v2 = dpp_d<CTRL>(v); else v2 = dpp_f<CTRL>(v);
  const int i2 = dpp_i<CTRL>(i);
  if (comes_before(v2, i2, v, i)) {
    v = v2;
    i = i2;
  }
}
// best (value, index) pair of an aligned group of LANES lanes, in every lane of the group
template <int LANES, typename V>
__device__ __forceinline__ void group_best(V &v, int &i) {
  best_step<kDppXor1>(v, i);
  best_step<kDppXor2>(v, i);
  if constexpr (LANES >= 8) best_step<kDppHalfMirror>(v, i);
  if constexpr (LANES >= 16) best_step<kDppMirror>(v, i);
}

// ---- candidates packed into one sortable word ---------------------------------
// (key, index) -> 64 bits whose unsigned order is the candidate order: larger key first, then
// smaller index.  One compare instead of three, and a pair moves as two DPP words.
__device__ __forceinline__ uint32_t orderable(float f) {
  const uint32_t u = __float_as_uint(f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float from_orderable(uint32_t u) {
  return __uint_as_float(u ^ (((u >> 31) - 1u) | 0x80000000u));
}
__device__ __forceinline__ uint64_t pack_cand(float key, int idx) {
  return ((uint64_t)orderable(key) << 32) | (uint32_t)(0x7fffffff - idx);
}
__device__ __forceinline__ float cand_key(uint64_t c) { return from_orderable((uint32_t)(c >> 32)); }
__device__ __forceinline__ int cand_idx(uint64_t c) { return 0x7fffffff - (int)(uint32_t)c; }
// "no candidate": key -inf, index 0x7fffffff; every real candidate is larger
__device__ __forceinline__ uint64_t no_cand() { return pack_cand(-INFINITY, 0x7fffffff); }

template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
  const int lo = dpp_i<CTRL>((int)(uint32_t)v), hi = dpp_i<CTRL>((int)(uint32_t)(v >> 32));
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}
template <int CTRL>
__device__ __forceinline__ uint64_t max_step(uint64_t v) {
  const uint64_t w = dpp_u64<CTRL>(v);
  return w > v ? w : v;
}
// largest packed candidate of an aligned group of LANES lanes, in every lane of the group
template <int LANES>
__device__ __forceinline__ uint64_t group_max_u64(uint64_t v) {
  v = max_step<kDppXor1>(v);
  v = max_step<kDppXor2>(v);
  if constexpr (LANES >= 8) v = max_step<kDppHalfMirror>(v);
  if constexpr (LANES >= 16) v = max_step<kDppMirror>(v);
  return v;
}
// wave-wide max of packed candidates, in every lane
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  v = group_max_u64<16>(v);
  uint64_t best = 0;
#pragma unroll
  for (int r = 0; r < 64; r += 16) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, r);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), r);
    const uint64_t w = ((uint64_t)hi << 32) | lo;
    best = w > best ? w : best;
  }
  return best;
}

template <int LANES>
__device__ __forceinline__ int group_min_i(int v) {
  v = min(v, dpp_i<kDppXor1>(v));
  v = min(v, dpp_i<kDppXor2>(v));
  if constexpr (LANES >= 8) v = min(v, dpp_i<kDppHalfMirror>(v));
  if constexpr (LANES >= 16) v = min(v, dpp_i<kDppMirror>(v));
  return v;
}

// wave-wide versions: reduce inside the four rows, then combine the rows through scalar reads
__device__ __forceinline__ float wave_max(float v) {
  v = group_max<16>(v);
  return fmaxf(fmaxf(readlane_f(v, 0), readlane_f(v, 16)), fmaxf(readlane_f(v, 32), readlane_f(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = group_sum<16>(v);
  return (readlane_f(v, 0) + readlane_f(v, 16)) + (readlane_f(v, 32) + readlane_f(v, 48));
}
__device__ __forceinline__ int wave_sum_i(int v) {
  v += dpp_i<kDppXor1>(v);
  v += dpp_i<kDppXor2>(v);
  v += dpp_i<kDppHalfMirror>(v);
  v += dpp_i<kDppMirror>(v);
  return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
         (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
__device__ __forceinline__ void wave_best(float &v, int &i) {
  group_best<16>(v, i);
  float bv = readlane_f(v, 0);
  int bi = __builtin_amdgcn_readlane(i, 0);
#pragma unroll
  for (int r = 16; r < 64; r += 16) {
    const float v2 = readlane_f(v, r);
    const int i2 = __builtin_amdgcn_readlane(i, r);
    if (comes_before(v2, i2, bv, bi)) {
      bv = v2;
      bi = i2;
    }
  }
  v = bv;
  i = bi;
}
__device__ __forceinline__ void wave_best(double &v, int &i) {
  group_best<16>(v, i);
  double bv = readlane_d(v, 0);
  int bi = __builtin_amdgcn_readlane(i, 0);
#pragma unroll
  for (int r = 16; r < 64; r += 16) {
    const double v2 = readlane_d(v, r);
    const int i2 = __builtin_amdgcn_readlane(i, r);
    if (comes_before(v2, i2, bv, bi)) {
      bv = v2;
      bi = i2;
    }
  }
  v = bv;
  i = bi;
}

// ---- arithmetic of the LSTM cell
// n / d by Newton's iteration on the reciprocal and two corrections of the quotient by its residual (Markstein, IBM Journal of Research
// and Development 34, 1990), for n from 0 to 1 and d from 1/4 to below 2^126, whose reciprocal is normal: the correctly rounded quotient, a
// subnormal one too.  The compiler's division scales its operands for the others, by way of the one condition register, which keeps
// divisions from overlapping.  FIXUP: d may be infinite.  (It comes negated: a residual is then one instruction with n as a literal, where the
// other sign would take a move of n to a register first; one utterance 0.7 % slower.)
template <bool FIXUP>
__device__ __forceinline__ float div_unit_f(float n, float minus_d) {
  float r = __builtin_amdgcn_rcpf(-minus_d);
  r = fmaf(fmaf(minus_d, r, 1.f), r, r);
  float q = n * r;
  q = fmaf(fmaf(minus_d, q, n), r, q);
  q = fmaf(fmaf(minus_d, q, n), r, q);
  return FIXUP ? __builtin_amdgcn_div_fixupf(q, -minus_d, 1.f) : q;  // (any n that is a number does)
}
// 1 / (1 + e) for e from 0 to infinity: numerator and denominator are quarters (the rounding of 1 + e is the same), since 1 + e may be
// beyond 2^126 and its reciprocal, flushed to zero, would make the quotient 0 there instead of some 2^-127
__device__ __forceinline__ float sigmoid_of(float e) { return div_unit_f<true>(0.25f, fmaf(e, -0.25f, -0.25f)); }
// (1 - e) / (1 + e) for e from 0 to 1
__device__ __forceinline__ float tanh_of(float e) { return div_unit_f<false>(1.f - e, -1.f - e); }
__device__ __forceinline__ float sigmoid_f(float x) { return sigmoid_of(__expf(-x)); }
__device__ __forceinline__ float tanh_f(float x) {
  const float r = tanh_of(__expf(-2.f * fabsf(x)));
  return x < 0.f ? -r : r;
}
// gates (i, f, g, o) = recurrent part r4 + token part g4; c: the unit's old cell state in, the new one out; returns h
__device__ __forceinline__ float lstm_unit(float4 r4, float4 g4, float &c) {
  c = sigmoid_f(r4.y + g4.y) * c + sigmoid_f(r4.x + g4.x) * tanh_f(r4.z + g4.z);
  return sigmoid_f(r4.w + g4.w) * tanh_f(c);
}

}  // namespace rb
