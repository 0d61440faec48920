// The encoder's per-block network (learned encoder control): inference,
// batch gradient and Adam update, hand-written for CDNA4.
//
// 16 features -> 64 ReLU -> 64 ReLU -> 37 logits (10 threshold classes, 27
// range classes).  Parameters W1[64][16], b1[64], W2[64][64], b2[64],
// W3[37][64], b3[37]; inference and gradients read them as bfloat16 and
// accumulate in float32.  The network is tiny (7,653 parameters).
// Every contraction runs on the matrix cores: inference keeps the weights in
// registers and takes 32 rows at a time, the gradient kernel keeps a tile of
// 128 rows' activations in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>

#include "internal.h"

namespace {

constexpr int kIn = 16, kH = 64, kOut = 37, kCls = 10, kRng = 27;
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kOut * kH, kParams = oB3 + kOut;
static_assert(kParams == LFC_MLP_PARAMS, "parameter count");
constexpr int kThreads = 256;
constexpr int kTile = 128;   // rows per gradient workgroup
constexpr int kCus = 256;    // compute units of the device

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// float32 -> bfloat16, round to nearest, ties to even (NaN stays NaN)
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

struct InferArgs {
  const uint16_t *w;
  const float *x;
  int64_t n;
  int8_t *cls, *rng;
  float *conf, *logits;
};

// ---------------------------------------------------------------------------
// inference on the matrix cores: bf16 operands, fp32 accumulation
// ---------------------------------------------------------------------------
// What bounds it: vector issue (the bias, ReLU and rounding of 128 hidden
// values a row, the two heads), which overlaps the matrix products of other
// waves only in part; the rows' 70 bytes from and to HBM would allow twice
// the rate.  Each wave runs tiles of 32 rows through
// v_mfma_f32_32x32x16_bf16 with the weights as the first operand (units x
// rows): lane l supplies unit l%32 with K elements 8 (l/32)..+7 and row l%32
// with the same K elements, and receives units 8 (r/4) + 4 (l/32) + r%4 of row
// l%32 in its register r.  A row's values thus stay in its two lanes l and
// l+32: after the bias they are rounded and packed, clamped at zero two at a
// time, and one exchange of register halves between the two lanes per pair of
// packed words (v_permlane32_swap) gives the next layer's operand with its K
// elements in their order, so no layer goes through LDS.  The weights stay in
// registers for the wave's life, the biases are read from LDS, and the next
// tile's features are requested before this tile's layers.  (The bias as a
// product with one, in an fp32 MFMA, costs more than the additions: those
// share the vector unit.)
// Measured over 18.2 M rows: 466 us, 2.7 TB/s of rows (936 us with each layer's
// output exchanged through LDS and the heads on half of the lanes); four waves
// per SIMD with part of the weights in LDS 504 us, two 490 us.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kMfmaWaves = 4;
constexpr int kMfmaWgs = 3;   // workgroups per compute unit that the registers allow

__device__ __forceinline__ bf16x8 load_bf16x8(const uint16_t *p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}

// op of a value over the lanes whose numbers differ in the bits from LOW up
// (through LDS: the register exchanges between halves cost more issue).
template <int LOW, typename T, typename Op>
__device__ __forceinline__ T across(T v, Op op) {
#pragma unroll
  for (int d = 32; d >= LOW; d >>= 1) v = op(v, __shfl_xor(v, d));
  return v;
}

// Argmax of a head whose logits are spread over the lanes of a row (which
// differ in the bits from LOW up), as one pass over its units in order gives
// it: a unit wins only with a larger logit, so ties go to the lower class and
// a NaN loses, unless it is the first unit's.  z: this lane's logits, -inf
// where it has none; at: each one's class less shift, rising.  holds: this
// lane has the head's first unit, z[first].  m: the row's largest logit.
template <int N, int LOW>
__device__ __forceinline__ int head_argmax(const float (&z)[N], const int (&at)[N], int shift, int first, bool holds,
                                           float &m) {
  m = z[0];
#pragma unroll
  for (int k = 1; k + 1 < N; k += 2) m = fmaxf(fmaxf(z[k], z[k + 1]), m);
  if constexpr (N % 2 == 0) m = fmaxf(m, z[N - 1]);
  m = across<LOW>(m, [](float u, float v) { return fmaxf(u, v); });
  int i = 64;
#pragma unroll
  for (int k = N - 1; k >= 0; k--) i = z[k] == m ? at[k] : i;
  if (holds && z[first] != z[first]) i = -64;
  i = across<LOW>(i + shift, [](int u, int v) { return min(u, v); });
  return max(i, 0);   // (below 0: the first unit's NaN, or no logit above -inf)
}

// 1 / x for 1 <= x <= 10 (a softmax denominator): the hardware reciprocal and
// one Newton step.
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}

// e^x for x <= 0 as 2^(x log2 e): the product's rounding moves the result by
// at most |x| e^x 2^-24, below 3e-8 of a softmax sum.
__device__ __forceinline__ float exp_neg(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504f); }

// The wave's 32 x 37 logits, staged in LDS as the output holds them.
__device__ __forceinline__ void put_logits(const float *sz, float *out, int rows, int lane) {
  __builtin_amdgcn_s_waitcnt(0xc07f);   // this wave's LDS writes are done
  __builtin_amdgcn_wave_barrier();
  for (int i = lane; i < rows * kOut; i += 64) out[i] = sz[i];
  __builtin_amdgcn_wave_barrier();
}

// The biases as float32 in LDS, zero past the last unit of a layer.
__device__ __forceinline__ void load_biases(const uint16_t *w, float (*sb)[kH]) {
  for (int i = threadIdx.x; i < 3 * kH; i += 64 * kMfmaWaves) {
    const int l = i / kH, j = i % kH;
    sb[l][j] = l == 0 ? bf16_to_f32(w[oB1 + j]) : (l == 1 ? bf16_to_f32(w[oB2 + j]) : (j < kOut ? bf16_to_f32(w[oB3 + j]) : 0.0f));
  }
  __syncthreads();
}

template <bool LOGITS>
__global__ __launch_bounds__(64 * kMfmaWaves, kMfmaWgs) void k_mlp_infer_mfma(InferArgs a) {
  __shared__ __attribute__((aligned(16))) float sb[3][kH];
  __shared__ float sz[LOGITS ? kMfmaWaves : 1][LOGITS ? 32 * kOut : 1];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, h = lane >> 5;
  load_biases(a.w, sb);
  // weights: W1 (K 16) as 2 unit tiles; W2, W3 (K 64) as 4 K steps x 2 tiles
  // (units from 37 on are zero)
  bf16x8 w1[2], w2[4][2], w3[4][2];
  const bf16x8 zero8 = {};
#pragma unroll
  for (int t = 0; t < 2; t++) {
    const int j = t * 32 + col;
    w1[t] = load_bf16x8(a.w + oW1 + j * kIn + h * 8);
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      w2[ks][t] = load_bf16x8(a.w + oW2 + j * kH + ks * 16 + h * 8);
      w3[ks][t] = j < kOut ? load_bf16x8(a.w + oW3 + j * kH + ks * 16 + h * 8) : zero8;
    }
  }
  auto products = [&](const bf16x8 (&w)[4][2], const bf16x8 (&x)[4], f32x16 (&d)[2]) {
    d[0] = d[1] = f32x16{};
#pragma unroll
    for (int ks = 0; ks < 4; ks++)
#pragma unroll
      for (int t = 0; t < 2; t++) d[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[ks][t], x[ks], d[t], 0, 0, 0);
  };
  // bias, ReLU, rounding to bf16, and the next layer's operand of each K
  // step.  The ReLU takes a NaN to 0.  FAST clamps the rounded pairs as signed
  // 16-bit numbers instead, which keeps a positive NaN: it makes every sum of its
  // row in the next layer NaN, of whatever sign, so each layer's sums are tested
  // before they are clamped, and the tile is then done again without FAST.
  auto next_operand = [&](auto fast, const f32x16 (&d)[2], const float *b, bf16x8 (&o)[4]) {
    constexpr bool FAST = decltype(fast)::value;
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef short i16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      uint32_t pk[4];   // units 16 ks + 4 h ..+3, then 16 ks + 8 + 4 h ..+3
#pragma unroll
      for (int g = 0; g < 2; g++) {
        const f32x4 bb = *reinterpret_cast<const f32x4 *>(b + 16 * ks + 8 * g);
#pragma unroll
        for (int p = 0; p < 2; p++) {
          const int r = 8 * (ks & 1) + 4 * g + 2 * p;
          float v0 = d[ks >> 1][r] + bb[2 * p], v1 = d[ks >> 1][r + 1] + bb[2 * p + 1];
          if constexpr (!FAST) v0 = fmaxf(v0, 0.0f), v1 = fmaxf(v1, 0.0f);
          const bf16x2 v = {(__bf16)v0, (__bf16)v1};
          uint32_t w = __builtin_bit_cast(uint32_t, v);
          if constexpr (FAST) {
            asm("" : "+v"(w));   // (keeps the two conversions one packed one)
            w = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, w), i16x2{0, 0}));
          }
          pk[2 * g + p] = w;
        }
      }
      // lane l keeps units 16 ks ..+7, lane l + 32 units 16 ks + 8 ..+7
      const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
      const u32x4 q = {s0[0], s1[0], s0[1], s1[1]};
      o[ks] = __builtin_bit_cast(bf16x8, q);
    }
  };
  const int64_t tiles = (a.n + 31) / 32, stride = (int64_t)gridDim.x * kMfmaWaves;
  f32x4 xu = {}, xv = {};   // this lane's half of its row, requested a tile ahead
  auto request = [&](int64_t tile) {
    const int64_t row = tile * 32 + col;
    if (row < a.n) {
      xu = *reinterpret_cast<const f32x4 *>(a.x + row * kIn + h * 8);
      xv = *reinterpret_cast<const f32x4 *>(a.x + row * kIn + h * 8 + 4);
    }
  };
  bf16x8 x;
  auto take_request = [&] {
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = (__bf16)xu[k], x[4 + k] = (__bf16)xv[k];
  };
  int64_t tile = (int64_t)blockIdx.x * kMfmaWaves + wv;
  request(tile);
  take_request();
  for (; tile < tiles; tile += stride) {
    request(tile + stride);
    f32x16 d[2];
    bool nan2 = false;   // a sum of layer 2 is NaN (all of its row are, if a NaN was kept)
    auto layers = [&](auto fast) {
      // (the biases are read anew for each tile: kept in registers, their 160
      // values would halve the waves per SIMD)
      int hb = 4 * h;
      asm volatile("" : "+v"(hb));
      const float *bias = &sb[0][0] + hb;
      bf16x8 o[4];
#pragma unroll
      for (int t = 0; t < 2; t++) d[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[t], x, f32x16{}, 0, 0, 0);
      next_operand(fast, d, bias, o);
      products(w2, o, d);
      if constexpr (decltype(fast)::value) nan2 = d[0][0] != d[0][0];
      next_operand(fast, d, bias + kH, o);
      products(w3, o, d);
#pragma unroll
      for (int g = 0; g < 5; g++) {
        const f32x4 bb = *reinterpret_cast<const f32x4 *>(bias + 2 * kH + 8 * g);
#pragma unroll
        for (int j = 0; j < 4; j++) d[g >> 2][(4 * g + j) & 15] += bb[j];
      }
    };
    layers(std::true_type{});
    if (__builtin_expect(__any(nan2 || d[0][0] != d[0][0]), 0)) layers(std::false_type{});
    // this lane's logits of its row: units 8 g + 4 h + j (d[0][4 g + j]), g = 0..3, and 32 + 4 h + j
    const int64_t r0 = tile * 32;
    const int rows = (int)min((int64_t)32, a.n - r0);
    const float ninf = -__builtin_inff();
    // threshold head: units 0..9 (lane l: 0-3, 8, 9; lane l + 32: 4-7)
    const float zc[6] = {d[0][0], d[0][1], d[0][2], d[0][3], h ? ninf : d[0][4], h ? ninf : d[0][5]};
    constexpr int ic[6] = {0, 1, 2, 3, 8, 9};
    float mc, mr;
    const int c = head_argmax<6, 32>(zc, ic, 4 * h, 0, !h, mc);
    // range head: units 10..36 (lane l: 10, 11, 16-19, 24-27, 32-35; lane l + 32: 12-15, 20-23, 28-31, 36)
    const float zr[16] = {h ? d[0][4] : ninf, h ? d[0][5] : ninf, d[0][6], d[0][7], d[0][8], d[0][9], d[0][10], d[0][11],
                          d[0][12], d[0][13], d[0][14], d[0][15], d[1][0], h ? ninf : d[1][1], h ? ninf : d[1][2],
                          h ? ninf : d[1][3]};
    constexpr int ir[16] = {-2, -1, 0, 1, 6, 7, 8, 9, 14, 15, 16, 17, 22, 23, 24, 25};
    const int q = head_argmax<16, 32>(zr, ir, 4 * h, 2, !h, mr);
    float den = 0.0f;
#pragma unroll
    for (int j = 0; j < 6; j++) den += exp_neg(zc[j] - mc);
    den = across<32>(den, [](float u, float v) { return u + v; });
    // the next tile's features are taken before this tile's stores: a wait for
    // loads also waits for every store issued before it is reached
    take_request();
    __builtin_amdgcn_sched_barrier(0);
    if (a.conf && !h && col < rows) a.conf[r0 + col] = recip(den);
    if (!h && col < rows) {
      a.cls[r0 + col] = (int8_t)c;
      a.rng[r0 + col] = (int8_t)q;
    }
    if constexpr (LOGITS) {
      float *sw = sz[wv];
#pragma unroll
      for (int k = 0; k < 20; k++) {
        const int u = 8 * (k / 4) + 4 * h + k % 4;
        if (u < kOut) sw[col * kOut + u] = d[k >> 4][k & 15];
      }
      put_logits(sw, a.logits + r0 * kOut, rows, lane);
    }
  }
}

// The parameters as bf16 in LDS.  The weights' row strides put the rows of an
// operand in different banks.
constexpr int kLdW1 = kIn + 4, kLdW = kH + 4;
constexpr int kLdsW = kH * kLdW1 + (kH + kOut) * kLdW + 2 * kH + kOut + 1;
struct LdsWeights {
  uint16_t *w1, *w2, *w3, *b1, *b2, *b3;   // [kH][kLdW1], [kH][kLdW], [kOut][kLdW], biases
  __device__ explicit LdsWeights(uint16_t *p)
      : w1(p), w2(w1 + kH * kLdW1), w3(w2 + kH * kLdW), b1(w3 + kOut * kLdW), b2(b1 + kH), b3(b2 + kH) {}
  // two parameters at a time (every part starts at an even offset); T threads
  template <int T>
  __device__ __forceinline__ void fill(const uint16_t *w, int t) const {
    const bool words = reinterpret_cast<uintptr_t>(w) % 4 == 0;
    auto copy2 = [&](uint16_t *dst, int o) {
      *reinterpret_cast<uint32_t *>(dst) =
          words ? *reinterpret_cast<const uint32_t *>(w + o) : (uint32_t)w[o] | (uint32_t)w[o + 1] << 16;
    };
#pragma unroll
    for (int i = t; i < kH * kIn / 2; i += T) copy2(w1 + i / (kIn / 2) * kLdW1 + i % (kIn / 2) * 2, oW1 + 2 * i);
#pragma unroll
    for (int i = t; i < kH * kH / 2; i += T) copy2(w2 + i / (kH / 2) * kLdW + i % (kH / 2) * 2, oW2 + 2 * i);
#pragma unroll
    for (int i = t; i < kOut * kH / 2; i += T) copy2(w3 + i / (kH / 2) * kLdW + i % (kH / 2) * 2, oW3 + 2 * i);
    if (t < kH / 2) copy2(b1 + 2 * t, oB1 + 2 * t);
    else if (t < kH) copy2(b2 + 2 * (t - kH / 2), oB2 + 2 * (t - kH / 2));
    else if (t < kH + kOut) b3[t - kH] = w[oB3 + t - kH];
  }
};

// ---------------------------------------------------------------------------
// inference in float32
// ---------------------------------------------------------------------------
// What bounds it: the fp32 matrix rate (the fp32 MFMAs share the vector unit,
// so the heads and the ReLU add to it).  Each wave runs tiles of 32 rows with
// the weights, widened to float32, as the first operand: layers 1 and 2 through
// v_mfma_f32_32x32x2_f32, layer 3 (37 units) through v_mfma_f32_16x16x4_f32,
// which pads it to 48 units instead of 64.  An fp32 MFMA accumulates its K
// elements as a chain of fused multiply-adds, so with the bias as the initial
// value and K in order a logit has the bits of a loop of fmas over the units.
// As in the bf16 kernel a row's values stay in its lanes; exchanges of register
// halves and quarters put the K elements where the next product wants them.
// The 128 weight registers allow two waves per SIMD, which fill the unit.
// Measured over 1.57 M rows: 229 us, 103 TFLOP/s (394 us with one row per lane
// and the weights through the scalar unit: unpacked fp32 fmas reach half of
// the matrix rate).
constexpr int kF32Wgs = 2;   // workgroups per compute unit that the registers allow

// max(x, 0), a NaN to 0, as one operation: the median of x, 0 and infinity
// (fmaxf of a matrix product is canonicalised by a second operation first, as
// is a median whose infinity the compiler can see)
__device__ __forceinline__ float opaque_inf() {
  float v = __builtin_inff();
  asm("" : "+s"(v));
  return v;
}
__device__ __forceinline__ void swap32(float &u, float &v) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(v), false, false);
  u = __uint_as_float(s[0]);
  v = __uint_as_float(s[1]);
}
__device__ __forceinline__ void swap16(float &u, float &v) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(u), __float_as_uint(v), false, false);
  u = __uint_as_float(s[0]);
  v = __uint_as_float(s[1]);
}

template <bool LOGITS>
__global__ __launch_bounds__(64 * kMfmaWaves, kF32Wgs) void k_mlp_infer(InferArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t sw[kLdsW];
  __shared__ __attribute__((aligned(16))) float sb[3][kH];
  __shared__ float sz[LOGITS ? kMfmaWaves : 1][LOGITS ? 32 * kOut : 1];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, h = lane >> 5, c16 = lane & 15, kq = lane >> 4;
  const float inf = opaque_inf(), ninf = -inf;
  const LdsWeights lw(sw);
  lw.fill<64 * kMfmaWaves>(a.w, threadIdx.x);
  load_biases(a.w, sb);
  float w1[2][kIn / 2], w2[2][kH / 2], w3[3][kH / 4];
#pragma unroll
  for (int t = 0; t < 2; t++) {
#pragma unroll
    for (int s = 0; s < kIn / 2; s++) w1[t][s] = bf16_to_f32(lw.w1[(t * 32 + col) * kLdW1 + 2 * s + h]);
#pragma unroll
    for (int s = 0; s < kH / 2; s++) w2[t][s] = bf16_to_f32(lw.w2[(t * 32 + col) * kLdW + 2 * s + h]);
  }
#pragma unroll
  for (int t = 0; t < 3; t++)
#pragma unroll
    for (int s = 0; s < kH / 4; s++)
      w3[t][s] = t * 16 + c16 < kOut ? bf16_to_f32(lw.w3[min(t * 16 + c16, kOut - 1) * kLdW + 4 * s + kq]) : 0.0f;
  const int64_t tiles = (a.n + 31) / 32, stride = (int64_t)gridDim.x * kMfmaWaves;
  f32x4 xu = {}, xv = {};   // this lane's half of its row, requested a tile ahead
  auto request = [&](int64_t tile) {
    const int64_t row = tile * 32 + col;
    if (row < a.n) {
      xu = *reinterpret_cast<const f32x4 *>(a.x + row * kIn + h * 8);
      xv = *reinterpret_cast<const f32x4 *>(a.x + row * kIn + h * 8 + 4);
    }
  };
  float x[kIn / 2];   // features 2 s + h of row col
  auto take_request = [&] {
    float u[8] = {xu[0], xu[1], xu[2], xu[3], xv[0], xv[1], xv[2], xv[3]};
#pragma unroll
    for (int p = 0; p < 4; p++) {
      swap32(u[2 * p], u[2 * p + 1]);
      x[p] = u[2 * p];
      x[4 + p] = u[2 * p + 1];
    }
  };
  int64_t tile = (int64_t)blockIdx.x * kMfmaWaves + wv;
  request(tile);
  take_request();
  for (; tile < tiles; tile += stride) {
    request(tile + stride);
    int hb = 4 * h, kb = 4 * kq;   // (the biases are read anew for each tile, not kept in registers)
    asm volatile("" : "+v"(hb), "+v"(kb));
    auto bias_tile = [&](int l, int t) {
      f32x16 d;
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const f32x4 b = *reinterpret_cast<const f32x4 *>(&sb[l][0] + hb + t * 32 + 8 * g);
#pragma unroll
        for (int j = 0; j < 4; j++) d[4 * g + j] = b[j];
      }
      return d;
    };
    f32x16 d[2] = {bias_tile(0, 0), bias_tile(0, 1)};
#pragma unroll
    for (int s = 0; s < kIn / 2; s++)
#pragma unroll
      for (int t = 0; t < 2; t++) d[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[t][s], x[s], d[t], 0, 0, 0);
    f32x16 e[2] = {bias_tile(1, 0), bias_tile(1, 1)};
    float v[kH / 2];   // units 2 s + h of row col
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        float u[4];
#pragma unroll
        for (int j = 0; j < 4; j++) u[j] = __builtin_amdgcn_fmed3f(d[t][4 * g + j], 0.0f, inf);
        swap32(u[0], u[1]);
        swap32(u[2], u[3]);
        float *o = v + 16 * t + 4 * g;
        o[0] = u[0], o[1] = u[2], o[2] = u[1], o[3] = u[3];
      }
#pragma unroll
    for (int s = 0; s < kH / 2; s++)
#pragma unroll
      for (int t = 0; t < 2; t++) e[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(w2[t][s], v[s], e[t], 0, 0, 0);
    // layer 3: rows 16 nt..+15, unit tile t; lane = row c16, K quarter kq
    f32x4 z[2][3];
#pragma unroll
    for (int t = 0; t < 3; t++) z[0][t] = z[1][t] = *reinterpret_cast<const f32x4 *>(&sb[2][0] + kb + 16 * t);
#pragma unroll
    for (int g = 0; g < 8; g++) {
      float u[4];
#pragma unroll
      for (int j = 0; j < 4; j++) u[j] = __builtin_amdgcn_fmed3f(e[g >> 2][4 * (g & 3) + j], 0.0f, inf);
      swap32(u[0], u[2]);
      swap32(u[1], u[3]);
      swap16(u[0], u[1]);
      swap16(u[2], u[3]);
#pragma unroll
      for (int k = 0; k < 2; k++)
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
          for (int nt = 0; nt < 2; nt++)
            z[nt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w3[t][2 * g + k], u[2 * k + nt], z[nt][t], 0, 0, 0);
    }
    // heads: this lane's logits of rows c16 and 16 + c16 are units 16 t + 4 kq + r
    const int64_t r0 = tile * 32;
    const int rows = (int)min((int64_t)32, a.n - r0);
    int cls[2], rng[2];
    float den[2];
#pragma unroll
    for (int nt = 0; nt < 2; nt++) {
      float zc[4], zr[12];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const bool is_cls = 4 * kq + r < kCls;
        zc[r] = is_cls ? z[nt][0][r] : ninf;
        zr[r] = is_cls ? ninf : z[nt][0][r];
        zr[4 + r] = z[nt][1][r];
        zr[8 + r] = 32 + 4 * kq + r < kOut ? z[nt][2][r] : ninf;
      }
      constexpr int ic[4] = {0, 1, 2, 3}, ir[12] = {-10, -9, -8, -7, 6, 7, 8, 9, 22, 23, 24, 25};
      float mc, mr;
      cls[nt] = head_argmax<4, 16>(zc, ic, 4 * kq, 0, kq == 0, mc);
      rng[nt] = head_argmax<12, 16>(zr, ir, 4 * kq, 2, kq == 2, mr);
      float s = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; r++) s += exp_neg(zc[r] - mc);
      den[nt] = across<16>(s, [](float p, float q) { return p + q; });
    }
    // the next tile's features are taken before this tile's stores: a wait for
    // loads also waits for every store issued before it is reached
    take_request();
    __builtin_amdgcn_sched_barrier(0);
    if (lane < rows) {   // (lane < 32: row lane, of half kq)
      a.cls[r0 + lane] = (int8_t)(kq ? cls[1] : cls[0]);
      a.rng[r0 + lane] = (int8_t)(kq ? rng[1] : rng[0]);
      if (a.conf) a.conf[r0 + lane] = recip(kq ? den[1] : den[0]);
    }
    if constexpr (LOGITS) {
      float *so = sz[wv];
#pragma unroll
      for (int nt = 0; nt < 2; nt++)
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
          for (int r = 0; r < 4; r++)
            if (16 * t + 4 * kq + r < kOut) so[(16 * nt + c16) * kOut + 16 * t + 4 * kq + r] = z[nt][t][r];
      put_logits(so, a.logits + r0 * kOut, rows, lane);
    }
  }
}

// ---------------------------------------------------------------------------
// batch gradient: 128 rows per workgroup, all contractions on the matrix cores
// ---------------------------------------------------------------------------
// What bounds it: at a training batch (1,024 rows, eight 128-row tiles) the
// latency of one workgroup's chain of layers, at large batches the fp32 matrix
// rate.  Every contraction (three layers forward, two back, three weight
// gradients) runs as fp32 MFMAs (fp32 operands and accumulation, the bf16
// weights widened).  Activations and deltas live in LDS as [row][unit] with a
// row stride of 68 words: a lane reads four consecutive units of its row in one
// 16-byte read (the operand of four MFMAs; K is taken in that order), and the
// weight gradients, which contract over rows, read 32 consecutive units of two
// rows 8 apart, which fall in different halves of the 64 banks.  The layers
// are computed transposed (units x rows), so the softmax of a row needs two
// exchanges between lanes and no LDS.  Each weight gradient is contracted over
// the two halves of the rows by different waves and the halves added.
// Measured: gradient and reduction at 1,024 rows 18 us (505 us with one
// output per lane as scalar LDS dot products), at 60,000 rows 61 us.
constexpr int kGradThreads = 512;
constexpr int kLd = kH + 4;     // row stride of the activations and deltas
constexpr int kLdX = kIn + 4;   // row stride of the features
constexpr int kRedTile = 16 * 64 + 64;      // one wave's tile and its column sums

struct GradArgs {
  const uint16_t *w;
  const float *x;
  const int8_t *cls, *rng;
  int n;
  float *part;   // [ceil(n/128)][kParams + 1]: partial gradient sums, then the partial loss
  int split;     // blockIdx.y computes one layer's gradient (else every workgroup all three)
};

__device__ __forceinline__ f32x4 lds4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }

// One wave's 32 x 32 tile of sum_r P[r][m] Q[r][n] over 64 rows, and (in
// psum) its lane's share of the column sums of P.
__device__ __forceinline__ f32x16 outer_tile(const float *P, const float *Q, int h, float &psum) {
  f32x16 d = {};
  psum = 0.0f;
#pragma unroll 8
  for (int i = 0; i < 32; i++) {
    const int r = (i >> 3) * 16 + (i & 7) + 8 * h;
    const float p = P[r * kLd], q = Q[r * kLd];
    psum += p;
    d = __builtin_amdgcn_mfma_f32_32x32x2f32(p, q, d, 0, 0, 0);
  }
  return d;
}

// A layer's weight gradient [M][64] and bias gradient [M] of the tile: four
// 32 x 32 tiles, each by two waves over half of the rows.
__device__ __forceinline__ void weight_grad(const float *P, const float *Q, int M, float *gw, float *gb, float *red,
                                            int wave, int lane) {
  const int col = lane & 31, h = lane >> 5, mt = wave & 1, nt = (wave >> 1) & 1, half = wave >> 2;
  float psum;
  const f32x16 d = outer_tile(P + half * 64 * kLd + mt * 32 + col, Q + half * 64 * kLd + nt * 32 + col, h, psum);
  float *mine = red + (wave & 3) * kRedTile + lane;
  if (half) {
#pragma unroll
    for (int r = 0; r < 16; r++) mine[r * 64] = d[r];
    mine[16 * 64] = psum;
  }
  __syncthreads();
  if (!half) {
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int m = mt * 32 + 8 * (r / 4) + 4 * h + r % 4;
      if (m < M) gw[m * kH + nt * 32 + col] = d[r] + mine[r * 64];
    }
    psum += mine[16 * 64];
    psum += __shfl_xor(psum, 32);
    if (nt == 0 && h == 0 && mt * 32 + col < M) gb[mt * 32 + col] = psum;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kGradThreads) void k_mlp_grad(GradArgs a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float *X = smem;                       // [kTile][kLdX]
  float *H1 = X + kTile * kLdX;          // [kTile][kLd], later dL/d(pre-activation 1)
  float *H2 = H1 + kTile * kLd;          // [kTile][kLd], later dL/d(pre-activation 2)
  float *Z = H2 + kTile * kLd;           // [kTile][kLd], dL/dz, zero from column 37
  float *red = Z + kTile * kLd;          // [4][kRedTile] tiles of the second row halves
  float *rloss = red + 4 * kRedTile;     // [8] loss of each wave's rows
  uint16_t *sw = reinterpret_cast<uint16_t *>(rloss + 8);   // the parameters
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r0 = blockIdx.x * kTile, rows = min(kTile, a.n - r0);
  const int roles = a.split ? 1 << blockIdx.y : 7;   // 1: layer 3 and the loss, 2: layer 2, 4: layer 1
  const float inv_n = 1.0f / (float)a.n;
  const LdsWeights lw(sw);
  lw.fill<kGradThreads>(a.w, t);
#pragma unroll
  for (int i = t; i < kTile * kIn; i += kGradThreads) {
    const int r = i / kIn;
    X[r * kLdX + i % kIn] = r < rows ? a.x[(size_t)r0 * kIn + i] : 0.0f;
  }
  // this lane's row in the softmax below: its labels, read early
  const int srow = wave * 16 + (lane & 15);
  int yc = 0, yr = 0;
  if (srow < rows) {
    yc = a.cls[r0 + srow];
    yr = a.rng[r0 + srow];
  }
  __syncthreads();
  // layers 1 and 2: wave = (rows 32 rt.., units 32 ut..); lane = row col, K half h
  const int col = lane & 31, h = lane >> 5, rt = wave & 3, ut = wave >> 2;
  const int row = rt * 32 + col;
  auto store_units = [&](float *dst, const f32x16 &d) {   // ReLU, four consecutive units at a time
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const f32x4 v = {fmaxf(d[4 * g], 0.0f), fmaxf(d[4 * g + 1], 0.0f), fmaxf(d[4 * g + 2], 0.0f),
                       fmaxf(d[4 * g + 3], 0.0f)};
      *reinterpret_cast<f32x4 *>(dst + row * kLd + ut * 32 + 8 * g + 4 * h) = v;
    }
  };
  auto bias_units = [&](const uint16_t *b) {
    f32x16 d;
#pragma unroll
    for (int r = 0; r < 16; r++) d[r] = bf16_to_f32(b[ut * 32 + 8 * (r / 4) + 4 * h + r % 4]);
    return d;
  };
  {
    f32x16 d = bias_units(lw.b1);
#pragma unroll
    for (int c = 0; c < kIn / 8; c++) {
      const f32x4 b = lds4(X + row * kLdX + 8 * c + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; j++)
        d = __builtin_amdgcn_mfma_f32_32x32x2f32(bf16_to_f32(lw.w1[(ut * 32 + col) * kLdW1 + 8 * c + 4 * h + j]), b[j],
                                                 d, 0, 0, 0);
    }
    store_units(H1, d);
  }
  __syncthreads();
  {
    f32x16 d = bias_units(lw.b2);
#pragma unroll
    for (int c = 0; c < kH / 8; c++) {
      const f32x4 b = lds4(H1 + row * kLd + 8 * c + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; j++)
        d = __builtin_amdgcn_mfma_f32_32x32x2f32(bf16_to_f32(lw.w2[(ut * 32 + col) * kLdW + 8 * c + 4 * h + j]), b[j],
                                                 d, 0, 0, 0);
    }
    store_units(H2, d);
  }
  __syncthreads();
  // layer 3 and both softmax cross-entropies: wave = 16 rows, lane = row
  // lane%16 and, in each of three 16-unit tiles, units 4 (lane/16) ..+3
  {
    const int c16 = lane & 15, kq = lane >> 4;
    f32x4 z[3];
#pragma unroll
    for (int tt = 0; tt < 3; tt++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int o = 16 * tt + 4 * kq + r;
        z[tt][r] = o < kOut ? bf16_to_f32(lw.b3[o]) : 0.0f;
      }
#pragma unroll
    for (int c = 0; c < kH / 16; c++) {
      const f32x4 b = lds4(H2 + srow * kLd + 16 * c + 4 * kq);
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int tt = 0; tt < 3; tt++) {
          const int o = 16 * tt + c16;
          const float w = o < kOut ? bf16_to_f32(lw.w3[o * kLdW + 16 * c + 4 * kq + j]) : 0.0f;
          z[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, b[j], z[tt], 0, 0, 0);
        }
    }
    // (a row's 37 logits are spread over the four lanes c16 + 16 kq)
    auto fmax2 = [](float u, float v) { return fmaxf(u, v); };
    auto add2 = [](float u, float v) { return u + v; };
    float mx[2] = {-__builtin_inff(), -__builtin_inff()}, den[2] = {0.0f, 0.0f}, zy[2] = {0.0f, 0.0f};
    const int y[2] = {yc, kCls + yr};
#pragma unroll
    for (int tt = 0; tt < 3; tt++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int o = 16 * tt + 4 * kq + r;
        if (o < kCls) mx[0] = fmaxf(mx[0], z[tt][r]);
        else if (o < kOut) mx[1] = fmaxf(mx[1], z[tt][r]);
      }
    mx[0] = across<16>(mx[0], fmax2);
    mx[1] = across<16>(mx[1], fmax2);
    f32x4 p[3];
#pragma unroll
    for (int tt = 0; tt < 3; tt++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int o = 16 * tt + 4 * kq + r, hd = o < kCls ? 0 : 1;
        p[tt][r] = o < kOut ? expf(z[tt][r] - (hd ? mx[1] : mx[0])) : 0.0f;
        (hd ? den[1] : den[0]) += p[tt][r];
        if (o == y[0]) zy[0] = z[tt][r];
        if (o == y[1]) zy[1] = z[tt][r];
      }
    float loss = 0.0f;
    const bool live = srow < rows, good = yc >= 0 && yc < kCls && yr >= 0 && yr < kRng;
#pragma unroll
    for (int hd = 0; hd < 2; hd++) {
      den[hd] = across<16>(den[hd], add2);
      zy[hd] = across<16>(zy[hd], add2);   // (one lane holds the label's logit, the others 0)
      loss += logf(den[hd]) + mx[hd] - zy[hd];
    }
    const float inv[2] = {1.0f / den[0], 1.0f / den[1]};
#pragma unroll
    for (int tt = 0; tt < 4; tt++) {
      f32x4 dz = {};
      if (tt < 3 && live && good)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int o = 16 * tt + 4 * kq + r;
          if (o < kOut) dz[r] = (p[tt < 3 ? tt : 0][r] * (o < kCls ? inv[0] : inv[1]) - (o == y[0] || o == y[1] ? 1.0f : 0.0f)) * inv_n;
        }
      *reinterpret_cast<f32x4 *>(Z + srow * kLd + 16 * tt + 4 * kq) = dz;
    }
    loss = !live ? 0.0f : (good ? loss : __builtin_nanf(""));
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) loss += __shfl_xor(loss, d);
    if (lane == 0) rloss[wave] = loss;
  }
  __syncthreads();
  float *part = a.part + (size_t)blockIdx.x * (kParams + 1);
  if (roles & 1) {
    if (t == 0) {
      float l = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; k++) l += rloss[k];
      part[kParams] = l * inv_n;
    }
    weight_grad(Z, H2, kOut, part + oW3, part + oB3, red, wave, lane);
  }
  if (!(roles & 6)) return;
  // back through a layer and the ReLU below it, in place over the activations
  auto back = [&](const f32x16 &d, float *act) {
#pragma unroll
    for (int g = 0; g < 4; g++) {
      f32x4 *p = reinterpret_cast<f32x4 *>(act + row * kLd + ut * 32 + 8 * g + 4 * h);
      f32x4 v = *p;
#pragma unroll
      for (int j = 0; j < 4; j++) v[j] = v[j] > 0.0f ? d[4 * g + j] : 0.0f;
      *p = v;
    }
  };
  {
    f32x16 d = {};
#pragma unroll
    for (int c = 0; c < (kOut + 7) / 8; c++) {
      const f32x4 b = lds4(Z + row * kLd + 8 * c + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int o = 8 * c + 4 * h + j;
        const float w = o < kOut ? bf16_to_f32(lw.w3[o * kLdW + ut * 32 + col]) : 0.0f;
        d = __builtin_amdgcn_mfma_f32_32x32x2f32(w, b[j], d, 0, 0, 0);
      }
    }
    back(d, H2);
  }
  __syncthreads();
  if (roles & 2) weight_grad(H2, H1, kH, part + oW2, part + oB2, red, wave, lane);
  if (!(roles & 4)) return;
  {
    f32x16 d = {};
#pragma unroll
    for (int c = 0; c < kH / 8; c++) {
      const f32x4 b = lds4(H2 + row * kLd + 8 * c + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; j++)
        d = __builtin_amdgcn_mfma_f32_32x32x2f32(bf16_to_f32(lw.w2[(8 * c + 4 * h + j) * kLdW + ut * 32 + col]), b[j],
                                                 d, 0, 0, 0);
    }
    back(d, H1);
  }
  __syncthreads();
  // layer 1: [64][16] as four 16 x 16 tiles, each by two waves over half of the rows
  {
    const int c16 = lane & 15, kq = lane >> 4, mt = wave & 3, half = wave >> 2;
    const float *P = H1 + half * 64 * kLd + mt * 16 + c16, *Q = X + half * 64 * kLdX + c16;
    f32x4 d = {};
    float psum = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const int r = (i >> 2) * 16 + (i & 3) + 4 * kq;
      const float p = P[r * kLd];
      psum += p;
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(p, Q[r * kLdX], d, 0, 0, 0);
    }
    float *mine = red + mt * kRedTile + lane;
    if (half) {
#pragma unroll
      for (int r = 0; r < 4; r++) mine[r * 64] = d[r];
      mine[4 * 64] = psum;
    }
    __syncthreads();
    if (!half) {
#pragma unroll
      for (int r = 0; r < 4; r++) part[oW1 + (mt * 16 + 4 * kq + r) * kIn + c16] = d[r] + mine[r * 64];
      psum += mine[4 * 64];
      psum += __shfl_xor(psum, 16);
      psum += __shfl_xor(psum, 32);
      if (kq == 0) part[oB1 + mt * 16 + c16] = psum;
    }
  }
}

// sum of the workgroups' partials, parameter by parameter (and the loss): 64
// parameters per workgroup, each wave a quarter of the partials, so that a
// batch of few partials costs one short chain of reads
__global__ __launch_bounds__(kThreads) void k_mlp_reduce(const float *part, int nwg, float *grad, float *loss) {
  __shared__ float sums[kThreads / 64][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
  float acc = 0.0f;
  if (p <= kParams)
#pragma unroll 4
    for (int w = wv; w < nwg; w += kThreads / 64) acc += part[(size_t)w * (kParams + 1) + p];
  sums[wv][lane] = acc;
  __syncthreads();
  if (wv || p > kParams) return;
  acc = (sums[0][lane] + sums[1][lane]) + (sums[2][lane] + sums[3][lane]);
  if (p < kParams)
    grad[p] = acc;
  else
    loss[0] = acc;
}

struct AdamArgs {
  float *master;
  uint16_t *w;
  float *m, *v;
  const float *grad;
  float lr, beta1, beta2, eps, c1, c2;   // c1 = 1/(1-beta1^t), c2 = 1/(1-beta2^t)
};

__global__ __launch_bounds__(kThreads) void k_mlp_adam(AdamArgs a) {
  const int p = blockIdx.x * kThreads + threadIdx.x;
  if (p >= kParams) return;
  const float g = a.grad[p];
  const float m = a.beta1 * a.m[p] + (1.0f - a.beta1) * g;
  const float v = a.beta2 * a.v[p] + (1.0f - a.beta2) * g * g;
  a.m[p] = m;
  a.v[p] = v;
  const float w = a.master[p] - a.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
  a.master[p] = w;
  a.w[p] = f32_to_bf16(w);
}

lfc_status mlp_check(const void *p, size_t need, size_t align, const char *who, const char *what) {
  if (!p) return lfc::fail(LFC_E_INVALID, std::string(who) + ": null " + what);
  if (reinterpret_cast<uintptr_t>(p) % align)
    return lfc::fail(LFC_E_INVALID, std::string(who) + ": " + what + " is not " + std::to_string(align) + "-byte aligned");
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) != hipSuccess || !base) {
    (void)hipGetLastError();
    return lfc::fail(LFC_E_INVALID, std::string(who) + ": " + what + " is not device memory");
  }
  const size_t off = static_cast<const char *>(p) - static_cast<const char *>(base);
  if (off + need > size) return lfc::fail(LFC_E_INVALID, std::string(who) + ": " + what + " is too small");
  return LFC_OK;
}

lfc_status mlp_launched(const char *who) {
  const hipError_t he = hipGetLastError();
  if (he != hipSuccess) return lfc::fail(LFC_E_HIP, std::string(who) + ": launch failed: " + hipGetErrorString(he));
  return LFC_OK;
}

constexpr size_t kGradLds = sizeof(float) * (kTile * (kLdX + 3 * kLd) + 4 * kRedTile + 8) + sizeof(uint16_t) * kLdsW;

lfc_status infer_launch(const uint16_t *w, const float *x, int64_t n, int8_t *cls, int8_t *rng, float *conf,
                        float *logits, int32_t precision, hipStream_t s) {
  if (n == 0) return LFC_OK;
  InferArgs a{w, x, n, cls, rng, conf, logits};
  const bool bf16 = precision == LFC_MLP_BF16;
  // resident workgroups whose waves take tiles in turn
  const int64_t groups = ((n + 31) / 32 + kMfmaWaves - 1) / kMfmaWaves;
  const dim3 grid((unsigned)std::min<int64_t>(groups, (int64_t)(bf16 ? kMfmaWgs : kF32Wgs) * kCus));
  const auto kern = bf16 ? (logits ? k_mlp_infer_mfma<true> : k_mlp_infer_mfma<false>)
                         : (logits ? k_mlp_infer<true> : k_mlp_infer<false>);
  hipLaunchKernelGGL(kern, grid, dim3(64 * kMfmaWaves), 0, s, a);
  return mlp_launched("lfc_mlp_infer");
}

}  // namespace

extern "C" lfc_status lfc_mlp_infer(const uint16_t *d_w, const float *d_x, int64_t n, int8_t *d_cls, int8_t *d_rng,
                                    float *d_conf, float *d_logits, hipStream_t s) {
  return lfc_mlp_infer_ex(d_w, d_x, n, d_cls, d_rng, d_conf, d_logits, LFC_MLP_FP32, s);
}

extern "C" lfc_status lfc_mlp_infer_ex(const uint16_t *d_w, const float *d_x, int64_t n, int8_t *d_cls, int8_t *d_rng,
                                       float *d_conf, float *d_logits, int32_t precision, hipStream_t s) {
  const char *who = "lfc_mlp_infer";
  if (precision != LFC_MLP_FP32 && precision != LFC_MLP_BF16)
    return lfc::fail(LFC_E_INVALID, "lfc_mlp_infer: unknown precision");
  if (n < 0) return lfc::fail(LFC_E_INVALID, "lfc_mlp_infer: n < 0");
  if (lfc_status st = mlp_check(d_w, sizeof(uint16_t) * kParams, 2, who, "d_w")) return st;
  if (n == 0) return LFC_OK;
  if (lfc_status st = mlp_check(d_x, sizeof(float) * kIn * (size_t)n, 16, who, "d_x")) return st;
  if (lfc_status st = mlp_check(d_cls, (size_t)n, 1, who, "d_cls")) return st;
  if (lfc_status st = mlp_check(d_rng, (size_t)n, 1, who, "d_rng")) return st;
  if (d_conf)
    if (lfc_status st = mlp_check(d_conf, sizeof(float) * (size_t)n, 4, who, "d_conf")) return st;
  if (d_logits)
    if (lfc_status st = mlp_check(d_logits, sizeof(float) * kOut * (size_t)n, 4, who, "d_logits")) return st;
  if (precision == LFC_MLP_BF16 && reinterpret_cast<uintptr_t>(d_w) % 16)
    return lfc::fail(LFC_E_INVALID, "lfc_mlp_infer: bf16 inference needs 16-byte aligned weights");
  return infer_launch(d_w, d_x, n, d_cls, d_rng, d_conf, d_logits, precision, s);
}

extern "C" lfc_status lfc_mlp_grad(const uint16_t *d_w, const float *d_x, const int8_t *d_cls, const int8_t *d_rng,
                                   int32_t n, float *d_part, float *d_grad, float *d_loss, hipStream_t s) {
  const char *who = "lfc_mlp_grad";
  if (n < 1) return lfc::fail(LFC_E_INVALID, "lfc_mlp_grad: n < 1");
  const int nwg = (n + kTile - 1) / kTile;
  if (lfc_status st = mlp_check(d_w, sizeof(uint16_t) * kParams, 2, who, "d_w")) return st;
  if (lfc_status st = mlp_check(d_x, sizeof(float) * kIn * (size_t)n, 4, who, "d_x")) return st;
  if (lfc_status st = mlp_check(d_cls, (size_t)n, 1, who, "d_cls")) return st;
  if (lfc_status st = mlp_check(d_rng, (size_t)n, 1, who, "d_rng")) return st;
  if (lfc_status st = mlp_check(d_part, sizeof(float) * (kParams + 1) * (size_t)nwg, 4, who, "d_part")) return st;
  if (lfc_status st = mlp_check(d_grad, sizeof(float) * kParams, 4, who, "d_grad")) return st;
  if (lfc_status st = mlp_check(d_loss, sizeof(float), 4, who, "d_loss")) return st;
  // While three workgroups per tile fit the chip at once, each takes one
  // layer's gradient and repeats the forward pass: the chain of one workgroup
  // is what a small batch waits for (1,024 rows: 18.1 us split, 24.2 not;
  // 10,880: 21.0, 26.9).  Beyond that the repeated work costs throughput
  // (10,881 rows: 32.4 us split, 26.7 not; 60,000: 103, 61).
  const bool split = 3 * nwg <= kCus;
  GradArgs a{d_w, d_x, d_cls, d_rng, n, d_part, split};
  hipLaunchKernelGGL(k_mlp_grad, dim3(nwg, split ? 3 : 1), dim3(kGradThreads), kGradLds, s, a);
  if (lfc_status st = mlp_launched(who)) return st;
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kParams + 1 + 63) / 64), dim3(kThreads), 0, s,
                     (const float *)d_part, nwg, d_grad, d_loss);
  return mlp_launched(who);
}

extern "C" lfc_status lfc_mlp_adam(float *d_master, uint16_t *d_w, float *d_m, float *d_v, const float *d_grad,
                                   int32_t step, float lr, float beta1, float beta2, float eps, hipStream_t s) {
  const char *who = "lfc_mlp_adam";
  if (step < 1) return lfc::fail(LFC_E_INVALID, "lfc_mlp_adam: step < 1");
  if (lfc_status st = mlp_check(d_master, sizeof(float) * kParams, 4, who, "d_master")) return st;
  if (lfc_status st = mlp_check(d_w, sizeof(uint16_t) * kParams, 2, who, "d_w")) return st;
  if (lfc_status st = mlp_check(d_m, sizeof(float) * kParams, 4, who, "d_m")) return st;
  if (lfc_status st = mlp_check(d_v, sizeof(float) * kParams, 4, who, "d_v")) return st;
  if (lfc_status st = mlp_check(d_grad, sizeof(float) * kParams, 4, who, "d_grad")) return st;
  const double c1 = 1.0 / (1.0 - std::pow((double)beta1, step)), c2 = 1.0 / (1.0 - std::pow((double)beta2, step));
  AdamArgs a{d_master, d_w, d_m, d_v, d_grad, lr, beta1, beta2, eps, (float)c1, (float)c2};
  hipLaunchKernelGGL(k_mlp_adam, dim3((kParams + kThreads - 1) / kThreads), dim3(kThreads), 0, s, a);
  return mlp_launched(who);
}

namespace lfc {

// The encoder's inference over host rows: staged through stream-ordered
// device memory, then back to the host.
lfc_status mlp_infer_rows(const void *d_w, const float *feat, int64_t n, int8_t *cls, int8_t *rng, float *conf,
                          hipStream_t s) {
  if (n == 0) return LFC_OK;
  if (lfc_status st = mlp_check(d_w, sizeof(uint16_t) * kParams, 2, "lfc_encode_ctl", "d_mlp")) return st;
  char *d = nullptr;
  const size_t fx = sizeof(float) * kIn * (size_t)n, bytes = fx + sizeof(float) * (size_t)n + 2 * (size_t)n;
  if (hipMallocAsync(reinterpret_cast<void **>(&d), bytes, s) != hipSuccess) {
    (void)hipGetLastError();
    return fail(LFC_E_NOMEM, "lfc_encode_ctl: device memory for the network's rows");
  }
  float *dx = reinterpret_cast<float *>(d), *dconf = reinterpret_cast<float *>(d + fx);
  int8_t *dcls = reinterpret_cast<int8_t *>(d + fx + sizeof(float) * (size_t)n), *drng = dcls + n;
  lfc_status st = LFC_OK;
  if (hipMemcpyAsync(dx, feat, fx, hipMemcpyHostToDevice, s) != hipSuccess)
    st = fail(LFC_E_HIP, "lfc_encode_ctl: copy of the features");
  if (st == LFC_OK) st = infer_launch(static_cast<const uint16_t *>(d_w), dx, n, dcls, drng, dconf, nullptr, LFC_MLP_FP32, s);
  if (st == LFC_OK && (hipMemcpyAsync(cls, dcls, (size_t)n, hipMemcpyDeviceToHost, s) != hipSuccess ||
                       hipMemcpyAsync(rng, drng, (size_t)n, hipMemcpyDeviceToHost, s) != hipSuccess ||
                       hipMemcpyAsync(conf, dconf, sizeof(float) * (size_t)n, hipMemcpyDeviceToHost, s) != hipSuccess))
    st = fail(LFC_E_HIP, "lfc_encode_ctl: copy of the classes");
  if (hipFreeAsync(d, s) != hipSuccess && st == LFC_OK) st = fail(LFC_E_HIP, "lfc_encode_ctl: release");
  if (hipStreamSynchronize(s) != hipSuccess && st == LFC_OK) st = fail(LFC_E_HIP, "lfc_encode_ctl: synchronize");
  return st;
}

}  // namespace lfc
