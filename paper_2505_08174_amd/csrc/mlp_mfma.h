// The seeded kernel MLP (3 -> 64 -> 64 -> 64 -> 9, tanh) on BF16 MFMA
// (v_mfma_f32_32x32x16_bf16, FP32 accumulation) for one wave-tile of 32 pairs.
//
// Lane l works on pair p = l % 32; lanes l and l + 32 hold the same pair and
// split the K dimension of every product (K slots 8 h .. 8 h + 7, h = l / 32).
// Hidden layers are computed transposed, H^T[64 x 32] = W[64 x 64] H_in^T, so
// the pairs are the MFMA columns. An MFMA result register v of lane l holds
// row 8 (v / 4) + 4 h + v % 4 of column p; the next layer's K index is
// permuted to exactly that order (the weights are stored pre-permuted), so a
// layer's tanh output is the next layer's B operand without any data motion:
// K step s (features 16 s .. 16 s + 15) takes result registers 8 (s % 2) ..
// 8 (s % 2) + 7 of M tile s / 2.
//
// Precision: every weight W is stored as W_hi + W_lo (two BF16 numbers) and
// multiplied in two MFMAs, which removes the systematic error of rounding
// the weights to BF16; activations are rounded to BF16 once (near field) or
// carried as BF16 hi + lo with a third MFMA per K step (ACA samples, whose
// error must stay far below the cross-approximation tolerance). Layer 1 takes
// the input v = v_hi + v_lo split the same way, with the bias in spare K
// slots (K = 16: v_hi W_hi, v_lo W_hi, b_hi, b_lo, v_hi W_lo). The biases of
// layers 2-4 enter through one extra K step whose B operand is the constant
// column (1, 1, 0, ...). Accumulation is FP32.
#pragma once

#include <hip/hip_runtime.h>

#include "devmath.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Fragment table (16 bytes per lane and fragment) in LDS.
#define FR_L1 0                                // [mo 2][lane 64]
#define FR_L2 (FR_L1 + 2 * 64)                 // [mo 2][s 4][part 2][lane]; bias [mo 2][lane]
#define FR_L3 (FR_L2 + (2 * 4 * 2 + 2) * 64)
#define FR_L4 (FR_L3 + (2 * 4 * 2 + 2) * 64)   // [s 4][part 2][lane]; bias [lane]
#define FR_TOTAL (FR_L4 + (4 * 2 + 1) * 64)
#define FR_BYTES (FR_TOTAL * 16)

__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// tanh of 8 consecutive result registers -> one BF16 B operand (and, for
// the accurate tile, the BF16 remainder as a second operand). Layers 1-3 are
// stored scaled by 2 log2(e), so a result register y holds 2 log2(e) times
// the pre-activation x and tanh(x) = 1 - 2 / (2^y + 1). The accurate tile
// adds the remainder t - hi, rounded to BF16. Values go in pairs through one
// two-way BF16 conversion.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float tanh_scaled(float y) {
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(y) + 1.0f);
}

template <bool ACC>
__device__ __forceinline__ void act8(const f32x16& a, int base, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int u = 0; u < 8; u += 2) {
    const f32x2 t = {tanh_scaled(a[base + u]), tanh_scaled(a[base + u + 1])};
    const bf16x2 h = __builtin_convertvector(t, bf16x2);
    hi[u] = h[0];
    hi[u + 1] = h[1];
    if (ACC) {
      const uint32_t hb = __builtin_bit_cast(uint32_t, h);
      const f32x2 r = {t[0] - __uint_as_float(hb << 16), t[1] - __uint_as_float(hb & 0xffff0000u)};
      const bf16x2 l = __builtin_convertvector(r, bf16x2);
      lo[u] = l[0];
      lo[u + 1] = l[1];
    }
  }
}

// One hidden layer (64 -> 64) of NT independent tiles: B[t][4] in, Bo[t][4]
// out (after tanh). Each weight fragment is read once for all NT tiles, and
// the tiles' MFMA chains are independent, so one tile's MFMAs overlap the
// other's activations. ACC adds the products of the activation remainders
// (W_hi a_lo), for samples whose error must stay far below the
// cross-approximation tolerance.
template <bool ACC, int NT>
__device__ __forceinline__ void hidden_layer(const bf16x8* __restrict__ fr, int base, int lane,
                                             const bf16x8 (&B)[NT][4], const bf16x8 (&Bl)[NT][4],
                                             const bf16x8& Bone, bf16x8 (&Bo)[NT][4],
                                             bf16x8 (&Bol)[NT][4]) {
#pragma unroll
  for (int mo = 0; mo < 2; ++mo) {
    f32x16 acc[NT];
    const bf16x8 wb = fr[base + (2 * 4 * 2) * 64 + mo * 64 + lane];   // bias
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = mfma_bf16(wb, Bone, f32x16{});
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bf16x8 wh = fr[base + ((mo * 4 + s) * 2 + 0) * 64 + lane];
      const bf16x8 wl = fr[base + ((mo * 4 + s) * 2 + 1) * 64 + lane];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc[t] = mfma_bf16(wh, B[t][s], acc[t]);
        acc[t] = mfma_bf16(wl, B[t][s], acc[t]);
        if (ACC) acc[t] = mfma_bf16(wh, Bl[t][s], acc[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      act8<ACC>(acc[t], 0, Bo[t][2 * mo], Bol[t][2 * mo]);
      act8<ACC>(acc[t], 8, Bo[t][2 * mo + 1], Bol[t][2 * mo + 1]);
    }
  }
}

// Input of the kernel MLP at displacement (rx, ry, rz), |r|^-1, and the
// symmetrised entry K(r) = (O + O^T)/2 / (8 pi |r|). The roundings are spelled
// out (which product of |r|^2 is rounded, which remainder of v is taken), so
// that every kernel that samples a pair gets the same bits: the ACA's pivots
// and stopping tests hang on them, and a replay reproduces a build exactly.
struct PairIn {
  float v0, v1, v2, rs;
  float l0, l1, l2;   // v minus its BF16 rounding, before its own rounding to BF16
};
__device__ __forceinline__ float pair_norm2(float rx, float ry, float rz) {
  return __builtin_fmaf(rz, rz, __builtin_fmaf(rx, rx, ry * ry));
}
// exact = true: the remainder of the unrounded product r |r|^-1, else of v. Neither
// is the better one (both are rounded to BF16 next); which one a pair takes is part of
// what the BF16 forms have always computed (the compiler contracted one of two inlined
// copies), and ranks and pivots that callers saved from earlier builds hang on it.
__device__ __forceinline__ float pair_rest(float v, float r, float sc, bool exact) {
#pragma clang fp contract(off)
  const float h = (float)(__bf16)v;
  const float d = v - h;
  return exact ? __builtin_fmaf(r, sc, -h) : d;
}
__device__ __forceinline__ PairIn pair_in(int mode, float rx, float ry, float rz, bool exact) {
  PairIn in;
  in.rs = hh_rsqrt(pair_norm2(rx, ry, rz));
  const float sc = mode == HH_MLP_INPUT_DIRECTION ? in.rs : 1.0f;
  in.v0 = rx * sc;
  in.v1 = ry * sc;
  in.v2 = rz * sc;
  in.l0 = pair_rest(in.v0, rx, sc, exact);
  in.l1 = pair_rest(in.v1, ry, sc, exact);
  in.l2 = pair_rest(in.v2, rz, sc, exact);
  return in;
}
__device__ __forceinline__ void pair_entry(const float (&o)[9], float rs, float K[9]) {
  const float s = rs * (float)(1.0 / (16.0 * HH_PI));
  K[0] = 2.0f * o[0] * s; K[1] = (o[1] + o[3]) * s; K[2] = (o[2] + o[6]) * s;
  K[3] = K[1];            K[4] = 2.0f * o[4] * s;   K[5] = (o[5] + o[7]) * s;
  K[6] = K[2];            K[7] = K[5];              K[8] = 2.0f * o[8] * s;
}
// (K(r) f)_d of one pair; sc = |r|^-1 / (16 pi), or 0 for a pair that adds nothing
__device__ __forceinline__ void pair_apply(const float (&q)[9], float sc, float f0, float f1,
                                           float f2, double& u0, double& u1, double& u2) {
  const float a = q[1] + q[3], b = q[2] + q[6], c = q[5] + q[7];
  u0 += (double)(sc * __builtin_fmaf(b, f2, __builtin_fmaf(2.0f * q[0], f0, a * f1)));
  u1 += (double)(sc * __builtin_fmaf(c, f2, __builtin_fmaf(a, f0, 2.0f * q[4] * f1)));
  u2 += (double)(sc * __builtin_fmaf(2.0f * q[8], f2, __builtin_fmaf(b, f0, c * f1)));
}

// Result registers acc[t] of the output layer for NT independent tiles with
// layer-1 operands b1[t] (K slots (v_hi, v_lo, 1, 1) in lanes 0-31, (v_hi, 0..)
// in lanes 32-63). ACC = false: activations rounded to BF16 once (relative
// error ~1e-4 of a sample); ACC = true: activations carried as BF16 hi + lo
// (~3e-6), used where samples must resolve a 1e-4 cross-approximation.
template <bool ACC, int NT>
__device__ __forceinline__ void mlp_core_bf16(const bf16x8* __restrict__ fr,
                                              const bf16x8 (&b1)[NT], f32x16 (&acc)[NT]) {
  // the fragments are re-read from LDS for every call: hoisting them out of
  // a caller's loop would pin 192 VGPRs and cut the occupancy to one wave
  __asm__ volatile("" ::: "memory");
  const int lane = threadIdx.x & 63;
  const bool h1 = lane >= 32;
  const __bf16 z = (__bf16)0.0f, one = (__bf16)1.0f;
  bf16x8 Bone;
#pragma unroll
  for (int u = 0; u < 8; ++u) Bone[u] = (!h1 && u < 2) ? one : z;
  bf16x8 B[NT][4], Bn[NT][4], Bl[NT][4], Bnl[NT][4];
#pragma unroll
  for (int mo = 0; mo < 2; ++mo) {
    const bf16x8 w1 = fr[FR_L1 + mo * 64 + lane];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = mfma_bf16(w1, b1[t], f32x16{});
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      act8<ACC>(acc[t], 0, B[t][2 * mo], Bl[t][2 * mo]);
      act8<ACC>(acc[t], 8, B[t][2 * mo + 1], Bl[t][2 * mo + 1]);
    }
  }
  hidden_layer<ACC, NT>(fr, FR_L2, lane, B, Bl, Bone, Bn, Bnl);
  hidden_layer<ACC, NT>(fr, FR_L3, lane, Bn, Bnl, Bone, B, Bl);
  const bf16x8 w4b = fr[FR_L4 + (4 * 2) * 64 + lane];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = mfma_bf16(w4b, Bone, f32x16{});
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const bf16x8 wh = fr[FR_L4 + (s * 2 + 0) * 64 + lane];
    const bf16x8 wl = fr[FR_L4 + (s * 2 + 1) * 64 + lane];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc[t] = mfma_bf16(wh, B[t][s], acc[t]);
      acc[t] = mfma_bf16(wl, B[t][s], acc[t]);
      if (ACC) acc[t] = mfma_bf16(wh, Bl[t][s], acc[t]);
    }
  }
}

// Raw outputs o[0..8] for one tile of 32 pairs. Must be called by all 64 lanes
// of the wave with lanes l and l + 32 holding the same input.
template <bool ACC>
__device__ __forceinline__ void mlp_tile_bf16(const bf16x8* __restrict__ fr, const PairIn& in,
                                              float (&o)[9]) {
  const bool h1 = (threadIdx.x & 63) >= 32;
  const __bf16 z = (__bf16)0.0f, one = (__bf16)1.0f;
  bf16x8 b1[1];
  b1[0][0] = (__bf16)in.v0;
  b1[0][1] = (__bf16)in.v1;
  b1[0][2] = (__bf16)in.v2;
  b1[0][3] = h1 ? z : (__bf16)in.l0;
  b1[0][4] = h1 ? z : (__bf16)in.l1;
  b1[0][5] = h1 ? z : (__bf16)in.l2;
  b1[0][6] = h1 ? z : one;
  b1[0][7] = h1 ? z : one;
  f32x16 acc[1];
  mlp_core_bf16<ACC, 1>(fr, b1, acc);
  // rows 0-3 and 8 live in lanes 0-31 (registers 0-3, 4); rows 4-7 in 32-63
  const f32x16& c = acc[0];
  const float t0 = __shfl_xor(c[0], 32, 64), t1 = __shfl_xor(c[1], 32, 64);
  const float t2 = __shfl_xor(c[2], 32, 64), t3 = __shfl_xor(c[3], 32, 64);
  const float t4 = __shfl_xor(c[4], 32, 64);
  o[0] = h1 ? t0 : c[0]; o[1] = h1 ? t1 : c[1]; o[2] = h1 ? t2 : c[2];
  o[3] = h1 ? t3 : c[3]; o[4] = h1 ? c[0] : t0; o[5] = h1 ? c[1] : t1;
  o[6] = h1 ? c[2] : t2; o[7] = h1 ? c[3] : t3; o[8] = h1 ? t4 : c[4];
}

// v_permlane32_swap_b32: lo = (a of lanes 0-31, b of lanes 0-31), hi = (a of
// lanes 32-63, b of lanes 32-63)
struct HalfSwap {
  uint32_t lo, hi;
};
__device__ __forceinline__ HalfSwap half_swap(uint32_t a, uint32_t b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return HalfSwap{r[0], r[1]};
}

// Outputs of two tiles' result registers for 64 different pairs: lanes 0-31
// take the pairs of tile 0, lanes 32-63 those of tile 1. Rows 0-3 and 8 of a
// tile sit in its lanes 0-31 (registers 0-3, 4), rows 4-7 in its lanes 32-63.
__device__ __forceinline__ void pair_outputs(const float (&c0)[5], const float (&c1)[5],
                                             float (&o)[9]) {
#pragma unroll
  for (int e = 0; e < 5; ++e) {
    const HalfSwap r = half_swap(__float_as_uint(c0[e]), __float_as_uint(c1[e]));
    if (e < 4) {
      o[e] = __uint_as_float(r.lo);
      o[4 + e] = __uint_as_float(r.hi);
    } else {
      o[8] = __uint_as_float(r.lo);
    }
  }
}

// Raw outputs o[0..8] for 64 different pairs, one per lane: two tiles, lanes
// 0-31 and lanes 32-63. Each lane prepares the input of its own pair and takes
// the outputs of its own pair; half-wave swaps move them to and from the two
// tiles' operand layout, so nothing outside the tiles is computed twice (a
// single tile spends both halves of the wave on the same 32 pairs).
template <bool ACC>
__device__ __forceinline__ void mlp_pairs_bf16(const bf16x8* __restrict__ fr, const PairIn& in,
                                               float (&o)[9]) {
  const bool h1 = (threadIdx.x & 63) >= 32;
  const uint32_t w0 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)in.v0, (__bf16)in.v1});
  const uint32_t w1 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)in.v2, (__bf16)in.l0});
  const uint32_t w2 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)in.l1, (__bf16)in.l2});
  const HalfSwap s0 = half_swap(w0, w0), s1 = half_swap(w1, w1), s2 = half_swap(w2, w2);
  const uint32_t ones = h1 ? 0u : 0x3f803f80u;   // (1, 1) in the bias slots
  const uint32_t m1 = h1 ? 0x0000ffffu : 0xffffffffu, m2 = h1 ? 0u : 0xffffffffu;
  const uint4 q0 = make_uint4(s0.lo, s1.lo & m1, s2.lo & m2, ones);
  const uint4 q1 = make_uint4(s0.hi, s1.hi & m1, s2.hi & m2, ones);
  const bf16x8 b1[2] = {__builtin_bit_cast(bf16x8, q0), __builtin_bit_cast(bf16x8, q1)};
  f32x16 acc[2];
  mlp_core_bf16<ACC, 2>(fr, b1, acc);
  float c0[5], c1[5];
#pragma unroll
  for (int e = 0; e < 5; ++e) {
    c0[e] = acc[0][e];
    c1[e] = acc[1][e];
  }
  pair_outputs(c0, c1, o);
}

// Stage the fragment table (global -> LDS) by the whole workgroup.
__device__ __forceinline__ void stage_frags(bf16x8* __restrict__ lds, const uint4* __restrict__ g,
                                            int nthreads) {
  uint4* d = reinterpret_cast<uint4*>(lds);
  for (int i = threadIdx.x; i < FR_TOTAL; i += nthreads) d[i] = g[i];
}

// ------------------------------------------------------------ FP32 MFMA tile
//
// The same MLP for one wave-tile of 32 pairs on FP32 MFMA
// (v_mfma_f32_32x32x2_f32: FP32 operands and accumulation, the plain FP32
// form). Lane l works on pair l % 32 and supplies K slot h = l / 32 of every
// product. A result register r of lane l holds row 8 (r / 4) + 4 h + r % 4
// of its M tile; K step (mo, r) of the next layer contracts the two features
// 32 mo + 8 (r / 4) + r % 4 + 4 h, h = 0, 1, which are exactly what the two
// halves of the wave hold in register r, so a layer's tanh output is the next
// layer's B operand with no data motion (the weights are stored permuted to
// that order, one float per lane and step). Layer 1 contracts (v0, v1) and
// (v2, 1), the 1 carrying the bias; layers 2-4 take their bias through one
// extra step whose B operand is (1, 0). Layers 1-3 are stored scaled by
// 2 log2(e) (see tanh_scaled).
#define F32_L1 0                               // [mo 2][step 2]
#define F32_L2 (F32_L1 + 4)                    // [mo' 2][mo 2][r 16], bias [mo' 2]
#define F32_L3 (F32_L2 + 66)
#define F32_L4 (F32_L3 + 66)                   // [mo 2][r 16], bias
#define F32_FRAGS (F32_L4 + 33)
#define F32_BYTES (F32_FRAGS * 64 * 4)

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// One hidden layer (64 -> 64, then tanh) of NT tiles from h[t] into g[t]; the
// output M tiles of every tile are independent MFMA chains, and a weight is
// read once for all tiles.
template <int NT>
__device__ __forceinline__ void hidden_f32(const float* __restrict__ fr, int base, int lane,
                                           float bone, const float (&h)[NT][2][16],
                                           float (&g)[NT][2][16]) {
  f32x16 a0[NT], a1[NT];
  const float wb0 = fr[(base + 64) * 64 + lane], wb1 = fr[(base + 65) * 64 + lane];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    a0[t] = mfma_f32(wb0, bone, f32x16{});
    a1[t] = mfma_f32(wb1, bone, f32x16{});
  }
#pragma unroll
  for (int mo = 0; mo < 2; ++mo)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float w0 = fr[(base + (0 * 2 + mo) * 16 + r) * 64 + lane];
      const float w1 = fr[(base + (1 * 2 + mo) * 16 + r) * 64 + lane];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        a0[t] = mfma_f32(w0, h[t][mo][r], a0[t]);
        a1[t] = mfma_f32(w1, h[t][mo][r], a1[t]);
      }
    }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      g[t][0][r] = tanh_scaled(a0[t][r]);
      g[t][1][r] = tanh_scaled(a1[t][r]);
    }
}

__device__ __forceinline__ void hidden_f32(const float* __restrict__ fr, int base, int lane,
                                           float bone, const float (&h)[2][16],
                                           float (&g)[2][16]) {
  hidden_f32<1>(fr, base, lane, bone, reinterpret_cast<const float(&)[1][2][16]>(h),
                reinterpret_cast<float(&)[1][2][16]>(g));
}

// Result registers c[t][0..4] of the output layer (rows 0-3 and 8 in lanes
// 0-31, rows 4-7 in lanes 32-63) of NT tiles with the layer-1 operands b0 =
// (v0 | v1) and b1 = (v2 | 1) of the two lane halves. Called by all 64 lanes.
// fr: the FP32 fragment table (F32_FRAGS x 64 floats).
template <int NT>
__device__ __forceinline__ void mlp_core_f32(const float* __restrict__ fr, const float (&b0)[NT],
                                             const float (&b1)[NT], float (&c)[NT][5]) {
  __asm__ volatile("" ::: "memory");
  const int lane = threadIdx.x & 63;
  const float bone = lane >= 32 ? 0.0f : 1.0f;
  float h[NT][2][16], g[NT][2][16];
#pragma unroll
  for (int mo = 0; mo < 2; ++mo) {
    const float w0 = fr[(F32_L1 + 2 * mo) * 64 + lane], w1 = fr[(F32_L1 + 2 * mo + 1) * 64 + lane];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x16 a = mfma_f32(w0, b0[t], f32x16{});
      a = mfma_f32(w1, b1[t], a);
#pragma unroll
      for (int r = 0; r < 16; ++r) h[t][mo][r] = tanh_scaled(a[r]);
    }
  }
  hidden_f32<NT>(fr, F32_L2, lane, bone, h, g);
  hidden_f32<NT>(fr, F32_L3, lane, bone, g, h);
  // layer 4: two chains (features of M tile 0 and 1), summed at the end
  f32x16 c0[NT], c1[NT];
  const float wb = fr[(F32_L4 + 32) * 64 + lane];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    c0[t] = mfma_f32(wb, bone, f32x16{});
    c1[t] = f32x16{};
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float w0 = fr[(F32_L4 + r) * 64 + lane], w1 = fr[(F32_L4 + 16 + r) * 64 + lane];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      c0[t] = mfma_f32(w0, h[t][0][r], c0[t]);
      c1[t] = mfma_f32(w1, h[t][1][r], c1[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 5; ++e) c[t][e] = c0[t][e] + c1[t][e];
}

// Raw outputs o[0..8] of the MLP at input (v0, v1, v2) for this lane's pair.
// Must be called by all 64 lanes with lanes l and l + 32 holding the same
// input.
__device__ __forceinline__ void mlp_tile_f32(const float* __restrict__ fr, float v0, float v1,
                                             float v2, float o[9]) {
  const bool h1 = (threadIdx.x & 63) >= 32;
  const float b0[1] = {h1 ? v1 : v0}, b1[1] = {h1 ? 1.0f : v2};
  float cc[1][5];
  mlp_core_f32<1>(fr, b0, b1, cc);
  const float(&c)[5] = cc[0];
  const float t0 = __shfl_xor(c[0], 32, 64), t1 = __shfl_xor(c[1], 32, 64);
  const float t2 = __shfl_xor(c[2], 32, 64), t3 = __shfl_xor(c[3], 32, 64);
  const float t4 = __shfl_xor(c[4], 32, 64);
  o[0] = h1 ? t0 : c[0]; o[1] = h1 ? t1 : c[1]; o[2] = h1 ? t2 : c[2];
  o[3] = h1 ? t3 : c[3]; o[4] = h1 ? c[0] : t0; o[5] = h1 ? c[1] : t1;
  o[6] = h1 ? c[2] : t2; o[7] = h1 ? c[3] : t3; o[8] = h1 ? t4 : c[4];
}

// Raw outputs for 64 different pairs, one per lane (two tiles: lanes 0-31 and
// lanes 32-63), with half-wave swaps as in mlp_pairs_bf16.
__device__ __forceinline__ void mlp_pairs_f32(const float* __restrict__ fr, float v0, float v1,
                                              float v2, float (&o)[9]) {
  // .lo: (v0 | v1) and (v2 | 1) of lanes 0-31's pairs, .hi: of lanes 32-63's
  const HalfSwap a = half_swap(__float_as_uint(v0), __float_as_uint(v1));
  const HalfSwap b = half_swap(__float_as_uint(v2), __float_as_uint(1.0f));
  const float b0[2] = {__uint_as_float(a.lo), __uint_as_float(a.hi)};
  const float b1[2] = {__uint_as_float(b.lo), __uint_as_float(b.hi)};
  float c[2][5];
  mlp_core_f32<2>(fr, b0, b1, c);
  pair_outputs(c[0], c[1], o);
}

// Entry of this lane's pair from one FP32 tile (all 64 lanes call it; lanes l
// and l + 32 hold the same r).
__device__ __forceinline__ void entry_f32tile(const float* __restrict__ fr, int mode, double dx,
                                              double dy, double dz, float K[9]) {
  const PairIn in = pair_in(mode, (float)dx, (float)dy, (float)dz, false);
  float o[9];
  mlp_tile_f32(fr, in.v0, in.v1, in.v2, o);
  pair_entry(o, in.rs, K);
}

// Stage the FP32 fragment table (global -> LDS) by the whole workgroup.
__device__ __forceinline__ void stage_frags_f32(float* __restrict__ lds,
                                                const float4* __restrict__ g, int nthreads) {
  float4* d = reinterpret_cast<float4*>(lds);
  for (int i = threadIdx.x; i < F32_FRAGS * 16; i += nthreads) d[i] = g[i];
}

// --------------------------------------------- FP32 values on FP16 MFMA, in parts
//
// The FP32 near field (the ACA's samples stay on the FP32 tile: factors, pivots
// and gradients through them have to reproduce). Layers 2-4 contract operands
// written as sums of FP16 numbers on v_mfma_f32_32x32x16_f16 (FP32 accumulation).
// An activation is hi + lo: two roundings to 11 bits with a sign keep 23 to 24 bits.
// A weight has three parts, 33 bits, so no bit of its FP32 value is lost (and so has a
// bias, in spare K slots): its error is common to all pairs and does not average out of
// a sum as an activation's does. The products W1 a_hi + W1 a_lo +
// W2 a_hi + W3 a_hi are exact, and the largest one left out, W2 a_lo, is below 2^-24
// of the product. Nothing may fall under FP16's range: activations are carried
// times 2^10, and every row of weights (its bias with it) times the power of two
// that takes its largest entry to [2^14, 2^15); one multiplication with the row's
// factor gives the FP32 result back. (A weight below 2^-15 of its row's largest is off by
// up to 2^-39 of that; an activation is off by 2^-24 and more, so its product with the
// largest is off by more than this, unless it is zero always: such columns are left out.) The small products are summed before the
// large ones, so a result has 5 roundings at full size (the FP32 tile: 66, one per
// K step). Measured against 64 bits over 654 networks and sizes (both inputs, Glorot
// weights times 0.3, 1 and 3, 2 to 6,000 sources), geometric mean of the ratio to the
// FP32 tile's error: single entries 0.84, sums with random forces 0.86, with gravity
// 0.86, with equal forces 0.86. With weights in two parts the last one was 0.98, and
// 1.04 to 1.12 over 500 and more sources: more than FP32, so the third part is not
// optional. It costs an eighth of the near field (31.3 -> 35.0 ms at 60,000 particles).
//
// Layer 1 (3 -> 64) is the FP32 tile's. The operand layout is the BF16 tile's.
// Cost per 32 pairs: 85 FP16 and 4 FP32 MFMAs (2,980 cycles; the FP32 tile
// 10,800) next to 6,144 activations of 9 issue slots each (3,460 cycles).
#define X2_L1 0                                    // 4 x 64 floats = 4 x 16 fragments
#define X2_SC (X2_L1 + 4 * 16)                     // row factors of layers 2-4: 3 x 64 floats
#define X2_L2 (X2_SC + 3 * 16)                     // [mo 2][s 4][part 3][lane]; bias [mo 2][lane]
#define X2_L3 (X2_L2 + (2 * 4 * 3 + 2) * 64)
#define X2_L4 (X2_L3 + (2 * 4 * 3 + 2) * 64)       // [s 4][part 3][lane]; bias [lane]
#define X2_TOTAL (X2_L4 + (4 * 3 + 1) * 64)
#define X2_ACT 1024.0f                             // activations are carried times this

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma_f16(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// 2^10 tanh of two scaled results -> elements u, u + 1 of the next layer's
// operands. neg1 is -1, kept from the compiler so that the remainder is one
// mixed-precision fma.
__device__ __forceinline__ void act_x2(float y0, float y1, float neg1, int u, f16x8& hi,
                                       f16x8& lo) {
  const float r0 = __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(y0) + 1.0f);
  const float r1 = __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(y1) + 1.0f);
  const f32x2 t = {__builtin_fmaf(-2.0f * X2_ACT, r0, X2_ACT),
                   __builtin_fmaf(-2.0f * X2_ACT, r1, X2_ACT)};
  const f16x2 h = __builtin_convertvector(t, f16x2);
  const f32x2 d = {__builtin_fmaf((float)h[0], neg1, t[0]), __builtin_fmaf((float)h[1], neg1, t[1])};
  const f16x2 l = __builtin_convertvector(d, f16x2);
  hi[u] = h[0];
  hi[u + 1] = h[1];
  lo[u] = l[0];
  lo[u + 1] = l[1];
}

// Product sums of M tile mo of the layer at fr + base (nmo M tiles) for NT tiles.
template <int NT>
__device__ __forceinline__ void layer_x2(const uint4* __restrict__ fr, int base, int mo, int nmo,
                                         int lane, const f16x8 (&Bh)[NT][4],
                                         const f16x8 (&Bl)[NT][4], const f16x8& bone,
                                         f32x16 (&acc)[NT]) {
  auto w = [&](int s, int part) {
    return __builtin_bit_cast(f16x8, fr[base + ((mo * 4 + s) * 3 + part) * 64 + lane]);
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x16{};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const f16x8 wh = w(s, 0), wl = w(s, 1), wt = w(s, 2);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = mfma_f16(wt, Bh[t][s], acc[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = mfma_f16(wl, Bh[t][s], acc[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = mfma_f16(wh, Bl[t][s], acc[t]);
  }
  const f16x8 wb = __builtin_bit_cast(f16x8, fr[base + nmo * 12 * 64 + mo * 64 + lane]);
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = mfma_f16(wb, bone, acc[t]);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const f16x8 wh = w(s, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = mfma_f16(wh, Bh[t][s], acc[t]);
  }
}

// One hidden layer (64 -> 64, then tanh) of NT tiles; sc: its row factors.
template <int NT>
__device__ __forceinline__ void hidden_x2(const uint4* __restrict__ fr, int base,
                                          const float4* __restrict__ sc, int lane, float neg1,
                                          const f16x8& bone, const f16x8 (&Bh)[NT][4],
                                          const f16x8 (&Bl)[NT][4], f16x8 (&Oh)[NT][4],
                                          f16x8 (&Ol)[NT][4]) {
#pragma unroll
  for (int mo = 0; mo < 2; ++mo) {
    f32x16 acc[NT];
    layer_x2<NT>(fr, base, mo, 2, lane, Bh, Bl, bone, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 c = sc[8 * mo + 2 * q + (lane >> 5)];   // rows 32 mo + 8 q + 4 h ..
      const int s = 2 * mo + q / 2, u = 4 * (q % 2);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        act_x2(acc[t][4 * q] * c.x, acc[t][4 * q + 1] * c.y, neg1, u, Oh[t][s], Ol[t][s]);
        act_x2(acc[t][4 * q + 2] * c.z, acc[t][4 * q + 3] * c.w, neg1, u + 2, Oh[t][s], Ol[t][s]);
      }
    }
  }
}

// Raw outputs for 64 different pairs, one per lane (as mlp_pairs_f32).
// fr: the table of X2_TOTAL fragments in LDS.
__device__ __forceinline__ void mlp_pairs_x2(const uint4* __restrict__ fr, float v0, float v1,
                                             float v2, float (&o)[9]) {
  __asm__ volatile("" ::: "memory");   // weights stay in LDS (see mlp_core_bf16)
  const int lane = threadIdx.x & 63;
  float neg1 = -1.0f;
  __asm__("" : "+s"(neg1));
  f16x8 bone;
#pragma unroll
  for (int u = 0; u < 8; ++u) bone[u] = (_Float16)(lane < 32 && u < 3 ? X2_ACT : 0.0f);
  const HalfSwap a = half_swap(__float_as_uint(v0), __float_as_uint(v1));
  const HalfSwap b = half_swap(__float_as_uint(v2), __float_as_uint(1.0f));
  const float b0[2] = {__uint_as_float(a.lo), __uint_as_float(a.hi)};
  const float b1[2] = {__uint_as_float(b.lo), __uint_as_float(b.hi)};
  const float* w1 = reinterpret_cast<const float*>(fr + X2_L1) + lane;
  const float4* sc = reinterpret_cast<const float4*>(fr + X2_SC);
  f16x8 Ah[2][4], Al[2][4], Bh[2][4], Bl[2][4];
#pragma unroll
  for (int mo = 0; mo < 2; ++mo)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16 c = mfma_f32(w1[64 * 2 * mo], b0[t], f32x16{});
      c = mfma_f32(w1[64 * (2 * mo + 1)], b1[t], c);
#pragma unroll
      for (int r = 0; r < 16; r += 2)
        act_x2(c[r], c[r + 1], neg1, r % 8, Ah[t][2 * mo + r / 8], Al[t][2 * mo + r / 8]);
    }
  hidden_x2<2>(fr, X2_L2, sc, lane, neg1, bone, Ah, Al, Bh, Bl);
  hidden_x2<2>(fr, X2_L3, sc + 16, lane, neg1, bone, Bh, Bl, Ah, Al);
  f32x16 acc[2];
  layer_x2<2>(fr, X2_L4, 0, 1, lane, Ah, Al, bone, acc);
  const float4 c = sc[32 + (lane >> 5)];   // rows 4 h ..; row 8 in lanes 0-31
  const float c8 = reinterpret_cast<const float*>(sc)[128 + 8];
  const float o0[5] = {acc[0][0] * c.x, acc[0][1] * c.y, acc[0][2] * c.z, acc[0][3] * c.w,
                       acc[0][4] * c8};
  const float o1[5] = {acc[1][0] * c.x, acc[1][1] * c.y, acc[1][2] * c.z, acc[1][3] * c.w,
                       acc[1][4] * c8};
  pair_outputs(o0, o1, o);
}

// Stage the table (global -> LDS) by the whole workgroup.
__device__ __forceinline__ void stage_frags_x2(uint4* __restrict__ lds,
                                               const uint4* __restrict__ g, int nthreads) {
  for (int i = threadIdx.x; i < X2_TOTAL; i += nthreads) lds[i] = g[i];
}
