// Which channels a wavefront's calls can need: one matrix product per round of
// calls bounds every channel's Gaussian exponent from below, and a channel
// whose terms cannot change f or g on any lane is left out of the channel
// loop.
//
// Brass, Kilian, Reuter, arXiv:1811.09711, Sec. 3.5, eq. g(p): g sums a term
// per channel.  The exponent of channel c's Gaussian axes is a quadratic form
//   S_c(p) = sum_k (ga_k p_k + gb_k)^2 = sum_k A_k q_k^2 + B_k q_k + C,
// q_k = p_k - 1/2, so the exponents of 64 calls and 32 channels are a
// 64 x (2d+1) by (2d+1) x 32 product: a few v_mfma_f32_32x32x16_f16 per round
// in place of two to three vector instructions per channel and axis.  The
// product only decides what is left out: its inputs are rounded to FP16, the
// rounding is bounded per channel (k_setup_mask) and added to the threshold,
// and every channel that the bound does not rule out is evaluated as ever, so
// f, g and w are the same bit for bit.
//
// Feature order of a kernel for MAXD axes (MaskForm): where the general form
// fits 16 features, q_0 .. q_{A-1}, e, their squares (A = MAXD up to 6; 7 in
// the 8-axis kernel of problems with fewer axes); else q_0 .. q_{MAXD-1},
// sum_k q_k^2, e, in which only channels that are Gaussian on every axis can
// be bounded (with their smallest ga for every axis).  e: the call's exponent
// (below).  Sixteen features are one product step and keep 8 registers; the
// general form for 10 axes needs two and spilled the pass's registers.
// Coefficients are scaled by 2^-s per channel so that the largest lies in
// FP16's normal range.
#pragma once

#include "mcv_point.h"

namespace mcv {

typedef _Float16 Half8 __attribute__((ext_vector_type(8)));
typedef float Acc16 __attribute__((ext_vector_type(16)));
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));

// The form for a problem of d axes: axes of its general form (0: the other
// form), index of e, product steps (0: no masks).
struct MaskForm {
  int axes, q2, e, steps;
};
constexpr MaskForm mask_form(int maxd, bool exact) {
  return maxd <= 6 ? MaskForm{maxd, maxd + 1, maxd, 1}
         : maxd == 8 && !exact ? MaskForm{7, 8, 7, 1}
         : maxd <= 16 ? MaskForm{0, maxd, maxd + 1, (maxd + 2 + 15) / 16} : MaskForm{0, 0, 0, 0};
}
inline MaskForm mask_form_of(int d) {
  const int m = d <= 2 ? 2 : d <= 4 ? 4 : d <= 6 ? 6 : d <= 8 ? 8 : d <= 10 ? 10 : d <= 12 ? 12
                                                                           : d <= 16 ? 16 : 32;
  return mask_form(m, d == m);
}

// The features of one call at p.  In the second form an axis beyond d, where p
// is 0, must add nothing: its q = -1/2 would enter the sum of squares, which
// bounds the exponent from below over the d axes alone.  In the first form its
// coefficients are 0.
template <int MAXD, bool EXACT, typename T, int N>
__device__ __forceinline__ void mask_features(const T (&p)[MAXD], int d, float ee, float (&x)[N]) {
  constexpr MaskForm F = mask_form(MAXD, EXACT);
  static_assert(N == 16 * F.steps, "whole product steps");
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] = 0.0f;
  x[F.e] = ee;
#pragma unroll
  for (int k = 0; k < MAXD; ++k) {
    float q = (float)p[k] - 0.5f;
    if constexpr (F.axes > 0) {
      if (k < F.axes) {
        x[k] = q;
        x[F.q2 + k] = q * q;
      }
    } else {
      if (!EXACT && k >= d) q = 0.0f;
      x[k] = q;
      x[F.q2] = fmaf(q, q, x[F.q2]);
    }
  }
}

// Bit j: channel 32 tile + j may change f or g on some lane of the wavefront.
// Every lane takes part (the product ignores the execution mask).  ee: the
// call's e = min(floor log2 f, floor log2 g), from which both sums only grow
// (fpos: no negative peak), or the least exponent; the channel's terms stay
// below half an ulp of both sums where S_c + e reaches its threshold.
//
// Operand layout of the 32x32x16 product: lane l holds features 8 (l / 32) ..
// + 7 of row l mod 32 (first operand: calls) or column l mod 32 (second:
// channels); a swap of the halves of two registers turns "all 16 features of
// call l" into the operands of calls 0..31 and 32..63.  Results: lane l holds
// column l mod 32, so a lane's minimum over its registers is its channel's
// minimum over half the calls, and the ballot's two halves join them.
template <int MAXD, bool EXACT, typename T>
__device__ __forceinline__ uint32_t channel_mask(const T (&p)[MAXD], int d, float ee,
                                                 const void* coef, const float* thr, int tile) {
  constexpr int MS = mask_form(MAXD, EXACT).steps;
  float x[16 * MS];
  mask_features<MAXD, EXACT>(p, d, ee, x);
  const int lane = (int)__lane_id();
  // an opaque offset, so that the loads stay in the loop over the calls
  // (cached) instead of occupying registers across it
  uint32_t off = (uint32_t)((tile * MS * 64 + lane) * 16);
  asm("" : "+v"(off));
  Half8 B[MS];
#pragma unroll
  for (int s = 0; s < MS; ++s) B[s] = *(GP<Half8>)((GP<char>)coef + (off + (uint32_t)(s * 1024)));
  const float t = *(GP<float>)((GP<char>)thr + (uint32_t)((tile * 32 + (lane & 31)) * 4));
  Half8 lo[MS], hi[MS];
#pragma unroll
  for (int s = 0; s < MS; ++s) {
    U32x4 l, h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto a = __builtin_amdgcn_cvt_pkrtz(x[16 * s + 2 * i], x[16 * s + 2 * i + 1]);
      const auto b = __builtin_amdgcn_cvt_pkrtz(x[16 * s + 8 + 2 * i], x[16 * s + 9 + 2 * i]);
      const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a),
                                                      __builtin_bit_cast(uint32_t, b), false, false);
      l[i] = r[0];
      h[i] = r[1];
    }
    lo[s] = __builtin_bit_cast(Half8, l);
    hi[s] = __builtin_bit_cast(Half8, h);
  }
  // one half of the calls after the other: 16 accumulator registers at a time
  Acc16 acc = {};
#pragma unroll
  for (int s = 0; s < MS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(lo[s], B[s], acc, 0, 0, 0);
  float m = acc[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) m = __builtin_fminf(m, acc[i]);
  __builtin_amdgcn_sched_barrier(0);
  acc = Acc16{};
#pragma unroll
  for (int s = 0; s < MS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(hi[s], B[s], acc, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < 16; ++i) m = __builtin_fminf(m, acc[i]);
  const uint64_t b = __ballot(!(m >= t));
  return (uint32_t)b | (uint32_t)(b >> 32);
}

}  // namespace mcv
