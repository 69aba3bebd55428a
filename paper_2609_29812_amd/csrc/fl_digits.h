// Dot products of bf16 vectors as integer sums on the i8 matrix instructions, for the fp64 statistics.
//
// Sixteen vectors are taken as integers X_e = rint(x_e / u), u = 2^(E - 31) a power of two with |X| <= 0x7F7F7F7F (2^E
// the first power of two above max|x|, or the one after where max|x| has a significand of eight ones), and X as four
// balanced base-256 digits: X = sum_s d_s 256^s, d_s in [-128, 127].  A bf16 value has 8 significant
// bits, so X_e is exact unless 0 < |x_e| < 2^(E - 23).  The dot product is the sum over digit pairs (s, t) of
// 256^(s + t) sum_e d_s d'_t, each inner sum exact in int32, and pairs of one weight share an accumulator.  The
// pairs of weight 256 and 1 (a digit 0, which only elements below 2^(E - 15) have, with a digit 1 or 0) are left out.
// What these and the rounded elements can amount to is bounded from the values at hand (DigitStat, digits_serve).
//
// Thirteen 8-bit products at twice the bf16 rate replace the fp64 product at 1/32 of it (2.5 PFLOP/s against
// 78.6 TFLOP/s): about 5 times the rate of the fp64 matrix instructions for the same sums.
#pragma once
#include "fl_attn_util.h"

namespace fl {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// What 16 vectors hold: the largest sum over one vector of the absolute roundings |x_e - u X_e|, the largest 2-norms of a
// vector's digits 0 and 1 (times u), the largest |x_e| (+inf if one is not finite) and the largest 2-norm of a vector.
struct DigitStat {
  float res, low0, low1, top, norm;
  int e;                    // u = 2^e
};

// the larger of each figure (not of the exponents)
__device__ __forceinline__ void join_stat(DigitStat& a, const DigitStat& b) {
  a.res = fmaxf(a.res, b.res);
  a.low0 = fmaxf(a.low0, b.low0);
  a.low1 = fmaxf(a.low1, b.low1);
  a.top = fmaxf(a.top, b.top);
  a.norm = fmaxf(a.norm, b.norm);
}

// Digits of 8 consecutive elements per uint4 of bf16 pairs: out[s][0..1] = digit s of elements 0-3 and 4-7.
__device__ __forceinline__ void digits8(uint4 w, float scale, uint32_t (&out)[4][2], float& res) {
  const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
  uint32_t y[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const float v = bf16_to_f32((t & 1) ? ws[t >> 1] >> 16 : ws[t >> 1] & 0xFFFFu) * scale;   // a power of two
    const float n = rintf(v);
    res += fabsf(v - n);
    // X + 0x80808080 has the bytes d_s + 128, and flipping their high bits gives d_s
    y[t] = ((uint32_t)(int)n + 0x80808080u) ^ 0x80808080u;
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {             // 4 x 4 byte transpose
    const uint32_t lo01 = __builtin_amdgcn_perm(y[4 * q + 1], y[4 * q], 0x05010400u);   // d0 d0 d1 d1
    const uint32_t lo23 = __builtin_amdgcn_perm(y[4 * q + 3], y[4 * q + 2], 0x05010400u);
    const uint32_t hi01 = __builtin_amdgcn_perm(y[4 * q + 1], y[4 * q], 0x07030602u);   // d2 d2 d3 d3
    const uint32_t hi23 = __builtin_amdgcn_perm(y[4 * q + 3], y[4 * q + 2], 0x07030602u);
    out[0][q] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    out[1][q] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
    out[2][q] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    out[3][q] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
  }
}

__device__ __forceinline__ uint32_t max_abs_bits(uint4 w, uint32_t m) {
  const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int t = 0; t < 4; ++t) m = max(m, max(ws[t] & 0x7FFFu, (ws[t] >> 16) & 0x7FFFu));
  return m;
}

// The exponent of u for a largest |bf16| pattern of m, kept where u and 1 / u are normal floats (also for infinities and
// NaN, whose digits are not used).
__device__ __forceinline__ int digit_exponent(uint32_t m) { return max((int)((m + 1) >> 7) - 126, -90) - 31; }
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }

// Digits of 16 vectors as one wave holds them: lane (l16, g) = (lane % 16, lane / 16) holds dims 64 ks + 16 g ..
// + 15 of vector l16 (any split of the dims over g serves, being the same on both sides of a product).
// d[s][ks] is the lane's operand of v_mfma_i32_16x16x64_i8 for digit 3 - s.
template <int D>
struct DigitBlock {
  i32x4 d[4][D / 64];
};

// max over the 16 lanes of a row (rotations within the row, no LDS)
__device__ __forceinline__ float row16_max(float x) {
#define FL_ROR(n) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + (n), 0xf, 0xf, false))
  x = fmaxf(x, FL_ROR(8));
  x = fmaxf(x, FL_ROR(4));
  x = fmaxf(x, FL_ROR(2));
  x = fmaxf(x, FL_ROR(1));
#undef FL_ROR
  return x;
}

// w: the lane's 2 KS loads of 8 elements.  stat: of the 16 vectors, the same in every lane.
template <int D>
__device__ __forceinline__ DigitBlock<D> make_digits(const uint4 (&w)[2 * (D / 64)], DigitStat& stat) {
  constexpr int KS = D / 64;
  DigitBlock<D> o;
  uint32_t m = 0;
#pragma unroll
  for (int x = 0; x < 2 * KS; ++x) m = max_abs_bits(w[x], m);
  m = (uint32_t)row4_max(row16_max((float)m));              // (15 bits: exact as floats)
  const int e = digit_exponent(m);
  const bool finite = m < 0x7F80u;
  const float scale = pow2f(-e);
  float res = 0.0f, n2 = 0.0f;
  int q0 = 0, q1 = 0;                       // squares of the digits 0 and 1
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint32_t q[4][2];
      digits8(w[2 * ks + half], scale, q, res);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        o.d[s][ks][2 * half] = (int)q[3 - s][0];
        o.d[s][ks][2 * half + 1] = (int)q[3 - s][1];
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        q0 = __builtin_amdgcn_sdot4((int)q[0][t], (int)q[0][t], q0, false);
        q1 = __builtin_amdgcn_sdot4((int)q[1][t], (int)q[1][t], q1, false);
      }
      const uint32_t ws[4] = {w[2 * ks + half].x, w[2 * ks + half].y, w[2 * ks + half].z, w[2 * ks + half].w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float a = bf16_to_f32(ws[t] & 0xFFFFu), c = bf16_to_f32(ws[t] >> 16);
        n2 = fmaf(a, a, fmaf(c, c, n2));
      }
    }
  }
  const float unit = pow2f(e);
  res = row16_max(row4_add(res));
  stat.res = res * unit;
  // (square roots to an ulp: digits_serve allows for it; sums of at most 128 squares of digits are exact as floats)
  stat.low0 = __builtin_amdgcn_sqrtf(row16_max(row4_add((float)q0))) * unit;
  stat.low1 = __builtin_amdgcn_sqrtf(row16_max(row4_add((float)q1))) * unit;
  stat.top = finite ? __uint_as_float(m << 16) : INFINITY;
  stat.norm = finite ? __builtin_amdgcn_sqrtf(row16_max(row4_add(n2))) : INFINITY;
  stat.e = e;
  return o;
}

// Whether the digits serve all dot products between the vectors of two sides: with `scale` the factor from dot
// product to natural exponent, what the digits leave out moves an exponent by at most 2^-25, so exp(l - lse) and the
// sums of it by at most 2^-24 of themselves (half an fp32 ulp at most), and no exponent leaves +-330 (its base-2 form
// stays far inside the doubles' range without a running maximum).  False for infinities and NaN.
// The pairs of digits left out are bounded by the norms of those digits, the roundings of one side by their sum times
// the largest element of the other.  For standard normal vectors of 128 dims, 32K of either side, the two come to
// 2^-34 and 2^-30; with one key channel offset by 32 to 2^-30 and 2^-26.5.
__device__ __forceinline__ bool digits_serve(const DigitStat& a, const DigitStat& b, float scale) {
  const float pairs = 256.0f * (a.low0 * b.low1 + a.low1 * b.low0) + a.low0 * b.low0;
  const float off = (a.res * b.top + b.res * (a.top + a.res) + pairs) * scale;
  const float most = a.norm * b.norm * scale;
  return off <= 0x1p-25f * 0.9999f && most <= 330.0f;     // (beyond fp32's range: false)
}

// Integer sums of a 16 x 16 block of dot products (rows 4 g + t of `a`, column l16 of `b`), by weight 256^(n + 2).
struct DigitSums {
  i32x4 s[5];
};

template <int D>
__device__ __forceinline__ void digit_sums(const i32x4 (&a)[4][D / 64], const DigitBlock<D>& b, DigitSums& o) {
  i32x4 s6 = {0, 0, 0, 0}, s5 = s6, s4 = s6, s3 = s6, s2 = s6;
#define FL_DIG(acc, x, y) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[3 - (x)][ks], b.d[3 - (y)][ks], acc, 0, 0, 0)
#pragma unroll
  for (int ks = 0; ks < D / 64; ++ks) {
    FL_DIG(s6, 3, 3);
    FL_DIG(s5, 3, 2);
    FL_DIG(s4, 3, 1);
    FL_DIG(s3, 3, 0);
    FL_DIG(s2, 2, 0);
    FL_DIG(s5, 2, 3);
    FL_DIG(s4, 2, 2);
    FL_DIG(s3, 2, 1);
    FL_DIG(s2, 1, 1);
    FL_DIG(s4, 1, 3);
    FL_DIG(s3, 1, 2);
    FL_DIG(s2, 0, 2);
    FL_DIG(s3, 0, 3);
  }
#undef FL_DIG
  o.s[0] = s2; o.s[1] = s3; o.s[2] = s4; o.s[3] = s5; o.s[4] = s6;
}

// The lane's dot product t in units of 2^16 u u'.  |s6| <= 2^21, |s4| < 2^22.6 and |s3| <= 2^23 for 128 dims, so each
// shifted pair fits int32; the doubles hold the sum exactly below 2^53 (beyond only for vectors whose elements are nearly
// all at the bound, then rounded once).
__device__ __forceinline__ double digit_dot(const DigitSums& o, int t) {
  const double p = fma((double)(o.s[4][t] * 256 + o.s[3][t]), 65536.0, (double)(o.s[2][t] * 256 + o.s[1][t]));
  return fma(p, 256.0, (double)o.s[0][t]);
}

constexpr int kDigStage = 4;              // 16-vector blocks staged in LDS per step

// The STG staged blocks (dig: as 16-byte pieces by block, digit 3 .. 0, 64 dims and lane) against a wave's own ones
// FIRST .. FIRST + NB - 1: add(sums, staged block, own block) for each pair.  The products of a pair are issued between the vector
// instructions of the add before: a product's matrix cycles cover four of them.
template <int D, int NB, int STG = kDigStage, int FIRST = 0, int OWN, typename Add>
__device__ __forceinline__ void digit_stage(const uint4* dig, const DigitBlock<D> (&own)[OWN], Add add) {
  static_assert(FIRST + NB <= OWN, "own blocks FIRST .. FIRST + NB - 1");
  constexpr int KS = D / 64;
  const i32x4* src = reinterpret_cast<const i32x4*>(dig) + (threadIdx.x & 63);
  i32x4 d[4][KS];
  DigitSums o[2];
#pragma unroll
  for (int i = -1; i < STG * NB; ++i) {
    if (i + 1 < STG * NB) {
      if ((i + 1) % NB == 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) d[s][ks] = src[((i + 1) / NB * 4 * KS + s * KS + ks) * 64];
      }
      digit_sums<D>(d, own[FIRST + (i + 1) % NB], o[(i + 1) & 1]);
    }
    if (i < 0) continue;
    add(o[i & 1], i / NB, FIRST + i % NB);
#pragma unroll
    for (int y = 0; y < 13 * KS; ++y) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, KS == 2 ? 4 : 7, 0);
    }
  }
}

// 2^x for |x| <= 1000: 2^rint(x) times a degree-10 polynomial of the rest (the Chebyshev interpolant of 2^r on
// [-1/2, 1/2]; relative error below 4e-16 before rounding).
__device__ __forceinline__ double exp2_f64(double x) {
  const double big = 0x1.8p52;
  const double y = x + big;                    // the low word of y is the nearest integer to x
  const double r = x - (y - big);
  double p = 0x1.e606343d16a96p-28;
  p = fma(p, r, 0x1.b675bc52c98b0p-24);
  p = fma(p, r, 0x1.62bfd47ecba29p-20);
  p = fma(p, r, 0x1.ffcb540682f51p-17);
  p = fma(p, r, 0x1.430913096c64ap-13);
  p = fma(p, r, 0x1.5d87fe9d7a3b5p-10);
  p = fma(p, r, 0x1.3b2ab6fba1defp-7);
  p = fma(p, r, 0x1.c6b08d703ce4ap-5);
  p = fma(p, r, 0x1.ebfbdff82c598p-3);
  p = fma(p, r, 0x1.62e42fefa3a19p-1);
  p = fma(p, r, 1.0);
  return __builtin_ldexp(p, (int)(uint32_t)__double_as_longlong(y));
}

}  // namespace fl
