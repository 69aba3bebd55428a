// Cross-loop K/V residual codec: Section 4.3, Eq. 4; Appendix D.3, Eq. 8; quantizer of Appendix E.
//
// All kernels stream rows with 16-byte loads: one thread owns 8 consecutive channels of a row, so codes
// of those channels form one 2/4/8-byte word (LSB-first packing) and metadata loads are 2 or 16 bytes.
//   quant_token   (keys, per-channel groups of G packed rows): a 256-thread workgroup owns one group of
//                 rows x 64 channels (256 at G = 8, 128 at G = 16); its row slices (G of them, at most 32)
//                 reduce min/max in registers and LDS, then the same threads encode their rows from registers
//                 (no second pass over HBM).
//   quant_channel (values, per-token groups of G channels): the G/8 lanes of a group reduce min/max by DPP.
//   dequant       rebuilds bf16(x_hat + z + q*s) rows, compact or in place.
// Both quantizers optionally write the reconstructed rows (fusing the compact dequantization).
//
// The quantizers are bound by vector instructions as much as by HBM (a 32K base of 16 heads x 128 in 4 bits moves
// 620 MB, 118 us at the rate of a large copy): 42 vector instructions a value, a third of them
// for the group's metadata in fp64 and a 64-bit division for the row, took 150 us; 31 a value, the count now, take 132.
#include "fl_attn_util.h"

namespace fl {

struct Row8 {
  float v[8];
};

// NT: marked non-temporal, for the new state, which is read once (a 32K base 134 -> 130 us)
template <bool NT = false>
__device__ __forceinline__ Row8 load_bf16x8(const uint16_t* p) {
  u32x4 w0;
  if constexpr (NT) w0 = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  else w0 = *reinterpret_cast<const u32x4*>(p);
  const uint4 w = make_uint4(w0[0], w0[1], w0[2], w0[3]);
  const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
  Row8 r;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    r.v[2 * t] = __uint_as_float(ws[t] << 16);
    r.v[2 * t + 1] = __uint_as_float(ws[t] & 0xFFFF0000u);
  }
  return r;
}

// Eight values rounded to bf16 (to nearest even, v_cvt_pk_bf16_f32), packed.
__device__ __forceinline__ uint4 to_bf16x8(const Row8& r) {
  return make_uint4(pack_bf16x2(r.v[0], r.v[1]), pack_bf16x2(r.v[2], r.v[3]), pack_bf16x2(r.v[4], r.v[5]),
                    pack_bf16x2(r.v[6], r.v[7]));
}

// Eight bf16 values (as packed bits) to fp16.
__device__ __forceinline__ uint4 bf16x8_to_f16(uint4 w) {
  const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
  uint32_t o[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) o[t] = pack_f16x2(__uint_as_float(ws[t] << 16), __uint_as_float(ws[t] & 0xFFFF0000u));
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// Reciprocal of a metadata scale for encode1 (within 1 ulp; s is an fp16 value, so 1/s is a normal fp32), 0 for s = 0.
__device__ __forceinline__ float scale_rcp(float s) { return s == 0.0f ? 0.0f : __builtin_amdgcn_rcpf(s); }

// Encode one value: q = clamp(rint(fp32(fp32(delta - z) / s)), 0, qmax), 0 when s == 0, with rs = scale_rcp(s).
// No division: q1 = a rs, e = a - q1 s (one fma, exact), q2 = e rs + q1 (one fma) is Markstein's correction
// step (P. Markstein, IBM J. Res. Dev. 34(1), 1990), within |a/s| 2^-45 of a/s.  The scale s is an fp16
// value (at most 11 significant bits) and a an fp32 value, so a - (m + 1/2) s is a multiple of a power of
// two that keeps a/s either exactly at a half-integer m + 1/2 or more than half an ulp away from it (by
// 2^-11 of that half ulp at least): rint(q2) is rint of the correctly rounded quotient, the IEEE division's
// code, bit for bit (checked in exact arithmetic on the host, ties and fp32 neighbours of every boundary).
// Returned as a float.
__device__ __forceinline__ float encode1(float delta, float z, float s, float rs, int qmax) {
  const float a = delta - z;
  const float q1 = a * rs;
  const float e = __builtin_fmaf(-q1, s, a);
  // (a median with 0 and qmax: the clamp in one step, 0 for NaN)
  return __builtin_amdgcn_fmed3f(__builtin_rintf(__builtin_fmaf(e, rs, q1)), 0.0f, (float)qmax);
}

template <int BITS>
__device__ __forceinline__ void store_codes8(uint8_t* dst, const uint32_t q[8]) {
  if constexpr (BITS == 8) {
    uint32_t lo = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
    uint32_t hi = q[4] | (q[5] << 8) | (q[6] << 16) | (q[7] << 24);
    *reinterpret_cast<uint2*>(dst) = make_uint2(lo, hi);
  } else {
    uint32_t w = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) w |= q[t] << (t * BITS);
    if constexpr (BITS == 4) *reinterpret_cast<uint32_t*>(dst) = w;
    else *reinterpret_cast<uint16_t*>(dst) = (uint16_t)w;
  }
}

template <int BITS>
__device__ __forceinline__ void load_codes8(const uint8_t* src, uint32_t q[8]) {
  constexpr uint32_t mask = (1u << BITS) - 1u;
  if constexpr (BITS == 8) {
    uint2 w = *reinterpret_cast<const uint2*>(src);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      q[t] = (w.x >> (8 * t)) & mask;
      q[t + 4] = (w.y >> (8 * t)) & mask;
    }
  } else {
    uint32_t w = (BITS == 4) ? *reinterpret_cast<const uint32_t*>(src)
                             : (uint32_t)*reinterpret_cast<const uint16_t*>(src);
#pragma unroll
    for (int t = 0; t < 8; ++t) q[t] = (w >> (t * BITS)) & mask;
  }
}

// Group metadata from fp32 min/max: z = the largest fp16 <= min, s = the smallest fp16 >= fp64((max - z) / qmax), both
// saturating at +-65504, zeros as +0.
//
// Without fp64: z is the fp16 towards zero, a step further down if that is above min.  With d = max - z exact in fp32
// and not negative, s is the smallest fp16 with s qmax >= d (s qmax has at most 19 significant bits, exact in fp32, and
// d 24, so d / qmax is s itself or further than an fp64 rounding from it): the fp16 towards zero of d / qmax by the
// reciprocal (off by less than a step), moved up while s qmax < d.  Otherwise the fp64 form (a rare branch).
struct GroupMeta {
  float z, s;
  uint32_t zb, sb;      // their fp16 bits
};

__device__ __forceinline__ uint32_t f16_towards_zero(float x) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x, 0.0f)) & 0xFFFFu;
}

template <int QMAX>
__device__ __forceinline__ GroupMeta group_meta(float mn, float mx) {
  GroupMeta m;
  const float x = __builtin_amdgcn_fmed3f(mn, -65504.0f, 65504.0f);
  m.zb = f16_towards_zero(x);
  m.zb += f16_bits_to_f32(m.zb) > x ? 1u : 0u;             // (only below zero: a step away from it)
  if (m.zb == 0x8000u) m.zb = 0u;
  m.z = f16_bits_to_f32(m.zb);
  const float d = mx - m.z;
  const float bb = d - mx;                                 // TwoSum: the rounding error of d
  const float err = (mx - (d - bb)) + (-m.z - bb);
  constexpr float q = (float)QMAX, rq = 1.0f / q;
  m.sb = f16_towards_zero(fminf(d * rq, 65504.0f)) & 0x7FFFu;   // (a group of -0 has d = -0)
  m.sb += f16_bits_to_f32(m.sb) * q < d ? 1u : 0u;
  m.sb += f16_bits_to_f32(m.sb) * q < d ? 1u : 0u;
  m.sb = min(m.sb, 0x7BFFu);
  if (!(err == 0.0f && d >= 0.0f)) {
    const double zd = f16_down_value((double)mn);
    const double sd = f16_up_value(((double)mx - zd) / (double)QMAX);
    m.zb = f16_bits_of_exact(zd);
    m.sb = f16_bits_of_exact(sd);
    m.z = (float)zd;
  }
  m.s = f16_bits_to_f32(m.sb);
  return m;
}

// min / max with a lane of the same 16-lane row (DPP, no LDS).  As medians with an infinity: a plain fminf adds a
// NaN-quieting step per operand, and no NaN gets here (the running min and max start at the infinities and drop them).
#define FL_DPP_F(x, ctrl) \
  __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), (ctrl), 0xf, 0xf, false))
#define FL_DPP_MINMAX(mn, mx, ctrl, inf)                            \
  do {                                                              \
    mn = __builtin_amdgcn_fmed3f(mn, FL_DPP_F(mn, ctrl), -(inf));   \
    mx = __builtin_amdgcn_fmed3f(mx, FL_DPP_F(mx, ctrl), (inf));    \
  } while (0)
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror8 = 0x141, kMirror16 = 0x140, kXor8 = 0x128;   // (xor 8: rotate by 8)

// ---- keys: per-channel groups along packed rows ----------------------------------------------------
// A workgroup of 256 threads = S row slices x CH chunks of 8 channels; each slice holds RPS = G/S rows.
// S = min(G, 32), so a group of 64 rows spreads over 32 slices and a workgroup covers 64 channels.

// out_rows: compact [B, k, HD] rows, or (commit) the cache rows idx of x_ref itself, written in place
// (every element is read before the same thread writes it, after the workgroup's reduction).
// Body of one workgroup: channel block bx, row group g, batch b.
template <int BITS, int S, int RPS>
__device__ __forceinline__ void quant_token_body(
    const uint16_t* __restrict__ x_cur, const uint16_t* x_ref,
    const int32_t* __restrict__ idx, int k, int N, int HD, int G, uint8_t* __restrict__ codes,
    uint16_t* __restrict__ scale, uint16_t* __restrict__ zero, uint16_t* out_rows, bool commit,
    int bx, int g, int b, float pinf) {
  constexpr int CH = 256 / S;          // chunks of 8 channels per workgroup
  // CH = 8: lanes l and l ^ 8 of a wave hold two slices of the same channels, joined in registers first
  constexpr int JOIN = CH == 8 ? 2 : 1, P = S / JOIN;
  constexpr int PARTS = CH == 8 ? 4 : 1;   // threads that reduce one channel
  __shared__ float s_mn[P][CH * 8 + 16 * (PARTS > 1)];
  __shared__ float s_mx[P][CH * 8 + 16 * (PARTS > 1)];
  __shared__ float s_z[CH * 8];
  __shared__ float s_s[CH * 8];
  __shared__ float s_r[CH * 8];
  constexpr int qmax = (1 << BITS) - 1;
  const int slice = threadIdx.x / CH, chunk = threadIdx.x % CH;
  const int c0 = bx * (CH * 8) + chunk * 8;
  const bool ch_ok = c0 < HD;
  const int ng = (k + G - 1) / G;

  float dl[RPS][8];
  uint4 ref_raw[RPS];
  int64_t roff[RPS];                   // element offset of each row in x_ref
  float mn[8], mx[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) { mn[t] = INFINITY; mx[t] = -INFINITY; }
  // (past the group's last row that row again, past the last channel the last ones: neither moves a minimum or
  // maximum that is used, and nothing branches)
  const int cl = min(c0, HD - 8);
#pragma unroll
  for (int j = 0; j < RPS; ++j) {
    const int p = min(g * G + slice * RPS + j, k - 1);
    const int64_t i = idx ? (int64_t)idx[(int64_t)b * k + p] : (int64_t)p;
    const int64_t off = ((int64_t)b * N + i) * HD + cl;
    roff[j] = off;
    const Row8 c = load_bf16x8<true>(x_cur + off);
    Row8 r{};
    ref_raw[j] = make_uint4(0, 0, 0, 0);
    if (x_ref) {
      ref_raw[j] = *reinterpret_cast<const uint4*>(x_ref + off);
      r = load_bf16x8(x_ref + off);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) dl[j][t] = c.v[t] - r.v[t];
  }
#pragma unroll
  for (int j = 0; j < RPS; ++j)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      mn[t] = fminf(mn[t], dl[j][t]);
      mx[t] = fmaxf(mx[t], dl[j][t]);
    }
  if constexpr (JOIN == 2) {
#pragma unroll
    for (int t = 0; t < 8; ++t) FL_DPP_MINMAX(mn[t], mx[t], kXor8, pinf);
  }
  if (JOIN == 1 || (slice & 1) == 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      s_mn[slice / JOIN][chunk * 8 + t] = mn[t];
      s_mx[slice / JOIN][chunk * 8 + t] = mx[t];
    }
  }
  __syncthreads();
  if (threadIdx.x < CH * 8 * PARTS) {
    const int ch = threadIdx.x / PARTS, part = threadIdx.x % PARTS;   // PARTS adjacent threads per channel
    const int c = bx * (CH * 8) + ch;
    float a = INFINITY, bb = -INFINITY;
#pragma unroll
    for (int sl = 0; sl < P / PARTS; ++sl) {
      a = fminf(a, s_mn[sl * PARTS + part][ch]);
      bb = fmaxf(bb, s_mx[sl * PARTS + part][ch]);
    }
    if constexpr (PARTS == 4) {
      FL_DPP_MINMAX(a, bb, kXor1, pinf);
      FL_DPP_MINMAX(a, bb, kXor2, pinf);
    }
    GroupMeta gm = {};
    if (c < HD) gm = group_meta<qmax>(a, bb);
    if (c < HD && part == 0) {
      const int64_t m = ((int64_t)b * ng + g) * HD + c;
      zero[m] = (uint16_t)gm.zb;
      scale[m] = (uint16_t)gm.sb;
    }
    if (part == 0) {
      s_z[ch] = gm.z;
      s_s[ch] = gm.s;
      s_r[ch] = scale_rcp(gm.s);
    }
  }
  __syncthreads();
  if (!ch_ok) return;
  float z8[8], s8[8], r8[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    z8[t] = s_z[chunk * 8 + t];
    s8[t] = s_s[chunk * 8 + t];
    r8[t] = s_r[chunk * 8 + t];
  }
  const int row_bytes = HD * BITS / 8;
#pragma unroll
  for (int j = 0; j < RPS; ++j) {
    const int p = g * G + slice * RPS + j;
    if (p >= k) break;
    float f[8];
    uint32_t q[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      f[t] = encode1(dl[j][t], z8[t], s8[t], r8[t], qmax);
      q[t] = (uint32_t)f[t];
    }
    store_codes8<BITS>(codes + ((int64_t)b * k + p) * row_bytes + c0 * BITS / 8, q);
    if (out_rows) {
      const uint32_t rw[4] = {ref_raw[j].x, ref_raw[j].y, ref_raw[j].z, ref_raw[j].w};
      Row8 o;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float ref = (t & 1) ? __uint_as_float(rw[t >> 1] & 0xFFFF0000u) : __uint_as_float(rw[t >> 1] << 16);
        o.v[t] = ref + __builtin_fmaf(f[t], s8[t], z8[t]);     // q * s is exact in fp32: one rounding
      }
      *reinterpret_cast<uint4*>(out_rows + (commit ? roff[j] : ((int64_t)b * k + p) * HD + c0)) = to_bf16x8(o);
    }
  }
}

template <int BITS, int S, int RPS>
__global__ __launch_bounds__(256) void quant_token_kernel(
    const uint16_t* __restrict__ x_cur, const uint16_t* x_ref,
    const int32_t* __restrict__ idx, int k, int N, int HD, int G, uint8_t* __restrict__ codes,
    uint16_t* __restrict__ scale, uint16_t* __restrict__ zero, uint16_t* out_rows, bool commit, float pinf) {
  quant_token_body<BITS, S, RPS>(x_cur, x_ref, idx, k, N, HD, G, codes, scale, zero, out_rows, commit,
                                 blockIdx.x, blockIdx.y, blockIdx.z, pinf);
}

// ---- values: per-token groups of G channels ----------------------------------------------------------
// out_rows as for quant_token_kernel (each element is read and written by one thread).
// Body of one thread: 8-channel chunk `local` of the k * HD / 8 chunks of batch b.
template <int BITS>
__device__ __forceinline__ void quant_channel_body(
    const uint16_t* __restrict__ x_cur, const uint16_t* x_ref,
    const int32_t* __restrict__ idx, int k, int N, int HD, int G, uint8_t* __restrict__ codes,
    uint16_t* __restrict__ scale, uint16_t* __restrict__ zero, uint16_t* out_rows, bool commit,
    int64_t local, int b, float pinf, uint16_t* out_f16 = nullptr) {
  constexpr int qmax = (1 << BITS) - 1;
  const int chunks = HD / 8;
  const bool ok = local < (int64_t)k * chunks;         // (k HD < 2^31: 32-bit quotients)
  const int p = ok ? (int)((uint32_t)local / (uint32_t)chunks) : 0;
  const int chunk = ok ? (int)local - p * chunks : 0;
  const int c0 = chunk * 8;
  float dl[8];
  uint4 ref_raw = make_uint4(0, 0, 0, 0);
  float mn = INFINITY, mx = -INFINITY;
  int64_t roff = 0;
  if (ok) {
    const int64_t i = idx ? (int64_t)idx[(int64_t)b * k + p] : (int64_t)p;
    const int64_t off = ((int64_t)b * N + i) * HD + c0;
    roff = off;
    Row8 c = load_bf16x8<true>(x_cur + off);
    Row8 r{};
    if (x_ref) {
      ref_raw = *reinterpret_cast<const uint4*>(x_ref + off);
      r = load_bf16x8(x_ref + off);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      dl[t] = c.v[t] - r.v[t];
      mn = fminf(mn, dl[t]);
      mx = fmaxf(mx, dl[t]);
    }
  }
  // reduce across the G/8 consecutive lanes of the group (groups never straddle a wave)
  if (G > 8) FL_DPP_MINMAX(mn, mx, kXor1, pinf);
  if (G > 16) FL_DPP_MINMAX(mn, mx, kXor2, pinf);
  if (G > 32) FL_DPP_MINMAX(mn, mx, kMirror8, pinf);         // (quads are uniform by now)
  if (G > 64) FL_DPP_MINMAX(mn, mx, kMirror16, pinf);
  if (!ok) return;
  const GroupMeta gm = group_meta<qmax>(mn, mx);
  const int lg = __builtin_ctz(G);                       // (G is a power of two)
  if ((c0 & (G - 1)) == 0) {
    const int64_t m = ((int64_t)b * k + p) * (HD >> lg) + (c0 >> lg);
    zero[m] = (uint16_t)gm.zb;
    scale[m] = (uint16_t)gm.sb;
  }
  const float z32 = gm.z, s32 = gm.s, r32 = scale_rcp(s32);
  float f[8];
  uint32_t q[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    f[t] = encode1(dl[t], z32, s32, r32, qmax);
    q[t] = (uint32_t)f[t];
  }
  store_codes8<BITS>(codes + ((int64_t)b * k + p) * (HD * BITS / 8) + c0 * BITS / 8, q);
  if (out_rows) {
    const uint32_t rw[4] = {ref_raw.x, ref_raw.y, ref_raw.z, ref_raw.w};
    Row8 o;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float ref = (t & 1) ? __uint_as_float(rw[t >> 1] & 0xFFFF0000u) : __uint_as_float(rw[t >> 1] << 16);
      o.v[t] = ref + __builtin_fmaf(f[t], s32, z32);
    }
    const uint4 w = to_bf16x8(o);
    *reinterpret_cast<uint4*>(out_rows + (commit ? roff : ((int64_t)b * k + p) * HD + c0)) = w;
    if (out_f16) *reinterpret_cast<uint4*>(out_f16 + roff) = bf16x8_to_f16(w);   // (commit only: the cache row's copy)
  }
}

template <int BITS>
__global__ __launch_bounds__(256) void quant_channel_kernel(
    const uint16_t* __restrict__ x_cur, const uint16_t* x_ref,
    const int32_t* __restrict__ idx, int k, int N, int HD, int G, uint8_t* __restrict__ codes,
    uint16_t* __restrict__ scale, uint16_t* __restrict__ zero, uint16_t* out_rows, bool commit, float pinf) {
  quant_channel_body<BITS>(x_cur, x_ref, idx, k, N, HD, G, codes, scale, zero, out_rows, commit,
                           (int64_t)blockIdx.x * blockDim.x + threadIdx.x, blockIdx.y, pinf);
}

// ---- keys and values in one launch -------------------------------------------------------------------
// The first kx * ky * B workgroups run the key body (token axis), the rest the value body (channel
// axis), so the two short streams share one launch instead of two dependent ones.
struct QuantKV {
  const uint16_t* k_cur;
  const uint16_t* k_ref;
  const uint16_t* v_cur;
  const uint16_t* v_ref;
  const int32_t* idx;
  uint8_t* k_codes;
  uint16_t* k_scale;
  uint16_t* k_zero;
  uint8_t* v_codes;
  uint16_t* v_scale;
  uint16_t* v_zero;
  uint16_t* k_rows;
  uint16_t* v_rows;
  uint16_t* v_f16;     // optional (commit): fp16 copy of the value cache, rows idx rewritten
  int k, N, HD, G;
  int kx, ky, vx;      // key workgroups per (row group, batch) and row groups; value workgroups per batch
  int commit;
  float pinf;          // +inf (an argument, so that medians with it stay medians)
};

template <int BITS, int S, int RPS>
__global__ __launch_bounds__(256) void quant_kv_kernel(QuantKV a) {
  const int nkb = a.kx * a.ky;
  const int blk = blockIdx.x;
  const int b = blk / (nkb + a.vx);
  const int r = blk - b * (nkb + a.vx);
  if (r < nkb) {
    quant_token_body<BITS, S, RPS>(a.k_cur, a.k_ref, a.idx, a.k, a.N, a.HD, a.G, a.k_codes, a.k_scale,
                                   a.k_zero, a.k_rows, a.commit != 0, r % a.kx, r / a.kx, b, a.pinf);
  } else {
    quant_channel_body<BITS>(a.v_cur, a.v_ref, a.idx, a.k, a.N, a.HD, a.G, a.v_codes, a.v_scale, a.v_zero,
                             a.v_rows, a.commit != 0, (int64_t)(r - nkb) * 256 + threadIdx.x, b, a.pinf, a.v_f16);
  }
}

// ---- bits = 16: the payload is the raw state ---------------------------------------------------------
__global__ __launch_bounds__(256) void passthrough_kernel(const uint16_t* __restrict__ x_cur,
                                                          const int32_t* __restrict__ idx, int k,
                                                          int N, int HD, uint8_t* __restrict__ codes,
                                                          uint16_t* __restrict__ out_rows, bool commit) {
  const int chunks = HD / 8;
  const int64_t local = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (local >= (int64_t)k * chunks) return;
  const int p = (int)((uint32_t)local / (uint32_t)chunks), c0 = ((int)local - p * chunks) * 8;
  const int64_t i = idx ? (int64_t)idx[(int64_t)b * k + p] : (int64_t)p;
  uint4 w = *reinterpret_cast<const uint4*>(x_cur + ((int64_t)b * N + i) * HD + c0);
  *reinterpret_cast<uint4*>(codes + (((int64_t)b * k + p) * HD + c0) * 2) = w;
  if (out_rows)
    *reinterpret_cast<uint4*>(out_rows + (commit ? ((int64_t)b * N + i) * HD : ((int64_t)b * k + p) * HD) + c0) = w;
}

// ---- dequantization / reconstruction ------------------------------------------------------------------
// One thread: 8-channel chunk `local` of the k * HD / 8 chunks of batch b.
template <int BITS, int AXIS>
__device__ __forceinline__ void dequant_body(
    const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scale,
    const uint16_t* __restrict__ zero, const int32_t* __restrict__ idx, int k, int N, int HD, int G,
    uint16_t* x_hat, uint16_t* out_rows, int64_t local, int b) {
  const int chunks = HD / 8;
  if (local >= (int64_t)k * chunks) return;
  const int p = (int)((uint32_t)local / (uint32_t)chunks), c0 = ((int)local - p * chunks) * 8;
  const int64_t i = idx ? (int64_t)idx[(int64_t)b * k + p] : (int64_t)p;
  const int64_t xoff = ((int64_t)b * N + i) * HD + c0;
  uint16_t* dst = out_rows ? out_rows + ((int64_t)b * k + p) * HD + c0 : x_hat + xoff;
  if constexpr (BITS == 16) {
    *reinterpret_cast<uint4*>(dst) =
        *reinterpret_cast<const uint4*>(codes + (((int64_t)b * k + p) * HD + c0) * 2);
  } else {
    uint32_t q[8];
    load_codes8<BITS>(codes + ((int64_t)b * k + p) * (HD * BITS / 8) + c0 * BITS / 8, q);
    float z8[8], s8[8];
    if constexpr (AXIS == FL_AXIS_TOKEN) {
      const int ng = (k + G - 1) / G;
      const int64_t m = ((int64_t)b * ng + p / G) * HD + c0;
      uint4 zw = *reinterpret_cast<const uint4*>(zero + m);
      uint4 sw = *reinterpret_cast<const uint4*>(scale + m);
      const uint32_t za[4] = {zw.x, zw.y, zw.z, zw.w}, sa[4] = {sw.x, sw.y, sw.z, sw.w};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        z8[t] = f16_bits_to_f32((t & 1) ? (za[t >> 1] >> 16) : (za[t >> 1] & 0xFFFFu));
        s8[t] = f16_bits_to_f32((t & 1) ? (sa[t >> 1] >> 16) : (sa[t >> 1] & 0xFFFFu));
      }
    } else {
      const int64_t m = ((int64_t)b * k + p) * (HD / G) + c0 / G;
      const float z = f16_bits_to_f32(zero[m]), s = f16_bits_to_f32(scale[m]);
#pragma unroll
      for (int t = 0; t < 8; ++t) { z8[t] = z; s8[t] = s; }
    }
    Row8 x = load_bf16x8(x_hat + xoff);
    Row8 o;
#pragma unroll
    for (int t = 0; t < 8; ++t) o.v[t] = x.v[t] + (z8[t] + (float)q[t] * s8[t]);
    *reinterpret_cast<uint4*>(dst) = to_bf16x8(o);
  }
}

template <int BITS, int AXIS>
__global__ __launch_bounds__(256) void dequant_kernel(
    const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scale,
    const uint16_t* __restrict__ zero, const int32_t* __restrict__ idx, int k, int N, int HD, int G,
    uint16_t* x_hat, uint16_t* out_rows) {
  dequant_body<BITS, AXIS>(codes, scale, zero, idx, k, N, HD, G, x_hat, out_rows,
                           (int64_t)blockIdx.x * blockDim.x + threadIdx.x, blockIdx.y);
}

// Keys (token axis) in workgroups [0, half) and values (channel axis) in [half, 2 half) of one launch.
struct DequantKV {
  const uint8_t* k_codes;
  const uint16_t* k_scale;
  const uint16_t* k_zero;
  const uint8_t* v_codes;
  const uint16_t* v_scale;
  const uint16_t* v_zero;
  const int32_t* idx;
  uint16_t* k_hat;
  uint16_t* v_hat;
  uint16_t* k_rows;
  uint16_t* v_rows;
  int k, N, HD, G, half;
};

template <int BITS>
__global__ __launch_bounds__(256) void dequant_kv_kernel(DequantKV a) {
  const int bx = blockIdx.x;
  if (bx < a.half)
    dequant_body<BITS, FL_AXIS_TOKEN>(a.k_codes, a.k_scale, a.k_zero, a.idx, a.k, a.N, a.HD, a.G, a.k_hat,
                                      a.k_rows, (int64_t)bx * 256 + threadIdx.x, blockIdx.y);
  else
    dequant_body<BITS, FL_AXIS_CHANNEL>(a.v_codes, a.v_scale, a.v_zero, a.idx, a.k, a.N, a.HD, a.G, a.v_hat,
                                        a.v_rows, (int64_t)(bx - a.half) * 256 + threadIdx.x, blockIdx.y);
}

static int check_codec_args(const char* fn, const void* codes, const void* a, int k, int B, int N,
                            int H, int d, int bits, int group, int axis, bool need_meta,
                            const void* scale, const void* zero, const void* idx) {
  FL_REQUIRE((codes || k == 0) && a, FL_E_NULL, "%s: codes and the state pointer are required", fn);
  FL_REQUIRE(B >= 1 && N >= 1 && H >= 1, FL_E_SHAPE, "%s: need B, N, H >= 1", fn);
  FL_REQUIRE(d == 64 || d == 128, FL_E_SHAPE, "%s: head dim %d not in {64, 128}", fn, d);
  FL_REQUIRE((int64_t)N * H * d < ((int64_t)1 << 31), FL_E_SHAPE, "%s: N * H * d too large", fn);
  FL_REQUIRE(idx != nullptr || k == N || k == 0, FL_E_SHAPE, "%s: without idx, k must equal N", fn);
  FL_REQUIRE(k >= 0 && k <= N, FL_E_RANGE, "%s: k=%d outside [0, N]", fn, k);
  FL_REQUIRE(bits == 2 || bits == 4 || bits == 8 || bits == 16, FL_E_UNSUPPORTED,
             "%s: bits=%d not in {2, 4, 8, 16}", fn, bits);
  FL_REQUIRE(axis == FL_AXIS_TOKEN || axis == FL_AXIS_CHANNEL, FL_E_UNSUPPORTED, "%s: bad axis %d", fn, axis);
  if (bits != 16) {
    FL_REQUIRE(group >= 8 && group <= 128 && group % 8 == 0 && (group & (group - 1)) == 0,
               FL_E_UNSUPPORTED, "%s: group=%d must be a power of two in [8, 128]", fn, group);
    FL_REQUIRE(axis == FL_AXIS_TOKEN || d % group == 0, FL_E_SHAPE,
               "%s: CHANNEL axis needs group | d (group=%d, d=%d)", fn, group, d);
    if (need_meta && k > 0) FL_REQUIRE(scale && zero, FL_E_NULL, "%s: scale and zero are required", fn);
  }
  return FL_OK;
}

static int residual_quant(const char* fn, const uint16_t* x_cur, const uint16_t* x_ref, const int32_t* idx,
                          int k, int B, int N, int H, int d, int bits, int group, int axis, uint8_t* codes,
                          uint16_t* scale, uint16_t* zero, uint16_t* out_rows, bool commit, void* stream) {
  int rc = check_codec_args(fn, codes, x_cur, k, B, N, H, d, bits, group, axis, true, scale, zero, idx);
  if (rc != FL_OK) return rc;
  if (k == 0) return FL_OK;
  hipStream_t st = as_stream(stream);
  FL_CHECK_LIST(fn, "idx", idx, B, k, 0, N, st);
  const int HD = H * d;
  if (bits == 16) {
    dim3 grid((unsigned)(((int64_t)k * (HD / 8) + 255) / 256), B);
    passthrough_kernel<<<grid, 256, 0, st>>>(x_cur, idx, k, N, HD, codes, out_rows, commit);
    return check_launch("passthrough_kernel");
  }
  if (axis == FL_AXIS_TOKEN) {
    const int slices = group < 32 ? group : 32;
    const int cw = 256 / slices * 8;                      // channels per workgroup
    dim3 grid((HD + cw - 1) / cw, (k + group - 1) / group, B);
#define FL_QT(BB, SS, RR)                                                                          \
  quant_token_kernel<BB, SS, RR><<<grid, 256, 0, st>>>(x_cur, x_ref, idx, k, N, HD, group, codes, \
                                                       scale, zero, out_rows, commit, INFINITY)
#define FL_QT_BITS(BB)                                   \
  switch (group) {                                       \
    case 8: FL_QT(BB, 8, 1); break;                      \
    case 16: FL_QT(BB, 16, 1); break;                    \
    case 32: FL_QT(BB, 32, 1); break;                    \
    case 64: FL_QT(BB, 32, 2); break;                    \
    default: FL_QT(BB, 32, 4); break;                    \
  }
    if (bits == 2) { FL_QT_BITS(2) } else if (bits == 4) { FL_QT_BITS(4) } else { FL_QT_BITS(8) }
#undef FL_QT_BITS
#undef FL_QT
    return check_launch("quant_token_kernel");
  }
  dim3 grid((unsigned)(((int64_t)k * (HD / 8) + 255) / 256), B);
#define FL_QC(BB) \
  quant_channel_kernel<BB><<<grid, 256, 0, st>>>(x_cur, x_ref, idx, k, N, HD, group, codes, scale, zero, out_rows, commit, INFINITY)
  if (bits == 2) FL_QC(2);
  else if (bits == 4) FL_QC(4);
  else FL_QC(8);
#undef FL_QC
  return check_launch("quant_channel_kernel");
}

// Keys (token axis) and values (channel axis) with one bit width and group size.  out rows: compact
// k_rows / v_rows (each optional), or with commit the rows idx of k_ref / v_ref in place.
// ---- fp16 copy of rows of a bf16 [B, N, HD] tensor (all rows, or rows idx) ------------------------------
__global__ __launch_bounds__(256) void f16_rows_kernel(const uint16_t* __restrict__ x, const int32_t* __restrict__ idx,
                                                       int k, int N, int HD, uint16_t* __restrict__ y) {
  const int b = blockIdx.y;
  const int chunks = HD / 8;
  const int64_t local = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (local >= (int64_t)k * chunks) return;
  const int p = (int)(local / chunks), c = (int)(local % chunks);
  const int64_t i = idx ? (int64_t)idx[(int64_t)b * k + p] : (int64_t)p;
  const int64_t off = ((int64_t)b * N + i) * HD + (int64_t)c * 8;
  *reinterpret_cast<uint4*>(y + off) = bf16x8_to_f16(*reinterpret_cast<const uint4*>(x + off));
}

static int launch_f16_rows(const uint16_t* x, const int32_t* idx, int k, int B, int N, int HD, uint16_t* y,
                           hipStream_t st) {
  if (k == 0) return FL_OK;
  dim3 grid((unsigned)(((int64_t)k * (HD / 8) + 255) / 256), B);
  f16_rows_kernel<<<grid, 256, 0, st>>>(x, idx, k, N, HD, y);
  return check_launch("f16_rows_kernel");
}

static int residual_quant_kv(const char* fn, const uint16_t* k_cur, uint16_t* k_ref, const uint16_t* v_cur,
                             uint16_t* v_ref, const int32_t* idx, int k, int B, int N, int H, int d, int bits,
                             int group, uint8_t* k_codes, uint16_t* k_scale, uint16_t* k_zero, uint8_t* v_codes,
                             uint16_t* v_scale, uint16_t* v_zero, uint16_t* k_rows, uint16_t* v_rows, bool commit,
                             uint16_t* v_f16,
                             void* stream) {
  int rc = check_codec_args(fn, k_codes, k_cur, k, B, N, H, d, bits, group, FL_AXIS_TOKEN, true, k_scale,
                            k_zero, idx);
  if (rc != FL_OK) return rc;
  rc = check_codec_args(fn, v_codes, v_cur, k, B, N, H, d, bits, group, FL_AXIS_CHANNEL, true, v_scale, v_zero,
                        idx);
  if (rc != FL_OK) return rc;
  if (k == 0) return FL_OK;
  if (bits == 16) {   // raw payload: two copy launches
    rc = residual_quant(fn, k_cur, k_ref, idx, k, B, N, H, d, bits, group, FL_AXIS_TOKEN, k_codes, k_scale,
                        k_zero, commit ? k_ref : k_rows, commit, stream);
    if (rc != FL_OK) return rc;
    rc = residual_quant(fn, v_cur, v_ref, idx, k, B, N, H, d, bits, group, FL_AXIS_CHANNEL, v_codes, v_scale,
                        v_zero, commit ? v_ref : v_rows, commit, stream);
    if (rc != FL_OK || !v_f16) return rc;
    return launch_f16_rows(v_ref, idx, k, B, N, H * d, v_f16, as_stream(stream));
  }
  const int HD = H * d;
  const int slices = group < 32 ? group : 32;
  const int cw = 256 / slices * 8;
  QuantKV a;
  a.k_cur = k_cur; a.k_ref = k_ref; a.v_cur = v_cur; a.v_ref = v_ref; a.idx = idx;
  a.k_codes = k_codes; a.k_scale = k_scale; a.k_zero = k_zero;
  a.v_codes = v_codes; a.v_scale = v_scale; a.v_zero = v_zero;
  a.k_rows = commit ? k_ref : k_rows;
  a.v_rows = commit ? v_ref : v_rows;
  a.v_f16 = commit ? v_f16 : nullptr;
  a.k = k; a.N = N; a.HD = HD; a.G = group;
  a.kx = (HD + cw - 1) / cw;
  a.ky = (k + group - 1) / group;
  a.vx = (int)(((int64_t)k * (HD / 8) + 255) / 256);
  a.commit = commit ? 1 : 0;
  a.pinf = INFINITY;
  const int64_t blocks = ((int64_t)a.kx * a.ky + a.vx) * B;
  FL_REQUIRE(blocks < ((int64_t)1 << 31), FL_E_SHAPE, "%s: grid too large", fn);
  hipStream_t st = as_stream(stream);
  FL_CHECK_LIST(fn, "idx", idx, B, k, 0, N, st);
#define FL_QKV(BB, SS, RR) quant_kv_kernel<BB, SS, RR><<<(unsigned)blocks, 256, 0, st>>>(a)
#define FL_QKV_BITS(BB)                                   \
  switch (group) {                                        \
    case 8: FL_QKV(BB, 8, 1); break;                      \
    case 16: FL_QKV(BB, 16, 1); break;                    \
    case 32: FL_QKV(BB, 32, 1); break;                    \
    case 64: FL_QKV(BB, 32, 2); break;                    \
    default: FL_QKV(BB, 32, 4); break;                    \
  }
  if (bits == 2) { FL_QKV_BITS(2) } else if (bits == 4) { FL_QKV_BITS(4) } else { FL_QKV_BITS(8) }
#undef FL_QKV_BITS
#undef FL_QKV
  return check_launch("quant_kv_kernel");
}


// The most recent tokens stay in bf16 (Appendix E): rows i >= N - tail among the active rows are stored as
// the exact X^(r) rows, in the caches and/or the compact rows (their codes are formed with the others).
// idx ascends, so only its last min(k, tail) entries can be tail rows: one thread per 16-byte chunk of those.
__global__ __launch_bounds__(256) void keep_recent_kernel(const uint16_t* __restrict__ x_cur,
                                                          const int32_t* __restrict__ idx, int k, int N, int HD,
                                                          int lo, int n_last, uint16_t* cache, uint16_t* rows) {
  const int b = blockIdx.y;
  const int chunks = HD / 8;
  const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (x >= (int64_t)n_last * chunks) return;
  const int p = k - n_last + (int)(x / chunks);
  const int c = (int)(x % chunks);
  const int i = idx ? idx[(int64_t)b * k + p] : p;
  if (i < lo) return;
  const uint4 v = *reinterpret_cast<const uint4*>(x_cur + ((int64_t)b * N + i) * HD + c * 8);
  if (cache) *reinterpret_cast<uint4*>(cache + ((int64_t)b * N + i) * HD + c * 8) = v;
  if (rows) *reinterpret_cast<uint4*>(rows + ((int64_t)b * k + p) * HD + c * 8) = v;
}

}  // namespace fl

using namespace fl;

extern "C" int fl_kv_residual_quant(const uint16_t* x_cur, const uint16_t* x_ref, const int32_t* idx,
                                    int k, int B, int N, int H, int d, int bits, int group, int axis,
                                    uint8_t* codes, uint16_t* scale, uint16_t* zero,
                                    uint16_t* out_rows, void* stream) {
  FL_API_BEGIN
  FL_REQUIRE(!(out_rows && out_rows == x_ref && idx), FL_E_SHAPE,
             "fl_kv_residual_quant: out_rows may alias x_ref only when idx is NULL");
  return residual_quant("fl_kv_residual_quant", x_cur, x_ref, idx, k, B, N, H, d, bits, group, axis, codes,
                        scale, zero, out_rows, false, stream);
  FL_API_END
}

extern "C" int fl_kv_residual_quant_commit(const uint16_t* x_cur, uint16_t* x_hat, const int32_t* idx, int k,
                                           int B, int N, int H, int d, int bits, int group, int axis,
                                           uint8_t* codes, uint16_t* scale, uint16_t* zero, void* stream) {
  FL_API_BEGIN
  FL_REQUIRE(x_hat != nullptr, FL_E_NULL, "fl_kv_residual_quant_commit: x_hat is required");
  return residual_quant("fl_kv_residual_quant_commit", x_cur, x_hat, idx, k, B, N, H, d, bits, group, axis,
                        codes, scale, zero, x_hat, true, stream);
  FL_API_END
}

extern "C" int fl_kv_residual_quant_kv(const uint16_t* k_cur, uint16_t* k_ref, const uint16_t* v_cur,
                                       uint16_t* v_ref, const int32_t* idx, int k, int B, int N, int H, int d,
                                       int bits, int group, uint8_t* k_codes, uint16_t* k_scale, uint16_t* k_zero,
                                       uint8_t* v_codes, uint16_t* v_scale, uint16_t* v_zero, uint16_t* k_rows,
                                       uint16_t* v_rows, int mode, void* stream) {
  FL_API_BEGIN
  const char* fn = "fl_kv_residual_quant_kv";
  FL_REQUIRE(mode == FL_DQ_COMPACT || mode == FL_DQ_COMMIT, FL_E_UNSUPPORTED, "%s: bad mode %d", fn, mode);
  if (mode == FL_DQ_COMMIT) {
    FL_REQUIRE(k_ref && v_ref, FL_E_NULL, "%s: COMMIT needs k_ref and v_ref", fn);
    FL_REQUIRE(!k_rows && !v_rows, FL_E_NULL, "%s: COMMIT needs k_rows == v_rows == NULL", fn);
    FL_REQUIRE(k_ref != v_ref, FL_E_SHAPE, "%s: COMMIT needs distinct key and value caches", fn);
  } else {
    FL_REQUIRE(!(k_rows && k_rows == k_ref && idx) && !(v_rows && v_rows == v_ref && idx), FL_E_SHAPE,
               "%s: rows may alias the reference only when idx is NULL", fn);
  }
  FL_REQUIRE(k == 0 || k_codes != v_codes, FL_E_SHAPE, "%s: key and value codes must be distinct buffers", fn);
  return residual_quant_kv(fn, k_cur, k_ref, v_cur, v_ref, idx, k, B, N, H, d, bits, group, k_codes, k_scale,
                           k_zero, v_codes, v_scale, v_zero, k_rows, v_rows, mode == FL_DQ_COMMIT, nullptr, stream);
  FL_API_END
}

extern "C" int fl_kv_residual_quant_kv_v16(const uint16_t* k_cur, uint16_t* k_ref, const uint16_t* v_cur,
                                           uint16_t* v_ref, uint16_t* v_f16, const int32_t* idx, int k, int B, int N,
                                           int H, int d, int bits, int group, uint8_t* k_codes, uint16_t* k_scale,
                                           uint16_t* k_zero, uint8_t* v_codes, uint16_t* v_scale, uint16_t* v_zero,
                                           void* stream) {
  FL_API_BEGIN
  const char* fn = "fl_kv_residual_quant_kv_v16";
  FL_REQUIRE(k_ref && v_ref && v_f16, FL_E_NULL, "%s: k_ref, v_ref and v_f16 are required", fn);
  FL_REQUIRE(k_ref != v_ref && (const void*)v_f16 != (const void*)v_ref && (const void*)v_f16 != (const void*)k_ref,
             FL_E_SHAPE, "%s: the key cache, the value cache and its fp16 copy must be distinct", fn);
  FL_REQUIRE(k == 0 || k_codes != v_codes, FL_E_SHAPE, "%s: key and value codes must be distinct buffers", fn);
  return residual_quant_kv(fn, k_cur, k_ref, v_cur, v_ref, idx, k, B, N, H, d, bits, group, k_codes, k_scale,
                           k_zero, v_codes, v_scale, v_zero, nullptr, nullptr, true, v_f16, stream);
  FL_API_END
}

extern "C" int fl_kv_f16_rows(const uint16_t* x, const int32_t* idx, int k, int B, int N, int H, int d,
                              uint16_t* x_f16, void* stream) {
  FL_API_BEGIN
  const char* fn = "fl_kv_f16_rows";
  FL_REQUIRE(x && x_f16, FL_E_NULL, "%s: x and x_f16 are required", fn);
  FL_REQUIRE((const void*)x != (const void*)x_f16, FL_E_SHAPE, "%s: x_f16 may not alias x", fn);
  FL_REQUIRE(B >= 1 && N >= 1 && H >= 1 && d >= 8 && d % 8 == 0, FL_E_SHAPE,
             "%s: need B, N, H >= 1 and d a multiple of 8", fn);
  FL_REQUIRE(k >= 0 && k <= N, FL_E_RANGE, "%s: k=%d outside [0, N]", fn, k);
  if (k == 0) return FL_OK;               // (an empty index list may come as NULL)
  FL_REQUIRE(idx || k == N, FL_E_RANGE, "%s: k=%d with idx NULL (every row: k = N)", fn, k);
  const hipStream_t st = as_stream(stream);
  if (idx) FL_CHECK_LIST(fn, "idx", idx, B, k, 0, N, st);
  return launch_f16_rows(x, idx, k, B, N, H * d, x_f16, st);
  FL_API_END
}

extern "C" int fl_kv_residual_dequant_kv(const uint8_t* k_codes, const uint16_t* k_scale, const uint16_t* k_zero,
                                         const uint8_t* v_codes, const uint16_t* v_scale, const uint16_t* v_zero,
                                         const int32_t* idx, int k, int B, int N, int H, int d, int bits, int group,
                                         int mode, uint16_t* k_hat, uint16_t* v_hat, uint16_t* k_rows,
                                         uint16_t* v_rows, void* stream) {
  FL_API_BEGIN
  const char* fn = "fl_kv_residual_dequant_kv";
  int rc = check_codec_args(fn, k_codes, k_hat, k, B, N, H, d, bits, group, FL_AXIS_TOKEN, true, k_scale, k_zero,
                            idx);
  if (rc != FL_OK) return rc;
  rc = check_codec_args(fn, v_codes, v_hat, k, B, N, H, d, bits, group, FL_AXIS_CHANNEL, true, v_scale, v_zero, idx);
  if (rc != FL_OK) return rc;
  FL_REQUIRE(mode == FL_DQ_COMPACT || mode == FL_DQ_COMMIT, FL_E_UNSUPPORTED, "%s: bad mode %d", fn, mode);
  FL_REQUIRE(mode == FL_DQ_COMMIT ? (!k_rows && !v_rows) : (k_rows && v_rows), FL_E_NULL,
             "%s: COMPACT needs k_rows and v_rows, COMMIT needs both NULL", fn);
  FL_REQUIRE(mode == FL_DQ_COMPACT || k_hat != v_hat, FL_E_SHAPE, "%s: COMMIT needs distinct caches", fn);
  if (k == 0) return FL_OK;
  const int64_t half = ((int64_t)k * (H * d / 8) + 255) / 256;
  FL_REQUIRE(2 * half < ((int64_t)1 << 31), FL_E_SHAPE, "%s: grid too large", fn);
  DequantKV a;
  a.k_codes = k_codes; a.k_scale = k_scale; a.k_zero = k_zero;
  a.v_codes = v_codes; a.v_scale = v_scale; a.v_zero = v_zero;
  a.idx = idx; a.k_hat = k_hat; a.v_hat = v_hat;
  a.k_rows = mode == FL_DQ_COMMIT ? nullptr : k_rows;
  a.v_rows = mode == FL_DQ_COMMIT ? nullptr : v_rows;
  a.k = k; a.N = N; a.HD = H * d; a.G = group; a.half = (int)half;
  dim3 grid((unsigned)(2 * half), B);
  hipStream_t st = as_stream(stream);
  FL_CHECK_LIST("fl_kv_residual_dequant_kv", "idx", idx, B, k, 0, N, st);
  if (bits == 16) {   // raw payload: both axes copy the same way
    dequant_kv_kernel<16><<<grid, 256, 0, st>>>(a);
  } else if (bits == 2) {
    dequant_kv_kernel<2><<<grid, 256, 0, st>>>(a);
  } else if (bits == 4) {
    dequant_kv_kernel<4><<<grid, 256, 0, st>>>(a);
  } else {
    dequant_kv_kernel<8><<<grid, 256, 0, st>>>(a);
  }
  return check_launch("dequant_kv_kernel");
  FL_API_END
}

extern "C" int fl_kv_residual_dequant(const uint8_t* codes, const uint16_t* scale, const uint16_t* zero,
                                      const int32_t* idx, int k, int B, int N, int H, int d, int bits,
                                      int group, int axis, int mode, uint16_t* x_hat,
                                      uint16_t* out_rows, void* stream) {
  FL_API_BEGIN
  int rc = check_codec_args("fl_kv_residual_dequant", codes, x_hat, k, B, N, H, d, bits, group, axis,
                            true, scale, zero, idx);
  if (rc != FL_OK) return rc;
  FL_REQUIRE(mode == FL_DQ_COMPACT || mode == FL_DQ_COMMIT, FL_E_UNSUPPORTED,
             "fl_kv_residual_dequant: bad mode %d", mode);
  FL_REQUIRE(mode == FL_DQ_COMMIT ? out_rows == nullptr : out_rows != nullptr, FL_E_NULL,
             "fl_kv_residual_dequant: COMPACT needs out_rows, COMMIT needs out_rows == NULL");
  if (k == 0) return FL_OK;
  const int HD = H * d;
  dim3 grid((unsigned)(((int64_t)k * (HD / 8) + 255) / 256), B);
  hipStream_t st = as_stream(stream);
  FL_CHECK_LIST("fl_kv_residual_dequant", "idx", idx, B, k, 0, N, st);
#define FL_DQ(BB, AA) \
  dequant_kernel<BB, AA><<<grid, 256, 0, st>>>(codes, scale, zero, idx, k, N, HD, group, x_hat, out_rows)
  if (bits == 16) FL_DQ(16, 0);
  else if (axis == FL_AXIS_TOKEN) {
    if (bits == 2) FL_DQ(2, FL_AXIS_TOKEN); else if (bits == 4) FL_DQ(4, FL_AXIS_TOKEN); else FL_DQ(8, FL_AXIS_TOKEN);
  } else {
    if (bits == 2) FL_DQ(2, FL_AXIS_CHANNEL); else if (bits == 4) FL_DQ(4, FL_AXIS_CHANNEL); else FL_DQ(8, FL_AXIS_CHANNEL);
  }
#undef FL_DQ
  return check_launch("dequant_kernel");
  FL_API_END
}

extern "C" int fl_kv_keep_recent(const uint16_t* x_cur, const int32_t* idx, int k, int B, int N, int H, int d,
                                 int tail, uint16_t* cache, uint16_t* rows, void* stream) {
  FL_API_BEGIN
  FL_REQUIRE(x_cur, FL_E_NULL, "fl_kv_keep_recent: x_cur is required");
  FL_REQUIRE(cache || rows, FL_E_NULL, "fl_kv_keep_recent: cache or rows is required");
  FL_REQUIRE(B >= 1 && N >= 1 && H >= 1, FL_E_SHAPE, "fl_kv_keep_recent: need B, N, H >= 1");
  FL_REQUIRE(d >= 8 && d % 8 == 0, FL_E_SHAPE, "fl_kv_keep_recent: d=%d must be a positive multiple of 8", d);
  FL_REQUIRE((int64_t)N * H * d < ((int64_t)1 << 40), FL_E_SHAPE, "fl_kv_keep_recent: N * H * d too large");
  FL_REQUIRE(k >= 0 && k <= N, FL_E_RANGE, "fl_kv_keep_recent: k=%d outside [0, N]", k);
  FL_REQUIRE(idx || k == N, FL_E_SHAPE, "fl_kv_keep_recent: without idx, k must equal N");
  FL_REQUIRE(tail >= 0, FL_E_RANGE, "fl_kv_keep_recent: tail must be >= 0");
  const int n_last = std::min(k, tail);
  if (n_last == 0) return FL_OK;
  const int HD = H * d;
  const int64_t work = (int64_t)n_last * (HD / 8);
  dim3 grid((unsigned)((work + 255) / 256), B);
  FL_CHECK_LIST("fl_kv_keep_recent", "idx", idx, B, k, 0, N, as_stream(stream));
  keep_recent_kernel<<<grid, 256, 0, as_stream(stream)>>>(x_cur, idx, k, N, HD, std::max(0, N - tail), n_last,
                                                          cache, rows);
  return check_launch("keep_recent_kernel");
  FL_API_END
}
