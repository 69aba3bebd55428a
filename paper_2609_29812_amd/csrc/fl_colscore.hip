// Column statistics in 64 bits, whose fp32 keys a top-k ranks:
//   * the dense source loop's statistic (Appendix D.2, Eq. 6 with all causal keys and cached mass 1, summed
//     over the rows of a prefill), in two passes: the rows' log-normalisers, then the column sums;
//   * the statistic that prunes a list for a smaller budget (Section 4.2): the mass the updated rows give
//     each list entry, from their stored reference log-normalisers.
// The dot products are integer products of byte digits (fl_digits.h), or v_mfma_f64_16x16x4 products (products of bf16
// values are exact in fp64) where the digits do not hold the values.  Every sum runs in a fixed order (deterministic).
// Before its rounding to fp32 a key is the exact statistic to fp64 rounding with the fp64 products, and to 2^-24 of
// itself at worst with the digits, by what they leave out of the values at hand (digits_serve).  The rounded keys of the
// two are the same for normal values of deviation 1 to 4 and with key channels offset by up to 32 (2.5 million keys,
// prompts of 1009 to 32768); with 2 % of the elements scaled by 2^-17, 3 of 409 thousand keys differ, by one ulp.
#include "fl_attn_util.h"
#include "fl_digits.h"

#include <type_traits>

namespace fl {

constexpr int kCsRows = 32;               // vectors staged per step
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Which (row, column) of a v_mfma_f64_16x16x4 product each of a lane's four accumulator elements holds,
// read off two index products (A = row index in k-column 0 against B = 1 in k-row 0, and the transposed
// pair), clamped so that the indices stay in range whatever the products hold.
__device__ __forceinline__ void mfma_f64_layout(int l16, int kq, int (&row)[4], int (&col)[4]) {
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  const f64x4 r = __builtin_amdgcn_mfma_f64_16x16x4f64(kq == 0 ? (double)l16 : 0.0, kq == 0 ? 1.0 : 0.0, zero, 0, 0, 0);
  const f64x4 c = __builtin_amdgcn_mfma_f64_16x16x4f64(kq == 0 ? 1.0 : 0.0, kq == 0 ? (double)l16 : 0.0, zero, 0, 0, 0);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    row[t] = min(max((int)r[t], 0), 15);
    col[t] = min(max((int)c[t], 0), 15);
  }
}

// Dense column statistic by v_mfma_f64_16x16x4 (products of bf16 values are exact in fp64), for the (batch,
// head) pairs whose values the digits do not hold, in two passes.  A wave owns 16 vectors of one side in registers
// (lane l holds dim 4s + l / 16 of vector l % 16 for step s), the workgroup 64 of them from vector wg_first on;
// the other side is staged 32 vectors at a time in LDS as fp64.
// The next step's vectors are loaded into registers while a step is multiplied: 8192 x 16 heads x 128 8.88 -> 6.40 ms,
// 32768 x 16 x 64 75.8 -> 59.4 (11.5 and 69.5 in a kernel of their own that loaded them in place).
//   pass 1 (ROWS)  : the wave's 16 query rows against the staged K columns j <= i: per accumulator element
//                    an online (max, sum) in fp64; the 16 partial pairs of a row are merged in column order;
//   pass 2 (!ROWS) : the wave's 16 K columns against the staged query rows i >= j and their lse_i:
//                    col_j = sum exp(l_ij - lse_i), the 16 partials of a column added in row order.
// Every sum runs in a fixed order (deterministic).
template <int D>
struct CsWide {
  double st[kCsRows * (D + 1)];           // padded stride: the 16 vectors of a read spread over banks
  double lse[kCsRows];
};
struct CsMerge {
  double v[4][16][16];
};

template <int D, bool ROWS>
__device__ __forceinline__ void colscore_wide(const uint16_t* __restrict__ qbase, const uint16_t* __restrict__ kbase, int N, int H,
                              double sigma, double* __restrict__ lse_bh, float* __restrict__ col_bh, int wg_first,
                              CsWide<D>& wide, CsMerge& red_m, CsMerge& red_s) {
  constexpr int QS = D + 1;
  constexpr int KSTEPS = D / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const int64_t stride = (int64_t)H * D;
  const int v0 = wg_first + wave * 16;                  // first of the wave's own vectors
  const bool wave_ok = v0 < N;

  float reg[KSTEPS];                                    // own vectors (query rows or key columns), widened where used
  {
    const int v = v0 + l16;
    const uint16_t* src = (ROWS ? qbase : kbase) + (int64_t)(v < N ? v : 0) * stride + kq;
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) reg[s] = v < N ? bf16_to_f32(src[4 * s]) : 0.0f;
  }
  int el_r[4], el_c[4];                   // element t: staged vector el_r (A side), own vector el_c (B side)
  mfma_f64_layout(l16, kq, el_r, el_c);
  // staged range: pass 1 columns 0 .. last own row; pass 2 rows from the workgroup's first column on
  const int s_begin = ROWS ? 0 : wg_first;
  const int s_end = ROWS ? min(N, wg_first + 64) : N;
  double m[4], acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) { m[t] = -INFINITY; acc[t] = 0.0; }
  // the thread's elements of a step (of vectors r0, r0 + 256 / D, ..), loaded while the step before is multiplied
  constexpr int PER = kCsRows * D / 256;
  const int r0 = threadIdx.x / D, dd = threadIdx.x % D;
  const rsrc_t oth = make_rsrc(ROWS ? kbase : qbase, (uint32_t)((N - 1) * stride + D) * 2u);
  uint16_t nx[PER];
  double nlse = 0.0;
  auto fetch = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int v = t0 + r0 + x * (256 / D);            // (N H D < 2^31: 32-bit byte offsets; 0xFFFFFFFE reads zero)
      const uint32_t off = v < s_end ? ((uint32_t)v * (uint32_t)stride + dd) * 2u : 0xFFFFFFFEu;
      nx[x] = __builtin_amdgcn_raw_buffer_load_b16(oth, off, 0, 0);
    }
    if (!ROWS && threadIdx.x < kCsRows) {
      const int v = t0 + (int)threadIdx.x;
      nlse = v < s_end ? lse_bh[v] : 0.0;
    }
  };
  fetch(s_begin);
  __syncthreads();
  for (int t0 = s_begin; t0 < s_end; t0 += kCsRows) {
#pragma unroll
    for (int x = 0; x < PER; ++x) wide.st[(r0 + x * (256 / D)) * QS + dd] = (double)bf16_to_f32(nx[x]);
    if (!ROWS && threadIdx.x < kCsRows) wide.lse[threadIdx.x] = nlse;
    fetch(t0 + kCsRows);
    __syncthreads();
#pragma unroll
    for (int half = 0; half < kCsRows / 16; ++half) {
      const int sv0 = t0 + 16 * half;                   // first staged vector of this 16
      // uniform: pass 1 needs staged columns <= the wave's last row, pass 2 staged rows >= its first column
      const bool useful = wave_ok && sv0 < s_end && (ROWS ? sv0 <= v0 + 15 : sv0 + 15 >= v0);
      if (useful) {
        f64x4 d4 = {0.0, 0.0, 0.0, 0.0};
        const double* sa = wide.st + (16 * half + l16) * QS + kq;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) d4 = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[4 * s], (double)reg[s], d4, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int sv = sv0 + el_r[t];                  // staged vector
          const int ov = v0 + el_c[t];                   // own vector
          const double l = sigma * d4[t];
          if (ROWS) {
            if (sv < s_end && ov < N && sv <= ov) {      // column sv of row ov
              if (l > m[t]) {
                acc[t] = acc[t] * exp(m[t] - l) + 1.0;
                m[t] = l;
              } else {
                acc[t] += exp(l - m[t]);
              }
            }
          } else {
            if (sv < s_end && ov < N && sv >= ov) acc[t] += exp(l - wide.lse[16 * half + el_r[t]]);   // row sv
          }
        }
      }
    }
    __syncthreads();
  }
  // merge the 16 partials of each own vector in staged-slot order
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    red_m.v[wave][el_c[t]][el_r[t]] = m[t];
    red_s.v[wave][el_c[t]][el_r[t]] = acc[t];
  }
  __syncthreads();
  const int v = v0 + lane;
  if (lane < 16 && v < N) {
    if (ROWS) {
      double mm = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mm = fmax(mm, red_m.v[wave][lane][r]);
      double ss = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (red_s.v[wave][lane][r] > 0.0) ss += red_s.v[wave][lane][r] * exp(red_m.v[wave][lane][r] - mm);
      lse_bh[v] = mm + log(ss);
    } else {
      double ss = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) ss += red_s.v[wave][lane][r];
      col_bh[v] = (float)ss;
    }
  }
  __syncthreads();
}

// Digits of the queries (side 0) and keys (side 1) of n_seg (batch, head) pairs from seg0 on, in the order in which
// the statistic's waves take them: per 16-vector block, digit 3 .. 0, 64 dims and lane, 16 bytes.
struct CsArgs {
  const uint16_t *q, *k;
  int N, H, seg0, n_seg, nblk;            // nblk = ceil(N / 16)
  double sigma;
  double* lse;                            // [n_seg, lse_stride]; log2 of the row sums where the digits serve
  int64_t lse_stride;
  float* col_key;                         // [B, H, N]
  uint4* dig;                             // [2, n_seg, nblk, 4 D / 64, 64]; NULL: no workspace for digits
  int* exps;                              // [2, n_seg, nblk4]: each block's unit 2^e, nblk4 = nblk rounded up to 4
  DigitStat* stat;                        // [2, n_seg, nblk]
};

template <int D>
__global__ __launch_bounds__(256) void cs_digits_kernel(CsArgs a) {
  constexpr int KS = D / 64;
  const int lane = threadIdx.x & 63, blk = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int seg = blockIdx.y, side = blockIdx.z;
  if (blk >= a.nblk) return;
  const int b = (a.seg0 + seg) / a.H, h = (a.seg0 + seg) % a.H;
  const int v = blk * 16 + (lane & 15);
  uint4 w[2 * KS];
#pragma unroll
  for (int x = 0; x < 2 * KS; ++x) w[x] = make_uint4(0, 0, 0, 0);
  if (v < a.N) {
    const uint16_t* src = (side ? a.k : a.q) + (((int64_t)b * a.N + v) * a.H + h) * D + 16 * (lane >> 4);
#pragma unroll
    for (int x = 0; x < 2 * KS; ++x) w[x] = *reinterpret_cast<const uint4*>(src + 64 * (x >> 1) + 8 * (x & 1));
  }
  DigitStat stat;
  const DigitBlock<D> o = make_digits<D>(w, stat);
  const int64_t sb = ((int64_t)side * a.n_seg + seg) * a.nblk + blk;
  i32x4* out = reinterpret_cast<i32x4*>(a.dig) + sb * (4 * KS * 64) + lane;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) out[(s * KS + ks) * 64] = o.d[s][ks];
  if (lane == 0) {
    a.stat[sb] = stat;
    a.exps[((int64_t)side * a.n_seg + seg) * ((a.nblk + 3) & ~3) + blk] = stat.e;
  }
}

// largest of the blocks' figures of one side over the workgroup
__device__ __forceinline__ DigitStat cs_side_stat(const DigitStat* __restrict__ st, int nblk, DigitStat (&red)[4]) {
  DigitStat m = {};
  for (int x = threadIdx.x; x < nblk; x += 256) join_stat(m, st[x]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const DigitStat o = {__shfl_xor(m.res, off, 64), __shfl_xor(m.low0, off, 64), __shfl_xor(m.low1, off, 64),
                         __shfl_xor(m.top, off, 64), __shfl_xor(m.norm, off, 64), 0};
    join_stat(m, o);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) join_stat(m, red[w]);
  __syncthreads();
  return m;
}

// One stage of the other side: STG blocks of digits, their exponents and (pass 2) the rows' log2 sums.
template <int D, int STG>
struct __attribute__((aligned(16))) CsSlot {
  uint4 dig[STG * 4 * (D / 64) * 64];
  double lse[STG * 16];
  int exps[STG];
};

// Dense column statistic in two passes over the digits.  A wave owns NB blocks of 16 vectors of one side in
// registers, a workgroup 64 NB of them; the other side streams through two LDS slots, filled by LDS-DMA in the
// order in which the waves read it (no bank conflicts, no shuffles).
//   pass 1 (ROWS)  : own query rows against staged K columns j <= i: lse2_i = log2 sum 2^(l2_ij);
//   pass 2 (!ROWS) : own K columns against staged query rows i >= j: col_j = sum 2^(l2_ij - lse2_i),
// l2 = log2(e) l.  Exponents are bounded (digits_serve), so no running maximum is kept.
// Bound by issue on both pipes: per 16 x 16 block and wave, 26 i8 products (416 matrix cycles) and about 95 vector
// instructions (380 cycles) at d = 128, so the products of one block are issued between the exponentials of the
// one before.  At N = 8192, 16 heads x 128: 11.5 -> 1.43 ms for the statistic and its lists (a pass took 5.5 ms in fp64
// products, 0.7 now; 0.75 at least and 0.80 in the median under the profiler), vector ALU 65 % and matrix cores 56 % of
// the busy cycles at 1.9 GHz.  Nine products and a branch to four more where a digit 0 is present measured 0.95 ms:
// the branch ends the interleaving.
// (three workgroups a CU also for 64-wide rows, where the fp64 products would take the registers of one of them)
template <int D, int NB, bool ROWS>
__global__ __launch_bounds__(256, NB == 1 || (D == 64 && ROWS) ? 3 : 2) void colscore_kernel(CsArgs a, int n_wg) {
  constexpr int KS = D / 64, STG = NB == 1 ? 2 : 4;
  constexpr int BLK = 4 * KS * 64;        // 16-byte pieces of a block
  constexpr size_t kSlot = sizeof(CsSlot<D, STG>) > sizeof(CsWide<D>) ? sizeof(CsSlot<D, STG>) : sizeof(CsWide<D>);
  constexpr size_t kSlot1 = sizeof(CsSlot<D, STG>) > sizeof(CsMerge) ? sizeof(CsSlot<D, STG>) : sizeof(CsMerge);
  __shared__ __attribute__((aligned(16))) char slot0[kSlot];
  __shared__ __attribute__((aligned(16))) char slot1[kSlot1];
  __shared__ DigitStat red[4];
  // the workgroups of one (batch, head) go to one XCD (its digits stay in that L2), the longest ranges first
  const int id = blockIdx.x;
  int seg, rank;
  if (a.n_seg % 8 == 0) {
    const int per = a.n_seg / 8;
    seg = (id & 7) + 8 * ((id >> 3) % per);
    rank = (id >> 3) / per;
  } else {
    seg = id % a.n_seg;
    rank = id / a.n_seg;
  }
  const int wg = ROWS && NB == 1 ? n_wg - 1 - rank : rank;
  const int gs = a.seg0 + seg;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* lse = a.lse + seg * a.lse_stride;
  float* col = a.col_key + (int64_t)gs * a.N;
  bool serve = a.dig != nullptr;
  if (serve) {
    const DigitStat sq = cs_side_stat(a.stat + (int64_t)seg * a.nblk, a.nblk, red);
    const DigitStat sk = cs_side_stat(a.stat + ((int64_t)a.n_seg + seg) * a.nblk, a.nblk, red);
    serve = digits_serve(sq, sk, (float)a.sigma);
  }
  if (!serve) {                           // uniform
    const int64_t base = (int64_t)(gs / a.H) * a.N * a.H * D + (int64_t)(gs % a.H) * D;
    for (int x = 0; x < NB; ++x)
      if ((x ? 2 * n_wg - 1 - wg : wg) * 64 < a.N)
        colscore_wide<D, ROWS>(a.q + base, a.k + base, a.N, a.H, a.sigma, lse, col, (x ? 2 * n_wg - 1 - wg : wg) * 64,
                               *reinterpret_cast<CsWide<D>*>(slot0), *reinterpret_cast<CsMerge*>(slot0),
                               *reinterpret_cast<CsMerge*>(slot1));
    return;
  }
  CsSlot<D, STG>& s0 = *reinterpret_cast<CsSlot<D, STG>*>(slot0);
  CsSlot<D, STG>& s1 = *reinterpret_cast<CsSlot<D, STG>*>(slot1);
  const int64_t own_side = (int64_t)(ROWS ? 0 : a.n_seg) + seg, oth_side = (int64_t)(ROWS ? a.n_seg : 0) + seg;
  const int nblk4 = (a.nblk + 3) & ~3;
  // The workgroup's own blocks: four from block 4 wg on and, with two per wave, the four that lie as far from the
  // other end, so that every workgroup has the same length of the causal triangle to do.
  const int first = 4 * wg, second = 8 * n_wg - 4 - first;
  DigitBlock<D> own[NB];
  double f_own[NB], acc[NB];
  int ob[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    ob[nb] = (nb ? second : first) + wave;
    const int x = min(ob[nb], a.nblk - 1);
    const i32x4* src = reinterpret_cast<const i32x4*>(a.dig) + (own_side * a.nblk + x) * BLK + lane;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) own[nb].d[s][ks] = src[(s * KS + ks) * 64];
    // sigma log2(e), the unit of digit_dot and the own block's exponent
    f_own[nb] = __builtin_ldexp(a.sigma * 0x1.71547652b82fep+16, a.exps[own_side * nblk4 + x]);
    acc[nb] = 0.0;
  }
  const int s_begin = ROWS ? 0 : first;
  const int s_end = ROWS ? min(a.nblk, (NB == 2 ? second : first) + 4) : a.nblk;
  const rsrc_t digR = make_rsrc(a.dig + oth_side * a.nblk * BLK, (uint32_t)a.nblk * BLK * 16u);
  const rsrc_t expR = make_rsrc(a.exps + oth_side * nblk4, (uint32_t)nblk4 * 4u);
  const rsrc_t lseR = make_rsrc(lse, (uint32_t)a.nblk * 128u);
  auto fill = [&](CsSlot<D, STG>& sl, int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < STG * 4 * KS / 4; ++x) {
      const int piece = 4 * x + wave;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(digR, FL_LDS(sl.dig + piece * 64), 16,
                                               (uint32_t)(t0 * BLK + piece * 64 + lane) * 16u, 0, 0, 0);
    }
    if (wave == 0 && lane < STG)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(expR, FL_LDS(sl.exps), 4, (uint32_t)(t0 + lane) * 4u, 0, 0, 0);
    if (!ROWS && wave == 1 && lane < STG * 8)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(lseR, FL_LDS(sl.lse), 16, (uint32_t)t0 * 128u + lane * 16u, 0, 0, 0);
  };
  // the exponentials of one block, added to acc; edge: with the causal bound and the end of the rows
  auto add = [&](const CsSlot<D, STG>& sl, const DigitSums& o, int t0, int x, int nb, auto edge) __attribute__((always_inline)) {
    const double f = __builtin_ldexp(f_own[nb], sl.exps[x]);
    double e[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const double v = digit_dot(o, t);
      double z = ROWS ? v * f : fma(v, f, -sl.lse[x * 16 + 4 * (lane >> 4) + t]);
      if (edge.value) {
        const int sv = (t0 + x) * 16 + 4 * (lane >> 4) + t, ov = ob[nb] * 16 + (lane & 15);
        z = (ROWS ? sv <= ov : sv >= ov && sv < a.N) ? z : -1000.0;
      }
      e[t] = exp2_f64(z);
    }
    acc[nb] += (e[0] + e[1]) + (e[2] + e[3]);
  };
  // own blocks FIRST .. FIRST + COUNT - 1 against a stage
  auto stage = [&](const CsSlot<D, STG>& sl, int t0, auto first_own, auto count, bool full) __attribute__((always_inline)) {
    if (full)
      digit_stage<D, count.value, STG, first_own.value>(sl.dig, own, [&](const DigitSums& o, int x, int nb) __attribute__((always_inline)) {
        add(sl, o, t0, x, nb, std::false_type{});
      });
    else
      digit_stage<D, count.value, STG, first_own.value>(sl.dig, own, [&](const DigitSums& o, int x, int nb) __attribute__((always_inline)) {
        add(sl, o, t0, x, nb, std::true_type{});
      });
  };
  // whether some of a stage is visible to an own block, and all of it
  auto seen = [&](int t0, int o) __attribute__((always_inline)) { return o < a.nblk && (ROWS ? t0 <= o : t0 + STG - 1 >= o); };
  auto whole = [&](int t0, int o) __attribute__((always_inline)) {
    return ROWS ? t0 + STG - 1 < o : t0 > o && (t0 + STG) * 16 <= a.N;
  };
  auto work = [&](const CsSlot<D, STG>& sl, int t0) __attribute__((always_inline)) {
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    if constexpr (NB == 1) {
      if (seen(t0, ob[0])) stage(sl, t0, c0, c1, whole(t0, ob[0]));
    } else {
      // (the lower block sees a prefix of the columns that the upper one sees, and a superset of its rows)
      constexpr std::integral_constant<int, 2> c2{};
      constexpr int RARE = ROWS ? 0 : 1;
      if (seen(t0, ob[RARE])) stage(sl, t0, c0, c2, whole(t0, ob[RARE]));
      else if (seen(t0, ob[1 - RARE])) stage(sl, t0, std::integral_constant<int, 1 - RARE>{}, c1, whole(t0, ob[1 - RARE]));
    }
  };
  fill(s0, s_begin);
  FL_WAIT_VM(0);
  lds_barrier();
  for (int t0 = s_begin; t0 < s_end; t0 += 2 * STG) {
    if (t0 + STG < s_end) fill(s1, t0 + STG);
    work(s0, t0);
    FL_WAIT_VM(0);
    lds_barrier();
    if (t0 + 2 * STG < s_end) fill(s0, t0 + 2 * STG);
    if (t0 + STG < s_end) work(s1, t0 + STG);
    FL_WAIT_VM(0);
    lds_barrier();
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    double s = acc[nb];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    const int v = ob[nb] * 16 + lane;
    if (lane < 16 && ob[nb] < a.nblk) {
      if (ROWS) lse[v] = v < a.N ? log2(s) : 0.0;
      else if (v < a.N) col[v] = (float)s;
    }
  }
}

// Statistic of the list entries for pruning a shrinking list (Section 4.2; Appendix D.2, Eq. 6 with a
// sparse source): entry j of the (b, h) list gets sum_{i updated, i >= j} exp(sigma q_i . k_j - lse_ref_i),
// the loop-r probability mass it receives from the updated rows, each row's probabilities recovered from
// its reference log-normaliser.  A workgroup takes entries and one chunk of kPruneChunk updated rows; the chunk
// partials (fp64, fixed order) are added in chunk order by prune_sum_kernel.
constexpr int kPruneChunk = 256;
constexpr int kPruneEnt = 64;             // entries per workgroup and block of a wave (16 per wave)
constexpr int kPruneRows = 32;            // rows staged per step of the fp64 products

struct PruneArgs {
  const uint16_t *q, *k;
  const int32_t* rows;
  int n_rows;
  const int32_t* cols;
  int c_list, ns;
  const float* lse_ref;
  int N, H;
  double sigma;
  int n_chunks;
  double* part;                           // [B, H, n_chunks, c_list - ns]
  bool digits;                            // q and k are 16-byte aligned
};

template <int D>
struct PruneWide {
  double qt[kPruneRows * (D + 1)];        // padded row stride: the 16 rows of a read spread over banks
  double lse[kPruneRows];
  int row[kPruneRows];
};

// 64 entries of a chunk by fp64 MFMAs (v_mfma_f64_16x16x4): a wave owns 16 entries (their K rows as the B
// operand, in registers: lane l holds dim 4s + l / 16 of entry l % 16 for step s), the chunk's rows from `first` on are
// staged 32 at a time in LDS as fp64 (the A operand: row l % 16, dim 4s + l / 16).  Which accumulator element is which
// (row, entry) is read off two index products at the start, so the epilogue does not depend on the output layout.
template <int D>
__device__ __forceinline__ void prune_wide(const PruneArgs& a, int b, int h, int e_first, const int* s_rows, int p0,
                                           int first, int p_end, double* __restrict__ part, PruneWide<D>& w,
                                           double (*red)[16][17]) {
  constexpr int QS = D + 1;
  constexpr int KSTEPS = D / 4;
  const int n_ent = a.c_list - a.ns;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const int64_t stride = (int64_t)a.H * D;
  const int32_t* cl = a.cols + ((int64_t)b * a.H + h) * a.c_list + a.ns;
  const int e_wave = e_first + wave * 16;                    // first entry of this wave
  const bool wave_ok = e_wave < n_ent;
  const int j_first = wave_ok ? cl[e_wave] : INT_MAX;        // entries ascend
  float kb[KSTEPS];                        // dims 4s + kq of entry e_wave + l16 (zero past the list's end)
  {
    const int e = e_wave + l16;
    const bool ok = e < n_ent;
    const uint16_t* src = a.k + ((int64_t)b * a.N + (ok ? cl[e] : 0)) * stride + (int64_t)h * D + kq;
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) kb[s] = ok ? bf16_to_f32(src[4 * s]) : 0.0f;
  }
  int el_row[4], el_ent[4];
  mfma_f64_layout(l16, kq, el_row, el_ent);
  int el_j[4];                             // column id of each element's entry (INT_MAX past the end)
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int e = e_wave + el_ent[t];
    el_j[t] = e < n_ent ? cl[e] : INT_MAX;
  }
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  // the thread's elements of a step (of rows r0, r0 + 256 / D, ..), loaded while the step before is multiplied
  constexpr int PER = kPruneRows * D / 256;
  const int r0 = threadIdx.x / D, dd = threadIdx.x % D;
  const rsrc_t qb = make_rsrc(a.q + (int64_t)b * a.N * stride + (int64_t)h * D, (uint32_t)((a.N - 1) * stride + D) * 2u);
  uint16_t nx[PER];
  int nrow = -1;
  float nlse = 0.0f;
  auto fetch = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int p = t0 + r0 + x * (256 / D);
      // (N H D < 2^31: 32-bit byte offsets; 0xFFFFFFFE reads zero)
      const uint32_t off = p < p_end ? ((uint32_t)s_rows[p - p0] * (uint32_t)stride + dd) * 2u : 0xFFFFFFFEu;
      nx[x] = __builtin_amdgcn_raw_buffer_load_b16(qb, off, 0, 0);
    }
    if (threadIdx.x < kPruneRows) {
      const int p = t0 + (int)threadIdx.x;
      nrow = p < p_end ? s_rows[p - p0] : -1;
      nlse = p < p_end ? a.lse_ref[((int64_t)b * a.N + nrow) * a.H + h] : 0.0f;
    }
  };
  fetch(first);
  __syncthreads();
  for (int t0 = first; t0 < p_end; t0 += kPruneRows) {
#pragma unroll
    for (int x = 0; x < PER; ++x) w.qt[(r0 + x * (256 / D)) * QS + dd] = (double)bf16_to_f32(nx[x]);
    if (threadIdx.x < kPruneRows) {
      w.row[threadIdx.x] = nrow;
      w.lse[threadIdx.x] = (double)nlse;
    }
    fetch(t0 + kPruneRows);
    __syncthreads();
#pragma unroll
    for (int half = 0; half < kPruneRows / 16; ++half) {
      // uniform: skip 16 rows that all come before this wave's first entry
      const int last_row = w.row[min(16 * half + 15, p_end - t0 - 1)];
      if (wave_ok && last_row >= j_first) {
        f64x4 d4 = {0.0, 0.0, 0.0, 0.0};
        const double* qa = w.qt + (16 * half + l16) * QS + kq;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) d4 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[4 * s], (double)kb[s], d4, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int r = 16 * half + el_row[t];
          const int i = w.row[r];                                // -1 past the chunk's last row
          if (i >= el_j[t]) acc[t] += exp(a.sigma * d4[t] - w.lse[r]);
        }
      }
    }
    __syncthreads();
  }
  // ordered sum over the rows held by the wave's lanes: accumulators by (entry, row group), then entry-wise
#pragma unroll
  for (int t = 0; t < 4; ++t) red[wave][el_ent[t]][el_row[t]] = acc[t];
  __syncthreads();
  if (lane < 16 && wave_ok && e_wave + lane < n_ent) {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) s += red[wave][lane][r];
    part[e_wave + lane] = s;
  }
  __syncthreads();
}

// A wave owns NB blocks of 16 entries as digits in registers, a workgroup 64 NB entries; the chunk's rows are turned
// into digits 64 at a time (16 per wave) into LDS, the rows of the next 64 on their way while these are multiplied.
// Where the digits do not serve the rows and entries of the workgroup, or a log-normaliser is out of their range, the
// workgroup takes fp64 products.  At 1638 rows and 1532 entries of 16 heads x 128: 103 us by digits; by fp64 products
// after them 256 us (358 where a step's rows were loaded in place; 308 in a kernel of their own that did the same).
template <int D, int NB>
__global__ __launch_bounds__(256, 2) void prune_mass_kernel(PruneArgs a) {
  constexpr int KS = D / 64;
  constexpr size_t kDig = sizeof(uint4) * kDigStage * 4 * KS * 64;
  constexpr size_t kBuf = kDig > sizeof(PruneWide<D>) ? kDig : sizeof(PruneWide<D>);
  static_assert(sizeof(double) * 4 * 16 * 17 <= kBuf, "the fp64 path's sums reuse the buffer");
  __shared__ __attribute__((aligned(16))) char buf[kBuf];
  __shared__ int s_rows[kPruneChunk];     // the chunk's updated rows
  __shared__ int s_cnt[4];
  __shared__ DigitStat s_own[4];
  __shared__ int s_exp[kDigStage], s_ok[kDigStage];   // of each wave's rows: the unit's exponent, whether digits serve
  __shared__ double s_lse[kDigStage * 16];
  __shared__ int s_id[kDigStage * 16];
  const int h = blockIdx.y % a.H, chunk = blockIdx.y / a.H, b = blockIdx.z;
  const int n_ent = a.c_list - a.ns;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int64_t stride = (int64_t)a.H * D;
  const int32_t* cl = a.cols + ((int64_t)b * a.H + h) * a.c_list + a.ns;
  const int32_t* rp = a.rows + (int64_t)b * a.n_rows;
  const int p0 = chunk * kPruneChunk, p_end = min(a.n_rows, p0 + kPruneChunk);
  const int e_wg = blockIdx.x * kPruneEnt * NB;              // entry e_wg + 64 nb + 16 wave + l16 is the lane's
  double* part = a.part + (((int64_t)b * a.H + h) * a.n_chunks + chunk) * n_ent;
  // the chunk's rows into LDS, and the first one that can see the workgroup's first entry (rows and
  // entries ascend: the rows before it are counted with one ballot per wave)
  static_assert(kPruneChunk == 256, "one row of the chunk per thread");
  {
    const int p = p0 + (int)threadIdx.x;
    const int i = p < p_end ? rp[p] : INT_MAX;
    s_rows[threadIdx.x] = i;
    const uint64_t before = __builtin_amdgcn_ballot_w64(i < cl[e_wg]);
    if (lane == 0) s_cnt[wave] = __builtin_popcountll(before);
  }
  DigitBlock<D> own[NB];
  int j[NB], j_lo[NB], j_hi[NB];          // column of the lane's entry, and the first and last of the block
  double f_own[NB], acc[NB];
  DigitStat st_own = {};
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int e0 = e_wg + 64 * nb + 16 * wave, e = e0 + l16;
    j[nb] = e < n_ent ? cl[e] : INT_MAX;
    j_lo[nb] = e0 < n_ent ? cl[e0] : INT_MAX;
    j_hi[nb] = e0 + 15 < n_ent ? cl[e0 + 15] : INT_MAX;
    uint4 w[2 * KS];
#pragma unroll
    for (int x = 0; x < 2 * KS; ++x) w[x] = make_uint4(0, 0, 0, 0);
    if (a.digits && e < n_ent) {
      const uint16_t* src = a.k + ((int64_t)b * a.N + j[nb]) * stride + (int64_t)h * D + 16 * g;
#pragma unroll
      for (int x = 0; x < 2 * KS; ++x) w[x] = *reinterpret_cast<const uint4*>(src + 64 * (x >> 1) + 8 * (x & 1));
    }
    DigitStat st;
    own[nb] = make_digits<D>(w, st);
    f_own[nb] = __builtin_ldexp(a.sigma * 0x1.71547652b82fep+16, st.e);
    acc[nb] = 0.0;
    join_stat(st_own, st);
  }
  if (lane == 0) s_own[wave] = st_own;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) join_stat(st_own, s_own[w]);
  const int first = p0 + s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
  bool serve = a.digits;
  // the wave's rows of a stage: 16, row l16 of them the lane's
  uint4 w[2 * KS];
  int id = -1;
  float lse = 0.0f;
  auto fetch = [&](int t0) __attribute__((always_inline)) {
    const int p = t0 + 16 * wave + l16;
    id = p < p_end ? s_rows[p - p0] : -1;
    lse = id >= 0 ? a.lse_ref[((int64_t)b * a.N + id) * a.H + h] : 0.0f;
#pragma unroll
    for (int x = 0; x < 2 * KS; ++x) w[x] = make_uint4(0, 0, 0, 0);
    if (a.digits && id >= 0) {
      const uint16_t* src = a.q + ((int64_t)b * a.N + id) * stride + (int64_t)h * D + 16 * g;
#pragma unroll
      for (int x = 0; x < 2 * KS; ++x) w[x] = *reinterpret_cast<const uint4*>(src + 64 * (x >> 1) + 8 * (x & 1));
    }
  };
  uint4* dig = reinterpret_cast<uint4*>(buf);
  fetch(first);
  for (int t0 = first; serve && t0 < p_end; t0 += 16 * kDigStage) {
    {
      DigitStat st;
      const DigitBlock<D> o = make_digits<D>(w, st);
      const bool ok = digits_serve(st_own, st, (float)a.sigma) &&
                      __builtin_amdgcn_ballot_w64(!(fabsf(lse) <= 330.0f)) == 0;           // (false for NaN)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          reinterpret_cast<i32x4*>(dig)[((wave * 4 + s) * KS + ks) * 64 + lane] = o.d[s][ks];
      if (lane == 0) {
        s_exp[wave] = st.e;
        s_ok[wave] = ok;
      }
      if (lane < 16) {
        s_lse[16 * wave + lane] = (double)lse * 0x1.71547652b82fep+0;
        s_id[16 * wave + lane] = id;
      }
    }
    fetch(t0 + 16 * kDigStage);            // (past the last row: nothing is loaded)
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kDigStage; ++x) serve = serve && s_ok[x];
    const int row_lo = s_id[0], row_hi = s_rows[min(t0 + 16 * kDigStage, p_end) - 1 - p0];
    if (serve && row_hi >= j_lo[0]) {      // uniform in the wave
      auto add = [&](const DigitSums& o, int x, int nb, auto edge) __attribute__((always_inline)) {
        const double f = __builtin_ldexp(f_own[nb], s_exp[x]);
        double e[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int r = 16 * x + 4 * g + t;
          double z = fma(digit_dot(o, t), f, -s_lse[r]);
          if (edge.value) z = s_id[r] >= j[nb] ? z : -1000.0;
          e[t] = exp2_f64(z);
        }
        acc[nb] += (e[0] + e[1]) + (e[2] + e[3]);
      };
      if (row_lo >= j_hi[NB - 1] && t0 + 16 * kDigStage <= p_end)
        digit_stage<D, NB>(dig, own, [&](const DigitSums& o, int x, int nb) __attribute__((always_inline)) { add(o, x, nb, std::false_type{}); });
      else
        digit_stage<D, NB>(dig, own, [&](const DigitSums& o, int x, int nb) __attribute__((always_inline)) { add(o, x, nb, std::true_type{}); });
    }
    __syncthreads();
  }
  if (!serve) {                            // the same in every wave
    for (int nb = 0; nb < NB; ++nb)
      if (e_wg + 64 * nb < n_ent)
        prune_wide<D>(a, b, h, e_wg + 64 * nb, s_rows, p0, first, p_end, part, *reinterpret_cast<PruneWide<D>*>(buf),
                      reinterpret_cast<double (*)[16][17]>(buf));
    return;
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    double s = acc[nb];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    const int e = e_wg + 64 * nb + 16 * wave + lane;
    if (lane < 16 && e < n_ent) part[e] = s;
  }
}

// key[b, h, e] = fp32 of the chunks' partial sums of entry e, added in chunk order
__global__ __launch_bounds__(256) void prune_sum_kernel(const double* __restrict__ part, int n_chunks, int n_ent,
                                                        int64_t n_seg, float* __restrict__ key) {
  const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (x >= n_seg * n_ent) return;
  const int64_t seg = x / n_ent, e = x % n_ent;
  double s = 0.0;
  for (int c = 0; c < n_chunks; ++c) s += part[(seg * n_chunks + c) * n_ent + e];
  key[x] = (float)s;
}

}  // namespace fl

using namespace fl;

// Workspace of the dense statistic: the rows' log-normalisers and digits of n_seg (batch, head) pairs at a time.
// The digits take 4 bytes per element of q and of k, so the pairs go in groups of about 256 MB (a 32K prompt of 16
// heads x 128 in two groups of 8).
namespace {
struct CsWs {
  int n_seg;
  size_t dig, exps, stat, total;
};
constexpr size_t kCsGroupBytes = (size_t)256 << 20;
constexpr size_t kCsGroupPairs = 65528;   // a grid's y extent, and a multiple of 8

CsWs cs_ws(int B, int N, int H, int d) {
  const size_t nblk = ((size_t)N + 15) / 16;
  const size_t pair = 2 * nblk * 16 * (size_t)d * 4;
  const size_t all = (size_t)B * H;
  size_t n = kCsGroupBytes / pair;
  n = n < 1 ? 1 : n > kCsGroupPairs ? kCsGroupPairs : n;
  const size_t most = n;
  n = n > all ? all : n;
  const size_t groups = (all + n - 1) / n;
  n = (all + groups - 1) / groups;
  if (n > 8 && n < all) n = (n + 7) / 8 * 8 <= most ? (n + 7) / 8 * 8 : n / 8 * 8;
  CsWs w;
  w.n_seg = (int)n;
  size_t off = n * nblk * 16 * sizeof(double);          // lse [n_seg, 16 nblk]
  w.dig = off; off += n * pair;
  w.exps = off; off += 2 * n * ((nblk + 3) / 4 * 4) * sizeof(int);
  w.stat = off; off += 2 * n * nblk * sizeof(DigitStat);
  w.total = off;
  return w;
}

template <int D, int NB>
int launch_colscore(const CsArgs& a, hipStream_t st) {
  const int n_wg = (a.nblk + 4 * NB - 1) / (4 * NB);
  const unsigned grid = (unsigned)n_wg * (unsigned)a.n_seg;
  colscore_kernel<D, NB, true><<<grid, 256, 0, st>>>(a, n_wg);
  int rc = check_launch("colscore_kernel(rows)");
  if (rc != FL_OK) return rc;
  colscore_kernel<D, NB, false><<<grid, 256, 0, st>>>(a, n_wg);
  return check_launch("colscore_kernel(columns)");
}
}  // namespace

// The head dimension is not an argument, so the larger of the two layouts: where the pairs take more than one group,
// 64-wide heads put up to twice as many into each, with their normalisers, exponents and figures.
extern "C" size_t fl_column_scores_ws(int B, int N, int H) {
  if (B < 1 || N < 1 || H < 1) return 0;
  const size_t rows = (size_t)B * (size_t)H * (size_t)N * sizeof(double);
  return std::max(rows, std::max(cs_ws(B, N, H, 64).total, cs_ws(B, N, H, 128).total));
}

extern "C" int fl_column_scores(const uint16_t* q, const uint16_t* k_cache, int B, int N, int H, int d,
                                float* col_key, void* ws, size_t ws_bytes, void* stream) {
  FL_API_BEGIN
  FL_REQUIRE(q && k_cache && col_key, FL_E_NULL, "fl_column_scores: q, k_cache and col_key are required");
  FL_REQUIRE(B >= 1 && N >= 1 && H >= 1, FL_E_SHAPE, "fl_column_scores: need B, N, H >= 1");
  FL_REQUIRE(d == 64 || d == 128, FL_E_SHAPE, "fl_column_scores: head dim %d not in {64, 128}", d);
  FL_REQUIRE((int64_t)N * H * d < ((int64_t)1 << 31), FL_E_SHAPE, "fl_column_scores: N * H * d too large");
  // (the rows' log-normalisers alone are the least a call can work with)
  const size_t least = (size_t)B * (size_t)H * (size_t)N * sizeof(double);
  FL_REQUIRE(ws && ws_bytes >= least, FL_E_WORKSPACE, "fl_column_scores: workspace of %zu bytes required", least);
  hipStream_t st = as_stream(stream);
  CsArgs a{};
  a.q = q; a.k = k_cache; a.N = N; a.H = H; a.nblk = (N + 15) / 16;
  a.sigma = 1.0 / std::sqrt((double)d);
  a.col_key = col_key;
  a.lse = static_cast<double*>(ws);
  const CsWs w = cs_ws(B, N, H, d);
  // The digits: with the workspace that fl_column_scores_ws asks for, 16-byte aligned queries and keys, and digits of
  // one pair within a buffer descriptor's 2 GiB; otherwise every pair takes the fp64 products.
  const bool aligned = ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_cache) | reinterpret_cast<uintptr_t>(ws)) & 15) == 0;
  const bool digits = aligned && ws_bytes >= w.total && (int64_t)a.nblk * 64 * d < ((int64_t)1 << 31);
  const int all = B * H;
  int step = std::min<int>(all, kCsGroupPairs);
  a.lse_stride = N;
  if (digits) {
    char* base = static_cast<char*>(ws);
    a.dig = reinterpret_cast<uint4*>(base + w.dig);
    a.exps = reinterpret_cast<int*>(base + w.exps);
    a.stat = reinterpret_cast<DigitStat*>(base + w.stat);
    a.lse_stride = (int64_t)a.nblk * 16;
    step = w.n_seg;
  }
  for (int s0 = 0; s0 < all; s0 += step) {
    a.seg0 = s0;
    a.n_seg = std::min(step, all - s0);
    if (digits) {
      const dim3 grid((a.nblk + 3) / 4, a.n_seg, 2);
      if (d == 128) cs_digits_kernel<128><<<grid, 256, 0, st>>>(a);
      else cs_digits_kernel<64><<<grid, 256, 0, st>>>(a);
      int rc = check_launch("cs_digits_kernel");
      if (rc != FL_OK) return rc;
    }
    // Two blocks per wave, one from either end, make workgroups of equal length, two per CU, in rounds of 512; one block,
    // the longest first, three per CU.  Two where their last round is at least three quarters full (or one of many).
    // Two against one, 128-wide heads: N = 4096 x 16 (512 workgroups of two) 0.426 ms against 0.435, 8192 x 4 (512)
    // 0.473 against 0.531, 8192 x 16 (1024) 1.451 against 1.471; 6000 x 16 (752) 0.838 against 0.812, 3000 x 16 (384)
    // 0.311 against 0.281.
    const int64_t pairs = (int64_t)((a.nblk + 7) / 8) * a.n_seg;
    const bool wide = pairs >= 1536 || (pairs >= 512 && 4 * pairs >= 3 * 512 * ((pairs + 511) / 512));
    int rc;
    if (d == 128) rc = wide ? launch_colscore<128, 2>(a, st) : launch_colscore<128, 1>(a, st);
    else rc = wide ? launch_colscore<64, 2>(a, st) : launch_colscore<64, 1>(a, st);
    if (rc != FL_OK) return rc;
  }
  return FL_OK;
  FL_API_END
}

extern "C" size_t fl_prune_columns_ws(int B, int H, int k, int c_list, int n_sink) {
  if (B < 1 || H < 1 || k < 0 || c_list < 1 || n_sink < 0) return 0;
  const int n_ent = c_list - std::min(n_sink, c_list);
  const int n_chunks = std::max(1, (k + kPruneChunk - 1) / kPruneChunk);
  return (size_t)B * H * n_chunks * n_ent * sizeof(double);
}

extern "C" int fl_prune_columns(const uint16_t* q, const uint16_t* k_cache, const int32_t* rows, int k,
                                const int32_t* cols, int c_list, const float* lse_ref, int B, int N, int H,
                                int d, double sm_scale, int n_sink, int t_next, float* col_key,
                                int32_t* cols_next, void* ws, size_t ws_bytes, void* stream) {
  FL_API_BEGIN
  FL_REQUIRE(q && k_cache && cols && lse_ref && cols_next, FL_E_NULL,
             "fl_prune_columns: q, k_cache, cols, lse_ref and cols_next are required");
  FL_REQUIRE(B >= 1 && N >= 1 && H >= 1, FL_E_SHAPE, "fl_prune_columns: need B, N, H >= 1");
  FL_REQUIRE(d == 64 || d == 128, FL_E_SHAPE, "fl_prune_columns: head dim %d not in {64, 128}", d);
  FL_REQUIRE((int64_t)N * H * d < ((int64_t)1 << 31), FL_E_SHAPE, "fl_prune_columns: N * H * d too large");
  FL_REQUIRE(k >= 0 && k <= N, FL_E_RANGE, "fl_prune_columns: k=%d outside [0, N]", k);
  FL_REQUIRE(k == 0 || rows, FL_E_NULL, "fl_prune_columns: rows are required when k > 0");
  FL_REQUIRE(c_list >= 1 && c_list <= N, FL_E_RANGE, "fl_prune_columns: c_list=%d outside [1, N]", c_list);
  FL_REQUIRE(n_sink >= 0, FL_E_RANGE, "fl_prune_columns: n_sink must be >= 0");
  const int ns = std::min(n_sink, c_list);
  const int n_ent = c_list - ns;
  FL_REQUIRE(t_next >= 0 && t_next <= n_ent, FL_E_RANGE, "fl_prune_columns: t_next=%d outside [0, %d]", t_next,
             n_ent);
  FL_REQUIRE(n_ent <= 65536, FL_E_SHAPE, "fl_prune_columns: %d list entries after the sinks exceed 65536", n_ent);
  FL_REQUIRE(n_ent == 0 || col_key, FL_E_NULL, "fl_prune_columns: col_key is required when entries follow the sinks");
  FL_REQUIRE(sm_scale > 0.0 && std::isfinite(sm_scale), FL_E_RANGE, "fl_prune_columns: sm_scale must be > 0");
  const size_t need = fl_prune_columns_ws(B, H, k, c_list, n_sink);
  FL_REQUIRE(need == 0 || (ws && ws_bytes >= need), FL_E_WORKSPACE,
             "fl_prune_columns: workspace of %zu bytes required", need);
  hipStream_t st = as_stream(stream);
  FL_CHECK_LIST("fl_prune_columns", "rows", rows, B, k, 0, N, st);
  FL_CHECK_LIST("fl_prune_columns", "cols", cols, (int64_t)B * H, c_list, 0, N, st);
  if (n_ent == 0) {                       // the list is all sinks: it is kept as it is
    if (hipMemcpyAsync(cols_next, cols, (size_t)B * H * ns * sizeof(int32_t), hipMemcpyDeviceToDevice, st) !=
        hipSuccess)
      return set_error(FL_E_HIP, "fl_prune_columns: copy of the sinks failed");
    return FL_OK;
  }
  const int n_chunks = std::max(1, (k + kPruneChunk - 1) / kPruneChunk);
  FL_REQUIRE((int64_t)H * n_chunks <= 65535, FL_E_SHAPE, "fl_prune_columns: H * ceil(k / %d) above 65535",
             kPruneChunk);
  double* part = static_cast<double*>(ws);
  const bool digits = ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_cache)) & 15) == 0;
  const PruneArgs a{q, k_cache, rows, k, cols, c_list, ns, lse_ref, N, H, sm_scale, n_chunks, part, digits};
  // two blocks of entries per wave halve the conversions of the rows; one where that leaves less than two workgroups
  // per CU
  const int64_t wide = (int64_t)((n_ent + 2 * kPruneEnt - 1) / (2 * kPruneEnt)) * H * n_chunks * B;
  const int nb = wide >= 512 ? 2 : 1;
  const dim3 grid((n_ent + nb * kPruneEnt - 1) / (nb * kPruneEnt), H * n_chunks, B);
  if (d == 128) {
    if (nb == 2) prune_mass_kernel<128, 2><<<grid, 256, 0, st>>>(a);
    else prune_mass_kernel<128, 1><<<grid, 256, 0, st>>>(a);
  } else {
    if (nb == 2) prune_mass_kernel<64, 2><<<grid, 256, 0, st>>>(a);
    else prune_mass_kernel<64, 1><<<grid, 256, 0, st>>>(a);
  }
  int rc = check_launch("prune_mass_kernel");
  if (rc != FL_OK) return rc;
  const int64_t total = (int64_t)B * H * n_ent;
  prune_sum_kernel<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(part, n_chunks, n_ent, (int64_t)B * H, col_key);
  rc = check_launch("prune_sum_kernel");
  if (rc != FL_OK) return rc;
  return launch_topk(B * H, col_key, n_ent, n_ent, t_next, cols + ns, c_list, 0, cols_next, ns + t_next, ns,
                     nullptr, 0, st);
  FL_API_END
}
