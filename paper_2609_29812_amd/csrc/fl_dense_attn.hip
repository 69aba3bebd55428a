// The dense source loop (Eq. 2, causal): o_i = softmax(sigma q_i K^T) V over j <= i for every row, and lse_i.
//
// A workgroup of 4 waves takes 128 / SPLIT consecutive rows of one (batch, head), 32 per wave; with SPLIT = 2 the two
// waves of a 32-row group take the halves of a stage and merge their states at the end.  Stages of
// 64 columns go through two LDS buffers, the next one's K by LDS-DMA and its V through registers
// (converted to fp16 on the way, exact for |v| in [2^-14, 65504]) while this one is multiplied: one barrier a stage.
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, K rows as the A operand, so a lane holds 16 columns of one row per block;
//   O^T += V^T P^T  v_mfma_f32_32x32x16_f16, V read transposed (ds_read_b64_tr_b16), P rounded to fp16.
// The softmax reference moves only when a score exceeds it by more than 8 (log2 units).
//
// Bound by the vector ALU beside the matrix cores: per 32 rows x 64 columns at d = 128, 32 products (1024 matrix cycles)
// against about 170 vector instructions and 32 exponentials (1200 cycles), overlapped by two waves per SIMD of
// independent workgroups; at N = 16384, 16 heads the clock falls to 1.6 GHz, the matrix cores are busy 50 % of its cycles.
// 16 heads x 128: N = 16384 1.41 -> 1.15 ms (955 TFLOP/s), N = 4096 158 -> 103 us; 3 x 1009 rows of 8 heads x 64
// 25 -> 14 us, against 32-column stages of a four-slot ring with tables and an LDS conversion of V each step.
#include "fl_attn_util.h"

#include <algorithm>
#include <type_traits>

namespace fl {

struct DenseArgs {
  const uint16_t *q, *k, *v;
  float *lse, *o;
  int B, N, H;
  float scale_log2;          // sm_scale * log2(e)
  float pinf;                // +inf
};

template <int D, int COLS>
struct __attribute__((aligned(16))) DenseSlot {
  uint16_t k[COLS * D];      // blocks of 32 rows, 16-byte chunks permuted (swz32_f)
  uint16_t v[COLS * D];      // the same layout, fp16
};

template <int D, int SPLIT>
__global__ __launch_bounds__(256, 2) void dense_attn_kernel(DenseArgs a) {
  constexpr int GROUPS = 4 / SPLIT;       // 32-row groups of the workgroup
  constexpr int BM = 32 * GROUPS;
  constexpr int COLS = 64;
  constexpr int NBK = COLS / 32 / SPLIT;  // 32-column blocks of a wave per stage
  constexpr int KS = D / 16;              // k-steps of QK^T
  constexpr int DB = D / 32;              // 32-dim output blocks
  constexpr int CH = D / 8;               // 16-byte chunks per row
  constexpr int RPI = 64 / CH;            // rows of one 1 KB load instruction
  constexpr int NI = COLS / RPI / 4;      // load instructions per wave, tensor and stage
  __shared__ DenseSlot<D, COLS> s0, s1;
  __shared__ float s_ml[2][4][64];        // the merge: references and sums by wave

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hw = lane >> 5, r32 = lane & 31;
  const int group = wave / SPLIT, phase = wave % SPLIT;
  // the row tiles of one (batch, head) on one XCD, the longest first
  const int n_rt = (a.N + BM - 1) / BM;
  const int n_bh = a.B * a.H;
  int bh, rt;
  if ((n_bh & 7) == 0) {
    const int g = blockIdx.x & 7, s = blockIdx.x >> 3, per = n_bh >> 3;
    bh = g + 8 * (s % per);
    rt = n_rt - 1 - s / per;
  } else {
    bh = blockIdx.x % n_bh;
    rt = n_rt - 1 - blockIdx.x / n_bh;
  }
  const int b = bh / a.H, h = bh % a.H;
  const int64_t HD = (int64_t)a.H * D;
  const int p0 = rt * BM;
  const int last = min(p0 + BM, a.N) - 1;              // last row of the workgroup
  const int gmin = p0 + 32 * group;                    // first row of the wave's group
  const int gmax = min(gmin + 31, last);               // (below gmin: no rows)
  const int row = gmin + r32;
  const bool row_ok = row <= gmax;
  bf16x8 qf[KS];
  {
    const uint16_t* src = a.q + ((int64_t)b * a.N + (row_ok ? row : 0)) * HD + (int64_t)h * D + hw * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 w = row_ok ? *reinterpret_cast<const uint4*>(src + ks * 16) : make_uint4(0, 0, 0, 0);
      qf[ks] = __builtin_bit_cast(bf16x8, w);
    }
  }
  // loads: instruction x of the wave covers rows (wave NI + x) RPI .. of the stage; rows past N read zeros
  const uint32_t rb = (uint32_t)(HD * 2);
  const rsrc_t kR = make_rsrc(a.k + (int64_t)b * a.N * HD, (uint32_t)a.N * rb);
  const rsrc_t vR = make_rsrc(a.v + (int64_t)b * a.N * HD, (uint32_t)a.N * rb);
  uint32_t ofs[NI];
#pragma unroll
  for (int x = 0; x < NI; ++x) {
    const int c = (wave * NI + x) * RPI + lane / CH;
    ofs[x] = (uint32_t)c * rb + (uint32_t)(h * D * 2) + (uint32_t)((lane % CH) ^ swz32_f<D>(c & 31)) * 16u;
  }
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  v4u vw[NI];
  auto fetch = [&](DenseSlot<D, COLS>& sl, int c0) __attribute__((always_inline)) {
    const uint32_t at = (uint32_t)c0 * rb;
#pragma unroll
    for (int x = 0; x < NI; ++x) {
      const uint32_t off = ofs[x] + at;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kR, FL_LDS(sl.k + (wave * NI + x) * 512), 16, off, 0, 0, 0);
    }
#pragma unroll
    for (int x = 0; x < NI; ++x) vw[x] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(vR, ofs[x] + at, 0, 0));
  };
  auto store_v = [&](DenseSlot<D, COLS>& sl) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < NI; ++x) {
      u32x4 hv;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        hv[e] = pack_f16x2(__uint_as_float(vw[x][e] << 16), __uint_as_float(vw[x][e] & 0xFFFF0000u));
      *reinterpret_cast<u32x4*>(sl.v + (wave * NI + x) * 512 + lane * 8) = hv;
    }
  };
  // LDS read offsets (elements).  K (A operand): row r32, data chunk 2 ks + hw.  V (transposed reads): lane
  // (16 g + 4 t + q) points at V[col][dim0 + 4 q] of column 16 kb + 4 (g >> 1) + t (and the same + 8), dims
  // 32 db + 16 (g & 1) + 4 q, so the transpose hands lane m of the group V[col_t][dim0 + m].
  int koff[KS], voff[DB], voff8[DB];
  {
    const int g16 = lane >> 4, m16 = lane & 15;
    const int tq = m16 >> 2, q = m16 & 3;
    const int col0 = 4 * (g16 >> 1) + tq;
    const int c_lo = 2 * (g16 & 1) + (q >> 1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) koff[ks] = r32 * D + ((2 * ks + hw) ^ swz32_f<D>(r32)) * 8;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      voff[db] = col0 * D + ((4 * db + c_lo) ^ swz32_f<D>(col0)) * 8 + 4 * (q & 1);
      voff8[db] = (col0 + 8) * D + ((4 * db + c_lo) ^ swz32_f<D>(col0 + 8)) * 8 + 4 * (q & 1);
    }
  }
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
  float ref = -INFINITY, lsum = 0.0f;     // softmax reference (log2 units) and the lane's part of the row sum

  auto compute = [&](const DenseSlot<D, COLS>& sl, int c0) __attribute__((always_inline)) {
    const int first = c0 + 32 * NBK * phase;              // the wave's columns first .. first + 32 NBK - 1
    if (first > gmax) return;                             // uniform
    f32x16 s[NBK];
#pragma unroll
    for (int x = 0; x < NBK; ++x) s[x] = f32x16{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int x = 0; x < NBK; ++x) {
        const u32x4 kw = *reinterpret_cast<const u32x4*>(&sl.k[(NBK * phase + x) * 32 * D + koff[ks]]);
        s[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kw), qf[ks], s[x], 0, 0, 0);
      }
    if (first + 32 * NBK - 1 > gmin) {                    // uniform: some column is beyond some row
#pragma unroll
      for (int x = 0; x < NBK; ++x)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int c = first + 32 * x + 8 * (v >> 2) + 4 * hw + (v & 3);
          s[x][v] = c <= row ? s[x][v] : -INFINITY;
        }
    }
    float mx[4] = {s[0][0], s[0][1], s[0][2], s[0][3]};
#pragma unroll
    for (int x = 0; x < NBK; ++x)
#pragma unroll
      for (int v = x == 0 ? 4 : 0; v < 16; ++v) mx[v & 3] = fmax_nn(mx[v & 3], s[x][v], a.pinf);
    float tmax = fmax_nn(fmax_nn(mx[0], mx[1], a.pinf), fmax_nn(mx[2], mx[3], a.pinf), a.pinf);
    tmax = xor32_max(tmax) * a.scale_log2;
    const bool raise = tmax > ref + 8.0f;                 // false while both are -inf
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {        // uniform: rescale the rows that need it
      const float nm = raise ? tmax : ref;
      const float alpha = raise ? __builtin_amdgcn_exp2f(ref - nm) : 1.0f;     // exp2(-inf) = 0
      lsum *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] *= alpha;
      ref = nm;
    }
    const float sub = ref == -INFINITY ? 0.0f : ref;
    float ts[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int x = 0; x < NBK; ++x) {
      float pr[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        pr[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[x][v], a.scale_log2, -sub));
        ts[v & 3] += pr[v];
      }
      // A block that no row of the group sees: its probabilities are 0, but 0 times a value that is not finite in fp16
      // would be NaN.  (Leaving out its scores too, in a form of its own, took 1309 us against 1156 at N = 16384: spills.)
      if (x > 0 && first + 32 * x > gmax) break;          // uniform
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const u32x4 pw = {pack_f16x2(pr[8 * kb + 0], pr[8 * kb + 1]), pack_f16x2(pr[8 * kb + 2], pr[8 * kb + 3]),
                          pack_f16x2(pr[8 * kb + 4], pr[8 * kb + 5]), pack_f16x2(pr[8 * kb + 6], pr[8 * kb + 7])};
        const f16x8 pf = __builtin_bit_cast(f16x8, pw);
        const uint16_t* vt = sl.v + (NBK * phase + x) * 32 * D + 16 * kb * D;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const i16x4 va = __builtin_amdgcn_ds_read_tr16_b64_v4i16(FL_LDS4(vt + voff[db]));
          const i16x4 vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16(FL_LDS4(vt + voff8[db]));
          const i16x8 v8 = __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7);
          acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, v8), pf, acc[db], 0, 0, 0);
        }
      }
    }
    lsum += (ts[0] + ts[1]) + (ts[2] + ts[3]);
  };

  fetch(s0, 0);
  store_v(s0);
  FL_WAIT_VM(0);
  lds_barrier();
  auto step = [&](DenseSlot<D, COLS>& cur, DenseSlot<D, COLS>& nxt, int c0) __attribute__((always_inline)) {
    const bool more = c0 + COLS <= last;                  // uniform
    if (more) fetch(nxt, c0 + COLS);
    compute(cur, c0);
    if (more) store_v(nxt);
    FL_WAIT_VM(0);
    lds_barrier();
  };
  for (int c0 = 0; c0 <= last; c0 += 2 * COLS) {
    step(s0, s1, c0);
    if (c0 + COLS <= last) step(s1, s0, c0 + COLS);
  }
  lsum = xor32_add(lsum);                                 // the half-waves hold disjoint columns of a row
  if constexpr (SPLIT > 1) {
    // the phases' states of a group meet in its first wave, through the idle buffers (phase - 1 + group (SPLIT - 1):
    // 32 D floats each)
    float4* x0 = reinterpret_cast<float4*>(&s0);
    constexpr int PER = 32 * D / 4;                       // float4 of a state
    static_assert((4 - GROUPS) * PER * 16 <= sizeof(DenseSlot<D, COLS>), "the states of the other phases fit a buffer");
    s_ml[0][wave][lane] = ref;
    s_ml[1][wave][lane] = lsum;
    if (phase > 0) {
      float4* dst = x0 + (group * (SPLIT - 1) + phase - 1) * PER + lane;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          dst[(db * 4 + j) * 64] = make_float4(acc[db][4 * j], acc[db][4 * j + 1], acc[db][4 * j + 2], acc[db][4 * j + 3]);
    }
    lds_barrier();
    if (phase > 0) return;
    float m = ref;
#pragma unroll
    for (int x = 1; x < SPLIT; ++x) m = fmaxf(m, s_ml[0][wave + x][lane]);
    const float f0 = ref == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ref - m);
    lsum *= f0;
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] *= f0;
#pragma unroll
    for (int x = 1; x < SPLIT; ++x) {
      const float rx = s_ml[0][wave + x][lane];
      const float f = rx == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(rx - m);
      lsum = fmaf(f, s_ml[1][wave + x][lane], lsum);
      const float4* src = x0 + (group * (SPLIT - 1) + x - 1) * PER + lane;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 w = src[(db * 4 + j) * 64];
          acc[db][4 * j] = fmaf(f, w.x, acc[db][4 * j]);
          acc[db][4 * j + 1] = fmaf(f, w.y, acc[db][4 * j + 1]);
          acc[db][4 * j + 2] = fmaf(f, w.z, acc[db][4 * j + 2]);
          acc[db][4 * j + 3] = fmaf(f, w.w, acc[db][4 * j + 3]);
        }
    }
    ref = m;
  }
  if (!row_ok || !(lsum > 0.0f)) return;   // (column 0 is always causal)
  const float inv = 1.0f / lsum;
  float* out = a.o + ((int64_t)b * a.N + row) * HD + (int64_t)h * D + 4 * hw;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<float4*>(out + db * 32 + 8 * j) = make_float4(acc[db][4 * j] * inv, acc[db][4 * j + 1] * inv,
                                                                      acc[db][4 * j + 2] * inv, acc[db][4 * j + 3] * inv);
  if (hw == 0) a.lse[((int64_t)b * a.N + row) * a.H + h] = (ref + log2f(lsum)) * 0.6931471805599453f;
}

template <int SPLIT>
static void launch_split(const DenseArgs& a, int d, hipStream_t st) {
  const int bm = 128 / SPLIT;
  const unsigned grid = (unsigned)((a.N + bm - 1) / bm) * (unsigned)(a.B * a.H);
  if (d == 128) dense_attn_kernel<128, SPLIT><<<grid, 256, 0, st>>>(a);
  else dense_attn_kernel<64, SPLIT><<<grid, 256, 0, st>>>(a);
}

int launch_dense(const uint16_t* q, const uint16_t* k, const uint16_t* v, int B, int N, int H, int d, float sm_scale,
                 float* lse, float* o, hipStream_t st) {
  DenseArgs a{q, k, v, lse, o, B, N, H, sm_scale * 1.4426950408889634f, INFINITY};
  const int64_t wgs = (int64_t)((N + 127) / 128) * B * H;
  // 128 rows per workgroup where that fills the chip (two workgroups per CU at d = 128, four at d = 64), else 64 rows and
  // split columns, which halves a workgroup's chain of stages.  128 rows against 64, 16 heads x 128: N = 16384
  // 1.16 ms against 1.42, N = 4096 (512 workgroups) 103 us against 106, N = 3000 77 against 62; 64-wide heads:
  // N = 16384 x 16 0.66 ms against 0.76, N = 8192 x 16 (1024 workgroups) 193 us against 194, N = 16384 x 4 267 against 213
  if (wgs >= (d == 128 ? 512 : 1024)) launch_split<1>(a, d, st);
  else launch_split<2>(a, d, st);
  return check_launch("dense_attn_kernel");
}

}  // namespace fl
