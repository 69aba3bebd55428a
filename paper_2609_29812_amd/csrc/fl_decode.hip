// Decode step of one loop for the newest position (Appendix D.2, Eqs. (6) and (7) for one query row).
//
// For each (batch, head) the query of position t = T-1 attends over the column set S that the previous
// loop selected (or over every column 0..T-1 for a dense source loop), with the cached mass m:
//   p_j = m * exp(l_j - L), l_j = sm_scale * q . K_j, L = logsumexp over S,
//   o <- o - sub + sum_j p_j V_j          (dense: o = sum_j p_j V_j, m = 1),
// then selects the next loop's S' (sinks and window forced, then the largest p, ties to the lower
// column) and forms its mass m' = sum_{S'} p_j and subtract term sub' = sum_{S'} p_j V_j.  Within a row
// p_j grows with l_j, so the ranking key is fp32(l_j), available before L is known.
//
// One row per (b, h) is a GEMV: HBM-bound, split over columns.  Two launches, or three:
//   decode_partial   chunks of 128 positions: fp64 logits (exact bf16 products, fp64 sums) and their fp32
//                    ranking keys (forced columns +inf), the chunk's max and exp-sum, and the
//                    exp-weighted sum of its V rows (fp32); K and V rows are each read once, 16 bytes per
//                    lane, D/8 lanes per row.
//   decode_finalize  per (b, h), one workgroup merges the chunks into L and the output, and others form the next
//                    loop's columns, mass and subtract term by the radix top-k of fl_topk.h over the keys and a
//                    gather of the selected V rows (read once more); nothing to select when every column is kept.
//   decode_sum       adds the sums of several selecting workgroups.
#include "fl_common.h"
#include "fl_topk.h"

#include <mutex>

namespace fl {

constexpr int kDecChunk = 128;           // positions per partial workgroup
constexpr int kSelWin = 1024;            // selected positions gathered per round of the finalize

// 16-byte load marked non-temporal: the K and V rows of a step are streamed once
typedef uint32_t u32x4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream16(const uint16_t* p) {
  const u32x4d w = __builtin_nontemporal_load(reinterpret_cast<const u32x4d*>(p));
  return make_uint4(w[0], w[1], w[2], w[3]);
}

struct DecodeArgs {
  const uint16_t* q;         // [B, H, D]
  const uint16_t* k;         // [B, T, H, D]
  const uint16_t* v;
  const int32_t* cols;       // [B, H, c] or NULL (dense)
  const float* mass;         // [B, H]
  const float* sub;          // [B, H, D]
  float* o;                  // [B, H, D]
  float* lse;                // [B, H] optional
  double* logit;             // ws [B*H, n]
  double* pmax;              // ws [B*H, nch] chunk max
  double* psum;              // ws [B*H, nch] chunk exp-sum
  float* pacc;               // ws [B*H, nch, D]
  float* key;                // ws [B*H, n]
  const int32_t* sel;        // ws [B*H, c_next] selected positions (one selecting workgroup per (b, h)), or
  double* part_mass;         //    [B*H, n_sel] and
  float* part_sub;           //    [B*H, n_sel, D] sums of the shares (more than one)
  int32_t* cols_next;        // [B, H, c_next]
  float* mass_next;          // [B, H]
  float* sub_next;           // [B, H, D]
  int B, T, H, n, nch, c_next, n_sink, window;
  double scale;
};

__device__ __forceinline__ int dec_col(const DecodeArgs& a, int bh, int p) {
  return a.cols ? a.cols[(int64_t)bh * a.n + p] : p;
}

__device__ __forceinline__ double wave_max_f64(double x) {
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off, 64));
  return x;
}
__device__ __forceinline__ double wave_sum_f64_dec(double x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// ---- partial: one chunk of positions of one (b, h) -------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void decode_partial_kernel(DecodeArgs a) {
  constexpr int LPC = D / 8;                 // lanes per row (16 bytes each)
  constexpr int CPW = 64 / LPC;              // rows per wave instruction
  constexpr int PER_WAVE = kDecChunk / 4;    // positions per wave
  constexpr int IT = PER_WAVE / CPW;
  __shared__ double s_red[4];
  __shared__ float s_acc[4][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sl = lane % LPC, grp = lane / LPC;
  const int chunk = blockIdx.x, bh = blockIdx.y;
  const int b = bh / a.H, h = bh % a.H;
  const int64_t HD = (int64_t)a.H * D;
  double qd[8];
  {
    const uint4 w = *reinterpret_cast<const uint4*>(a.q + (int64_t)bh * D + 8 * sl);
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      qd[2 * t] = (double)bf16_to_f32(ws[t] & 0xFFFFu);
      qd[2 * t + 1] = (double)bf16_to_f32(ws[t] >> 16);
    }
  }
  // pass 1: logits (every lane of a row group ends with the row's full dot product).  All column ids,
  // then all K and V loads, are issued before any use, so a chunk costs two load latencies.
  double lg[IT];
  int colv[IT];
  uint4 kw[IT], vw[IT];
  double mx = -INFINITY;
  const int p0 = chunk * kDecChunk + wave * PER_WAVE + grp;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int p = p0 + it * CPW;
    colv[it] = p < a.n ? dec_col(a, bh, p) : 0;
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t off = ((int64_t)b * a.T + colv[it]) * HD + (int64_t)h * D + 8 * sl;
    kw[it] = stream16(a.k + off);
    vw[it] = stream16(a.v + off);
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int p = p0 + it * CPW;
    const bool ok = p < a.n;
    const int col = colv[it];
    const uint4 w = kw[it];
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      acc = fma((double)bf16_to_f32(ws[t] & 0xFFFFu), qd[2 * t], acc);
      acc = fma((double)bf16_to_f32(ws[t] >> 16), qd[2 * t + 1], acc);
    }
#pragma unroll
    for (int off = 1; off < LPC; off <<= 1) acc += __shfl_xor(acc, off, 64);
    const double l = ok ? a.scale * acc : -INFINITY;
    lg[it] = l;
    mx = fmax(mx, l);
    if (ok && sl == 0) {
      a.logit[(int64_t)bh * a.n + p] = l;
      if (a.c_next > 0) {
        const bool forced = col < a.n_sink || (a.window > 0 && col >= a.T - a.window);
        a.key[(int64_t)bh * a.n + p] = forced ? INFINITY : (float)l;
      }
    }
  }
  mx = wave_max_f64(mx);
  if (lane == 0) s_red[wave] = mx;
  __syncthreads();
  mx = fmax(fmax(s_red[0], s_red[1]), fmax(s_red[2], s_red[3]));
  __syncthreads();
  // pass 2: exp-weights against the chunk max, exp-sum and the weighted V rows
  // (every lane of a row group holds the same logits: lane sl of the group takes the exponential of the
  // group's position sl and the group shares them by shuffles, one fp64 exp per lane instead of IT)
  static_assert(IT <= LPC, "one position per lane of a row group");
  double mine = 0.0;
#pragma unroll
  for (int it = 0; it < IT; ++it) mine = sl % IT == it ? lg[it] : mine;
  mine = exp(mine - mx);                        // 0 for positions past the end
  double es = 0.0;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const double e = __shfl(mine, grp * LPC + it, 64);
    if (sl == 0) es += e;
    const float wf = (float)e;
    const uint4 w = vw[it];
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      acc[2 * t] = fmaf(wf, bf16_to_f32(ws[t] & 0xFFFFu), acc[2 * t]);
      acc[2 * t + 1] = fmaf(wf, bf16_to_f32(ws[t] >> 16), acc[2 * t + 1]);
    }
  }
  es = wave_sum_f64_dec(es);
  // rows of a wave -> lanes 0..LPC-1, then the four waves through LDS
#pragma unroll
  for (int t = 0; t < 8; ++t)
    for (int off = LPC; off < 64; off <<= 1) acc[t] += __shfl_xor(acc[t], off, 64);
  if (lane < LPC) {
#pragma unroll
    for (int t = 0; t < 8; ++t) s_acc[wave][8 * sl + t] = acc[t];
  }
  if (lane == 0) s_red[wave] = es;
  __syncthreads();
  const int64_t slot = (int64_t)bh * a.nch + chunk;
  if (threadIdx.x < D) {
    const int dd = threadIdx.x;
    a.pacc[slot * D + dd] = s_acc[0][dd] + s_acc[1][dd] + s_acc[2][dd] + s_acc[3][dd];
  }
  if (threadIdx.x == 0) {
    a.pmax[slot] = mx;
    a.psum[slot] = s_red[0] + s_red[1] + s_red[2] + s_red[3];
  }
}

// ---- finalize ------------------------------------------------------------------------------------------
// Workgroup y = 0 of each (b, h) merges the chunks into L and the output; when the next loop keeps every column
// (c_next = n) it also writes the columns themselves, m' = m (the probabilities over S sum to m) and sub' = the
// add term just formed.  Otherwise the workgroups y = 1 .. n_sel (the grid starts at y0) select the next loop's columns
// and sum their probabilities and values: each runs the radix top-k of fl_topk.h over all keys, writes its share of the selected
// positions (ascending) and gathers their logits and V rows (ids and weights in LDS, every V load issued before any
// use).  With one of them the positions go through the workspace in windows of kSelWin; with more, each has one
// window in LDS, and decode_sum_kernel adds their sums in order (deterministic).  The merge reads m and sub, which the
// one selecting workgroup replaces by m' and sub' where a caller updates them in place: then the two are launched one
// after the other (more selecting workgroups write sums of their own, and the merge alone touches m and sub).
//
// Bound by latency: a top-k over 32K keys takes about 20 us on one workgroup however few of them run, and the
// gather of 2048 rows by one workgroup as long again.  At 16 heads over 32K columns, c_next = 2048, one workgroup for
// all of it took 49 us, 32 us so (28 and 4 for the sum; the merge beside the selection, eight gathers side by side).

// L = M + log S over the chunks' maxima and exp-sums, in every wave
__device__ __forceinline__ void merge_normaliser(const DecodeArgs& a, int bh, double& Mx, double& S) {
  const int lane = threadIdx.x & 63;
  const double* pm = a.pmax + (int64_t)bh * a.nch;
  const double* ps = a.psum + (int64_t)bh * a.nch;
  double mx = -INFINITY;
  for (int c = lane; c < a.nch; c += 64) mx = fmax(mx, pm[c]);
  Mx = wave_max_f64(mx);
  double es = 0.0;
  for (int c = lane; c < a.nch; c += 64) es += ps[c] * exp(pm[c] - Mx);
  S = wave_sum_f64_dec(es);
}

template <int D>
__device__ __forceinline__ void decode_merge(const DecodeArgs& a, int bh, double m, float* s_f, float (*s_acc)[D]) {
  constexpr int PARTS = kTopkThreads / D;    // threads per output dimension
  const int tid = threadIdx.x;
  const bool dense = a.cols == nullptr;
  double Mx, S;
  merge_normaliser(a, bh, Mx, S);
  for (int c = tid; c < a.nch; c += kTopkThreads) s_f[c] = (float)(m * exp(a.pmax[(int64_t)bh * a.nch + c] - Mx) / S);
  __syncthreads();
  {
    // thread (part, dd) adds the chunks part, part + PARTS, ...; the parts are then added in order
    const int dd = tid % D, part = tid / D;
    const float* pa = a.pacc + (int64_t)bh * a.nch * D + dd;
    float add = 0.0f;
#pragma unroll 8
    for (int c = part; c < a.nch; c += PARTS) add = fmaf(s_f[c], pa[(int64_t)c * D], add);
    s_acc[part][dd] = add;
  }
  __syncthreads();
  const bool keep_all = a.c_next == a.n;
  if (tid < D) {
    float o_add = 0.0f;
#pragma unroll
    for (int q = 0; q < PARTS; ++q) o_add += s_acc[q][tid];
    const int64_t od = (int64_t)bh * D + tid;
    a.o[od] = dense ? o_add : a.o[od] - a.sub[od] + o_add;
    if (keep_all) a.sub_next[od] = o_add;
  }
  if (tid == 0 && a.lse) a.lse[bh] = (float)(Mx + log(S));
  if (keep_all) {
    for (int i = tid; i < a.n; i += kTopkThreads) a.cols_next[(int64_t)bh * a.n + i] = dec_col(a, bh, i);
    if (tid == 0) a.mass_next[bh] = (float)m;
  }
}

template <int D, int M, int NH>
__global__ __launch_bounds__(kTopkThreads) void decode_finalize_kernel(DecodeArgs a, int n_sel, int y0) {
  constexpr int NW = kTopkThreads / 64;      // waves
  constexpr int LPC = D / 8;                 // lanes per V row (16 bytes each)
  constexpr int CPW = 64 / LPC;              // rows per wave instruction
  constexpr int IT = kSelWin / (NW * CPW);   // window rows per lane
  static_assert(IT * NW * CPW == kSelWin && kSelWin == kTopkThreads, "one id per thread, IT rows per lane");
  constexpr int BUF = NW * D > 2 * kSelWin ? NW * D : 2 * kSelWin;
  typedef TopkShared<M, kTopkThreads, NH> Topk;
  __shared__ __attribute__((aligned(16))) Topk topk;
  static_assert(sizeof(topk.hist) >= BUF * sizeof(float), "the sums and a window's ids and weights take its place");
  __shared__ double s_m[NW];
  __shared__ float s_f[512];                 // chunk weights (nch <= 512)
  __shared__ int32_t s_sel[kSelWin];         // a window's selected positions
  float* s_buf = reinterpret_cast<float*>(topk.hist);
  float (*s_acc)[D] = reinterpret_cast<float (*)[D]>(s_buf);
  int32_t* s_col = reinterpret_cast<int32_t*>(s_buf);
  float* s_w = s_buf + kSelWin;
  const int bh = blockIdx.x;
  const int b = bh / a.H, h = bh % a.H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double m = a.cols ? (double)a.mass[bh] : 1.0;
  const int y = (int)blockIdx.y + y0 - 1;    // -1: the merge
  if (y < 0) {                               // uniform
    decode_merge<D>(a, bh, m, s_f, s_acc);
    return;
  }
  // this workgroup's share [lo0, hi0) of the selected positions
  const int share = (a.c_next + n_sel - 1) / n_sel;
  const int lo0 = y * share, hi0 = min(a.c_next, lo0 + share);
  int32_t* sel = const_cast<int32_t*>(a.sel) + (int64_t)bh * a.c_next;
  const float* keys = a.key + (int64_t)bh * a.n;
  if (n_sel == 1) {
    // the workgroup's writes are visible to its own threads after a workgroup-scope release and acquire around the
    // barrier
    topk_block<M, kTopkThreads, NH>(topk, keys, a.n, a.c_next, nullptr, 0, sel, 0, nullptr, 0);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  } else {
    topk_block<M, kTopkThreads, NH>(topk, keys, a.n, a.c_next, nullptr, 0, s_sel, 0, nullptr, 0, lo0, hi0);
  }
  double Mx, S;
  merge_normaliser(a, bh, Mx, S);
  const double L = Mx + log(S);
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const int sl = lane % LPC, grp = lane / LPC;
  const int64_t HD = (int64_t)a.H * D;
  double ms = 0.0;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int lo = lo0; lo < hi0; lo += kSelWin) {
    const int rows = min(kSelWin, hi0 - lo);
    // ids, weights p_j = m exp(l_j - L) and the next loop's columns of the window (thread t: entry t)
    {
      const bool ok = tid < rows;
      const int p = ok ? (n_sel == 1 ? sel[lo + tid] : s_sel[tid]) : 0;
      const int col = dec_col(a, bh, p);
      const double pr = ok ? m * exp(a.logit[(int64_t)bh * a.n + p] - L) : 0.0;
      if (ok) a.cols_next[(int64_t)bh * a.c_next + lo + tid] = col;
      ms += pr;
      s_col[tid] = col;
      s_w[tid] = (float)pr;
    }
    __syncthreads();
    // their V rows: wave w, row group g takes window entries (w * CPW + g) + it * NW * CPW
    uint4 vw[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int e = wave * CPW + grp + it * NW * CPW;
      vw[it] = make_uint4(0, 0, 0, 0);
      if (it * NW * CPW < rows)              // uniform
        vw[it] = *reinterpret_cast<const uint4*>(a.v + ((int64_t)b * a.T + s_col[e]) * HD + (int64_t)h * D + 8 * sl);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      if (it * NW * CPW >= rows) continue;   // uniform
      const int e = wave * CPW + grp + it * NW * CPW;
      const float wf = s_w[e];               // 0 past the end of the share
      const uint32_t ws[4] = {vw[it].x, vw[it].y, vw[it].z, vw[it].w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        acc[2 * t] = fmaf(wf, bf16_to_f32(ws[t] & 0xFFFFu), acc[2 * t]);
        acc[2 * t + 1] = fmaf(wf, bf16_to_f32(ws[t] >> 16), acc[2 * t + 1]);
      }
    }
    __syncthreads();                         // the window's ids and weights are no longer read
  }
  ms = wave_sum_f64_dec(ms);
#pragma unroll
  for (int t = 0; t < 8; ++t)
    for (int off = LPC; off < 64; off <<= 1) acc[t] += __shfl_xor(acc[t], off, 64);
  if (lane < LPC) {
#pragma unroll
    for (int t = 0; t < 8; ++t) s_acc[wave][8 * sl + t] = acc[t];
  }
  if (lane == 0) s_m[wave] = ms;
  __syncthreads();
  float* sub = n_sel == 1 ? a.sub_next + (int64_t)bh * D : a.part_sub + ((int64_t)bh * n_sel + y) * D;
  if (tid < D) {
    float sacc = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) sacc += s_acc[w][tid];
    sub[tid] = sacc;
  }
  if (tid == 0) {
    double mt = 0.0;
    for (int w = 0; w < NW; ++w) mt += s_m[w];
    if (n_sel == 1) a.mass_next[bh] = (float)mt;
    else a.part_mass[(int64_t)bh * n_sel + y] = mt;
  }
}

// sub' and m' of each (b, h) from the selecting workgroups' sums, in their order
template <int D>
__global__ __launch_bounds__(D) void decode_sum_kernel(DecodeArgs a, int n_sel) {
  const int bh = blockIdx.x, tid = threadIdx.x;
  float s = 0.0f;
  double m = 0.0;
  for (int y = 0; y < n_sel; ++y) {
    s += a.part_sub[((int64_t)bh * n_sel + y) * D + tid];
    m += a.part_mass[(int64_t)bh * n_sel + y];
  }
  a.sub_next[(int64_t)bh * D + tid] = s;
  if (tid == 0) a.mass_next[bh] = (float)m;
}

// Workgroups that select for one (b, h).  One top-k per CU at most, each of them all over the keys, so more only where
// CUs are idle otherwise; shares of at most kSelWin rows and at least d + 2 (their sums take the place of the selected
// positions in the workspace) and 128 (below, the gather is not what a share waits for).
static int select_workgroups(int bh, int d, int n, int c_next) {
  if (c_next == 0 || c_next == n) return 0;
  const int most = std::min(std::min(256 / std::max(bh, 1), 8), c_next / std::max(d + 2, 128));
  if (most < 2 || (c_next + most - 1) / most > kSelWin) return 1;
  return most;
}

// whether two arrays of the same size share memory
static bool overlap(const void* a, const void* b, size_t bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + bytes && y < x + bytes;
}

// workspace regions, each 256-byte aligned
struct DecodeWs {
  size_t logit, pmax, psum, pacc, key, sel, total;
};
static DecodeWs decode_ws(int B, int H, int d, int n, int c_next) {
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t bh = (size_t)B * H;
  const size_t nch = ((size_t)n + kDecChunk - 1) / kDecChunk;
  DecodeWs w;
  size_t off = 0;
  w.logit = off; off += al(bh * n * sizeof(double));
  w.pmax = off; off += al(bh * nch * sizeof(double));
  w.psum = off; off += al(bh * nch * sizeof(double));
  w.pacc = off; off += al(bh * nch * d * sizeof(float));
  w.key = off; off += al(bh * n * sizeof(float));
  w.sel = off; off += al(bh * (size_t)c_next * sizeof(int32_t));
  w.total = off;
  return w;
}

}  // namespace fl

using namespace fl;

extern "C" size_t fl_decode_step_ws(int B, int T, int H, int d, int c, int c_next) {
  if (B < 1 || T < 1 || H < 1 || (d != 64 && d != 128) || c < 0 || c_next < 0) return 0;
  const int n = c > 0 ? c : T;
  return decode_ws(B, H, d, n, c_next).total;
}

static int decode_scratch(void** out);

// ws == nullptr with use_scratch: the library's own scratch array, looked up after the arguments pass
static int decode_step(const char* fn, bool use_scratch, const uint16_t* q, const uint16_t* k_cache,
                       const uint16_t* v_cache, const int32_t* cols, int c, const float* mass, const float* sub,
                       int B, int T, int H, int d, float sm_scale, float* o, float* lse, int n_sink, int window, int c_next,
                       int32_t* cols_next, float* mass_next, float* sub_next, void* ws, size_t ws_bytes,
                       void* stream) {
  FL_REQUIRE(q && k_cache && v_cache && o, FL_E_NULL, "%s: q, k_cache, v_cache and o are required", fn);
  FL_REQUIRE(B >= 1 && T >= 1 && H >= 1, FL_E_SHAPE, "%s: need B, T, H >= 1", fn);
  FL_REQUIRE(d == 64 || d == 128, FL_E_SHAPE, "%s: head dim %d not in {64, 128}", fn, d);
  FL_REQUIRE((int64_t)T * H * d < ((int64_t)1 << 31), FL_E_SHAPE, "%s: T * H * d too large", fn);
  FL_REQUIRE(sm_scale > 0.0f && std::isfinite(sm_scale), FL_E_RANGE, "%s: sm_scale must be > 0", fn);
  const bool dense = cols == nullptr;
  if (dense) {
    FL_REQUIRE(c == 0 || c == T, FL_E_SHAPE, "%s: without cols, c must be 0 or T", fn);
  } else {
    FL_REQUIRE(c >= 1 && c <= T, FL_E_RANGE, "%s: c=%d outside [1, T]", fn, c);
    FL_REQUIRE(mass && sub, FL_E_NULL, "%s: a sparse loop needs its cached mass and subtract term", fn);
  }
  const int n = dense ? T : c;
  FL_REQUIRE(n <= 65536, FL_E_SHAPE, "%s: %d columns exceed the 65536 the selection supports", fn, n);
  FL_REQUIRE(c_next >= 0 && c_next <= n, FL_E_RANGE, "%s: c_next=%d outside [0, %d]", fn, c_next, n);
  FL_REQUIRE(c_next == 0 || (cols_next && mass_next && sub_next), FL_E_NULL,
             "%s: cols_next, mass_next and sub_next are required when c_next > 0", fn);
  FL_REQUIRE(n_sink >= 0 && window >= 0, FL_E_RANGE, "%s: n_sink and window must be >= 0", fn);
  const DecodeWs L = decode_ws(B, H, d, n, c_next);
  if (use_scratch) {
    FL_REQUIRE(L.total <= (size_t)FL_DECODE_SCRATCH_BYTES, FL_E_RANGE,
               "%s: the step needs %zu bytes of scratch, above the %zu available (use fl_decode_step with a "
               "workspace)", fn, L.total, (size_t)FL_DECODE_SCRATCH_BYTES);
    const int rc = decode_scratch(&ws);
    if (rc != FL_OK) return rc;
    ws_bytes = (size_t)FL_DECODE_SCRATCH_BYTES;
  }
  FL_REQUIRE(ws && ws_bytes >= L.total, FL_E_WORKSPACE, "%s: workspace of %zu bytes required", fn, L.total);
  hipStream_t st = as_stream(stream);
  FL_CHECK_LIST(fn, "cols", cols, (int64_t)B * H, c, 0, T, st);
  char* base = static_cast<char*>(ws);
  DecodeArgs a{};
  a.q = q; a.k = k_cache; a.v = v_cache; a.cols = cols; a.mass = mass; a.sub = sub; a.o = o; a.lse = lse;
  a.logit = reinterpret_cast<double*>(base + L.logit);
  a.pmax = reinterpret_cast<double*>(base + L.pmax);
  a.psum = reinterpret_cast<double*>(base + L.psum);
  a.pacc = reinterpret_cast<float*>(base + L.pacc);
  a.key = reinterpret_cast<float*>(base + L.key);
  a.sel = reinterpret_cast<const int32_t*>(base + L.sel);
  a.cols_next = cols_next; a.mass_next = mass_next; a.sub_next = sub_next;
  a.B = B; a.T = T; a.H = H; a.n = n; a.nch = (n + kDecChunk - 1) / kDecChunk; a.c_next = c_next;
  a.n_sink = n_sink; a.window = window; a.scale = (double)sm_scale;
  const int BH = B * H;
  dim3 gp(a.nch, BH);
  if (d == 128) decode_partial_kernel<128><<<gp, 256, 0, st>>>(a);
  else decode_partial_kernel<64><<<gp, 256, 0, st>>>(a);
  int rc = check_launch("decode_partial_kernel");
  if (rc != FL_OK) return rc;
  // finalize: the top-k's register depth follows the number of keys (as in the selection kernels)
  const int n_sel = select_workgroups(BH, d, n, c_next);
  a.part_mass = reinterpret_cast<double*>(base + L.sel);
  a.part_sub = reinterpret_cast<float*>(a.part_mass + (int64_t)BH * n_sel);
  const int keys = n_sel > 0 ? n : 0;
  int y0 = 0;
  dim3 gf(BH, 1 + n_sel);
#define FL_FIN(MM, HH)                                                                              \
  do {                                                                                              \
    if (d == 128) decode_finalize_kernel<128, MM, HH><<<gf, kTopkThreads, 0, st>>>(a, n_sel, y0);   \
    else decode_finalize_kernel<64, MM, HH><<<gf, kTopkThreads, 0, st>>>(a, n_sel, y0);             \
  } while (0)
  if (n_sel == 1 && !dense &&
      (overlap(sub, sub_next, (size_t)BH * d * sizeof(float)) || overlap(mass, mass_next, (size_t)BH * sizeof(float)))) {
    gf.y = 1;
    FL_FIN(1, 1);                          // the merge
    rc = check_launch("decode_finalize_kernel(merge)");
    if (rc != FL_OK) return rc;
    y0 = 1;
  }
  if (keys <= 1024) FL_FIN(1, 1);
  else if (keys <= 2048) FL_FIN(2, 1);
  else if (keys <= 4096) FL_FIN(4, 1);
  else if (keys <= 8192) FL_FIN(8, 1);
  else if (keys <= 16384) FL_FIN(16, 1);
  else if (keys <= 32768) FL_FIN(32, 1);
  else FL_FIN(32, 2);
#undef FL_FIN
  rc = check_launch("decode_finalize_kernel");
  if (rc != FL_OK || n_sel < 2) return rc;
  if (d == 128) decode_sum_kernel<128><<<BH, 128, 0, st>>>(a, n_sel);
  else decode_sum_kernel<64><<<BH, 64, 0, st>>>(a, n_sel);
  return check_launch("decode_sum_kernel");
}

extern "C" int fl_decode_step(const uint16_t* q, const uint16_t* k_cache, const uint16_t* v_cache,
                              const int32_t* cols, int c, const float* mass, const float* sub, int B, int T,
                              int H, int d, float sm_scale, float* o, float* lse, int n_sink, int window,
                              int c_next, int32_t* cols_next, float* mass_next, float* sub_next, void* ws,
                              size_t ws_bytes, void* stream) {
  FL_API_BEGIN
  return decode_step("fl_decode_step", false, q, k_cache, v_cache, cols, c, mass, sub, B, T, H, d, sm_scale, o, lse,
                     n_sink, window, c_next, cols_next, mass_next, sub_next, ws, ws_bytes, stream);
  FL_API_END
}

// ---- the decode step without a caller workspace ----------------------------------------------------------
// The workspace lives in a file-scope device array of FL_DECODE_SCRATCH_BYTES, one copy per GPU, held
// until the process ends.  Host code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol): the device address of each GPU's copy is looked up once with
// hipGetSymbolAddress, with that GPU current, and that address is what the kernels receive.  Every region
// of the workspace is written before it is read within one call, so nothing needs clearing between calls.
static __device__ __align__(256) unsigned char scratch[FL_DECODE_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];
}  // namespace

static int decode_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  FL_REQUIRE(e == hipSuccess && dev >= 0 && dev < kMaxDevices, FL_E_HIP,
             "fl_decode_step_noalloc: no current device (%s)", hipGetErrorString(e));
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    FL_REQUIRE(e == hipSuccess && p != nullptr, FL_E_HIP,
               "fl_decode_step_noalloc: hipGetSymbolAddress failed on device %d (%s)", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return FL_OK;
}

extern "C" int fl_decode_step_noalloc(const uint16_t* q, const uint16_t* k_cache, const uint16_t* v_cache,
                                      const int32_t* cols, int c, const float* mass, const float* sub, int B,
                                      int T, int H, int d, float sm_scale, float* o, float* lse, int n_sink,
                                      int window, int c_next, int32_t* cols_next, float* mass_next,
                                      float* sub_next, void* stream) {
  FL_API_BEGIN
  return decode_step("fl_decode_step_noalloc", true, q, k_cache, v_cache, cols, c, mass, sub, B, T, H, d, sm_scale,
                     o, lse, n_sink, window, c_next, cols_next, mass_next, sub_next, nullptr, 0, stream);
  FL_API_END
}
