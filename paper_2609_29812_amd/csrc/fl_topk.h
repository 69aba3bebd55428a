// Radix top-k of one segment by one workgroup, shared by the selection kernels and the decode step (Appendix D.1,
// Eq. 5; Appendix D.2, Eq. 6: the largest keys, ties to the lower position, emitted in ascending position order).
//
// Keys are mapped to order-preserving uint32 and held in registers: thread t of NT holds the M consecutive positions
// from t M on (two such blocks, NH = 2, above 32K keys), read coalesced and turned round in LDS, so that a thread's
// selected positions are bits of one word and one block scan gives their places in the output.  The k-th largest key is
// found by an LDS histogram over the keys' range, whose bin is compacted into LDS and resolved by digit histograms.
//
// Bound by latency: one workgroup, a chain of barriers.  32K keys (k = 1638, with the slot map): 18.7 us, 23 with keys
// held in stripes, whose output order took ballot bitmaps through LDS, and LDS-permute scans (8K keys 10.2 against 15.7,
// 256 keys 4.5 against 7.9).
#pragma once
#include "fl_common.h"

#include <climits>

namespace fl {

constexpr int kTopkThreads = 1024;

// ---- wave and workgroup helpers -------------------------------------------------------------------
#define FL_DPP(old, x, ctrl, rows) __builtin_amdgcn_update_dpp((old), (x), (ctrl), (rows), 0xf, false)
// inclusive prefix sum over the wave's lanes (row shifts, then the rows' totals broadcast to the rows after)
__device__ __forceinline__ int wave_scan(int v) {
  v += FL_DPP(0, v, 0x111, 0xf);
  v += FL_DPP(0, v, 0x112, 0xf);
  v += FL_DPP(0, v, 0x114, 0xf);
  v += FL_DPP(0, v, 0x118, 0xf);
  v += FL_DPP(0, v, 0x142, 0xa);
  v += FL_DPP(0, v, 0x143, 0xc);
  return v;
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#define FL_STEP(ctrl, rows) v = min(v, (uint32_t)FL_DPP(-1, (int)v, ctrl, rows))
  FL_STEP(0x111, 0xf); FL_STEP(0x112, 0xf); FL_STEP(0x114, 0xf); FL_STEP(0x118, 0xf); FL_STEP(0x142, 0xa);
  FL_STEP(0x143, 0xc);
#undef FL_STEP
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
#undef FL_DPP

template <int NT>
struct TopkScan {
  int2 total[2][NT / 64];
};

// Exclusive prefix sums of two values over the workgroup's threads, and their totals.  Alternate `parity` between
// calls: the next call's writes then never race this one's reads.
template <int NT>
__device__ __forceinline__ int2 block_scan2(int a, int b, TopkScan<NT>& sc, int parity, int2& all) {
  const int w = threadIdx.x >> 6;
  const int ia = wave_scan(a), ib = wave_scan(b);
  if ((threadIdx.x & 63) == 63) sc.total[parity][w] = make_int2(ia, ib);
  __syncthreads();
  int2 before = make_int2(0, 0);
  all = make_int2(0, 0);
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    const int2 s = sc.total[parity][i];
    before.x += i < w ? s.x : 0;
    before.y += i < w ? s.y : 0;
    all.x += s.x;
    all.y += s.y;
  }
  return make_int2(before.x + ia - a, before.y + ib - b);
}

// Histogram of one digit per lane and round, for keys that crowd into few bins: the bin of the wave's
// first key of the first round is counted in a register with ballots (one LDS atomic at the end), the
// other keys add with LDS atomics.  Same-address LDS atomics from many waves serialize; this keeps them
// to one per wave for the crowded bin.
struct WaveHist {
  uint32_t lead = 0;
  int count = 0;
  bool started = false;
  __device__ __forceinline__ void add(int* hist, uint32_t bin, bool want) {
    if (!started) {                                        // uniform
      lead = __builtin_amdgcn_readfirstlane(bin);
      started = true;
    }
    const bool same = want && bin == lead;
    count += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(same));
    if (want && !same) atomicAdd(&hist[bin], 1);
  }
  __device__ __forceinline__ void flush(int* hist) {
    if ((threadIdx.x & 63) == 0 && count > 0) atomicAdd(&hist[lead], count);
  }
};

__device__ __forceinline__ uint32_t orderable(float f) {
  const uint32_t u = __float_as_uint(f + 0.0f);   // -0 and +0 are the same key
  return max((u & 0x80000000u) ? ~u : (u | 0x80000000u), 1u);   // (0 is no key: only the lowest NaN moves)
}

template <int M, int NT, int NH>
struct TopkShared {
  static constexpr int kBins = 4 * NT;
  static constexpr int kBuf = NT * (M + 1);   // rows of M keys, one word apart: strided reads spread over the banks
  TopkScan<NT> scan;
  uint32_t lo[NT / 64], hi[NT / 64];
  int meta[3];                                // the threshold's bin, keys still to take from it, its size
  int n_in;
  int hist[kBins];
  uint32_t buf[kBuf];                         // the keys by position, then the keys of the threshold's bin
};

// The bin, scanning bins from the highest, where the running count of keys first reaches krem; hist holds nbins
// counts, PER per thread.  Result in meta; ends with a barrier.
template <int PER, int NT>
__device__ __forceinline__ void find_bin(const int* hist, int nbins, int krem, TopkScan<NT>& sc, int parity, int* meta) {
  int hb[PER], local = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int bin = nbins - 1 - PER * (int)threadIdx.x - q;
    hb[q] = bin >= 0 ? hist[bin] : 0;
    local += hb[q];
  }
  int2 all;
  const int above = block_scan2<NT>(local, 0, sc, parity, all).x;
  if (above < krem && above + local >= krem) {
    int acc = above;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (acc < krem && acc + hb[q] >= krem) {
        meta[0] = nbins - 1 - PER * (int)threadIdx.x - q;
        meta[1] = krem - acc;
        meta[2] = hb[q];
      }
      acc += hb[q];
    }
  }
  __syncthreads();
}

// One workgroup of NT threads selects the top k of n <= M NT NH keys kp[0..n).  Position p has id cp[p]
// (cp != NULL) or id_base + p.  Selected ids are written ascending at op[n_prefix + pos]; ids
// 0..n_prefix-1 are written first (column sinks).  Optional slot map: sp[id] = pos (or -1), sp holding
// slot_n entries.  Only output positions pos in [out_lo, out_hi) are written, at op[n_prefix + pos -
// out_lo] (the sink ids only when out_lo == 0): a workgroup that needs one window of the selection keeps
// it in LDS.  Ends with the ids written by this workgroup's threads (no trailing barrier).
template <int M, int NT, int NH>
__device__ __forceinline__ void topk_block(TopkShared<M, NT, NH>& sh, const float* __restrict__ kp, int n, int k,
                                           const int32_t* __restrict__ cp, int id_base,
                                           int32_t* __restrict__ op, int n_prefix,
                                           int32_t* __restrict__ sp, int slot_n, int out_lo = 0,
                                           int out_hi = INT_MAX) {
  static_assert(M <= 32 && (NH == 1 || M == 32), "a thread's selected positions of one block are one word");
  constexpr int kBins = TopkShared<M, NT, NH>::kBins;
  constexpr int kHistBits = __builtin_ctz(kBins), kDigit = __builtin_ctz(NT);
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  int32_t* slot = sp;
  if (slot) {
    for (int i = t; i < slot_n; i += NT) sp[i] = -1;
  }
  if (out_lo == 0)
    for (int i = t; i < n_prefix; i += NT) op[i] = i;
#pragma unroll
  for (int q = 0; q < kBins / NT; ++q) sh.hist[q * NT + t] = 0;
  if (t == 0) sh.n_in = 0;

  // (buffer loads: out-of-range positions read 0 without a branch, so all loads are in flight at once;
  // a bounds-checked pointer load puts each one behind its own branch and wait)
  uint32_t u[NH][M];                          // codes; 0 past the last key, below every key
  {
    const __amdgpu_buffer_rsrc_t kr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kp), (short)0, n * 4, 0x00020000);
#pragma unroll
    for (int q = 0; q < NH; ++q) {
      uint32_t x[M];
#pragma unroll
      for (int j = 0; j < M; ++j)
        x[j] = __builtin_amdgcn_raw_buffer_load_b32(kr, (uint32_t)(q * NT * M + NT * j + t) * 4u, 0, 0);
      if (q > 0) __syncthreads();
#pragma unroll
      for (int j = 0; j < M; ++j) {
        const int p = NT * j + t;
        sh.buf[p + p / M] = q * NT * M + p < n ? orderable(__uint_as_float(x[j])) : 0u;
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < M; ++j) u[q][j] = sh.buf[t * (M + 1) + j];
    }
  }

  // k-th largest key.  The keys' range (lo, hi], lo below every key: the codes become offsets v = u - lo (order kept;
  // 0 past the last key, so below the k-th largest), and the first histogram takes the kHistBits bits of v from the highest bit the range needs (shift0 up),
  // so the bins cover the keys' actual range and the bin that holds the k-th largest is small.  With
  // k == n every position is taken and no threshold is needed.
  const bool take_all = k == n;
  uint32_t prefix = 0, mask = 0;
  int krem = 0;
  if (k > 0 && !take_all) {                               // uniform
    uint32_t lo = 0xFFFFFFFFu, nhi = 0xFFFFFFFFu;         // (the largest as the smallest complement)
#pragma unroll
    for (int q = 0; q < NH; ++q)
#pragma unroll
      for (int j = 0; j < M; ++j) {
        lo = min(lo, u[q][j] - 1u);                       // (of 0, past the last key: no effect)
        nhi = min(nhi, ~u[q][j]);
      }
    lo = wave_min_u32(lo);
    nhi = wave_min_u32(nhi);
    if (lane == 0) {
      sh.lo[wave] = lo;
      sh.hi[wave] = nhi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      lo = min(lo, sh.lo[w]);
      nhi = min(nhi, sh.hi[w]);
    }
    const uint32_t span = ~nhi - lo;
    const int shift0 = span >> kHistBits ? 32 - __builtin_clz(span) - kHistBits : 0;   // span >> shift0 < kBins
    WaveHist wh;
#pragma unroll
    for (int q = 0; q < NH; ++q)
#pragma unroll
      for (int j = 0; j < M; ++j) {
        u[q][j] = max(u[q][j], lo) - lo;
        wh.add(sh.hist, u[q][j] >> shift0, true);
      }
    wh.flush(sh.hist);
    __syncthreads();
    find_bin<kBins / NT, NT>(sh.hist, kBins, k, sh.scan, 0, sh.meta);
    const uint32_t bin = (uint32_t)sh.meta[0];
    const int cnt = sh.meta[2];
    krem = sh.meta[1];
    prefix = bin << shift0;
    mask = ~0u << shift0;
    if (shift0 == 0) {
      // every offset is its own bin: the threshold is known
    } else if (NH == 1 || cnt <= NT * M) {
      // that bin's keys into LDS (any order), then the low shift0 bits with digit histograms of up to kDigit bits
      int n_in = 0;
#pragma unroll
      for (int q = 0; q < NH; ++q)
#pragma unroll
        for (int j = 0; j < M; ++j) n_in += (u[q][j] & mask) == prefix ? 1 : 0;
      const int incl = wave_scan(n_in);
      int off = 0;
      if (lane == 63 && incl > 0) off = atomicAdd(&sh.n_in, incl);
      off = __builtin_amdgcn_readlane(off, 63) + incl - n_in;
#pragma unroll
      for (int q = 0; q < NH; ++q)
#pragma unroll
        for (int j = 0; j < M; ++j)
          if ((u[q][j] & mask) == prefix) sh.buf[off++] = u[q][j];
      int shift = shift0, parity = 1;
      while (shift > 0) {                                 // uniform
        const int passes = (shift + kDigit - 1) / kDigit;
        const int nb = (shift + passes - 1) / passes;
        shift -= nb;
        if (t < (1 << nb)) sh.hist[t] = 0;
        __syncthreads();                                  // also orders the compaction writes
        WaveHist dh;
        for (int i0 = 0; i0 < cnt; i0 += NT) {
          const int i = i0 + t;
          const uint32_t v = i < cnt ? sh.buf[i] : 0u;
          dh.add(sh.hist, (v >> shift) & ((1u << nb) - 1), i < cnt && (v & mask) == prefix);
        }
        dh.flush(sh.hist);
        __syncthreads();
        find_bin<1, NT>(sh.hist, 1 << nb, krem, sh.scan, parity, sh.meta);
        parity ^= 1;
        prefix |= (uint32_t)sh.meta[0] << shift;
        mask |= ((1u << nb) - 1) << shift;
        krem = sh.meta[1];
      }
    } else {
      // too many keys in one bin for the LDS buffer: resolve the low bits over the registers
      for (int bit = shift0 - 1; bit >= 0; --bit) {
        const uint32_t want = prefix | (1u << bit), m2 = mask | (1u << bit);
        int c = 0;
#pragma unroll
        for (int q = 0; q < NH; ++q)
#pragma unroll
          for (int j = 0; j < M; ++j) c += (u[q][j] & m2) == want ? 1 : 0;
        int2 all;
        block_scan2<NT>(c, 0, sh.scan, bit & 1, all);
        if (all.x >= krem) prefix = want; else krem -= all.x;
        mask = m2;
      }
      __syncthreads();
    }
  }
  // The selected positions: keys above the threshold, and the krem lowest positions of those equal to it.
  uint32_t gt[NH], eq[NH];
#pragma unroll
  for (int q = 0; q < NH; ++q) {
    gt[q] = eq[q] = 0u;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      gt[q] |= u[q][j] > prefix ? 1u << j : 0u;
      eq[q] |= u[q][j] == prefix ? 1u << j : 0u;
    }
    if (take_all || k == 0) {                             // (the codes themselves, no threshold)
      const int nv = min(max(n - q * NT * M - t * M, 0), M);
      gt[q] = k == 0 ? 0u : nv >= 32 ? ~0u : (1u << nv) - 1u;
      eq[q] = 0u;
    }
  }
  // the -1 fill above is complete before positions are written (same workgroup: a workgroup-scope
  // release suffices; a device-scope fence would also write back the L2)
  if (slot) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  int2 base = make_int2(0, 0);
#pragma unroll
  for (int q = 0; q < NH; ++q) {
    int2 all;
    // (find_bin's last barrier lies between its last scan and this one)
    int2 at = block_scan2<NT>(__builtin_popcount(gt[q]), __builtin_popcount(eq[q]), sh.scan, q & 1, all);
    at.x += base.x;
    at.y += base.y;
    base.x += all.x;
    base.y += all.y;
    int pos = at.x + min(at.y, krem);
    int take = krem - at.y;                               // equal keys this thread still takes
    uint32_t both = gt[q] | eq[q];
    while (both != 0) {
      const int j = __builtin_ctz(both);
      both &= both - 1;
      if ((eq[q] >> j) & 1u) {
        if (take <= 0) continue;
        --take;
      }
      if (pos < k) {                // exactly k positions are selected; the bound is a safety net
        const int p = q * NT * M + t * M + j;
        const int id = cp ? cp[p] : id_base + p;
        if (pos >= out_lo && pos < out_hi) op[n_prefix + pos - out_lo] = id;
        if (slot) sp[id] = pos;
      }
      ++pos;
    }
  }
}

}  // namespace fl
