// Small kernels that finish the two streamed contractions.  They run one or a few workgroups of
// 16 waves on a chip of 256 CUs, so what they cost is latency and instruction count, not
// bandwidth: loads are issued together and never consumed right behind their issue, loops over
// per-thread slots are branch-free, and selections run as wave-wide maxima over the DPP network.
//
// rel_finalize:    cosines from the split dot products / squared norms, then the mean of the
//                  Top-N largest cosines per draft row (paper Eq. 8).  The N-th largest value
//                  is found exactly (duplicates count by value) and the sum is taken in fixed
//                  point, so the result does not depend on thread scheduling.
// accept_finalize: merges the per-workgroup (max, sum exp, top-k candidates) of lm_head into the
//                  greedy target token and the k most probable tokens per draft row
//                  (optionally the row's softmax entropy), then the paper's Eq. 9 (loosened
//                  set), Eq. 10/11 (verdicts incl. position-shift tolerance) and Eq. 2 (accepted
//                  length = longest accepted prefix); the chains of a draft tree share a
//                  workgroup, which then keeps the longest one (long trees: in a launch of its own).
#include "lvspec_dev.h"
#include "lvspec_kernels.h"

namespace lvspec {

namespace {

constexpr int kFinThreads = 1024;
constexpr int kMaxBranches = 8;   // chains of a draft tree (one wave each)

constexpr int kCandCap = 4096;       // candidates kept in LDS for the exact selection

struct SelectScratch {
  uint32_t hist[kFinThreads / 64][256];   // one histogram per wave: 16x less contention
  uint32_t wave_tot[4];
  uint32_t prefix, remaining;
};

// Exact n-th largest of `count` keys (key_at(idx), idx < count), 1 <= n <= count, by a 4-pass
// most-significant-digit radix select.  Returns the key; *need_eq = how many keys equal to it
// belong to the n largest.  All threads of the block must call it.
template <class KeyAt>
LVS_DEV uint32_t radix_select(int count, int n, KeyAt key_at, SelectScratch& sc,
                              uint32_t* need_eq) {
  const int tid = threadIdx.x;
  if (tid == 0) {
    sc.prefix = 0;
    sc.remaining = (uint32_t)n;
  }
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    for (int t = tid; t < (kFinThreads / 64) * 256; t += kFinThreads) (&sc.hist[0][0])[t] = 0;
    __syncthreads();
    const uint32_t prefix = sc.prefix;
    const uint32_t rem = sc.remaining;
    const uint32_t hi_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
    for (int idx = tid; idx < count; idx += kFinThreads) {
      const uint32_t k = key_at(idx);
      if ((k & hi_mask) == prefix) atomicAdd(&sc.hist[tid >> 6][(k >> shift) & 0xffu], 1u);
    }
    __syncthreads();
    // suffix sums S[t] = sum_{u >= t} hist[u]; the selected digit is the t with
    // S[t] >= rem > S[t+1]
    uint32_t own = 0, suf = 0;
    if (tid < 256) {
#pragma unroll
      for (int w = 0; w < kFinThreads / 64; ++w) own += sc.hist[w][tid];
      suf = own;
      const int lane = tid & 63;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_down(suf, off, 64);
        if (lane + off < 64) suf += o;
      }
      if (lane == 0) sc.wave_tot[tid >> 6] = suf;
    }
    __syncthreads();
    if (tid < 256) {
      for (int w = (tid >> 6) + 1; w < 4; ++w) suf += sc.wave_tot[w];
      if (suf >= rem && suf - own < rem) {
        sc.prefix = prefix | ((uint32_t)tid << shift);
        sc.remaining = rem - (suf - own);   // copies of the selected digit still needed
      }
    }
    __syncthreads();
  }
  const uint32_t key = sc.prefix;
  *need_eq = sc.remaining;
  __syncthreads();   // the scratch may be reused by the next call
  return key;
}

// Cosines of the rows j = jr + 1024 * u + tid, u < U, from the split partial sums.  Written for
// instruction count (16 waves share four SIMDs here): the row index is clamped instead of
// predicated, every split pointer is uniform (scalar base + one 32-bit lane offset per row), all
// loads of the round are issued before the first is used, splits past n_ds re-read split 0 with
// weight 0, and the cosine is dot * rsqrt(max(|v|^2, 1e-16)) / |h_d| (rsqrt of the clamped
// square = 1 / max(|v|, 1e-8)).  Writes the cosines to cosb and returns the largest key.
// pre: nbase holds the rows' prepared inverse norms (one plane, nstep = 0) instead of squared
// norms per split (planes nstep apart).
template <int U, int NS>
LVS_DEV uint32_t cos_round(int jr, int tid, int lv, int n_ds, const float* dbase,
                           const float* nbase, int64_t dstep, int64_t nstep, bool pre,
                           float inv_nd, float* cosb) {
  float dv[U][NS], nv[U][NS];
  uint32_t off[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = jr + u * kFinThreads + tid;
    off[u] = (uint32_t)(j < lv ? j : lv - 1) * 4u;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int sc = s < n_ds ? s : 0;                                     // uniform
      const char* dp = reinterpret_cast<const char*>(dbase + sc * dstep);   // uniform
      const char* np = reinterpret_cast<const char*>(nbase + sc * nstep);   // uniform
      dv[u][s] = *reinterpret_cast<const float*>(dp + off[u]);
      nv[u][s] = *reinterpret_cast<const float*>(np + off[u]);
    }
  }
  uint32_t mk = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = jr + u * kFinThreads + tid;
    float dot = dv[u][0], n2 = nv[u][0];
#pragma unroll
    for (int s = 1; s < NS; ++s) {
      const float ws = s < n_ds ? 1.f : 0.f;                               // uniform
      dot = __builtin_fmaf(dv[u][s], ws, dot);
      n2 = __builtin_fmaf(nv[u][s], pre ? 0.f : ws, n2);
    }
    const float c = dot * (pre ? n2 : __builtin_amdgcn_rsqf(fmaxf(n2, 1e-16f))) * inv_nd;
    if (j < lv) *reinterpret_cast<float*>(reinterpret_cast<char*>(cosb) + off[u]) = c;
    mk = max(mk, j < lv ? order_key(c) : 0u);
  }
  return mk;
}

constexpr float kFixScale = 1099511627776.0f;   // 2^40: cosines as 64-bit fixed point

constexpr int kSmallN = 16;          // Top-N sizes served by the shuffle-based selection
constexpr int kSmallCand = 256;      // candidates wave 0 can hold (4 per lane)

// One round of "largest remaining key" over NK keys per lane: returns the key (0 = none
// left), counts its copies and retires them.  Wave-uniform result.
template <int NK>
LVS_DEV uint32_t take_largest(uint32_t (&k)[NK], int& copies) {
  uint32_t best = k[0];
#pragma unroll
  for (int j = 1; j < NK; ++j) best = max(best, k[j]);
  const uint32_t w = wave_max_u32(best);
  copies = 0;
#pragma unroll
  for (int j = 0; j < NK; ++j) {
    copies += __popcll(__ballot(k[j] == w));
    k[j] = k[j] == w ? 0u : k[j];
  }
  return w;
}

// SMALL: top_n <= kSmallN.  The two selections (the bound from the per-thread maxima, then the
// exact Top-N among the candidates) are then done by wave-wide maxima over the DPP network, a
// handful of instructions per round and five barriers in the whole kernel, instead of two
// 4-pass radix selects (about 36 barriers of 16 waves).  Rows with more than kSmallCand
// candidates (many values at the bound) continue on the general path.
template <bool SMALL>
__global__ __launch_bounds__(kFinThreads) void rel_finalize_kernel(const RelFinalizeArgs p) {
  __shared__ float red[16];
  __shared__ SelectScratch sc;
  __shared__ uint32_t tmax[kFinThreads];
  __shared__ float cand[kCandCap];
  __shared__ int cand_count;
  __shared__ long long fix_part[kFinThreads / 64];
  __shared__ uint32_t sm_top[4][kSmallN];
  __shared__ uint32_t sm_t0;
  const int i = blockIdx.x;
  const int b = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  LVS_TRACE_BEGIN;
  LVS_TRACE(0);
  int lv = p.l_v[b];
  if (lv > p.lv_max) lv = (int)p.lv_max;
  float* rel_out = p.relevance + (int64_t)b * p.gamma + i;
  if (lv <= 0) {
    if (tid == 0) *rel_out = 0.f;
    return;
  }
  // |h_d row|^2 (rows are 16-byte aligned and d is a multiple of 128: eight elements per load)
  const uint16_t* hd = p.h_d + (int64_t)b * p.hd_sb + (int64_t)i * p.hd_sg;
  float part = 0.f;
  for (int t = tid * 8; t < p.d; t += kFinThreads * 8) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(hd + t);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __builtin_bit_cast(float, w[e] << 16);
      const float hi = __builtin_bit_cast(float, w[e] & 0xffff0000u);
      part = __builtin_fmaf(lo, lo, part);
      part = __builtin_fmaf(hi, hi, part);
    }
  }
  part = wave_sum(part);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  float nd2 = 0.f;
#pragma unroll
  for (int w = 0; w < kFinThreads / 64; ++w) nd2 += red[w];
  const float inv_nd = 1.0f / fmaxf(sqrtf(nd2), 1e-8f);
  LVS_TRACE(1);
  float* cosb = p.cosbuf + ((int64_t)b * p.gamma + i) * p.ld;
  const float* dbase = p.dots + (((int64_t)b * p.n_ds) * p.gamma + i) * p.ld;
  const bool pre = p.inv_norm != nullptr;
  const float* nbase = pre ? p.inv_norm + (int64_t)b * p.lv_max
                           : p.nv2 + ((int64_t)b * p.n_ds) * p.ld;
  const int64_t nstep = pre ? 0 : p.ld;
  const int64_t dstep = (int64_t)p.gamma * p.ld;
  const int n_eff = p.top_n < lv ? p.top_n : lv;

  // ---- pass 1: cosines to the workspace (split partial sums added in split order), largest
  // value of every thread kept
  uint32_t mk = 0;
  if (p.n_ds == 1) {
    for (int jr = 0; jr < lv; jr += 16 * kFinThreads)
      mk = max(mk, cos_round<16, 1>(jr, tid, lv, 1, dbase, nbase, dstep, nstep, pre, inv_nd, cosb));
  } else if (p.n_ds == 2) {
    for (int jr = 0; jr < lv; jr += 8 * kFinThreads)
      mk = max(mk, cos_round<8, 2>(jr, tid, lv, 2, dbase, nbase, dstep, nstep, pre, inv_nd, cosb));
  } else {
    for (int jr = 0; jr < lv; jr += 2 * kFinThreads)
      mk = max(mk, cos_round<2, 8>(jr, tid, lv, p.n_ds, dbase, nbase, dstep, nstep, pre, inv_nd, cosb));
  }
  LVS_TRACE(2);
  // ---- lower bound of the answer: the n-th largest of the per-thread maxima.  At least n
  // values are >= it, so only values >= it can be among the n largest.
  uint32_t need_eq;
  uint32_t t0key;
  if (tid == 0) cand_count = 0;
  if constexpr (SMALL) {
    // the thread maxima go through LDS to waves 0..3 (four per lane, one wave per SIMD), each
    // of which lists the n_eff largest of its 256 (copies included) ...
    tmax[tid] = mk;
    __syncthreads();
    if (wave < 4) {
      uint32_t k4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) k4[j] = tmax[wave * 256 + 64 * j + lane];
      int got = 0;
      while (got < n_eff) {
        int copies;
        const uint32_t w = take_largest(k4, copies);
        if (w == 0u) break;
        if (lane < copies && got + lane < n_eff) sm_top[wave][got + lane] = w;
        got += copies;
      }
      if (lane < kSmallN && lane >= got) sm_top[wave][lane] = 0u;
    }
    __syncthreads();
    // ... and wave 0 takes the n_eff-th largest of the four lists
    if (wave == 0) {
      uint32_t cur = (lane & (kSmallN - 1)) < n_eff ? sm_top[lane / kSmallN][lane & (kSmallN - 1)]
                                                    : 0u;
      uint32_t t0 = 0u;
      for (int got = 0; got < n_eff;) {
        const uint32_t w = wave_max_u32(cur);
        if (w == 0u) break;
        got += __popcll(__ballot(cur == w));
        cur = cur == w ? 0u : cur;
        t0 = w;
      }
      if (lane == 0) sm_t0 = t0;
    }
    __syncthreads();
    t0key = sm_t0;
  } else {
    tmax[tid] = mk;
    __syncthreads();
    t0key = radix_select(kFinThreads, n_eff, [&](int idx) { return tmax[idx]; }, sc, &need_eq);
  }
  LVS_TRACE(3);
  // ---- pass 2: every thread re-reads the cosines it wrote and keeps those >= the bound in
  // LDS (in no particular order: they are only counted, compared and summed exactly)
  for (int jr = 0; jr < lv; jr += 16 * kFinThreads) {
    float c[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int j = jr + u * kFinThreads + tid;
      c[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(cosb) +
                                             (uint32_t)(j < lv ? j : lv - 1) * 4u);
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int j = jr + u * kFinThreads + tid;
      if (j < lv && order_key(c[u]) >= t0key) {
        const int slot = atomicAdd(&cand_count, 1);
        if (slot < kCandCap) cand[slot] = c[u];
      }
    }
  }
  __syncthreads();
  LVS_TRACE(4);
  const int total = cand_count;
  if constexpr (SMALL) {
    if (total <= kSmallCand) {
      // exact Top-N among the candidates by wave 0: largest first, copies counted by value;
      // the sum is taken in 2^-40 fixed point like on the general path, so both give the same
      // bits
      if (wave != 0) return;
      uint32_t k4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int idx = lane + 64 * j;
        k4[j] = idx < total ? order_key(cand[idx]) : 0u;
      }
      long long tot = 0;
      for (int got = 0; got < n_eff;) {
        int copies;
        const uint32_t w = take_largest(k4, copies);
        if (w == 0u) break;
        const int take = copies < n_eff - got ? copies : n_eff - got;
        tot += (long long)take * (long long)(key_value(w) * kFixScale);
        got += copies;
      }
      if (lane == 0) *rel_out = (float)((double)tot / (double)kFixScale / (double)n_eff);
      LVS_TRACE(5);
      LVS_TRACE_END;
      return;
    }
  }
  uint32_t tkey;
  long long fix = 0;     // sum of the values above the n-th largest, exact in 2^-40 units
  if (total <= kCandCap) {
    tkey = radix_select(total, n_eff, [&](int idx) { return order_key(cand[idx]); }, sc, &need_eq);
    for (int idx = tid; idx < total; idx += kFinThreads)
      if (order_key(cand[idx]) > tkey) fix += (long long)(cand[idx] * kFixScale);
  } else {
    // (many equal values at the bound) select over the whole row in the workspace
    tkey = radix_select(lv, n_eff, [&](int idx) { return order_key(cosb[idx]); }, sc, &need_eq);
    for (int j = tid; j < lv; j += kFinThreads) {
      const float c = cosb[j];
      if (order_key(c) > tkey) fix += (long long)(c * kFixScale);
    }
  }
  // integer addition is associative: any reduction order gives the same bits
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) fix += __shfl_xor(fix, sft, 64);
  if ((tid & 63) == 0) fix_part[tid >> 6] = fix;
  __syncthreads();
  if (tid == 0) {
    long long tot = 0;
    for (int w = 0; w < kFinThreads / 64; ++w) tot += fix_part[w];
    tot += (long long)need_eq * (long long)(key_value(tkey) * kFixScale);
    *rel_out = (float)((double)tot / (double)kFixScale / (double)n_eff);
  }
}

// ------------------------------------------------------------------------------------------
constexpr int kAcceptOneKernelRows = 16;   // hidden rows of a sequence, a wave each
constexpr int kRecRegs = 8;            // records per lane: kAcceptMaxRecords / 64
constexpr int kPickedMax = 32;         // records the short way of the selection can take

// Largest T with at least k of the wave's keys >= T (0 = no key; fewer than k keys: T = 1), found
// bit by bit from the first bit in which the keys differ; exact unless it can stop early because
// exactly k keys are left.
template <int NV>
LVS_DEV uint32_t kth_bound(const uint32_t (&key)[NV], int k) {
  uint32_t hi = key[0], nlo = 0u;      // largest key; largest complement = smallest key
  int have = 0;
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    hi = max(hi, key[u]);
    nlo = max(nlo, key[u] != 0u ? ~key[u] : 0u);
    have += __popcll(__ballot(key[u] != 0u));
  }
  if (have <= k) return 1u;
  hi = wave_max_u32(hi);
  if (k == 1) return hi;
  const uint32_t lo = ~wave_max_u32(nlo);
  if (hi == lo) return hi;
  const int top = 31 - __clz((int)(hi ^ lo));
  uint32_t T = hi & ~((2u << top) - 1u);     // (top = 31: 2u << 31 = 0, T = 0)
  for (int bit = top; bit >= 0; --bit) {
    const uint32_t c = T | (1u << bit);
    int n = 0;
#pragma unroll
    for (int u = 0; u < NV; ++u) n += __popcll(__ballot(key[u] >= c));
    if (n >= k) T = c;
    if (n == k) break;
  }
  return T;
}

// ---- the two halves of the acceptance
// The merge, one wave per hidden row: the records lm_head left of the row (one per workgroup of that
// launch) become the greedy target token, the k most probable tokens and (optionally) the softmax
// entropy.  The k best candidates can only come from
// the k records with the largest maxima, and the maxima are needed for the softmax sum anyway: so
// the wave looks for the k-th largest maximum (kth_bound) and fetches the candidates of those
// records alone, k * k instead of all (5 rows, 476 records, k = 4: 16 of 1904).  What bounds it is
// the number of instructions and dependent loads of a wave.
// The rule, one wave per chain of the sequence's draft tree (a plain chain draft is a tree with one
// branch), one lane per draft position: loosened set (Eq. 9),
// verdicts (Eq. 10 / 11), accepted length (Eq. 2) per chain, then the chain with the longest
// accepted length (appendix on draft token trees).  Everything a position needs from the others
// comes through v_readlane in a loop over the positions.
//
// Up to kAcceptOneKernelRows hidden rows per sequence, one workgroup does both (accept_finalize_kernel;
// rocprofv3, against a merge over one record per 64 vocabulary rows followed by a launch of its own for
// the rule: 5 rows, V = 152064: k = 4 9.5 + 4.8 -> 7.0 us, k = 16 28.4 + 4.6 -> 11.4).  More rows
// would take turns on the waves of one CU: then the merge is spread over the chip and the rule waits
// for it in a launch of its own (accept_merge_kernel, accept_rule_kernel; 8 chains of 8, V = 8192:
// k = 4 31.9 -> 4.0 + 3.1 us, k = 16 60.0 -> 6.8 + 4.5; with V = 152064 31.1 -> 6.1 + 4.6 and
// 60.7 -> 8.7 + 4.6; 2 chains of 10, k = 4, V = 8192 12.2 -> 4.0 + 2.6, V = 152064 11.8 -> 6.5 + 4.5).

// What the rule needs of a merged row: in LDS, or where the row's records were.
struct RowsInLds {
  int (&top)[kAcceptOneKernelRows][16];
  float (&ent)[kAcceptOneKernelRows];
  LVS_DEV void put_top(int row, int lane, int id) const { top[row][lane] = id; }
  LVS_DEV void put_ent(int row, float e) const { ent[row] = e; }
  LVS_DEV int top_at(int row, int e) const { return top[row][e]; }
  LVS_DEV float ent_at(int row) const { return ent[row]; }
};

// A row's first candidates and its first maximum have been read by the wave that puts the results
// there, and no other wave looks at them.
struct RowsInRecords {
  const AcceptFinalizeArgs& p;
  int64_t col0;     // column of row 0
  LVS_DEV int* ids(int row) const {
    return reinterpret_cast<int*>(const_cast<uint64_t*>(p.cand) + (col0 + row) * p.n_rec * p.topk);
  }
  LVS_DEV float* stat(int row) const {
    return const_cast<float*>(p.stats) + (col0 + row) * p.n_rec * 2;
  }
  LVS_DEV void put_top(int row, int lane, int id) const { ids(row)[lane] = id; }
  LVS_DEV void put_ent(int row, float e) const { *stat(row) = e; }
  LVS_DEV int top_at(int row, int e) const { return ids(row)[e]; }
  LVS_DEV float ent_at(int row) const { return *stat(row); }
};

// NR: records per lane (n_rec <= 64 * NR).
template <int NR, class Rows>
LVS_DEV void merge_row(const AcceptFinalizeArgs& p, int64_t col, int row, int lane, int* pick,
                       const Rows& rows) {
  const bool want_z = p.stats_z != nullptr;
  const int n_rec = p.n_rec;
  const float2* st = reinterpret_cast<const float2*>(p.stats) + col * n_rec;
  const uint64_t* ck = p.cand + col * n_rec * p.topk;
  // ---- softmax statistics over the records
  float2 ms[NR];
  float z[NR];
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    const int i = 64 * u + lane;
    const int ic = i < n_rec ? i : n_rec - 1;
    ms[u] = st[ic];
    z[u] = want_z ? p.stats_z[col * n_rec + ic] : 0.f;
  }
  float mx = -INFINITY;
  uint32_t mkey[NR];
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    const bool on = 64 * u + lane < n_rec;
    ms[u].x = on ? ms[u].x : -INFINITY;
    mkey[u] = ms[u].x != -INFINITY ? order_key(ms[u].x) : 0u;
    mx = fmaxf(mx, ms[u].x);
  }
  // ---- records that can hold one of the k best
  const uint32_t bound = kth_bound<NR>(mkey, p.topk);
  int picked = 0;
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    const bool q = mkey[u] >= bound;
    const unsigned long long mask = __ballot(q);
    const int slot = picked + __popcll(mask & ((1ull << lane) - 1ull));
    if (q && slot < kPickedMax) pick[slot] = 64 * u + lane;
    picked += __popcll(mask);
  }
  uint64_t top = 0ull;
  if (picked <= kPickedMax) {
    const int nk = picked * p.topk;
    for (int k0 = 0; k0 < nk; k0 += 256) {
      uint64_t key[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = k0 + 64 * u + lane;
        const int ic = i < nk ? i : nk - 1;
        const int t = (int)fast_div((uint32_t)ic, p.div_topk);
        const int e = ic - t * p.topk;
        key[u] = ck[(int64_t)pick[t] * p.topk + e];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) key[u] = k0 + 64 * u + lane < nk ? key[u] : 0ull;
      if (p.topk > kSortTopk)
        topk_take<4, true>(top, key, p.topk, lane);
      else
        topk_take<4, false>(top, key, p.topk, lane);
    }
  } else {
    // (many records share the k-th largest maximum) all candidates
    const int nk = n_rec * p.topk;
    for (int k0 = 0; k0 < nk; k0 += 256) {
      uint64_t key[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = k0 + 64 * u + lane;
        key[u] = i < nk ? ck[i] : 0ull;
      }
      if (p.topk > kSortTopk)
        topk_take<4, true>(top, key, p.topk, lane);
      else
        topk_take<4, false>(top, key, p.topk, lane);
    }
  }
  // ---- results of the row
  mx = wave_max(mx);
  float se = 0.f, sz = 0.f;
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    const float f = ms[u].x == -INFINITY ? 0.f : fast_exp2((ms[u].x - mx) * kLog2e);
    se += ms[u].y * f;
    sz += z[u] * f;
  }
  se = wave_sum(se);
  if (want_z) {
    // H = -sum p ln p with p = exp(z - max) / se:  ln se + max - (sum exp(z - max) z) / se
    sz = wave_sum(sz);
    const float ent = __logf(se) + mx - sz / se;
    if (lane == 0) {
      rows.put_ent(row, ent);
      if (p.entropy) p.entropy[col] = ent;
    }
  }
  if (lane < p.topk) {
    const bool none = top == 0ull;
    const float win_v = key_value((uint32_t)(top >> 32));
    const int id = none ? -1 : 0x7fffffff - (int)(uint32_t)top;
    const float prob = none ? 0.f : __expf(win_v - mx) / se;
    if (lane == 0) p.target_ids[col] = id;
    rows.put_top(row, lane, id);
    if (p.topk_ids) p.topk_ids[col * p.topk + lane] = id;
    if (p.topk_probs) p.topk_probs[col * p.topk + lane] = prob;
  }
}

// br: the branch of this wave.  All waves of the workgroup call it.
template <class Rows>
LVS_DEV void apply_rule(const AcceptFinalizeArgs& p, int seq, int br, int lane, const Rows& rows,
                        int (&sh_tau)[kMaxBranches]) {
  if (br < p.n_branches) {
    const int b = seq * p.n_branches + br;                 // chain index
    const int g = p.gamma;
    const bool on = lane < g;
    const int idx = b * g + (on ? lane : 0);                      // draft position of this lane
    const int row = br * p.rows + (lane < p.rows ? lane : 0);     // hidden row of this lane
    const int dk = p.draft_ids[idx];
    const int yk = rows.top_at(row, 0);
    unsigned char vd = 0;
    if (p.rule == 0) {
      const float ak = p.relevance[idx];
      int gate_ok = 1;
      if (p.gate > 0) {
        gate_ok = 0;
        for (int e = 0; e < p.gate; ++e) gate_ok |= (rows.top_at(row, e) == dk);
      }
      // position of this lane in the stable ascending order of the relevance scores (Eq. 9: the
      // n_loose first are loosened), and whether its target token occurs among the other drafts
      // within the shift window (Eq. 11)
      int rank = 0;
      bool shifted = false;
      for (int j = 0; j < g; ++j) {
        const float aj = __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ak), j));
        const int dj = __builtin_amdgcn_readlane(dk, j);
        rank += ((aj < ak) | ((aj == ak) & (j < lane))) ? 1 : 0;
        const int dist = j > lane ? j - lane : lane - j;
        shifted |= (j != lane) & (dist <= p.pst_window) & (dj == yk);
      }
      if (dk == yk) {
        vd = 1;
      } else if (rank < p.n_loose && gate_ok) {
        vd = 2;
      } else if (p.pst_window > 0 && shifted) {
        vd = 3;
      }
    } else {
      // Entropy-gated rules of the text-only loose methods the paper compares against: a
      // mismatch passes when its row's entropy exceeds the threshold and (rule 2) the w
      // positions behind it are all draft positions that match exactly.
      const float hk = rows.ent_at(row);
      const unsigned long long exact = __ballot(on && dk == yk);
      const int w = p.rule == 2 ? p.defer_window : 0;
      const unsigned long long need = ((1ull << w) - 1ull) << (on ? lane + 1 : 0);   // < 2^33
      const bool confirmed = (lane + w <= g - 1) && ((exact & need) == need);
      if (dk == yk) {
        vd = 1;
      } else if (hk > p.ent_threshold && confirmed) {
        vd = 4;
      }
    }
    if (on) p.verdict[idx] = vd;
    const unsigned long long rejected = __ballot(on && vd == 0);
    const int tau = rejected ? __ffsll((long long)rejected) - 1 : g;   // first rejected position
    // the target's token at the first rejected position, or the one after the last draft when
    // the chain brought that row
    const int bonus = __builtin_amdgcn_readlane(yk, tau < p.rows ? tau : 0);
    if (lane == 0) {
      p.accept_len[b] = tau;
      p.bonus_id[b] = tau < p.rows ? bonus : -1;
      sh_tau[br] = tau;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && p.best_branch != nullptr) {
    int best = 0;
    for (int a = 1; a < p.n_branches; ++a)
      if (sh_tau[a] > sh_tau[best]) best = a;
    p.best_branch[seq] = best;
  }
}

template <int NR>
__global__ __launch_bounds__(64 * kAcceptOneKernelRows) void accept_finalize_kernel(
    const AcceptFinalizeArgs p) {
  __shared__ int sm_pick[kAcceptOneKernelRows][kPickedMax];
  __shared__ int sh_top[kAcceptOneKernelRows][16];
  __shared__ float sh_ent[kAcceptOneKernelRows];
  __shared__ int sh_tau[kMaxBranches];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowsInLds rows{sh_top, sh_ent};
  const int R = p.n_branches * p.rows;      // hidden rows of this sequence, one per wave
  merge_row<NR>(p, (int64_t)blockIdx.x * R + wave, wave, lane, sm_pick[wave], rows);
  __syncthreads();
  apply_rule(p, blockIdx.x, wave, lane, rows, sh_tau);
}

constexpr int kMergeWaves = 4;         // one per SIMD

template <int NR>
__global__ __launch_bounds__(64 * kMergeWaves) void accept_merge_kernel(const AcceptFinalizeArgs p) {
  __shared__ int sm_pick[kMergeWaves][kPickedMax];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x * kMergeWaves + wave;
  if (row < p.B * p.rows) merge_row<NR>(p, row, row, lane, sm_pick[wave], RowsInRecords{p, 0});
}

__global__ __launch_bounds__(64 * kMaxBranches) void accept_rule_kernel(const AcceptFinalizeArgs p) {
  __shared__ int sh_tau[kMaxBranches];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int R = p.n_branches * p.rows;
  apply_rule(p, blockIdx.x, wave, lane, RowsInRecords{p, (int64_t)blockIdx.x * R}, sh_tau);
}

// ------------------------------------------------------------------------------------------
// Two-kernel Top-N for N <= 16 and up to 65536 video rows: the row is cut into slices of 1024
// video tokens, one small workgroup per (slice, draft row) keeps the slice's N largest scores
// (rel_cand_kernel, hundreds of workgroups spread over the chip), and one workgroup per draft
// row takes the N largest of the slices' lists (rel_merge_kernel).  The single-workgroup kernel
// above does all of a row's work on one CU, which at 63488 video rows is 54 us of mostly
// serial latency.
//
// Scores are ranked as s = dot * rsqrt(max(|v|^2, 1e-16)); the cosine is s / |h_d| with
// |h_d| > 0 constant over the row, so the order is the same, and the merge kernel applies the
// factor to the N winners (the same floating-point operations, in the same order, as the
// single-kernel path: both give the same bits).
template <int NS, bool MULTI>
__global__ __launch_bounds__(256) void rel_cand_kernel(const RelFinalizeArgs p) {
  __shared__ uint32_t sm_top[4][kRelSmallN];
  const int part = blockIdx.x;
  const int i = blockIdx.y;
  const int b = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lv = p.l_v[b];
  if (lv > p.lv_max) lv = (int)p.lv_max;
  const int n = p.top_n;
  uint32_t* out = p.cand_keys + (((int64_t)b * p.gamma + i) * p.n_parts + part) * kRelSmallN;
  const int j0 = part * p.slice_rows;
  if (j0 >= lv) {   // slice past the sequence's video tokens: an empty list
    if (tid < kRelSmallN) out[tid] = 0u;
    return;
  }
  const float* dbase = p.dots + (((int64_t)b * p.n_ds) * p.gamma + i) * p.ld;
  const bool pre = p.inv_norm != nullptr;   // prepared inverse norms instead of squared norms
  const float* nbase = pre ? p.inv_norm + (int64_t)b * p.lv_max
                           : p.nv2 + ((int64_t)b * p.n_ds) * p.ld;
  const int64_t nstep = pre ? 0 : p.ld;
  const int64_t dstep = (int64_t)p.gamma * p.ld;
  // The slice is taken 1024 rows (four per thread) at a time; MULTI: slices of several such
  // chunks (more than 65536 video rows), each wave carrying its list of the n largest so far
  // (one entry per lane) into the selection of the next chunk.
  constexpr int NK = MULTI ? 5 : 4;
  const int jend = j0 + p.slice_rows < lv ? j0 + p.slice_rows : lv;
  for (int jc = j0; jc < jend; jc += kRelSliceRows) {
    float dv[4][NS], nv[4][NS];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = jc + u * 256 + tid;
      const uint32_t off = (uint32_t)(j < lv ? j : lv - 1) * 4u;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int sc = s < p.n_ds ? s : 0;
        dv[u][s] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(dbase + sc * dstep) + off);
        nv[u][s] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(nbase + sc * nstep) + off);
      }
    }
    uint32_t k[NK];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float dot = dv[u][0], n2 = nv[u][0];
#pragma unroll
      for (int s = 1; s < NS; ++s) {
        const float ws = s < p.n_ds ? 1.f : 0.f;
        dot = __builtin_fmaf(dv[u][s], ws, dot);
        n2 = __builtin_fmaf(nv[u][s], pre ? 0.f : ws, n2);
      }
      const float sc = dot * (pre ? n2 : __builtin_amdgcn_rsqf(fmaxf(n2, 1e-16f)));
      k[u] = jc + u * 256 + tid < jend ? order_key(sc) : 0u;
    }
    if constexpr (MULTI) k[4] = (jc > j0 && lane < n) ? sm_top[wave][lane] : 0u;
    // the n largest of this wave's scores so far (copies included) ...
    int got = 0;
    while (got < n) {
      int copies;
      const uint32_t w = take_largest(k, copies);
      if (w == 0u) break;
      if (lane < copies && got + lane < n) sm_top[wave][got + lane] = w;
      got += copies;
    }
    if (lane < kRelSmallN && lane >= got) sm_top[wave][lane] = 0u;
    if constexpr (!MULTI) break;
  }
  __syncthreads();
  if (wave != 0) return;
  // ... and of the four waves' lists
  uint32_t cur = (lane & (kRelSmallN - 1)) < n ? sm_top[lane / kRelSmallN][lane & (kRelSmallN - 1)]
                                               : 0u;
  int got = 0;
  while (got < n) {
    const uint32_t w = wave_max_u32(cur);
    if (w == 0u) break;
    const int copies = __popcll(__ballot(cur == w));
    if (lane < copies && got + lane < n) out[got + lane] = w;
    cur = cur == w ? 0u : cur;
    got += copies;
  }
  if (lane < kRelSmallN && lane >= (got < n ? got : n)) out[lane] = 0u;
}

__global__ __launch_bounds__(256) void rel_merge_kernel(const RelFinalizeArgs p) {
  __shared__ float red[4];
  __shared__ uint32_t sm_top[4][kRelSmallN];
  const int i = blockIdx.x;
  const int b = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lv = p.l_v[b];
  if (lv > p.lv_max) lv = (int)p.lv_max;
  float* rel_out = p.relevance + (int64_t)b * p.gamma + i;
  if (lv <= 0) {
    if (tid == 0) *rel_out = 0.f;
    return;
  }
  const int n_eff = p.top_n < lv ? p.top_n : lv;
  // the slices' lists: n_parts * 16 keys, four per thread (n_parts <= 64)
  const uint32_t* keys = p.cand_keys + ((int64_t)b * p.gamma + i) * p.n_parts * kRelSmallN;
  const int total = p.n_parts * kRelSmallN;
  uint32_t k4[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int idx = u * 256 + tid;
    k4[u] = keys[idx < total ? idx : total - 1];
  }
  // |h_d row| while the keys are on their way
  const uint16_t* hd = p.h_d + (int64_t)b * p.hd_sb + (int64_t)i * p.hd_sg;
  float part = 0.f;
  for (int t = tid * 8; t < p.d; t += 256 * 8) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(hd + t);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __builtin_bit_cast(float, w[e] << 16);
      const float hi = __builtin_bit_cast(float, w[e] & 0xffff0000u);
      part = __builtin_fmaf(lo, lo, part);
      part = __builtin_fmaf(hi, hi, part);
    }
  }
  part = wave_sum(part);
  if (lane == 0) red[wave] = part;
#pragma unroll
  for (int u = 0; u < 4; ++u) k4[u] = u * 256 + tid < total ? k4[u] : 0u;
  int got = 0;
  while (got < n_eff) {
    int copies;
    const uint32_t w = take_largest(k4, copies);
    if (w == 0u) break;
    if (lane < copies && got + lane < n_eff) sm_top[wave][got + lane] = w;
    got += copies;
  }
  if (lane < kRelSmallN && lane >= got) sm_top[wave][lane] = 0u;
  __syncthreads();
  if (wave != 0) return;
  const float inv_nd = 1.0f / fmaxf(sqrtf(((red[0] + red[1]) + red[2]) + red[3]), 1e-8f);
  uint32_t cur = (lane & (kRelSmallN - 1)) < n_eff
                     ? sm_top[lane / kRelSmallN][lane & (kRelSmallN - 1)]
                     : 0u;
  long long tot = 0;
  got = 0;
  while (got < n_eff) {
    const uint32_t w = wave_max_u32(cur);
    if (w == 0u) break;
    const int copies = __popcll(__ballot(cur == w));
    const int take = copies < n_eff - got ? copies : n_eff - got;
    tot += (long long)take * (long long)(key_value(w) * inv_nd * kFixScale);
    cur = cur == w ? 0u : cur;
    got += copies;
  }
  if (lane == 0) *rel_out = (float)((double)tot / (double)kFixScale / (double)n_eff);
}

// ------------------------------------------------------------------------------------------
constexpr int kRelKeepN = 128;
constexpr int kRelOneKernelRows = 4096;

// Two-kernel Top-N for 16 < N <= 128 and 4097 to 65536 video rows.  One CU that reads a row's dot products
// and norms alone is bound by its own requests in flight (rel_finalize_kernel: 230 KB at 14336 rows
// in two splits), and the scores are needed once: so a workgroup per (slice, draft row) makes the
// scores of 1024 (4096) video rows and leaves those that can be among the N largest, and one
// workgroup per draft row selects among these.  At least N scores reach the N-th largest of the
// threads' maxima (all scores, where there are fewer maxima than N).  The kept keys take the slice's
// places of the cosine plane, their number the place of the slice's first dot product, which no one
// else reads.  Scores rank like cosines and the N winners are the same, see rel_cand_kernel.
// Both kernels are chains of latencies.  Per call against rel_finalize_kernel, N = 100: 14336 rows,
// d = 5120, 5 draft rows (two splits) 42.6 -> 38.1 us; d = 1024: 8192 rows 20.5 -> 18.8, 63488 rows
// 49.8 -> 34.4, 8 x 30000 rows with 8 draft rows each 100 -> 92; also where few of the rows are in use
// (100 of 14336: 17.0 -> 12.7).  Up to 4096 rows the kernels gain about 1 us (4096 rows 18.7 -> 17.6)
// and a caller that is bound by its launches loses more on the third (234 rows from Python 18.5 ->
// 20.2).  N > 128: a slice would keep most of its scores, and selecting among more than are held in
// LDS costs more than the one kernel (N = 1000, 14336 rows: 26.7 us there, 34.3 here).
template <int NS, int M>
__global__ __launch_bounds__(256) void rel_keep_kernel(const RelFinalizeArgs p) {
  __shared__ uint32_t tmax[256];
  __shared__ int kept;
  const int part = blockIdx.x;
  const int i = blockIdx.y;
  const int b = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  int lv = p.l_v[b];
  if (lv > p.lv_max) lv = (int)p.lv_max;
  const int j0 = part * M * kRelSliceRows;
  if (j0 >= lv) return;
  float* dbase = const_cast<float*>(p.dots) + (((int64_t)b * p.n_ds) * p.gamma + i) * p.ld;
  const bool pre = p.inv_norm != nullptr;   // prepared inverse norms instead of squared norms
  const float* nbase = pre ? p.inv_norm + (int64_t)b * p.lv_max
                           : p.nv2 + ((int64_t)b * p.n_ds) * p.ld;
  const int64_t nstep = pre ? 0 : p.ld;
  const int64_t dstep = (int64_t)p.gamma * p.ld;
  uint32_t k[4 * M];
#pragma unroll
  for (int c = 0; c < M; ++c) {
    const int jc = j0 + c * kRelSliceRows;
    float dv[4][NS], nv[4][NS];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = jc + u * 256 + tid;
      const uint32_t off = (uint32_t)(j < lv ? j : lv - 1) * 4u;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int sc = s < p.n_ds ? s : 0;
        dv[u][s] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(dbase + sc * dstep) + off);
        nv[u][s] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(nbase + sc * nstep) + off);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float dot = dv[u][0], n2 = nv[u][0];
#pragma unroll
      for (int s = 1; s < NS; ++s) {
        const float ws = s < p.n_ds ? 1.f : 0.f;
        dot = __builtin_fmaf(dv[u][s], ws, dot);
        n2 = __builtin_fmaf(nv[u][s], pre ? 0.f : ws, n2);
      }
      const float sc = dot * (pre ? n2 : __builtin_amdgcn_rsqf(fmaxf(n2, 1e-16f)));
      k[4 * c + u] = jc + u * 256 + tid < lv ? order_key(sc) : 0u;
    }
  }
  uint32_t most = k[0];
#pragma unroll
  for (int u = 1; u < 4 * M; ++u) most = max(most, k[u]);
  tmax[tid] = most;
  if (tid == 0) kept = 0;
  __syncthreads();
  uint32_t m4[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) m4[u] = tmax[64 * u + lane];
  const uint32_t bound = kth_bound<4>(m4, p.top_n);
  unsigned long long mask[4 * M];
  int n = 0;
#pragma unroll
  for (int u = 0; u < 4 * M; ++u) {
    mask[u] = __ballot(k[u] >= bound);       // bound >= 1: no row past the last
    n += __popcll(mask[u]);
  }
  int at = 0;
  if (lane == 0) at = atomicAdd(&kept, n);
  at = __builtin_amdgcn_readfirstlane(at);
  uint32_t* out = reinterpret_cast<uint32_t*>(p.cosbuf + ((int64_t)b * p.gamma + i) * p.ld) + j0;
#pragma unroll
  for (int u = 0; u < 4 * M; ++u) {
    if ((mask[u] >> lane) & 1ull) out[at + __popcll(mask[u] & ((1ull << lane) - 1ull))] = k[u];
    at += __popcll(mask[u]);
  }
  __syncthreads();                           // every dot product of the slice has been read
  if (tid == 0) dbase[j0] = __builtin_bit_cast(float, kept);
}

// As radix_select, for keys in LDS between lo and hi: the digits start at the first bit in which keys
// differ, one wave adds a histogram up over the DPP network, and the search ends when all keys of
// the digit it is down to are among the n largest (after two digits as a rule): the key returned is
// then the largest one below, with none of its copies needed.  hi, lo: the same in all threads.
LVS_DEV uint32_t select_in_lds(const uint32_t* keys, int count, int n, uint32_t hi, uint32_t lo,
                               SelectScratch& sc, uint32_t* need_eq) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  uint32_t* hist = &sc.hist[0][0];                 // four histograms, by wave
  if (hi == lo) {
    *need_eq = (uint32_t)n;
    return hi;
  }
  const int top = 31 - __clz((int)(hi ^ lo));
  uint32_t mask = top == 31 ? 0u : 0xffffffffu << (top + 1);   // bits that are settled
  uint32_t prefix = hi & mask;
  uint32_t rem = (uint32_t)n;
  int shift = top > 7 ? top - 7 : 0;
  while (true) {
    hist[tid] = 0u;
    __syncthreads();
    for (int idx = tid; idx < count; idx += kFinThreads) {
      const uint32_t k = keys[idx];
      if ((k & mask) == prefix)
        atomicAdd(&hist[((tid >> 6) & 3) * 256 + ((k >> shift) & 0xffu)], 1u);
    }
    __syncthreads();
    if (tid < 64) {
      // lane l: digits 255 - 4 l .. 252 - 4 l
      uint32_t own[4], sum = 0u;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int d = 255 - 4 * lane - u;
        own[u] = (hist[d] + hist[256 + d]) + (hist[512 + d] + hist[768 + d]);
        sum += own[u];
      }
      uint32_t upto = sum;
      upto += dpp_move<0x111, 0xf>(0u, upto);    // inclusive sums: row shifts, row broadcasts
      upto += dpp_move<0x112, 0xf>(0u, upto);
      upto += dpp_move<0x114, 0xf>(0u, upto);
      upto += dpp_move<0x118, 0xf>(0u, upto);
      upto += dpp_move<0x142, 0xa>(0u, upto);
      upto += dpp_move<0x143, 0xc>(0u, upto);
      uint32_t above = upto - sum;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (above < rem && above + own[u] >= rem) {
          sc.prefix = prefix | ((uint32_t)(255 - 4 * lane - u) << shift);
          sc.remaining = rem - above;              // keys of this digit still needed
          sc.wave_tot[0] = own[u];                 // keys of this digit
        }
        above += own[u];
      }
    }
    __syncthreads();
    prefix = sc.prefix;
    rem = sc.remaining;
    const uint32_t in_digit = sc.wave_tot[0];
    if (shift == 0) {
      *need_eq = rem;
      return prefix;
    }
    if (rem == in_digit) {
      *need_eq = 0u;
      return prefix != 0u ? prefix - 1u : 0u;      // (keys are above 0)
    }
    mask = 0xffffffffu << shift;
    shift = shift > 8 ? shift - 8 : 0;
  }
}

// Slices of `rows` video rows.
__global__ __launch_bounds__(kFinThreads) void rel_take_kernel(const RelFinalizeArgs p, int rows) {
  constexpr int kWaves = kFinThreads / 64;
  constexpr int kOwn = kRelMaxParts / kWaves;   // slices of a wave
  constexpr int kAtOnce = 4;                    // keys per lane and slice asked for together
  __shared__ float red[kWaves];
  __shared__ SelectScratch sc;
  __shared__ uint32_t sm_hi[kWaves], sm_nlo[kWaves];
  __shared__ uint32_t cand[kCandCap];
  __shared__ int sm_count[kRelMaxParts];
  __shared__ long long fix_part[kWaves];
  const int i = blockIdx.x;
  const int b = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lv = p.l_v[b];
  if (lv > p.lv_max) lv = (int)p.lv_max;
  float* rel_out = p.relevance + (int64_t)b * p.gamma + i;
  if (lv <= 0) {
    if (tid == 0) *rel_out = 0.f;
    return;
  }
  const int n_eff = p.top_n < lv ? p.top_n : lv;
  const int parts = (lv + rows - 1) / rows;      // at most kRelMaxParts
  const float* dbase = p.dots + (((int64_t)b * p.n_ds) * p.gamma + i) * p.ld;
  const uint32_t* keys = reinterpret_cast<const uint32_t*>(p.cosbuf + ((int64_t)b * p.gamma + i) * p.ld);
  // lane l: number of keys of slice l
  int count = __builtin_bit_cast(int, dbase[(int64_t)(lane < parts ? lane : 0) * rows]);
  // |h_d row|^2 as in rel_finalize_kernel, while the counts are on their way
  const uint16_t* hd = p.h_d + (int64_t)b * p.hd_sb + (int64_t)i * p.hd_sg;
  float part = 0.f;
  for (int t = tid * 8; t < p.d; t += kFinThreads * 8) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(hd + t);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __builtin_bit_cast(float, w[e] << 16);
      const float hi = __builtin_bit_cast(float, w[e] & 0xffff0000u);
      part = __builtin_fmaf(lo, lo, part);
      part = __builtin_fmaf(hi, hi, part);
    }
  }
  count = lane < parts ? count : 0;
  int end = count;                               // keys of slices 0 .. lane
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(end, off, 64);
    if (lane >= off) end += o;
  }
  const int total = __builtin_amdgcn_readlane(end, 63);
  if (wave == 0) sm_count[lane] = count;
  if (total <= kCandCap) {
    uint32_t key[kOwn][kAtOnce];
    uint32_t hi = 0u, nlo = 0u;      // largest key and largest complement
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      const int s = wave + kWaves * o;
      const int c = __builtin_amdgcn_readlane(count, s);
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u)
        if (64 * u + lane < c) key[o][u] = keys[s * rows + 64 * u + lane];
    }
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      const int s = wave + kWaves * o;
      const int c = __builtin_amdgcn_readlane(count, s);
      const int at = __builtin_amdgcn_readlane(end, s) - c;
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u)
        if (64 * u + lane < c) {
          cand[at + 64 * u + lane] = key[o][u];
          hi = max(hi, key[o][u]);
          nlo = max(nlo, ~key[o][u]);
        }
      for (int t = 64 * kAtOnce + lane; t < c; t += 64) {
        const uint32_t k = keys[s * rows + t];
        cand[at + t] = k;
        hi = max(hi, k);
        nlo = max(nlo, ~k);
      }
    }
    hi = wave_max_u32(hi);
    nlo = wave_max_u32(nlo);
    if (lane == 0) {
      sm_hi[wave] = hi;
      sm_nlo[wave] = nlo;
    }
  }
  part = wave_sum(part);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  float nd2 = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) nd2 += red[w];
  const float inv_nd = 1.0f / fmaxf(sqrtf(nd2), 1e-8f);
  uint32_t need_eq, tkey;
  long long fix = 0;     // sum of the values above the n-th largest, exact in 2^-40 units
  auto add = [&](uint32_t k) {
    if (k > tkey) fix += (long long)(key_value(k) * inv_nd * kFixScale);
  };
  if (total <= kCandCap) {
    uint32_t hi = 0u, nlo = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      hi = max(hi, sm_hi[w]);
      nlo = max(nlo, sm_nlo[w]);
    }
    tkey = select_in_lds(cand, total, n_eff, hi, ~nlo, sc, &need_eq);
    for (int idx = tid; idx < total; idx += kFinThreads) add(cand[idx]);
  } else {
    // (many equal values at the bounds) over the kept keys where they are
    const int shift = 31 - __clz(rows);            // rows: a power of two
    const int all = (parts - 1) * rows + sm_count[parts - 1];
    auto key_at = [&](int idx) {
      return (idx & (rows - 1)) < sm_count[idx >> shift] ? keys[idx] : 0u;
    };
    tkey = radix_select(all, n_eff, key_at, sc, &need_eq);
    for (int idx = tid; idx < all; idx += kFinThreads) add(key_at(idx));
  }
  // integer addition is associative: any reduction order gives the same bits
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) fix += __shfl_xor(fix, sft, 64);
  if (lane == 0) fix_part[wave] = fix;
  __syncthreads();
  if (tid == 0) {
    long long tot = 0;
    for (int w = 0; w < kWaves; ++w) tot += fix_part[w];
    tot += (long long)need_eq * (long long)(key_value(tkey) * inv_nd * kFixScale);
    *rel_out = (float)((double)tot / (double)kFixScale / (double)n_eff);
  }
}

}  // namespace

hipError_t launch_rel_finalize(const RelFinalizeArgs& a, hipStream_t stream) {
  static_assert(kRelSmallN == kSmallN, "same small-N bound on both paths");
  if (a.top_n <= kRelSmallN && a.n_parts >= 1 && a.n_parts <= kRelMaxParts &&
      a.slice_rows >= kRelSliceRows && a.slice_rows % kRelSliceRows == 0) {
    const dim3 grid(a.n_parts, a.gamma, a.B);
    const bool multi = a.slice_rows > kRelSliceRows;
    if (a.n_ds == 1) {
      if (multi) hipLaunchKernelGGL((rel_cand_kernel<1, true>), grid, dim3(256), 0, stream, a);
      else hipLaunchKernelGGL((rel_cand_kernel<1, false>), grid, dim3(256), 0, stream, a);
    } else if (a.n_ds == 2) {
      if (multi) hipLaunchKernelGGL((rel_cand_kernel<2, true>), grid, dim3(256), 0, stream, a);
      else hipLaunchKernelGGL((rel_cand_kernel<2, false>), grid, dim3(256), 0, stream, a);
    } else {
      if (multi) hipLaunchKernelGGL((rel_cand_kernel<8, true>), grid, dim3(256), 0, stream, a);
      else hipLaunchKernelGGL((rel_cand_kernel<8, false>), grid, dim3(256), 0, stream, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rel_merge_kernel, dim3(a.gamma, a.B), dim3(256), 0, stream, a);
    return hipGetLastError();
  }
  if (a.top_n > kSmallN && a.top_n <= kRelKeepN && a.lv_max > kRelOneKernelRows &&
      a.lv_max <= 16 * 4 * (int64_t)kRelSliceRows) {
    // longer slices where the kept keys of short ones (about 1.3 N each) would not fit
    const bool longer = a.lv_max > 20 * kRelSliceRows;
    const int rows = longer ? 4 * kRelSliceRows : kRelSliceRows;
    const dim3 grid((unsigned)((a.lv_max + rows - 1) / rows), a.gamma, a.B);
#define LVS_KEEP(NS)                                                                           \
  if (longer) hipLaunchKernelGGL((rel_keep_kernel<NS, 4>), grid, dim3(256), 0, stream, a);     \
  else hipLaunchKernelGGL((rel_keep_kernel<NS, 1>), grid, dim3(256), 0, stream, a)
    if (a.n_ds == 1) {
      LVS_KEEP(1);
    } else if (a.n_ds == 2) {
      LVS_KEEP(2);
    } else {
      LVS_KEEP(8);
    }
#undef LVS_KEEP
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rel_take_kernel, dim3(a.gamma, a.B), dim3(kFinThreads), 0, stream, a, rows);
    return hipGetLastError();
  }
  if (a.top_n <= kSmallN)
    hipLaunchKernelGGL(rel_finalize_kernel<true>, dim3(a.gamma, a.B), dim3(kFinThreads), 0, stream,
                       a);
  else
    hipLaunchKernelGGL(rel_finalize_kernel<false>, dim3(a.gamma, a.B), dim3(kFinThreads), 0,
                       stream, a);
  return hipGetLastError();
}

template <int NR>
static void launch_accept(const AcceptFinalizeArgs& a, hipStream_t stream) {
  const int R = a.n_branches * a.rows;
  if (R <= kAcceptOneKernelRows) {
    hipLaunchKernelGGL(accept_finalize_kernel<NR>, dim3(a.B / a.n_branches), dim3(64 * R), 0, stream,
                       a);
    return;
  }
  hipLaunchKernelGGL(accept_merge_kernel<NR>, dim3((a.B * a.rows + kMergeWaves - 1) / kMergeWaves),
                     dim3(64 * kMergeWaves), 0, stream, a);
  hipLaunchKernelGGL(accept_rule_kernel, dim3(a.B / a.n_branches), dim3(64 * a.n_branches), 0, stream,
                     a);
}

hipError_t launch_accept_finalize(const AcceptFinalizeArgs& a, hipStream_t stream) {
  static_assert(kRecRegs * 64 == kAcceptMaxRecords, "records per lane");
  const int R = a.n_branches * a.rows;
  if (R > kAcceptMaxRows || a.topk > 16 || a.n_rec > kAcceptMaxRecords || a.n_branches > kMaxBranches)
    return hipErrorInvalidValue;
  if (a.n_rec <= 64 * 2) launch_accept<2>(a, stream);
  else launch_accept<kRecRegs>(a, stream);
  return hipGetLastError();
}

}  // namespace lvspec
