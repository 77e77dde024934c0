// Attention of 65 to 128 query rows of a kv head by one workgroup (attn_segment32), on 32x32 MFMA tiles.
//
// HBM is the floor: it delivers the 32 KiB of a round (64 keys) in 2600 cycles.  By 128 rows that are 1090 cycles
// of each SIMD's matrix core and about 1200 of its vector unit, which fit under the copy only as far as they
// overlap it and each other; a round takes about 3000.  The 64-row variant of attn_segment takes such rows in
// two chunks, each a workgroup with copies of its own, and spends 5700 cycles on 128 keys by 64 rows, waiting
// on one instruction chain after the other.  Here all rows share one copy of each tile:
//   Eight waves, four groups of 32 rows by two streams of keys; the lane layout of a 32x32 result
//   (one query row and sixteen keys per lane) is the operand layout of the second product up to an
//   order of the keys that both of its operands share, so probabilities stay in their lane.
//   V tiles are read transposed (ds_read_b64_tr_b16): no byte permutes.
//   The reads and the softmax of a round, and the products behind them (scores of the next round, then
//   the output), are two halves; the second four waves, one on each SIMD next to one of the first four,
//   run half a round late, so that one wave's products cover the other's vector work.
// Per call, in two chunks and here: tree of 2 x 10 rows, 40 / 8 heads, 16384 keys 27.5 -> 25.1 us (23.7 with
// attn_combine32_kernel), 65536 keys 76.6 -> 59.8; 4 x 30000 keys, 64 / 8 heads, 10 rows 113.7 -> 95.0; 24
// sequences of 3000 to 8750 keys, 28 / 4 heads, 14 rows 83.2 -> 65.6.  Tried on the 4 x 30000 keys: 64 rows per
// wave and four waves (113), both halves behind barriers of their own (116), waves without the half-round offset (100), a
// running maximum with slack 8 (the branch below is then rare: 92, but the probabilities lose the exact
// one of their largest, error against 64 bits 2.15e-3 -> 2.32e-3), the same with probabilities split into
// two bf16 (1.66e-3, 107 us); the rescaling of the output among the matrix instructions of the scores (96).
// Only K(0), V(0) and K(1) are requested before K(0) has landed: 16384 keys, 128 rows 26.9 -> 26.0 us.
#pragma once

#include "lvspec_dev.h"
#include "lvspec_kernels.h"

namespace lvspec {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// D[m][n] += sum_k A[m][k] * B[k][n], 32x32 output, 16-deep, bf16 in, fp32 accumulate.  Lane l: A holds
// row m = l % 32, k = 8*(l/32) .. +7; B holds column n = l % 32, same k; D holds column n = l % 32,
// element r is row m = 8*(r/4) + 4*(l/32) + r%4.
LVS_DEV f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Sixteen lanes read a block of 4 rows x 16 columns (lane i: row i / 4, columns 4*(i%4) .. +3) and get
// it transposed: lane i column i, element j row j.
LVS_DEV u32x2 lds_load_tr(uint32_t a) {
  return __builtin_bit_cast(
      u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)a));
}

// The 16-byte chunk c of tile row r sits at c ^ rows32_swz(r).  A transposed read takes four
// consecutive rows by four chunks per half wave: bits 2-3 of the key separate the rows (the four
// quarters of 64 banks).  The K operand reads take one chunk of 16 rows that differ in r & 15: any
// key that is one-to-one there serves them.
LVS_DEV constexpr int rows32_swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// RG: row groups of 32 (waves with rows of their own); KS: streams (waves with keys of their own);
// SL: ring slots of K and of V.  A round is a tile of 32 keys per stream.
template <int RG, int KS, int SL>
struct Rows32 {
  static constexpr int kWaves = RG * KS;
  static constexpr int kTile = 32 * kRowBytes;          // K or V rows of one stream
  static constexpr int kHalf = KS * kTile;              // K or V rows of a round
  static constexpr int kRing = 2 * SL * kHalf;
  static constexpr int kCopies = 8 / RG;                // copy instructions per wave, round and K / V
  static constexpr int kRows = 32 * RG;
  static constexpr int kMergeStride = 132;
  static constexpr size_t kMerge = sizeof(float) * KS * kRows * (3 + kMergeStride);
  static constexpr size_t kLds = kRing > (int)kMerge ? (size_t)kRing : kMerge;
  static_assert(kLds <= 160 * 1024, "LDS of one CU");
};

// wait until at most n halves' copies (STEP each) of this wave are under way; uniform n >= 0
template <int STEP, int MAXN>
LVS_DEV void wait_copies_upto(int n) {
  if constexpr (MAXN <= 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    if (n >= MAXN)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAXN * STEP) : "memory");
    else
      wait_copies_upto<STEP, MAXN - 1>(n);
  }
}

// As attn_segment: tiles t_begin .. t_end - 1 of one unit by the whole workgroup.  The ring's start is
// aligned to 256 bytes (chunk numbers are exchanged in addresses).
template <int RG, int KS, int SL, class Args, class Record>
LVS_DEV void attn_segment32(const Args& p, uint8_t* smem, int lane, int wave, int b, int kvh,
                            int rc, int L, int gamma, int t_begin, int t_end,
                            const uint8_t* kbase, const uint8_t* vbase, int64_t rsb,
                            Record&& record) {
  using W = Rows32<RG, KS, SL>;
  constexpr int NT = 64 * W::kWaves;
  const int stream = wave % KS;
  const int rg = wave / KS;
  const bool late = wave >= W::kWaves / 2;     // waves w and w + 4 share a SIMD
  const int n32 = lane & 31;
  const int h = lane >> 5;
  const int n16 = lane & 15;
  const int g4 = lane >> 4;
  const int rpad = p.rpad;
  const int n_rounds = (t_end - t_begin + KS - 1) / KS;
  // rows that this workgroup may copy: those of its tiles that exist
  const int n_keys = L + gamma;
  const int last_row = (t_end * 32 < n_keys ? t_end * 32 : n_keys) - 1;
  const uint32_t ring = lds_addr(smem);

  // ---- copies: wave w takes rows w * 32 / RG .. of the round's 32 * KS
  const int crow = wave * (4 * W::kCopies) + g4;        // + 4 * jj
  const uint8_t* krow[W::kCopies];
#pragma unroll
  for (int jj = 0; jj < W::kCopies; ++jj)
    krow[jj] = kbase + (int64_t)(t_begin * 32 + crow + 4 * jj) * rsb +
               ((n16 ^ rows32_swz((crow + 4 * jj) & 15)) << 4);
  const int64_t v_minus_k = vbase - kbase;
  const int64_t step = (int64_t)(32 * KS) * rsb;
  const int n_full = (last_row + 1 - t_begin * 32) / (32 * KS);    // rounds whose rows all exist
  // K (which = 0) or V (1) of a round
  auto issue = [&](int which, int round) {
    const uint32_t dst = ring + (which * SL + round % SL) * W::kHalf + wave * (W::kCopies * 1024);
    if (round < n_full) {
      const int64_t off = round * step + (which ? v_minus_k : 0);
#pragma unroll
      for (int jj = 0; jj < W::kCopies; ++jj) dma16_untracked(krow[jj] + off, dst + jj * 1024);
    } else {
      int cr = crow, nn = n16;
      asm volatile("" : "+v"(cr), "+v"(nn));      // (runs once: keep its arithmetic out of the loop)
      const int row0 = (t_begin + round * KS) * 32;
#pragma unroll
      for (int jj = 0; jj < W::kCopies; ++jj) {
        int row = row0 + cr + 4 * jj;
        row = row < last_row ? row : last_row;
        dma16_untracked((which ? vbase : kbase) + (int64_t)row * rsb +
                      ((nn ^ rows32_swz((cr + 4 * jj) & 15)) << 4), dst + jj * 1024);
      }
    }
  };
  if (n_rounds > 0) issue(0, 0);

  // ---- query operand (rows past the last one read a valid row and become zero)
  u32x4 qreg[8];
  const int r = rc * rpad + rg * 32 + n32;
  const bool valid = rg * 32 + n32 < rpad && r < p.R;
  const int rcl = r < p.R ? r : p.R - 1;
  const int qi = (int)fast_div((uint32_t)rcl, FastDiv{p.div_g.mul, p.div_g.shift});
  const int draft_row = valid ? qi : -1;
  {
    const uint16_t* qp = p.q + (int64_t)b * p.q_sb + (int64_t)qi * p.q_sg +
                         (int64_t)(kvh * p.G + (rcl - qi * p.G)) * p.q_sh;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      qreg[ks] = *reinterpret_cast<const u32x4*>(qp + (2 * ks + h) * 8);
  }
  const float c = p.scale_log2e;
  int vis_b = 0, vis_e = 0;
  if (p.vis_begin != nullptr) {
    vis_b = p.vis_begin[b];
    vis_e = p.vis_end[b];
  }
  uint32_t rowmask = 0;
#pragma unroll
  for (int j = 0; j < 32; ++j) rowmask = (draft_row == j) ? p.draft_mask[j] : rowmask;
  rowmask &= 0xffffffffu >> (32 - gamma);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    qreg[ks] = draft_row >= 0 ? qreg[ks] : u32x4{0u, 0u, 0u, 0u};
    asm volatile("" : "+v"(qreg[ks]));
  }
  // (every load so far has been waited for: from here on the counters see copies only)
  int issued = 0;                       // halves behind K(0): V0 K1 | V1 K2 | ...
  auto request = [&](int round) {       // V of it and K of the next one
    if (round >= n_rounds) return;
    issue(1, round);
    ++issued;
    if (round + 1 >= n_rounds) return;
    issue(0, round + 1);
    ++issued;
  };
  request(0);

  // LDS addresses of the operand reads
  const uint32_t ka = (uint32_t)(stream * W::kTile + n32 * kRowBytes + ((h ^ rows32_swz(n32 & 15)) << 4));
  uint32_t va;
  {
    const int rr = (lane & 15) >> 2;
    const int g1 = (lane >> 4) & 1;
    const int chunk = (2 * g1 + ((lane & 3) >> 1)) ^ ((rr << 2) | h);
    va = (uint32_t)(SL * W::kHalf + stream * W::kTile + (4 * h + rr) * kRowBytes + (chunk << 4) + (lane & 1) * 8);
  }

  f32x16 acc[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
  float m = -1.0e30f, l = 0.f, lvis = 0.f;
  const bool has_rows = rg * 32 < rpad && rc * rpad + rg * 32 < p.R;

  f32x16 s;             // scores of the round at hand: element e is key 8*(e/4) + 4*h + e%4, row n32
  u32x4 kop[8];
  u32x4 vop[4][2];
  u32x4 pop[2];
  auto scores = [&] {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) s = mfma32(kop[ks], qreg[ks], s);
  };
  auto read_k = [&](int round) {
    const uint32_t a = ring + (round % SL) * W::kHalf + ka;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kop[ks] = lds_load16(a ^ (ks << 5));
  };
  // Interval t begins when V(t) and K(t+1) have landed and the slots of V(t-1) and K(t) are free.  In it
  // every wave reads V(t) and K(t+1) and takes the softmax of round t; the products behind that, scores
  // of round t+1 and output of round t, come last in it or, in the late waves, first in the next one.
  auto enter = [&](int t) {
    const int need = t + 1 < n_rounds ? 2 * t + 2 : 2 * t + 1;
    wait_copies_upto<W::kCopies, 2 * (SL - 2)>(issued - need);
    lds_barrier();
    request(t + SL - 1);
  };
  auto multiply = [&](int round) {
    if (!(has_rows && t_begin + round * KS + stream < t_end)) return;
    __builtin_amdgcn_sched_barrier(0);
    scores();        // of the next round (behind the last one: of stale operands, unused)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int db = 0; db < 4; ++db) acc[db] = mfma32(vop[db][kt], pop[kt], acc[db]);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (n_rounds > 0) {
    wait_copies_upto<W::kCopies, 2>(issued);
    asm volatile("s_barrier" ::: "memory");
    read_k(0);
#pragma unroll
    for (int i = 1; i < SL - 1; ++i) request(i);
    scores();
    if (late) enter(0);
  }
  for (int round = 0; round < n_rounds; ++round) {
    if (!late) enter(round);
    const int tile = t_begin + round * KS + stream;
    const int key0 = tile * 32;
    if (has_rows && tile < t_end) {     // (past the end: only in the last round)
      if (round + 1 < n_rounds) read_k(round + 1);
      const uint32_t a0 = ring + (round % SL) * W::kHalf + va;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int db = 0; db < 4; ++db) {
          const uint32_t a = a0 ^ (db << 6);
          const u32x2 lo = lds_load_tr(a + kt * (16 * kRowBytes));
          const u32x2 hi = lds_load_tr((a ^ 32) + (kt * 16 + 8) * kRowBytes);
          vop[db][kt] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
      if (key0 + 32 > L) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = key0 + 8 * (e >> 2) + 4 * h + (e & 3) - L;
          const int jc = j < 0 ? 0 : (j > 31 ? 31 : j);
          const uint32_t bit = (rowmask >> jc) & 1u;
          const bool vis = (j < 0) | ((j < 32) & (bit != 0u));
          s[e] = vis ? s[e] : -INFINITY;
        }
      }
      float tmax = s[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) tmax = fmaxf(tmax, s[e]);
      tmax *= c;
      if (__any(tmax > m)) {
        const float x = max_halves(fmaxf(m, tmax));
        const float alpha = fast_exp2(m - x);
        m = x;
        if (round > 0) {       // (nothing to rescale yet)
          l *= alpha;
          lvis *= alpha;
#pragma unroll
          for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[db][e] *= alpha;
        }
      }
      float pr[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) pr[e] = fast_exp2(__builtin_fmaf(s[e], c, -m));
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        pop[kt] = u32x4{pack_bf16(pr[8 * kt], pr[8 * kt + 1]), pack_bf16(pr[8 * kt + 2], pr[8 * kt + 3]),
                        pack_bf16(pr[8 * kt + 4], pr[8 * kt + 5]), pack_bf16(pr[8 * kt + 6], pr[8 * kt + 7])};
      float q4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        q4[e] = (pr[4 * e] + pr[4 * e + 1]) + (pr[4 * e + 2] + pr[4 * e + 3]);
      const float tsum = (q4[0] + q4[1]) + (q4[2] + q4[3]);
      l += tsum;
      const bool vis_all = key0 >= vis_b && key0 + 32 <= vis_e;
      const bool vis_any = key0 < vis_e && key0 + 32 > vis_b;
      float vs = vis_all ? tsum : 0.f;
      if (vis_any && !vis_all) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = key0 + 8 * (e >> 2) + 4 * h + (e & 3);
          vs += (key >= vis_b && key < vis_e) ? pr[e] : 0.f;
        }
      }
      lvis += vs;
    }
    if (late && round + 1 < n_rounds) enter(round + 1);
    multiply(round);
  }

  // ---- merge of the streams through LDS, in fixed order, as in attn_segment
  l += xor_shuffle(l, 32);
  lvis += xor_shuffle(lvis, 32);
  __syncthreads();
  float* sm_m = reinterpret_cast<float*>(smem);            // [KS][kRows]
  float* sm_l = sm_m + KS * W::kRows;
  float* sm_v = sm_l + KS * W::kRows;
  float* sm_o = sm_v + KS * W::kRows;                      // [KS][kRows][kMergeStride]
  {
    const int row = rg * 32 + n32;
    if (h == 0) {
      sm_m[stream * W::kRows + row] = m;
      sm_l[stream * W::kRows + row] = l;
      sm_v[stream * W::kRows + row] = lvis;
    }
    float* orow = sm_o + ((size_t)stream * W::kRows + row) * W::kMergeStride + 4 * h;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(orow + db * 32 + q * 8) =
            f32x4{acc[db][4 * q], acc[db][4 * q + 1], acc[db][4 * q + 2], acc[db][4 * q + 3]};
  }
  __syncthreads();
  float* part = record(b * p.Hkv + kvh);
  int rows_here = p.R - rc * rpad;
  rows_here = rows_here < rpad ? rows_here : rpad;
  for (int row = threadIdx.x; row < rows_here; row += NT) {
    float mm = sm_m[row];
#pragma unroll
    for (int k = 1; k < KS; ++k) mm = fmaxf(mm, sm_m[k * W::kRows + row]);
    float ls = 0.f, vs = 0.f;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const float f = fast_exp2(sm_m[k * W::kRows + row] - mm);
      ls += sm_l[k * W::kRows + row] * f;
      vs += sm_v[k * W::kRows + row] * f;
    }
    part[row] = mm;
    part[rpad + row] = ls;
    part[2 * rpad + row] = vs;
  }
  float* po = part + 3 * rpad;
  for (int idx = threadIdx.x; idx < rows_here * 32; idx += NT) {
    const int row = idx >> 5;
    const int c4 = (idx & 31) * 4;
    float mm = sm_m[row];
#pragma unroll
    for (int k = 1; k < KS; ++k) mm = fmaxf(mm, sm_m[k * W::kRows + row]);
    f32x4 o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k)
      o4 += *reinterpret_cast<const f32x4*>(sm_o + ((size_t)k * W::kRows + row) * W::kMergeStride + c4) *
            fast_exp2(sm_m[k * W::kRows + row] - mm);
    asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(po + (size_t)row * 128 + c4), "v"(o4)
                 : "memory");
  }
}

}  // namespace lvspec
