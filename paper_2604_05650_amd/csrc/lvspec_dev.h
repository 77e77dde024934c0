// Device-side building blocks shared by the gfx950 kernels: vector types, direct-to-LDS loads,
// LDS reads whose completion is waited for by hand, bf16 MFMA wrappers, cross-lane helpers.
//
// Memory pipeline used by every streaming kernel here
// ---------------------------------------------------
// Rows of 128 bf16 (256 bytes) are the unit.  A wave copies rows from HBM straight into LDS with
// global_load_lds_dwordx4 (no VGPR staging): one instruction moves four rows (64 lanes x 16 B),
// sixteen consecutive lanes cover one 256-byte row, so the HBM side is fully coalesced.  Inside
// LDS the sixteen 16-byte chunks of row r are stored at chunk position (c ^ key(r)), key(r) = r & 15
// in the GEMM kernels (the attention kernel, which also reads tiles row-wise, flips one more bit);
// an MFMA operand read, where sixteen lanes hold sixteen different rows at the same logical
// chunk, then touches sixteen different bank groups.  The permutation is applied on the *global* side of the
// copy (each lane fetches the chunk that belongs at its LDS position), which costs nothing.
//
// The compiler cannot see which LDS bytes such a copy writes and would wait for *all*
// outstanding copies before any LDS read.  LDS reads of streamed tiles are therefore written as
// inline assembly together with the exact s_waitcnt they need; copies complete in issue order,
// so "vmcnt(n)" means "everything except the youngest n copy instructions has landed".
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lvspec {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowBytes = 256;   // 128 bf16
constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;

#define LVS_DEV __device__ __forceinline__

// Optional in-kernel timeline hook for development builds; expands to nothing in the library.
#ifndef LVS_TRACE
#define LVS_TRACE(id)
#define LVS_TRACE_BEGIN
#define LVS_TRACE_END
#endif
#ifndef LVS_TRACE2          // same, for the second kernel of an entry point
#define LVS_TRACE2(id)
#define LVS_TRACE2_BEGIN
#define LVS_TRACE2_END
#endif

// 32-bit LDS byte address of a __shared__ object
LVS_DEV uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// Cache policy of a copy.  Data that is read exactly once (K/V tiles, video hidden states,
// lm_head rows) is fetched with the non-temporal hint: measured on MI355X, a pure streaming read
// sustains about 15 % more HBM bandwidth with it than without.  Small operands that every
// workgroup re-reads keep the default policy so they stay in L2.
constexpr int kCopyDefault = 0;
constexpr int kCopyStream = 2;   // "nt" bit of the gfx94x/gfx950 cache-policy field

// One direct-to-LDS copy instruction: lane l fetches 16 bytes from gptr (per lane) and the wave
// writes 1 KiB to lds_base + l*16.  lds_base must be wave-uniform.
template <int POLICY = kCopyStream>
LVS_DEV void dma16(const void* gptr, uint32_t lds_base) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)gptr,
      (__attribute__((address_space(3))) void*)(uintptr_t)__builtin_amdgcn_readfirstlane(lds_base),
      16, 0, POLICY);
}

// The same copy (kCopyStream) as a statement that the compiler does not know as an LDS write.  LDS reads
// are then ordinary loads with waits of their own, spread among the instructions that use them, instead of a
// wait for every copy under way; the kernel waits for copies (wait_copies) and separates reads and
// copies of a slot by barriers itself (lds_barrier).  m0 is as before behind it (the compiler takes no
// clobber of m0, and may keep a value there).
LVS_DEV void dma16_untracked(const void* gptr, uint32_t lds_base) {
  const uint32_t at = __builtin_amdgcn_readfirstlane(lds_base);
  uint32_t keep;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off nt\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(keep) : "s"(at), "v"(gptr));
}

LVS_DEV u32x4 lds_load16(uint32_t a) {
  return *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)a;
}

// Barrier behind this wave's LDS reads and writes; copies stay under way.
LVS_DEV void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0), for the compiler's own count ...
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");    // ... and with the barrier
}

// Wait until at most N copy instructions of this wave are outstanding, then read eight 16-byte
// values from LDS: r[j] from a[j & 3] + (j >> 2) * OFF, and wait for them.
template <int N, int OFF>
LVS_DEV void lds_read8_after(u32x4 (&r)[8], const uint32_t (&a)[4]) {
  asm volatile(
      "s_waitcnt vmcnt(%12)\n\t"
      "ds_read_b128 %0, %8\n\t"
      "ds_read_b128 %1, %9\n\t"
      "ds_read_b128 %2, %10\n\t"
      "ds_read_b128 %3, %11\n\t"
      "ds_read_b128 %4, %8 offset:%13\n\t"
      "ds_read_b128 %5, %9 offset:%13\n\t"
      "ds_read_b128 %6, %10 offset:%13\n\t"
      "ds_read_b128 %7, %11 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]),
        "=&v"(r[6]), "=&v"(r[7])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(N), "n"(OFF)
      : "memory");
}

// Four 16-byte LDS reads from a[0..3], no copy wait.
LVS_DEV void lds_read4(u32x4 (&r)[4], const uint32_t (&a)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4\n\t"
      "ds_read_b128 %1, %5\n\t"
      "ds_read_b128 %2, %6\n\t"
      "ds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
      : "memory");
}

template <int N>
LVS_DEV void wait_copies() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// D[m][n] += sum_k A[m][k] * B[k][n], 16x16 output, 32-deep, bf16 in, fp32 accumulate.
// Operand layout (lane l): A holds row m = l % 16, k = 8*(l/16) .. +7; B holds column n = l % 16,
// same k; D holds column n = l % 16, rows m = 4*(l/16) .. +3.
LVS_DEV f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// pack two fp32 into one dword of two bf16 (round to nearest even), lo = a, hi = b
LVS_DEV uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 t = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, t);
}

LVS_DEV float xor_shuffle(float x, int mask) { return __shfl_xor(x, mask, 64); }

// Maximum over the lane pairs l, l ^ 32 and l, l ^ 16 through the lane-swap instructions (a lane gets
// its own value and its partner's, in either order): no trip through the LDS queue, behind whatever
// reads wait there.  The running maximum of the attention kernels grows in most tiles of a short key
// range (32 rows, t tiles seen: some row's with probability 32 / t), so its exchange is on the way of
// every round: 16384 keys, 40 / 8 heads, 3 draft rows 16.9 -> 16.5 us per layer, 5 16.7 and 16.8,
// 12 20.2 -> 20.0, 20 in chunks of 64 rows 28.3 -> 27.5.
// (Assembly: this compiler takes the two results of the swap builtin for equal when its operands are.)
LVS_DEV float max_halves(float x) {
  float y;
  asm("v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1\n\tv_max_f32 %0, %0, %1"
      : "+v"(x), "=&v"(y));
  return x;
}
LVS_DEV float max_rows(float x) {
  float y;
  asm("v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1\n\tv_max_f32 %0, %0, %1"
      : "+v"(x), "=&v"(y));
  return x;
}

LVS_DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Order-preserving map from fp32 to unsigned integers (larger float = larger key) and back.
LVS_DEV uint32_t order_key(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

LVS_DEV float key_value(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __builtin_bit_cast(float, u);
}

// A (value, token id) candidate as one 64-bit key, larger = better in (value descending, id
// ascending) order; 0 = no candidate.  Ids are unique within a column, so equal keys are the
// same candidate.
LVS_DEV uint64_t cand_key(float v, int id) {
  return id < 0 ? 0ull : (((uint64_t)order_key(v) << 32) | (uint32_t)(0x7fffffff - id));
}

// Wave-wide reductions through the DPP lane network (no LDS traffic): two quad permutes, two
// row mirrors, then the row broadcasts of the gfx9 family; lane 63 ends up with the result,
// which is handed back through scalar registers (so the result is wave-uniform).  `ident` is
// the operation's identity; the order of the combination is fixed, so sums are reproducible.
template <int CTRL, int ROW_MASK>
LVS_DEV uint32_t dpp_move(uint32_t ident, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)ident, (int)v, CTRL, ROW_MASK, 0xf, false);
}

template <class Op>
LVS_DEV float wave_reduce(float x, float ident, Op op) {
  const uint32_t id = __builtin_bit_cast(uint32_t, ident);
  auto f = [](uint32_t u) { return __builtin_bit_cast(float, u); };
  auto u = [](float v) { return __builtin_bit_cast(uint32_t, v); };
  x = op(x, f(dpp_move<0xB1, 0xf>(id, u(x))));    // quad_perm [1,0,3,2]
  x = op(x, f(dpp_move<0x4E, 0xf>(id, u(x))));    // quad_perm [2,3,0,1]
  x = op(x, f(dpp_move<0x141, 0xf>(id, u(x))));   // row_half_mirror
  x = op(x, f(dpp_move<0x140, 0xf>(id, u(x))));   // row_mirror
  x = op(x, f(dpp_move<0x142, 0xa>(id, u(x))));   // row_bcast:15 into rows 1 and 3
  x = op(x, f(dpp_move<0x143, 0xc>(id, u(x))));   // row_bcast:31 into rows 2 and 3
  return f((uint32_t)__builtin_amdgcn_readlane((int)u(x), 63));
}

LVS_DEV float wave_max(float x) {
  return wave_reduce(x, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}

LVS_DEV float wave_sum(float x) {
  return wave_reduce(x, 0.f, [](float a, float b) { return a + b; });
}

// maximum of a 32-bit unsigned key over the wave (identity 0), same network
LVS_DEV uint32_t wave_max_u32(uint32_t x) {
  x = max(x, dpp_move<0xB1, 0xf>(0u, x));
  x = max(x, dpp_move<0x4E, 0xf>(0u, x));
  x = max(x, dpp_move<0x141, 0xf>(0u, x));
  x = max(x, dpp_move<0x140, 0xf>(0u, x));
  x = max(x, dpp_move<0x142, 0xa>(0u, x));
  x = max(x, dpp_move<0x143, 0xc>(0u, x));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// maximum of a 64-bit unsigned key over the wave (identity 0): of the upper halves, then, among the
// lanes that hold it, of the lower ones (mostly one lane: no second reduction).  The selection rounds of
// the candidate lists are a chain of these: against one network of 64-bit steps 96 hidden rows, k = 4,
// V = 152064, d = 5120 328 -> 318 us; 128 rows, V = 8192, d = 1024 36.6 -> 33.9.
LVS_DEV uint64_t wave_max_u64(uint64_t x) {
  const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
  const uint32_t top = wave_max_u32(hi);
  const unsigned long long at = __ballot(hi == top);
  uint32_t low;
  if ((at & (at - 1)) == 0ull)
    low = (uint32_t)__builtin_amdgcn_readlane((int)lo, __builtin_ctzll(at));
  else
    low = wave_max_u32(hi == top ? lo : 0u);
  return ((uint64_t)top << 32) | low;
}

LVS_DEV uint64_t read_lane64(uint64_t x, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// The k <= 16 largest of a wave's 64-bit keys (0 = none), the r-th in lane r.
template <int NV>
LVS_DEV uint64_t topk_of(uint64_t (&key)[NV], int k, int lane) {
  uint64_t top = 0ull;
  for (int r = 0; r < k; ++r) {
    uint64_t best = key[0];
#pragma unroll
    for (int j = 1; j < NV; ++j) best = key[j] > best ? key[j] : best;
    const uint64_t w = wave_max_u64(best);
#pragma unroll
    for (int j = 0; j < NV; ++j) key[j] = key[j] == w ? 0ull : key[j];
    top = lane == r ? w : top;
  }
  return top;
}

// Compare-exchange of 64-bit keys with the partner lane's: lanes without `bit` keep the larger.
LVS_DEV uint64_t keep_ordered(uint64_t x, uint64_t partner, int bit, int lane) {
  const bool other = (partner > x) != ((lane & bit) != 0);
  return other ? partner : x;
}
template <int CTRL>
LVS_DEV uint64_t dpp_move64(uint64_t x) {
  const uint32_t lo = dpp_move<CTRL, 0xf>(0u, (uint32_t)x);
  const uint32_t hi = dpp_move<CTRL, 0xf>(0u, (uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}
// partners within a row of 16 lanes
LVS_DEV uint64_t lane_xor1(uint64_t x) { return dpp_move64<0xB1>(x); }
LVS_DEV uint64_t lane_xor2(uint64_t x) { return dpp_move64<0x4E>(x); }
LVS_DEV uint64_t lane_xor3(uint64_t x) { return dpp_move64<0x1B>(x); }
LVS_DEV uint64_t lane_xor7(uint64_t x) { return dpp_move64<0x141>(x); }     // half mirror
LVS_DEV uint64_t lane_xor8(uint64_t x) { return dpp_move64<0x128>(x); }     // rotation by 8
LVS_DEV uint64_t lane_xor15(uint64_t x) { return dpp_move64<0x140>(x); }    // mirror
LVS_DEV uint64_t lane_xor4(uint64_t x) { return lane_xor3(lane_xor7(x)); }

// Every row of 16 lanes, a bitonic sequence, into descending order.
LVS_DEV uint64_t sort_bitonic16(uint64_t x, int lane) {
  x = keep_ordered(x, lane_xor8(x), 8, lane);
  x = keep_ordered(x, lane_xor4(x), 4, lane);
  x = keep_ordered(x, lane_xor2(x), 2, lane);
  return keep_ordered(x, lane_xor1(x), 1, lane);
}
// Every row of 16 lanes into descending order.
LVS_DEV uint64_t sort_row16(uint64_t x, int lane) {
  x = keep_ordered(x, lane_xor1(x), 1, lane);
  x = keep_ordered(x, lane_xor3(x), 2, lane);
  x = keep_ordered(x, lane_xor1(x), 1, lane);
  x = keep_ordered(x, lane_xor7(x), 4, lane);
  x = keep_ordered(x, lane_xor2(x), 2, lane);
  x = keep_ordered(x, lane_xor1(x), 1, lane);
  x = keep_ordered(x, lane_xor15(x), 8, lane);
  x = keep_ordered(x, lane_xor4(x), 4, lane);
  x = keep_ordered(x, lane_xor2(x), 2, lane);
  return keep_ordered(x, lane_xor1(x), 1, lane);
}
// The 16 largest of two descending rows, descending.
LVS_DEV uint64_t merge_rows16(uint64_t a, uint64_t b, int lane) {
  const uint64_t m = lane_xor15(b);
  return sort_bitonic16(m > a ? m : a, lane);
}
// x becomes its even rows (lower half) in both rows of a pair (both halves), y the odd ones (the upper).
// (Assembly for the reason given at max_halves.)
LVS_DEV void split_rows(uint32_t& x, uint32_t& y) {
  asm("v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "=&v"(y));
}
LVS_DEV void split_halves(uint32_t& x, uint32_t& y) {
  asm("v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "=&v"(y));
}

// Takes NV keys per lane into a wave's list of the 16 largest (lane r < 16 the r-th, 0 = none) by sorting
// networks over the lanes: rows of 16, then rows against rows.  Keys are unique (0 aside).
template <int NV>
LVS_DEV void topk_merge(uint64_t& top, const uint64_t (&key)[NV], int lane) {
  uint64_t x = sort_row16(key[0], lane);
#pragma unroll
  for (int j = 1; j < NV; ++j) x = merge_rows16(x, sort_row16(key[j], lane), lane);
  uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32), lo2, hi2;
  split_rows(lo, lo2);
  split_rows(hi, hi2);
  x = merge_rows16(((uint64_t)hi << 32) | lo, ((uint64_t)hi2 << 32) | lo2, lane);
  lo = (uint32_t)x;
  hi = (uint32_t)(x >> 32);
  split_halves(lo, lo2);
  split_halves(hi, hi2);
  x = merge_rows16(((uint64_t)hi << 32) | lo, ((uint64_t)hi2 << 32) | lo2, lane);
  x = merge_rows16(x, top, lane);
  top = lane < 16 ? x : 0ull;
}

// A wave's running list of the k <= 16 largest 64-bit keys, lane r < 16 holding the r-th largest
// (0 = none): take in NV keys per lane.  Only keys above the k-th so far cost a round, largest
// first; every round retires one key, so the loop ends.  Equal keys are the same candidate.
template <int NV>
LVS_DEV void topk_insert(uint64_t& top, uint64_t (&key)[NV], int k, int lane) {
  uint64_t kth = read_lane64(top, k - 1);
  while (true) {
    uint64_t best = key[0];
#pragma unroll
    for (int j = 1; j < NV; ++j) best = key[j] > best ? key[j] : best;
    if (__ballot(best > kth) == 0ull) break;
    const uint64_t w = wave_max_u64(best);
#pragma unroll
    for (int j = 0; j < NV; ++j) key[j] = key[j] == w ? 0ull : key[j];
    // lanes above w keep their key, the next one takes w, the others move down by one
    // (row_shr:1: the list lives in one DPP row)
    const int pos = __popcll(__ballot((lane < 16) & (top > w)));
    const uint32_t dlo = dpp_move<0x111, 0xf>(0u, (uint32_t)top);
    const uint32_t dhi = dpp_move<0x111, 0xf>(0u, (uint32_t)(top >> 32));
    const uint64_t down = ((uint64_t)dhi << 32) | dlo;
    top = lane < pos ? top : lane == pos ? w : lane < 16 ? down : 0ull;
    kth = read_lane64(top, k - 1);
  }
}

// A wave's list of the k <= 16 largest takes in NV keys per lane, whichever way is the shortest.  The
// first keys need no places found for them, a third of a round (a small vocabulary has only first rows:
// k = 16, d = 1024, 32 hidden rows, V = 8192 34.3 -> 27.4 us).  With many candidates asked for, more than
// a handful enter in the first tasks of a pass: sorted in at once they cost as much as about five rounds,
// however many enter.  All rounds against this, hidden rows, V / d, k: 128, 152064 / 3584, 16 393 -> 328 us;
// 100, 32000 / 2048, 16 89.5 -> 61.7 and 8 65.2 -> 61.1; 32, 8192 / 1024, 16 37.6 -> 23.2.  For k = 4 the
// rounds stay the shorter way (128 rows, d = 8192 533 us, sorted 563); 8 lanes as the bound are 4 % slower than
// 5 on the first of these, 3 the same.  The networks are not in the code where nobody asks for
// them: there they cost short passes 0.2 us (16 rows, k = 4, V = 8192 17.6 -> 17.8).
constexpr int kSortTopk = 6;
constexpr int kSortLanes = 5;
template <int NV, bool SORT>
LVS_DEV void topk_take(uint64_t& top, uint64_t (&key)[NV], int k, int lane) {
  if constexpr (SORT) {      // k > kSortTopk
    uint64_t best = key[0];
#pragma unroll
    for (int j = 1; j < NV; ++j) best = key[j] > best ? key[j] : best;
    if (__popcll(__ballot(best > read_lane64(top, k - 1))) > kSortLanes) {
      topk_merge<NV>(top, key, lane);
      return;
    }
  }
  if (read_lane64(top, 0) == 0ull)
    top = topk_of<NV>(key, k, lane);
  else
    topk_insert<NV>(top, key, k, lane);
}

}  // namespace lvspec
