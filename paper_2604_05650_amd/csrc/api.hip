// C ABI of the library: argument validation, launch planning (all on the host, no device access)
// and kernel launches on the caller's stream.
#include <hip/hip_runtime.h>

#include <atomic>

#include "../../include/lvspec.h"
#include "lvspec_kernels.h"

// Scratch of lvspec_verify_attn_static: part of the code object, one copy per GPU.  In host code
// the array's name is only a handle for the symbol lookup, never a device address: everything
// below works with the pointer that hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) unsigned char scratch[LVSPEC_STATIC_SCRATCH_BYTES];

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
  g_last_hip_error = (int)e;
  return LVSPEC_EHIP;
}

// compute units of the current device; 256 (MI355X) when no device can be queried.  Cached per
// device; the query is idempotent, so racing first calls store the same value.
int num_compute_units() {
  static std::atomic<int> cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return 256;
  }
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked) {
    const int c = cached[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) {
    if (tracked) cached[dev].store(n, std::memory_order_relaxed);
    return n;
  }
  (void)hipGetLastError();
  return 256;
}

size_t round_up(size_t x, size_t m) { return (x + m - 1) / m * m; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool stride_ok(int64_t s) { return s >= 0 && (s % 8) == 0; }

// ------------------------------------------------------------------------------ attention
// Rows of a kv head in chunks, and the two ways to divide the keys: equal splits per unit (sequence, kv
// head, row chunk), and equal stretches of one line over all sequences.
struct AttnCut {
  int rpad, n_rc, n_split;
  size_t split_bytes;      // partials of n_split workgroups per unit
  int flat_pos;            // stretches of the line over all sequences, 0: none
  size_t flat_bytes;       // partials of those
  size_t bytes() const { return flat_bytes > split_bytes ? flat_bytes : split_bytes; }
};

struct AttnPlan {
  int G, R;
  AttnCut cut;             // row chunks of up to 64 rows: what every workspace of cut.split_bytes serves
  AttnCut wide;            // row chunks of 65 to 128 rows, n_rc = 0: not for this shape
  size_t ws_bytes;         // what the caller is asked for
  // Wide row chunks for a workspace as large as asked for; one that holds no more than equal splits of
  // the narrow ones is served by those.
  const AttnCut& served_by(size_t have) const { return wide.n_rc > 0 && have >= ws_bytes ? wide : cut; }
};

// Equal splits and stretches for the row chunks that `c` holds; n_tiles of 32 keys at most.
void divide_keys(const lvspec_attn_args* a, int64_t n_tiles, AttnCut* c) {
  const int64_t units = (int64_t)a->B * a->Hkv * c->n_rc;
  int64_t ns = num_compute_units() / units;
  const int64_t cap_split = (n_tiles + 3) / 4;
  if (ns > cap_split) ns = cap_split;
  if (ns > 256) ns = 256;
  if (ns < 1) ns = 1;
  c->n_split = (int)ns;
  const size_t rec_bytes = (size_t)c->rpad * 131 * sizeof(float);
  c->split_bytes = (size_t)units * (size_t)ns * rec_bytes;
  // A batch that the caller says is short keeps attn_split_kernel: its combine kernel does not wait
  // for the lengths (2 x 2048 keys, 40 / 8 heads: 13.0 us against 14.1, 4 x 2048: 14.4 against 15.4;
  // but 16 x 512, two workgroups per unit: 19.5 against 15.1).  By cap where there is no max_kv_len;
  // the lengths themselves then ask for the same cut, see flat_equal_splits.
  // Shapes that the static scratch serves with equal splits stay within it: fewer stretches leave a
  // few CUs idle (one in sixteen for 256 units of 64 rows).
  c->flat_pos = lvspec::attn_flat_positions(a->B, a->Hkv, c->rpad, c->n_rc, a->cap, num_compute_units());
  if ((ns > 2 && n_tiles < lvspec::attn_short_tiles(a->B) * ns) || ns > 128) c->flat_pos = 0;
  auto flat_bytes = [&] {
    return ((size_t)c->flat_pos + (size_t)a->B * a->Hkv) * (size_t)c->n_rc * rec_bytes;
  };
  if (c->split_bytes <= (size_t)LVSPEC_STATIC_SCRATCH_BYTES) {
    const int least = c->flat_pos * 7 / 8;
    while (c->flat_pos > 0 && flat_bytes() > (size_t)LVSPEC_STATIC_SCRATCH_BYTES)
      c->flat_pos = c->flat_pos - 8 >= least ? c->flat_pos - 8 : 0;
  }
  c->flat_bytes = c->flat_pos > 0 ? flat_bytes() : 0;
}

// More than 64 query rows per kv head in chunks of 65 to 128 (attn_segment32).
void plan_wide(const lvspec_attn_args* a, int64_t n_tiles, AttnPlan* pl) {
  AttnCut& w = pl->wide;
  w = AttnCut{};
  // Without max_kv_len the sequences may be a small part of the cache: short ones go faster in narrow chunks.
  if (pl->R <= 64 || a->B > 64 || a->max_kv_len == 0) return;
  AttnCut c{};
  c.n_rc = (pl->R + 127) / 128;
  c.rpad = ((pl->R + c.n_rc - 1) / c.n_rc + 3) / 4 * 4;
  divide_keys(a, n_tiles, &c);
  // Splits that fill the static scratch to the brim: one in sixteen fewer fits 128 rows on 256 CUs.
  const size_t scratch = LVSPEC_STATIC_SCRATCH_BYTES;
  if (a->B == 1 && c.split_bytes > scratch) {
    const int most = (int)(scratch / (c.split_bytes / c.n_split));
    if (most >= c.n_split - c.n_split / 16) {
      c.split_bytes = c.split_bytes / c.n_split * most;
      c.n_split = most;
    }
  }
  if (a->B > 1 && c.flat_pos == 0) return;
  // More than 32 splits of one sequence: fewer than eight kv heads, whose records no longer lie in the L2
  // of the XCD that merges them.  28 / 4 heads, 98 rows, in chunks of up to 64 rows and here: 2034 keys under
  // a hint of 60000 12.4 and 19.1 us, 8178 keys 15.3 and 20.7; 8 / 2 heads, 80 rows, 57324 keys 21.2 and 26.2.
  if (a->B == 1 && c.n_split > 32) return;
  // Twice the rows mean twice the partial records per workgroup, and a round is a longer chain: worth it
  // from this many tiles of 32 keys per workgroup on.  In narrow chunks and here, us:
  //   one sequence, 8 kv heads, 100 rows 8 tiles 17.4 and 17.1, 16 tiles 24.3 and 22.2; 128 rows 12 tiles 21.3
  //   and 21.5, 16 tiles 24.5 and 23.4; three chunks against two, 150 rows 6 tiles 16.5 and 15.7; four against
  //   two, 240 rows 6 tiles 16.0 and 16.2, 12 tiles 21.2 and 20.0;
  //   the 48-row variant (65 to 96, 129 to 144 rows) holds its own for longer: 80 rows 16 tiles 20.6 and 20.9,
  //   28 tiles 29.2 and 28.1; batches of 4, 28 / 4 heads, 72 rows, equal lengths 16 tiles 0.98 times as long here,
  //   24 tiles 0.95.
  // max_kv_len is a bound of the lengths and no more, and which cut is used must not depend on where the
  // lengths are given: the lines lie where a hint that is right gains, and lengths far below it lose little.
  // Times as long as in the narrow chunks of the same shape: one sequence of 1000 to 3000 keys under a long
  // hint, 8 kv heads, 100 rows 1.03 to 1.06, 80 and 128 rows 1.08 to 1.12; batches whose lengths spread over 5
  // to 100 % of the hint, so that a stretch gets a third of the tiles that the hint promises, and that just pass
  // the line 0.9 to 1.1; 3 to 7 tiles per workgroup, under a hint many times too long, 0.84 to 1.16 (2 to 8
  // sequences, 2 to 8 kv heads, 80 to 100 rows).
  const int64_t parts = a->B > 1 ? c.flat_pos : c.n_split;
  const int64_t tiles = a->B > 1 ? n_tiles * a->B * a->Hkv : n_tiles;
  const bool rows48 = pl->cut.rpad == 48;
  int64_t least = pl->cut.n_rc > 2 ? 6 : 16;
  if (a->B == 1) {
    if (rows48 && pl->cut.n_rc == 2 && c.n_split > 16) least = 24;
  } else {
    least = rows48 && a->B * a->Hkv < 48 ? 32 : least * 3 / 2;
  }
  if (tiles < least * parts) return;
  // What the static scratch serves it goes on serving, with the same results.
  if (pl->cut.bytes() <= scratch && c.bytes() > scratch) return;
  w = c;
}

int plan_attn(const lvspec_attn_args* a, AttnPlan* pl) {
  if (a == nullptr) return LVSPEC_EINVAL;
  if (a->B < 1 || a->gamma < 1 || a->gamma > LVSPEC_MAX_DRAFT_ROWS || a->Hq < 1 || a->Hkv < 1 ||
      a->D < 1)
    return LVSPEC_EINVAL;
  if (a->Hq % a->Hkv != 0) return LVSPEC_EINVAL;
  if (a->D != LVSPEC_HEAD_DIM) return LVSPEC_EUNSUPPORTED;
  if (a->cap < a->gamma || a->max_kv_len < 0 || a->max_kv_len + a->gamma > a->cap)
    return LVSPEC_EINVAL;
  if (a->cap > (int64_t)1 << 30) return LVSPEC_EUNSUPPORTED;
  if (!(a->scale >= 0.f) || a->scale > 1.0e6f) return LVSPEC_EINVAL;
  const int64_t lmax = a->max_kv_len > 0 ? a->max_kv_len : a->cap - a->gamma;
  pl->G = a->Hq / a->Hkv;
  pl->R = pl->G * a->gamma;
  AttnCut& c = pl->cut;
  c.n_rc = (pl->R + 63) / 64;
  const int per_chunk = (pl->R + c.n_rc - 1) / c.n_rc;
  c.rpad = per_chunk <= 16 ? 16 : per_chunk <= 32 ? 32 : per_chunk <= 48 ? 48 : 64;
  const int64_t units = (int64_t)a->B * a->Hkv * c.n_rc;
  // block ids and row indices stay below 2^27, the range of the kernels' multiply-shift division
  if (units * 64 > (int64_t)1 << 27 || a->Hq > 65536) return LVSPEC_EUNSUPPORTED;
  const int64_t n_tiles = (lmax + a->gamma + 31) / 32;
  divide_keys(a, n_tiles, &c);
  plan_wide(a, n_tiles, pl);
  pl->ws_bytes = c.bytes();
  if (pl->wide.n_rc > 0 && pl->wide.bytes() > pl->ws_bytes) pl->ws_bytes = pl->wide.bytes();
  return LVSPEC_OK;
}

int check_attn_pointers(const lvspec_attn_args* a) {
  if (!a->q || !a->k || !a->v || !a->out) return LVSPEC_EINVAL;
  if (!a->kv_len && !(a->kv_len_host && a->B <= 32)) return LVSPEC_EINVAL;
  if (a->kv_len_host != nullptr) {
    const int64_t lmax = a->max_kv_len > 0 ? a->max_kv_len : a->cap - a->gamma;
    for (int b = 0; b < a->B; ++b)
      if (a->kv_len_host[b] < 0 || a->kv_len_host[b] > lmax) return LVSPEC_EINVAL;
  }
  if (!aligned16(a->q) || !aligned16(a->k) || !aligned16(a->v) || !aligned16(a->out))
    return LVSPEC_EINVAL;
  if (!stride_ok(a->q_sb) || !stride_ok(a->q_sg) || !stride_ok(a->q_sh) || !stride_ok(a->kv_sb) ||
      !stride_ok(a->kv_sh) || !stride_ok(a->kv_sl) || !stride_ok(a->o_sb) || !stride_ok(a->o_sg) ||
      !stride_ok(a->o_sh))
    return LVSPEC_EINVAL;
  if (a->kv_sl < a->D || a->q_sh < a->D || a->o_sh < a->D) return LVSPEC_EINVAL;
  if ((a->vis_begin == nullptr) != (a->vis_end == nullptr)) return LVSPEC_EINVAL;
  if (a->vis_mass != nullptr && a->vis_begin == nullptr) return LVSPEC_EINVAL;
  if (a->draft_mask != nullptr) {
    for (int i = 0; i < a->gamma; ++i) {
      if (!((a->draft_mask[i] >> i) & 1u)) return LVSPEC_EINVAL;   // a row always sees itself
      if (a->gamma < 32 && (a->draft_mask[i] >> a->gamma) != 0u) return LVSPEC_EINVAL;
    }
  }
  return LVSPEC_OK;
}

// ------------------------------------------------------------------------------ relevance
struct RelPlan {
  int rows, n_rb, n_ds, kc, row_bytes;
  int64_t ld;
  size_t off_nv2, off_cos, off_keys, ws_bytes;
  int n_parts, slice_rows;
};

int plan_rel(const lvspec_rel_args* a, RelPlan* pl) {
  if (a == nullptr) return LVSPEC_EINVAL;
  if (a->B < 1 || a->gamma < 1 || a->gamma > LVSPEC_MAX_DRAFT_ROWS || a->d < 1 ||
      a->top_n < 1 || a->top_n > LVSPEC_MAX_TOPN || a->lv_max < 0)
    return LVSPEC_EINVAL;
  if (a->d % 128 != 0) return LVSPEC_EUNSUPPORTED;
  if (a->lv_max > (int64_t)1 << 30) return LVSPEC_EUNSUPPORTED;
  // Stages of 64 rows x 512 bytes when the shape allows (up to 16 draft rows, d a multiple of
  // 256): longer contiguous row segments stream measurably faster from HBM than 256-byte ones.
  // Otherwise 256-byte stages: 128-row tasks (bigger stages, fewer barriers per byte) once they
  // fill the persistent workgroups without splitting the hidden dimension, 64-row tasks else.
  const int64_t wg_slots = 2 * (int64_t)num_compute_units();
  pl->row_bytes = (a->gamma <= 16 && a->d % 256 == 0) ? 512 : 256;
  const int big = (pl->row_bytes == 256 &&
                   (int64_t)a->B * ((a->lv_max + 127) / 128) >= wg_slots) ? 1 : 0;
  const int rows = lvspec::rel_rows_per_block(big);
  pl->rows = rows;
  pl->n_rb = (int)((a->lv_max + rows - 1) / rows);
  if (pl->n_rb < 1) pl->n_rb = 1;
  // task indices (row blocks x up to 8 splits x sequences) stay in 32-bit range, and the
  // sequence index is a grid dimension of the finalize kernels
  if (a->B > 65535 || (int64_t)a->B * pl->n_rb * 8 > (int64_t)1 << 30) return LVSPEC_EUNSUPPORTED;
  const int nchunks = a->d * 2 / pl->row_bytes;
  // Split the hidden dimension when the row blocks alone leave most of the persistent
  // workgroups (two per CU) without a task.  A split is not free: shorter tasks, partial results
  // per split and their sum in the finalize kernels cost about 9 % of the streaming rate per
  // doubling (measured at equal fill: 6.2 TB/s unsplit against 5.7 and 5.5 TB/s in two and four
  // splits on 4 GB of hidden states), so the fill of the last round is weighed against that;
  // among near-equal scores the fewest splits win.  At most 8 splits, at least 2 chunks each.
  const int64_t slots = 2 * (int64_t)num_compute_units();
  int best = 1;
  double best_score = 0.0;
  for (int ds = 1; ds <= nchunks && ds <= 8; ++ds) {
    if (nchunks % ds != 0) continue;
    if (nchunks / ds < 2 && ds != 1) break;
    const int64_t tasks = (int64_t)a->B * pl->n_rb * ds;
    const int64_t rounds = (tasks + slots - 1) / slots;
    const double fill = (double)tasks / (double)(rounds * slots);
    const double score = fill / (1.0 + 0.1 * __builtin_log2((double)ds));
    if (score > best_score + 0.03) {
      best = ds;
      best_score = score;
    }
  }
  pl->n_ds = best;
  pl->kc = nchunks / best;
  pl->ld = (int64_t)round_up((size_t)(a->lv_max > 0 ? a->lv_max : 1), 128);
  const size_t f = sizeof(float);
  const size_t dots = round_up((size_t)a->B * pl->n_ds * a->gamma * pl->ld * f, 256);
  const size_t nv2 = round_up((size_t)a->B * pl->n_ds * pl->ld * f, 256);
  const size_t cosb = round_up((size_t)a->B * a->gamma * pl->ld * f, 256);
  // slices of the two-kernel Top-N (small N): at most kRelMaxParts slices of as few 1024-row
  // chunks as that allows; n_parts = 0: not used (large N, or more than a million video rows)
  const int64_t per_slice = (int64_t)lvspec::kRelSliceRows * lvspec::kRelMaxParts;
  int64_t chunks = (a->lv_max + per_slice - 1) / per_slice;
  if (chunks < 1) chunks = 1;
  pl->slice_rows = (int)(chunks * lvspec::kRelSliceRows);
  const int64_t parts = (a->lv_max + pl->slice_rows - 1) / pl->slice_rows;
  pl->n_parts = (a->top_n <= lvspec::kRelSmallN && parts >= 1 && parts <= lvspec::kRelMaxParts &&
                 chunks <= lvspec::kRelMaxChunks)
                    ? (int)parts : 0;
  const size_t keys = round_up((size_t)a->B * a->gamma * (size_t)pl->n_parts *
                               lvspec::kRelSmallN * sizeof(uint32_t), 256);
  pl->off_nv2 = dots;
  pl->off_cos = dots + nv2;
  pl->off_keys = dots + nv2 + cosb;
  pl->ws_bytes = dots + nv2 + cosb + keys;
  return LVSPEC_OK;
}

// ------------------------------------------------------------------------------ accept
struct AccPlan {
  int n_tasks, n_cols;     // n_cols: columns of one (full) pass
  int per_pass;            // chains of one pass: one group, or two side by side
  int rows_per_block;      // vocabulary rows with one order of summation, 64 or 128
  int block_rows;          // vocabulary rows per pipeline stage
  int group;               // chains of a group (a multiple of the branches per sequence)
  int n_rec;               // records per column (workgroups of the lm_head launch)
  size_t off_cand, off_sz, ws_bytes;
};

// two: groups of chains share a pass in pairs, which takes records for twice the columns
int plan_acc(const lvspec_accept_args* a, AccPlan* pl, bool two = true) {
  if (a == nullptr) return LVSPEC_EINVAL;
  if (a->B < 1 || a->gamma < 1 || a->gamma > LVSPEC_MAX_GAMMA || a->d < 1 || a->V < 1 ||
      a->topk < 1 || a->topk > LVSPEC_MAX_TOPK)
    return LVSPEC_EINVAL;
  if (a->n_loose < 0 || a->n_loose > a->gamma || a->pst_window < 0 || a->loose_topk_gate < 0 ||
      a->loose_topk_gate > a->topk)
    return LVSPEC_EINVAL;
  if (a->n_branches < 0 || a->n_branches > LVSPEC_MAX_BRANCHES ||
      (a->n_branches > 1 && a->B % a->n_branches != 0))
    return LVSPEC_EINVAL;
  if (a->bonus_row != 0 && a->bonus_row != 1) return LVSPEC_EINVAL;
  if (a->rule < LVSPEC_RULE_VISUAL || a->rule > LVSPEC_RULE_ENTROPY_WINDOW) return LVSPEC_EINVAL;
  if (a->rule != LVSPEC_RULE_VISUAL &&
      (!(a->entropy_threshold >= 0.f) || a->defer_window < 0 || a->defer_window > LVSPEC_MAX_GAMMA))
    return LVSPEC_EINVAL;
  if (a->d % 128 != 0) return LVSPEC_EUNSUPPORTED;
  // Chains are taken in groups of whole sequences (the branches of a tree stay together) with at
  // most kMaxCols hidden rows, and two groups share one pass of the lm_head stream.
  constexpr int kMaxCols = 64;
  const int nbr = a->n_branches > 1 ? a->n_branches : 1;
  const int rpc = a->gamma + a->bonus_row;   // hidden rows per chain
  if (nbr * rpc > kMaxCols || a->B > 4096) return LVSPEC_EUNSUPPORTED;
  // Fewest groups first; among equal counts the smallest group whose columns fit the
  // narrower (faster) kernel variants.
  const int gmax = (kMaxCols / rpc) / nbr * nbr;
  const int groups = (a->B + gmax - 1) / gmax;
  pl->group = ((a->B + groups - 1) / groups + nbr - 1) / nbr * nbr;
  if (pl->group > a->B) pl->group = a->B;
  pl->per_pass = two && pl->group < a->B ? 2 * pl->group : pl->group;
  pl->n_cols = (pl->per_pass < a->B ? pl->per_pass : a->B) * rpc;
  // The block whose rows add their chunks of d up in one order (see issue_stage): 64 rows, except
  // 128 for up to 32 columns where the row pitch wants 128-row stages or many candidates are
  // asked for.  A pair of 64-row blocks is still streamed block by block: at k = 16 (d = 3584,
  // V = 152064) 163 us against 171 us in 128-row stages.
  const int64_t pitch = (a->w_sv > 0 ? a->w_sv : a->d) * 2;
  pl->rows_per_block = lvspec::lmh_order_rows(pl->n_cols, pitch, a->V, a->topk);
  pl->block_rows = lvspec::lmh_block_rows(pl->n_cols, pitch, a->V, num_compute_units());
  pl->n_tasks = (a->V + pl->block_rows - 1) / pl->block_rows;
  pl->n_rec = lvspec::lmh_records(pl->n_cols, pl->n_tasks, num_compute_units());
  const size_t rec = (size_t)pl->n_rec * pl->n_cols;
  pl->off_cand = round_up(rec * 2 * sizeof(float), 256);
  pl->off_sz = pl->off_cand + round_up(rec * a->topk * sizeof(uint64_t), 256);
  pl->ws_bytes = pl->off_sz + round_up(rec * sizeof(float), 256);
  return LVSPEC_OK;
}

int enqueue_attn(const lvspec_attn_args* a, const AttnPlan& pl, void* workspace, size_t have,
                 void* stream);

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(void** out) {
  static std::atomic<void*> cached[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  const bool tracked = dev >= 0 && dev < 64;
  void* ptr = tracked ? cached[dev].load(std::memory_order_acquire) : nullptr;
  if (ptr == nullptr) {
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e);
    if (ptr == nullptr) return hip_fail(hipErrorInvalidSymbol);
    if (tracked) cached[dev].store(ptr, std::memory_order_release);   // same value from any thread
  }
  *out = ptr;
  return LVSPEC_OK;
}

int check_ws(const void* ws, size_t have, size_t need) {
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 || have < need)
    return LVSPEC_EWORKSPACE;
  return LVSPEC_OK;
}

}  // namespace

extern "C" {

const char* lvspec_status_string(int status) {
  switch (status) {
    case LVSPEC_OK: return "ok";
    case LVSPEC_EINVAL: return "invalid argument";
    case LVSPEC_EUNSUPPORTED: return "unsupported shape";
    case LVSPEC_EWORKSPACE: return "workspace missing, misaligned or too small";
    case LVSPEC_EHIP: return "HIP error";
    case LVSPEC_ESCRATCH: return "static scratch too small for these shapes";
    default: return "unknown status";
  }
}

int lvspec_version(void) { return LVSPEC_VERSION; }
int lvspec_last_hip_error(void) { return g_last_hip_error; }

int lvspec_n_loose(float lambda, int gamma) {
  if (gamma < 0) return 0;
  int n = (int)__builtin_floor((double)lambda * (double)gamma + 1e-6);
  if (n < 0) n = 0;
  if (n > gamma) n = gamma;
  return n;
}

size_t lvspec_verify_attn_workspace(const lvspec_attn_args* args) {
  AttnPlan pl;
  return plan_attn(args, &pl) == LVSPEC_OK ? pl.ws_bytes : 0;
}

int lvspec_verify_attn(const lvspec_attn_args* a, void* stream) {
  AttnPlan pl;
  int rc = plan_attn(a, &pl);
  if (rc != LVSPEC_OK) return rc;
  rc = check_attn_pointers(a);
  if (rc != LVSPEC_OK) return rc;
  rc = check_ws(a->workspace, a->workspace_bytes, pl.cut.split_bytes);
  if (rc != LVSPEC_OK) return rc;
  return enqueue_attn(a, pl, a->workspace, a->workspace_bytes, stream);
}

int lvspec_verify_attn_static(const lvspec_attn_args* a, void* stream) {
  AttnPlan pl;
  int rc = plan_attn(a, &pl);
  if (rc != LVSPEC_OK) return rc;
  rc = check_attn_pointers(a);
  if (rc != LVSPEC_OK) return rc;
  if (pl.ws_bytes > (size_t)LVSPEC_STATIC_SCRATCH_BYTES) return LVSPEC_ESCRATCH;
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != LVSPEC_OK) return rc;
  return enqueue_attn(a, pl, ws, (size_t)LVSPEC_STATIC_SCRATCH_BYTES, stream);
}

}  // extern "C"

namespace {

int enqueue_attn(const lvspec_attn_args* a, const AttnPlan& pl, void* workspace, size_t have,
                 void* stream) {
  const AttnCut& cut = pl.served_by(have);
  lvspec::AttnKernelArgs k{};
  k.q = static_cast<const uint16_t*>(a->q);
  k.q_sb = a->q_sb; k.q_sg = a->q_sg; k.q_sh = a->q_sh;
  k.k = static_cast<const uint16_t*>(a->k);
  k.v = static_cast<const uint16_t*>(a->v);
  k.kv_sb = a->kv_sb; k.kv_sh = a->kv_sh; k.kv_sl = a->kv_sl;
  k.kv_len = a->kv_len;
  // lengths known to the host travel in the launch arguments: up to 6 in the lines the kernel's
  // prologue fetches anyway; a longer table only when there is no device array to read
  k.len_mode = (a->kv_len_host != nullptr && a->B <= 5) ? 1
               : (a->kv_len == nullptr && a->kv_len_host != nullptr && a->B <= 32) ? 2 : 0;
  for (int b = 0; b < 5; ++b)
    k.len_hot[b] = (k.len_mode == 1 && b < a->B) ? a->kv_len_host[b] : 0;
  for (int b = 0; b < 32; ++b)
    k.len_host[b] = (k.len_mode == 2 && b < a->B) ? a->kv_len_host[b] : 0;
  k.lmax = (int)(a->cap - a->gamma);
  k.vis_begin = a->vis_begin;
  k.vis_end = a->vis_end;
  k.B = a->B; k.gamma = a->gamma; k.Hq = a->Hq; k.Hkv = a->Hkv;
  k.G = pl.G; k.R = pl.R; k.rpad = cut.rpad; k.n_rc = cut.n_rc; k.n_split = cut.n_split;
  k.div_split = lvspec::make_fast_div((uint32_t)cut.n_split);
  k.div_rpad = lvspec::make_fast_div((uint32_t)cut.rpad);
  k.div_hkv = lvspec::make_fast_div((uint32_t)a->Hkv);
  k.div_rc = lvspec::make_fast_div((uint32_t)cut.n_rc);
  k.div_g = lvspec::make_fast_div((uint32_t)pl.G);
  const float scale = a->scale > 0.f ? a->scale : 1.0f / __builtin_sqrtf((float)a->D);
  k.xcd_map = ((int64_t)a->B * cut.n_rc * a->Hkv) % 8 == 0 ? 1 : 0;
  k.scale_log2e = scale * 1.4426950408889634f;
  k.ws = static_cast<float*>(workspace);
  // several sequences share one line of tiles; a workspace that holds only the partials of equal
  // splits is served by those.  The choice goes by the shapes, max_kv_len and the workspace, never
  // by kv_len_host: results are the same bits whether the host knows the lengths or not.
  constexpr int64_t kMaxStride = (int64_t)8 << 32;     // travels as a 32-bit number of 8 elements
  k.flat_pos = have >= cut.bytes() && a->kv_sb < kMaxStride && a->kv_sh < kMaxStride &&
                       a->kv_sl < kMaxStride ? cut.flat_pos : 0;
  for (int i = 0; i < 32; ++i)
    k.draft_mask[i] = a->draft_mask ? (i < a->gamma ? a->draft_mask[i] : 0u)
                                    : (0xffffffffu >> (31 - i));
  k.out = static_cast<uint16_t*>(a->out);
  k.o_sb = a->o_sb; k.o_sg = a->o_sg; k.o_sh = a->o_sh;
  k.lse = a->lse;
  k.vis_mass = a->vis_mass;
  hipError_t e = lvspec::launch_attn(k, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? LVSPEC_OK : hip_fail(e);
}

}  // namespace

extern "C" {

size_t lvspec_visual_relevance_workspace(const lvspec_rel_args* args) {
  RelPlan pl;
  return plan_rel(args, &pl) == LVSPEC_OK ? pl.ws_bytes : 0;
}

int lvspec_visual_relevance(const lvspec_rel_args* a, void* stream) {
  RelPlan pl;
  int rc = plan_rel(a, &pl);
  if (rc != LVSPEC_OK) return rc;
  if (!a->h_d || !a->l_v || !a->relevance || (a->lv_max > 0 && !a->h_v)) return LVSPEC_EINVAL;
  if (!aligned16(a->h_d) || !aligned16(a->h_v)) return LVSPEC_EINVAL;
  if (!stride_ok(a->hd_sb) || !stride_ok(a->hd_sg) || !stride_ok(a->hv_sb) ||
      !stride_ok(a->hv_sl) || a->hd_sg < a->d || a->hv_sl < a->d)
    return LVSPEC_EINVAL;
  rc = check_ws(a->workspace, a->workspace_bytes, pl.ws_bytes);
  if (rc != LVSPEC_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  uint8_t* ws = static_cast<uint8_t*>(a->workspace);
  float* dots = reinterpret_cast<float*>(ws);
  float* nv2 = reinterpret_cast<float*>(ws + pl.off_nv2);
  float* cosb = reinterpret_cast<float*>(ws + pl.off_cos);
  if (a->lv_max > 0) {
    lvspec::GemmKernelArgs g{};
    g.a = static_cast<const uint8_t*>(a->h_v);
    g.a_sb = a->hv_sb * 2;
    g.a_sr = a->hv_sl * 2;
    g.n_rows_dev = a->l_v;
    g.n_rows = (int)a->lv_max;
    g.x = static_cast<const uint8_t*>(a->h_d);
    g.x_sb = a->hd_sb * 2;
    g.x_sg = a->hd_sg * 2;
    g.gamma = a->gamma;
    g.n_cols = a->gamma;
    g.B = a->B;
    g.rows_per_block = pl.rows;
    g.row_bytes = pl.row_bytes;
    g.n_rb = pl.n_rb;
    g.n_ds = pl.n_ds;
    g.kc = pl.kc;
    g.n_tasks = a->B * pl.n_rb * pl.n_ds;
    g.dots = dots;
    g.nv2 = a->hv_inv_norm ? nullptr : nv2;   // prepared norms: dot products only
    g.ld = pl.ld;
    hipError_t e = lvspec::launch_rel_gemm(g, num_compute_units(), st);
    if (e != hipSuccess) return hip_fail(e);
  }
  lvspec::RelFinalizeArgs f{};
  f.h_d = static_cast<const uint16_t*>(a->h_d);
  f.hd_sb = a->hd_sb; f.hd_sg = a->hd_sg;
  f.d = a->d; f.gamma = a->gamma; f.B = a->B; f.top_n = a->top_n; f.n_ds = pl.n_ds;
  f.l_v = a->l_v;
  f.lv_max = a->lv_max;
  f.dots = dots; f.nv2 = nv2; f.ld = pl.ld; f.cosbuf = cosb;
  f.inv_norm = a->hv_inv_norm;
  f.cand_keys = reinterpret_cast<uint32_t*>(ws + pl.off_keys);
  f.n_parts = pl.n_parts;
  f.slice_rows = pl.slice_rows;
  f.relevance = a->relevance;
  hipError_t e = lvspec::launch_rel_finalize(f, st);
  return e == hipSuccess ? LVSPEC_OK : hip_fail(e);
}

int lvspec_hv_prepare(const lvspec_hv_args* a, void* stream) {
  if (a == nullptr) return LVSPEC_EINVAL;
  if (a->B < 1 || a->B > 65535 || a->d < 1 || a->lv_max < 0) return LVSPEC_EINVAL;
  if (a->d % 128 != 0 || a->lv_max > (int64_t)1 << 30) return LVSPEC_EUNSUPPORTED;
  if (!a->hv_inv_norm || (a->lv_max > 0 && !a->h_v)) return LVSPEC_EINVAL;
  if (!aligned16(a->h_v) || !stride_ok(a->hv_sb) || !stride_ok(a->hv_sl) || a->hv_sl < a->d)
    return LVSPEC_EINVAL;
  if (a->lv_max == 0) return LVSPEC_OK;
  lvspec::HvPrepareArgs k{};
  k.h_v = static_cast<const uint8_t*>(a->h_v);
  k.sb = a->hv_sb * 2; k.sl = a->hv_sl * 2;
  k.n_rows = a->lv_max; k.B = a->B; k.d = a->d;
  k.inv_norm = a->hv_inv_norm;
  hipError_t e = lvspec::launch_hv_prepare(k, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? LVSPEC_OK : hip_fail(e);
}

size_t lvspec_loose_accept_workspace(const lvspec_accept_args* args) {
  AccPlan pl;
  return plan_acc(args, &pl) == LVSPEC_OK ? pl.ws_bytes : 0;
}

int lvspec_loose_accept(const lvspec_accept_args* a, void* stream) {
  AccPlan pl;
  int rc = plan_acc(a, &pl);
  if (rc != LVSPEC_OK) return rc;
  if (!a->h_d || !a->lm_head || !a->draft_ids || !a->target_ids || !a->verdict ||
      !a->accept_len || !a->bonus_id)
    return LVSPEC_EINVAL;
  if (a->rule == LVSPEC_RULE_VISUAL && !a->relevance) return LVSPEC_EINVAL;
  if (!aligned16(a->h_d) || !aligned16(a->lm_head)) return LVSPEC_EINVAL;
  const int64_t w_sv = a->w_sv > 0 ? a->w_sv : a->d;
  if (!stride_ok(a->hd_sb) || !stride_ok(a->hd_sg) || !stride_ok(w_sv) || a->hd_sg < a->d ||
      w_sv < a->d)
    return LVSPEC_EINVAL;
  // a workspace too small for two groups in a pass is served group by group
  if (a->workspace_bytes < pl.ws_bytes && (rc = plan_acc(a, &pl, false)) != LVSPEC_OK) return rc;
  rc = check_ws(a->workspace, a->workspace_bytes, pl.ws_bytes);
  if (rc != LVSPEC_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  uint8_t* ws = static_cast<uint8_t*>(a->workspace);
  const int nbr = a->n_branches > 1 ? a->n_branches : 1;
  const int rpc = a->gamma + a->bonus_row;                         // hidden rows per chain
  for (int b0 = 0; b0 < a->B; b0 += pl.per_pass) {
    const int nb = a->B - b0 < pl.per_pass ? a->B - b0 : pl.per_pass;   // chains of this pass
    const int n_cols = nb * rpc;
    // a last, narrower pass has its own stage size and grid, within the records of a full pass
    int block_rows = pl.block_rows, n_tasks = pl.n_tasks, n_rec = pl.n_rec;
    if (n_cols < pl.n_cols) {
      block_rows = n_cols <= 32 && pl.rows_per_block == 64
                       ? 64 : lvspec::lmh_block_rows(n_cols, w_sv * 2, a->V, num_compute_units());
      n_tasks = (a->V + block_rows - 1) / block_rows;
      n_rec = lvspec::lmh_records(n_cols, n_tasks, num_compute_units());
      const int room = (int)((int64_t)pl.n_rec * pl.n_cols / n_cols);
      n_rec = n_rec < room ? n_rec : room;
    }
    const int64_t c0 = (int64_t)b0 * rpc;                          // first hidden row of this pass
    const int64_t t0 = (int64_t)b0 * a->gamma;                     // first draft token of this pass
    lvspec::GemmKernelArgs g{};
    g.a = static_cast<const uint8_t*>(a->lm_head);
    g.a_sb = 0;
    g.a_sr = w_sv * 2;
    g.n_rows_dev = nullptr;
    g.n_rows = a->V;
    g.x = static_cast<const uint8_t*>(a->h_d) + (int64_t)b0 * a->hd_sb * 2;
    g.x_sb = a->hd_sb * 2;
    g.x_sg = a->hd_sg * 2;
    g.gamma = rpc;
    g.n_cols = n_cols;
    g.half_cols = nb > pl.group ? pl.group * rpc : n_cols < 32 ? n_cols : 32;
    g.B = 1;
    g.rows_per_block = block_rows;
    g.rot_shift = pl.rows_per_block > block_rows ? 1 : 0;
    g.n_rb = n_tasks;
    g.n_ds = 1;
    g.kc = a->d / 128;
    g.row_bytes = 256;
    g.n_tasks = n_tasks;
    g.stats = reinterpret_cast<float*>(ws);
    g.cand = reinterpret_cast<uint64_t*>(ws + pl.off_cand);
    g.n_rec = n_rec;
    // the entropy rules read the row entropies, asked for or not
    const bool ent = a->entropy != nullptr || a->rule != LVSPEC_RULE_VISUAL;
    g.stats_z = ent ? reinterpret_cast<float*>(ws + pl.off_sz) : nullptr;
    g.topk = a->topk;
    g.logits = a->logits ? a->logits + c0 * a->V : nullptr;
    hipError_t e = lvspec::launch_lmh_gemm(g, num_compute_units(), st);
    if (e != hipSuccess) return hip_fail(e);
    lvspec::AcceptFinalizeArgs f{};
    f.B = nb; f.gamma = a->gamma; f.rows = rpc; f.V = a->V; f.topk = a->topk;
    f.n_rec = n_rec;
    f.div_topk = lvspec::make_fast_div((uint32_t)a->topk);
    f.stats = g.stats; f.stats_z = g.stats_z; f.cand = g.cand;
    f.entropy = a->entropy ? a->entropy + c0 : nullptr;
    f.rule = a->rule; f.ent_threshold = a->entropy_threshold; f.defer_window = a->defer_window;
    f.draft_ids = a->draft_ids + t0;
    f.relevance = a->relevance ? a->relevance + t0 : nullptr;
    f.n_loose = a->n_loose; f.pst_window = a->pst_window; f.gate = a->loose_topk_gate;
    f.n_branches = nbr;
    f.best_branch = a->best_branch ? a->best_branch + b0 / nbr : nullptr;
    f.target_ids = a->target_ids + c0;
    f.topk_ids = a->topk_ids ? a->topk_ids + c0 * a->topk : nullptr;
    f.topk_probs = a->topk_probs ? a->topk_probs + c0 * a->topk : nullptr;
    f.verdict = a->verdict + t0;
    f.accept_len = a->accept_len + b0;
    f.bonus_id = a->bonus_id + b0;
    e = lvspec::launch_accept_finalize(f, st);
    if (e != hipSuccess) return hip_fail(e);
  }
  return LVSPEC_OK;
}

int lvspec_kv_commit(const lvspec_commit_args* a, void* stream) {
  if (a == nullptr) return LVSPEC_EINVAL;
  const int nbr = a->n_branches > 1 ? a->n_branches : 1;
  if (a->B < 1 || a->B > 65535 || a->Hkv < 1 || a->D < 8 || a->D % 8 != 0 || a->n_layers < 1 ||
      a->n_layers > 65535 || a->n_branches < 0 || a->n_branches > LVSPEC_MAX_BRANCHES ||
      a->chain_len < 1 || a->chain_len > LVSPEC_MAX_GAMMA ||
      nbr * a->chain_len > LVSPEC_MAX_DRAFT_ROWS || a->cap < nbr * a->chain_len)
    return LVSPEC_EINVAL;
  if (!a->k || !a->v || !a->kv_len || !a->accept_len || !a->new_len ||
      a->new_len == a->kv_len)
    return LVSPEC_EINVAL;
  if (!aligned16(a->k) || !aligned16(a->v)) return LVSPEC_EINVAL;
  if (!stride_ok(a->kv_sb) || !stride_ok(a->kv_sh) || !stride_ok(a->kv_sl) || a->kv_sl < a->D ||
      (a->n_layers > 1 && (!stride_ok(a->kv_slayer) || a->kv_slayer < 1)))
    return LVSPEC_EINVAL;
  if ((int64_t)2 * a->Hkv * a->chain_len * (a->D / 8) > ((int64_t)1 << 30))
    return LVSPEC_EUNSUPPORTED;
  lvspec::CommitKernelArgs c{};
  c.k = static_cast<uint8_t*>(a->k);
  c.v = static_cast<uint8_t*>(a->v);
  c.slayer = a->n_layers > 1 ? a->kv_slayer * 2 : 0;
  c.sb = a->kv_sb * 2; c.sh = a->kv_sh * 2; c.sl = a->kv_sl * 2;
  c.B = a->B; c.Hkv = a->Hkv; c.n_layers = a->n_layers;
  c.n_branches = nbr; c.chain_len = a->chain_len;
  c.chunks = a->D / 8;
  c.cap = a->cap;
  c.kv_len = a->kv_len; c.accept_len = a->accept_len;
  c.best_branch = nbr > 1 ? a->best_branch : nullptr;
  c.new_len = a->new_len;
  hipError_t e = lvspec::launch_kv_commit(c, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? LVSPEC_OK : hip_fail(e);
}

int lvspec_describe_plan(const lvspec_attn_args* attn, const lvspec_rel_args* rel,
                         const lvspec_accept_args* accept, lvspec_plan_info* out) {
  if (out == nullptr) return LVSPEC_EINVAL;
  int first = LVSPEC_OK;
  if (attn != nullptr) {
    AttnPlan pl;
    const int rc = plan_attn(attn, &pl);
    if (rc == LVSPEC_OK) {
      const AttnCut& cut = pl.served_by(attn->workspace_bytes);
      out->attn_rows_padded = cut.rpad;
      out->attn_row_chunks = cut.n_rc;
      out->attn_splits = cut.n_split;
    } else if (first == LVSPEC_OK) {
      first = rc;
    }
  }
  if (rel != nullptr) {
    RelPlan pl;
    const int rc = plan_rel(rel, &pl);
    if (rc == LVSPEC_OK) {
      out->rel_splits = pl.n_ds;
      out->rel_stage_bytes = pl.row_bytes;
      out->rel_slices = pl.n_parts;
      out->rel_slice_rows = pl.slice_rows;
    } else if (first == LVSPEC_OK) {
      first = rc;
    }
  }
  if (accept != nullptr) {
    AccPlan pl;
    const int rc = plan_acc(accept, &pl);
    if (rc == LVSPEC_OK) {
      out->acc_rows_per_task = pl.rows_per_block;
      out->acc_chains_per_pass = pl.group;
      out->acc_passes = (accept->B + pl.group - 1) / pl.group;
    } else if (first == LVSPEC_OK) {
      first = rc;
    }
  }
  return first;
}

}  // extern "C"
