// Streamed skinny GEMM for gfx950: C[r][c] = sum_t A[r][t] X[c][t] with A a tall bf16 matrix read
// exactly once from HBM and X at most 128 bf16 rows.  Two users:
//   relevance (paper Eq. 8):  A = video hidden states H_V [l_v, d], X = draft hidden states
//       H_D [gamma, d]; the kernel emits raw dot products and squared row norms per split of d;
//       a finalize kernel turns them into cosines and the mean of the Top-N.
//   lm_head (paper Eq. 6):    A = lm_head [V, d], X = the B*gamma final hidden rows; the
//       epilogue folds each block of vocabulary rows into the workgroup's running (max, sum exp,
//       top-k candidates) per column, so the gamma x V logits never have to be re-read (they are
//       written only on request) and a column leaves one record per workgroup.
//
// Structure: persistent workgroups (two per CU, 4 waves each).  A workgroup walks its tasks (row
// block x split of d) as one uninterrupted sequence of stages; a stage is a slice of d of RB
// bytes per row (RB = 256 or 512: 128 or 256 elements).  Every wave copies its own 16*MB rows of
// A plus a share of the X slice straight into LDS (a ring of as many slots as fit into half of
// the CU's LDS: two to four), then all waves meet at one barrier per stage and feed 16x16x32
// bf16 MFMAs from LDS.  The ring keeps running across task boundaries, so there is no pipeline
// bubble between tasks.  Squared norms of the A rows come from the diagonal of A A^T on the
// same MFMA operands.
//
// Instances <MODE, MB, NBX, RB>: 64*MB rows of A per task, 16*NBX columns of X.
//   relevance: <1,1,512> (up to 16 draft rows, d % 256 == 0); otherwise <1|2, 1|2, 256>
//   lm_head:   <1,1,256> or <2,1,256> up to 16 columns, <1,2,256> or <2,2,256> up to 32, each with and
//              without the sorting networks of long candidate lists; more
//              columns (up to 128) take lm_head_wide_kernel below
#include "lvspec_dev.h"
#include "lvspec_kernels.h"

namespace lvspec {

namespace {

constexpr int MODE_REL = 0;    // relevance, squared row norms of A taken in the same pass
constexpr int MODE_LMH = 1;
constexpr int MODE_RELP = 2;   // relevance with the rows' inverse norms prepared by the caller
constexpr int MODE_LMHS = 3;   // lm_head with more than kSortTopk candidates asked for
constexpr bool is_rel(int mode) { return mode != MODE_LMH && mode != MODE_LMHS; }

template <int MB, int NBX, int RB>
struct Geo {
  static_assert(RB == 256 || RB == 512, "row bytes per stage");
  static constexpr int kKSteps = RB / 64;                  // 32-deep MFMA steps per stage
  static constexpr int kRowsPerInstr = 1024 / RB;          // rows one copy instruction covers
  static constexpr int kLanesPerRow = RB / 16;
  static constexpr int kAInstr = 16 * MB / kRowsPerInstr;  // A copy instructions per wave
  static constexpr int kXInstr = 16 * NBX / kRowsPerInstr / 4;   // X copy instructions per wave
  static constexpr int kInstrPerStage = kAInstr + kXInstr;
  static constexpr int kAWave = MB * 16 * RB;              // bytes of A per wave per stage
  static constexpr int kA = 4 * kAWave;
  static constexpr int kX = NBX * 16 * RB;
  static constexpr int kStage = kA + kX;
  // Two workgroups share a CU (80 KiB of LDS each): while one waits at its stage barrier or for
  // LDS, the other one issues copies and MFMAs.  Each gets as many ring slots as fit (at most
  // 8); the epilogue tile reuses the slot that has just been consumed.
  static constexpr int kWgPerCu = 2;
  static constexpr int kFit = (160 * 1024 / kWgPerCu) / kStage;
  static constexpr int kStages = kFit > 8 ? 8 : kFit;
  static constexpr int kRing = kStages * kStage;
  static constexpr int kRowsWg = 64 * MB;
  static constexpr int kZtStride = kRowsWg + 4;            // floats per column in the epilogue tile
  static constexpr int kZt = 16 * NBX * kZtStride * 4;     // bytes
};

struct Cursor {
  int task;   // global task index (strided by gridDim.x)
  int kc;     // chunk within the task
  int cb;     // batch whose row count is cached in cn (-1: none); consecutive tasks of a
  int cn;     // workgroup mostly share the batch, so the device read happens once per batch
};

template <int MODE>
LVS_DEV void decode_task(const GemmKernelArgs& p, int task, int& b, int& rb, int& ds) {
  if (is_rel(MODE)) {
    ds = task % p.n_ds;
    const int t2 = task / p.n_ds;
    rb = t2 % p.n_rb;
    b = t2 / p.n_rb;
  } else {
    ds = 0;
    rb = task;
    b = 0;
  }
}

template <int MODE>
LVS_DEV int rows_of(const GemmKernelArgs& p, Cursor& c, int b) {
  if (is_rel(MODE)) {
    if (b != c.cb) {
      const int n = __builtin_amdgcn_readfirstlane(p.n_rows_dev[b]);
      c.cb = b;
      c.cn = n < p.n_rows ? n : p.n_rows;
    }
    return c.cn;
  }
  return p.n_rows;
}

// skip tasks whose row block lies beyond the valid rows of their batch
template <int MODE, int ROWS_WG>
LVS_DEV void settle(const GemmKernelArgs& p, Cursor& c) {
  if (is_rel(MODE)) {
    while (c.task < p.n_tasks) {
      int b, rb, ds;
      decode_task<MODE>(p, c.task, b, rb, ds);
      if (rb * ROWS_WG < rows_of<MODE>(p, c, b)) break;
      c.task += gridDim.x;
    }
  }
}

template <int MODE, int ROWS_WG>
LVS_DEV void advance(const GemmKernelArgs& p, Cursor& c) {
  if (++c.kc == p.kc) {
    c.kc = 0;
    c.task += gridDim.x;
    settle<MODE, ROWS_WG>(p, c);
  }
}

// Per-lane source pointers of the task the issue cursor is in: computed once per task, so that a
// stage costs one 64-bit add per copy instruction instead of a multiply-add chain.
//
// Copy geometry: one instruction moves 1 KiB = kRowsPerInstr rows x RB bytes; lane l handles
// row (l / kLanesPerRow) of the instruction at LDS chunk position cpos = l % kLanesPerRow and
// fetches the global chunk cpos ^ (row & 15) of the stage's RB-byte row segment (the XOR stays
// inside a 256-byte half, so MFMA operand reads of 16 rows at one logical chunk hit 16
// different bank groups).
template <int MB, int NBX, int RB>
struct IssuePtrs {
  const uint8_t* arow[Geo<MB, NBX, RB>::kAInstr];   // A row of copy instruction j at the task's first column
  const uint8_t* xcol[Geo<MB, NBX, RB>::kXInstr];   // X row of copy instruction k
  int rot;                                          // task mod chunks per task: first chunk read
};

template <int MODE, int MB, int NBX, int RB>
LVS_DEV void setup_task(const GemmKernelArgs& p, Cursor& c, IssuePtrs<MB, NBX, RB>& ip,
                        int wave, int lane) {
  using G = Geo<MB, NBX, RB>;
  if (c.task >= p.n_tasks) return;
  int b, rb, ds;
  decode_task<MODE>(p, c.task, b, rb, ds);
  const int n_rows = rows_of<MODE>(p, c, b);
  ip.rot = (c.task >> p.rot_shift) % p.kc;
  const int rsub = lane / G::kLanesPerRow;
  const int cpos = lane % G::kLanesPerRow;
  const int64_t col_byte = (int64_t)ds * p.kc * RB;
  const uint8_t* abase = p.a + (int64_t)b * p.a_sb + col_byte;
  const int row0 = rb * G::kRowsWg + wave * 16 * MB;
#pragma unroll
  for (int j = 0; j < G::kAInstr; ++j) {
    const int rl = G::kRowsPerInstr * j + rsub;      // row within the wave's tile
    int row = row0 + rl;
    row = row < n_rows ? row : n_rows - 1;
    ip.arow[j] = abase + (int64_t)row * p.a_sr + ((cpos ^ (rl & 15)) << 4);
  }
#pragma unroll
  for (int k = 0; k < G::kXInstr; ++k) {
    const int jx = 4 * k + wave;
    const int cl = G::kRowsPerInstr * jx + rsub;     // LDS row of this lane in the X tile
    const int col = cl < p.n_cols ? cl : p.n_cols - 1;
    int xb, xi;
    if (is_rel(MODE)) {
      xb = b;
      xi = col;
    } else {
      xb = col / p.gamma;
      xi = col - xb * p.gamma;
    }
    ip.xcol[k] = p.x + (int64_t)xb * p.x_sb + (int64_t)xi * p.x_sg + col_byte +
                 ((cpos ^ (cl & 15)) << 4);
  }
}

// Stage kc of a task reads column chunk (kc + task) mod n_chunks of its slice: the workgroups
// walk the hidden dimension from different starting points, so at any moment their row
// segments spread over all HBM channels (with a power-of-two row pitch, e.g. d = 8192, all
// rows of a column chunk fall into the same few channels).  The order is a fixed function of
// the task, so results stay reproducible.  lm_head: of the block of 64 (rot_shift = 0) or 128
// vocabulary rows (lmh_order_rows), whatever the rows of a stage: a logit's bits, and with them the
// order of tokens that nearly tie, do not depend on the stage size or on which rows share the call.
template <int MB, int NBX, int RB>
LVS_DEV void issue_stage(const IssuePtrs<MB, NBX, RB>& ip, int kc, int n_chunks, uint32_t slot,
                         int wave) {
  using G = Geo<MB, NBX, RB>;
  int chunk = kc + ip.rot;
  chunk = chunk >= n_chunks ? chunk - n_chunks : chunk;
  const int64_t off = (int64_t)chunk * RB;
#pragma unroll
  for (int j = 0; j < G::kAInstr; ++j) dma16(ip.arow[j] + off, slot + wave * G::kAWave + j * 1024);
#pragma unroll
  for (int k = 0; k < G::kXInstr; ++k)
    dma16<kCopyDefault>(ip.xcol[k] + off, slot + G::kA + (4 * k + wave) * 1024);
}

// advance the issue cursor; recompute the source pointers when it enters a new task
template <int MODE, int MB, int NBX, int RB>
LVS_DEV void advance_issue(const GemmKernelArgs& p, Cursor& c, IssuePtrs<MB, NBX, RB>& ip,
                           int wave, int lane) {
  using G = Geo<MB, NBX, RB>;
  if (++c.kc == p.kc) {
    c.kc = 0;
    c.task += gridDim.x;
    settle<MODE, G::kRowsWg>(p, c);
    setup_task<MODE, MB, NBX, RB>(p, c, ip, wave, lane);
  }
}

// wait until at most `ahead` whole stages (IPS copy instructions each) of this wave are still
// outstanding; ahead is uniform and in [0, MAXA]
template <int IPS, int MAXA>
LVS_DEV void wait_stages(int ahead) {
  if constexpr (MAXA <= 0) {
    wait_copies<0>();
  } else {
    if (ahead >= MAXA) {
      wait_copies<(IPS * MAXA > 63 ? 63 : IPS * MAXA)>();
    } else {
      wait_stages<IPS, MAXA - 1>(ahead);
    }
  }
}


// ---- running softmax statistics and top-k of one logits column over the tasks of a workgroup ----
// The same wave serves a column in every task, so the state stays in its registers: lane l keeps
// the maximum and the sums of the rows it has seen (no cross-lane work per task), lane r the r-th
// best candidate of the whole wave.  Per task only the rows that beat the k-th best so far cost a
// selection round (about k/t of task t's rows do), where every task used to run k rounds of its own
// and write k candidates: five columns, V = 152064: 2376 records per column before, 476 now; the
// pass itself 228.5 -> 223.6 us at d = 5120, with 48 columns 333 -> 307, with k = 16 (d = 3584)
// 177 -> 163.
struct ColumnState {
  uint64_t top;   // lane r < k: r-th best (value, id) key, descending; 0 = none
  float m, s, sz; // this lane's rows: maximum, sum exp(z - m), sum exp(z - m) * z
};

LVS_DEV void column_init(ColumnState& c) {
  c.top = 0ull;
  c.m = -INFINITY;
  c.s = 0.f;
  c.sz = 0.f;
}

// v[j]: logit of vocabulary row id0 + 64 * j (lane's rows), to be ignored from n_rows on.
// The set of the k best under the total order (value descending, id ascending) does not depend
// on the order in which rows arrive, and the tasks of a workgroup are a fixed function of the
// shape: results are reproducible.
template <int NV, bool SORT>
LVS_DEV void column_fold(ColumnState& c, const float (&vin)[NV], int id0, int n_rows, int topk,
                         bool want_z, int lane) {
  float v[NV];
  uint64_t key[NV];
  float mn = c.m;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int id = id0 + 64 * j;
    v[j] = id < n_rows ? vin[j] : -INFINITY;
    key[j] = v[j] != -INFINITY ? cand_key(v[j], id) : 0ull;
    mn = fmaxf(mn, v[j]);
  }
  const float keep = c.m == -INFINITY ? 0.f : fast_exp2((c.m - mn) * kLog2e);
  float s = c.s * keep;
  float e[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    e[j] = v[j] == -INFINITY ? 0.f : fast_exp2((v[j] - mn) * kLog2e);
    s += e[j];
  }
  if (want_z) {
    float sz = c.sz * keep;
#pragma unroll
    for (int j = 0; j < NV; ++j) sz += v[j] == -INFINITY ? 0.f : e[j] * v[j];
    c.sz = sz;
  }
  c.m = mn;
  c.s = s;
  topk_take<NV, SORT>(c.top, key, topk, lane);
}

// the workgroup's record of a column
LVS_DEV void column_emit(const ColumnState& c, const GemmKernelArgs& p, int col, int lane) {
  const float mx = wave_max(c.m);
  const float f = c.m == -INFINITY ? 0.f : fast_exp2((c.m - mx) * kLog2e);
  const float s = wave_sum(c.s * f);
  const int64_t rec = (int64_t)col * p.n_rec + blockIdx.x;
  if (lane == 0) {
    // The merge ranks the records by this maximum.  The maximum of floats passes over NaN, the
    // candidates do not: a record whose best candidate is NaN (there is nothing else in it, or
    // the NaN ranks above the rest) says so, or the merge would not look at its candidates.
    const uint32_t best = (uint32_t)(c.top >> 32);
    const float v = key_value(best);
    p.stats[rec * 2] = best != 0u && v != v ? v : mx;
    p.stats[rec * 2 + 1] = s;
  }
  if (p.stats_z != nullptr) {
    const float sz = wave_sum(c.sz * f);
    if (lane == 0) p.stats_z[rec] = sz;
  }
  if (lane < p.topk) p.cand[rec * p.topk + lane] = c.top;
}

// Four columns' values of this lane's rows from the epilogue tile.  Assembly, like every LDS read
// of these kernels: an ordinary load would wait for all outstanding copies.
template <int NV>
LVS_DEV void read_columns4(float (&v)[4][NV], const uint32_t (&a)[4]) {
  static_assert(NV == 1 || NV == 2, "64 or 128 rows");
  if constexpr (NV == 1) {
    asm volatile(
        "ds_read_b32 %0, %4\n\tds_read_b32 %1, %5\n\tds_read_b32 %2, %6\n\tds_read_b32 %3, %7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0][0]), "=&v"(v[1][0]), "=&v"(v[2][0]), "=&v"(v[3][0])
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
        : "memory");
  } else {
    asm volatile(
        "ds_read_b32 %0, %8\n\tds_read_b32 %1, %8 offset:256\n\t"
        "ds_read_b32 %2, %9\n\tds_read_b32 %3, %9 offset:256\n\t"
        "ds_read_b32 %4, %10\n\tds_read_b32 %5, %10 offset:256\n\t"
        "ds_read_b32 %6, %11\n\tds_read_b32 %7, %11 offset:256\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0][0]), "=&v"(v[0][1]), "=&v"(v[1][0]), "=&v"(v[1][1]), "=&v"(v[2][0]),
          "=&v"(v[2][1]), "=&v"(v[3][0]), "=&v"(v[3][1])
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
        : "memory");
  }
}

// own LDS writes done, then the barrier; unlike __syncthreads it leaves copies in flight
LVS_DEV void barrier_after_lds_writes() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int MODE, int MB, int NBX, int RB>
__global__ __launch_bounds__(256, 2) void gemm_stream_kernel(const GemmKernelArgs p) {
  using G = Geo<MB, NBX, RB>;
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n16 = lane & 15;
  const int g4 = lane >> 4;
  const uint32_t ring = lds_addr(smem);

  // operand chunk 4*ks + g4 of row n16, for ks = 0..3; steps 4..7 (RB = 512) sit 256 bytes on
  uint32_t oaddr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) oaddr[i] = n16 * RB + (((4 * i + g4) ^ n16) << 4);

  f32x4 acc[MB][NBX];
  f32x4 accn[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    accn[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nx = 0; nx < NBX; ++nx) acc[mb][nx] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // lm_head: wave w serves columns w, w + 4, ...
  constexpr int kCols = is_rel(MODE) ? 1 : 4 * NBX;
  ColumnState cst[kCols];
  if constexpr (!is_rel(MODE)) {
#pragma unroll
    for (int t = 0; t < kCols; ++t) column_init(cst[t]);
  }

  Cursor cc{(int)blockIdx.x, 0, -1, 0};   // compute cursor
  settle<MODE, G::kRowsWg>(p, cc);
  Cursor ic = cc;                  // issue cursor
  IssuePtrs<MB, NBX, RB> ip;
  setup_task<MODE, MB, NBX, RB>(p, ic, ip, wave, lane);
  int ahead = -1;                  // stages issued beyond the one about to be consumed
  wait_copies<0>();
#pragma unroll
  for (int s = 0; s < G::kStages - 1; ++s) {
    if (ic.task < p.n_tasks) {
      issue_stage<MB, NBX, RB>(ip, ic.kc, p.kc, ring + s * G::kStage, wave);
      advance_issue<MODE, MB, NBX, RB>(p, ic, ip, wave, lane);
      ++ahead;
    }
  }

  int slot_c = 0;    // ring slot of the stage being consumed
  while (cc.task < p.n_tasks) {
    const uint32_t slot = ring + slot_c * G::kStage;
    // epilogue tile: the slot being consumed is free from the last operand read of this
    // iteration until the next iteration's barrier
    float* zt = reinterpret_cast<float*>(smem + slot_c * G::kStage);
    wait_stages<G::kInstrPerStage, G::kStages - 2>(ahead);
    __builtin_amdgcn_s_barrier();
    // refill the slot consumed in the previous iteration (it + kStages - 1 lands there)
    if (ic.task < p.n_tasks) {
      const int slot_i = slot_c == 0 ? G::kStages - 1 : slot_c - 1;
      issue_stage<MB, NBX, RB>(ip, ic.kc, p.kc, ring + slot_i * G::kStage, wave);
      advance_issue<MODE, MB, NBX, RB>(p, ic, ip, wave, lane);
    } else {
      ahead -= 1;
    }
    // ---- operands from LDS, four 32-deep steps at a time -------------------------------------
#pragma unroll
    for (int half = 0; half < G::kKSteps / 4; ++half) {
      u32x4 aop[MB][4];
      u32x4 xop[NBX][4];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        uint32_t a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          a[ks] = slot + wave * G::kAWave + mb * 16 * RB + half * 256 + oaddr[ks];
        lds_read4(aop[mb], a);
      }
#pragma unroll
      for (int nx = 0; nx < NBX; ++nx) {
        uint32_t a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          a[ks] = slot + G::kA + nx * 16 * RB + half * 256 + oaddr[ks];
        lds_read4(xop[nx], a);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
          for (int nx = 0; nx < NBX; ++nx)
            acc[mb][nx] = mfma16(aop[mb][ks], xop[nx][ks], acc[mb][nx]);
          if (MODE == MODE_REL) accn[mb] = mfma16(aop[mb][ks], aop[mb][ks], accn[mb]);
        }
      }
    }
    // ---- end of a task: epilogue -----------------------------------------------------------
    if (cc.kc == p.kc - 1) {
      int b, rb, ds;
      decode_task<MODE>(p, cc.task, b, rb, ds);
      const int row0 = rb * G::kRowsWg;
      if constexpr (is_rel(MODE)) {
        // acc[mb][nx][i] = dot(A row row0 + wave*16*MB + 16*mb + 4*g4 + i, X column 16*nx + n16)
#pragma unroll
        for (int nx = 0; nx < NBX; ++nx) {
          const int col = 16 * nx + n16;
          if (col < p.gamma) {
            float* dp = p.dots + (((int64_t)b * p.n_ds + ds) * p.gamma + col) * p.ld + row0 +
                        wave * 16 * MB + 4 * g4;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4*>(dp + 16 * mb) = acc[mb][nx];
          }
        }
        // squared norms sit on the diagonal of A A^T: lane (n16, g4 == n16/4), element n16 % 4
        if (MODE == MODE_REL && g4 == (n16 >> 2)) {
          float* np = p.nv2 + ((int64_t)b * p.n_ds + ds) * p.ld + row0 + wave * 16 * MB + n16;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const int e = n16 & 3;
            const float v = e == 0 ? accn[mb][0] : e == 1 ? accn[mb][1] : e == 2 ? accn[mb][2]
                                                                                 : accn[mb][3];
            np[16 * mb] = v;
          }
        }
      } else {
        const int n_rows = p.n_rows;
        // the tile overlays the slot just consumed: every wave must be done reading operands
        __builtin_amdgcn_s_barrier();
        // logits tile to LDS as [column][row]
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nx = 0; nx < NBX; ++nx)
            *reinterpret_cast<f32x4*>(zt + (16 * nx + n16) * G::kZtStride + wave * 16 * MB +
                                      16 * mb + 4 * g4) = acc[mb][nx];
        barrier_after_lds_writes();
        const uint32_t zl = slot + (uint32_t)lane * 4u;
#pragma unroll
        for (int t4 = 0; t4 < kCols; t4 += 4) {
          if (wave + 4 * t4 < p.n_cols) {
            uint32_t a[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t] = zl + (wave + 4 * (t4 + t)) * (G::kZtStride * 4);
            float v[4][MB];
            read_columns4<MB>(v, a);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int col = wave + 4 * (t4 + t);
              if (col < p.n_cols) {
                if (p.logits != nullptr) {
#pragma unroll
                  for (int j = 0; j < MB; ++j)
                    if (row0 + lane + 64 * j < n_rows)
                      p.logits[(int64_t)col * n_rows + row0 + lane + 64 * j] = v[t][j];
                }
                column_fold<MB, MODE == MODE_LMHS>(cst[t4 + t], v[t], row0 + lane, n_rows, p.topk,
                                p.stats_z != nullptr, lane);
              }
            }
          }
        }
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        accn[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nx = 0; nx < NBX; ++nx) acc[mb][nx] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    advance<MODE, G::kRowsWg>(p, cc);
    slot_c = slot_c + 1 == G::kStages ? 0 : slot_c + 1;
  }
  if constexpr (!is_rel(MODE)) {
#pragma unroll
    for (int t = 0; t < kCols; ++t)
      if (wave + 4 * t < p.n_cols) column_emit(cst[t], p, wave + 4 * t, lane);
  }
}

// ---- lm_head for 33 to 128 hidden rows ------------------------------------------------------------
// A server's batch brings more hidden rows than the kernel above can hold next to its ring: with more
// than 32 columns half of a CU's LDS would leave room for one stage in flight (two slots).  Here
// one workgroup of eight waves has the CU to itself: 64 * MB vocabulary rows by two
// column halves of 16 * NB2, waves 4 (row groups of 16 * MB) x 2 (halves), so that a wave feeds
// MB * NB2 independent accumulators from MB + NB2 operands per step and every X byte in LDS is
// read by four waves instead of eight.  No unit is what bounds it: with 96 columns (4.8 TB/s) the
// counters show the LDS active for 15 % of the cycles, without bank conflicts, and the matrix cores busy
// for 18 %.  (Read from the code, not measured: a stage is 32 KiB of lm_head and 24 KiB of X per CU and
// ends on a barrier that waits for the slowest of eight waves' copies, with two stages in flight.)
//
// Rings: three slots of A (two stages in flight) and two of X (it comes from L2).  Copies complete
// in issue order, so X(i+1) is issued ahead of A(i+2) and the wait for X(i) leaves A(i+1) out.
// Two groups of chains with up to 64 columns each share a pass, one in each half; a single group of
// more than 32 columns is split over the halves.
//
// A block of 64 vocabulary rows adds its chunks up from chunk (block mod n_chunks) on, as in
// gemm_stream_kernel.  The second block of a 128-row task thus starts one chunk later than the
// first: it joins in at the task's second stage and ends one stage behind, while the X chunk of
// a stage serves both (n_chunks + 1 stages; with one start for both blocks the logits are other
// 32-bit sums, and tokens that tie within 6e-6 change places: 2 of 576 ids at k = 16).
// 96 rows, d = 5120, V = 152064: 689 us in two passes of 48 columns, 335 here (328 without the
// extra stage).
template <int MB, int NB2>
struct Wide {
  static constexpr int kRowsWg = 64 * MB;
  static constexpr int kASlot = kRowsWg * kRowBytes;
  static constexpr int kXSlot = 2 * NB2 * 16 * kRowBytes;
  static constexpr int kXOff = 3 * kASlot;
  static constexpr int kLds = kXOff + 2 * kXSlot;
  static constexpr int kAInstr = 2 * MB;        // copy instructions per wave and stage
  static constexpr int kXInstr = NB2;
  static constexpr int kZtStride = kRowsWg + 4; // floats per column of the epilogue tile
  static constexpr int kLate = MB == 2 ? 1 : 0; // stages the second 64-row block starts late
  static_assert(kLds <= 160 * 1024, "LDS of one CU");
  static_assert(32 * kZtStride * 4 <= kASlot, "epilogue tile of 32 columns in one A slot");
};

template <int MB, int NB2, bool SORT>
__global__ __launch_bounds__(512, 2) void lm_head_wide_kernel(const GemmKernelArgs p) {
  using W = Wide<MB, NB2>;
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave & 3;       // row group
  const int wc = wave >> 2;      // column half
  const int n16 = lane & 15;
  const int g4 = lane >> 4;
  const uint32_t ring = lds_addr(smem);
  const int n_chunks = p.kc;     // 256-byte chunks of a row
  const int n_stages = n_chunks + W::kLate;
  // the stages of a task in which this wave copies, and computes, rows of its block
  const int copy_from = wave >= 4 ? W::kLate : 0;
  const int comp_from = wr >= 2 ? W::kLate : 0;

  uint32_t oaddr[4];             // operand chunk 4*ks + g4 of row n16
#pragma unroll
  for (int i = 0; i < 4; ++i) oaddr[i] = n16 * kRowBytes + (((4 * i + g4) ^ n16) << 4);

  // X sources: LDS row cl of half h = cl / (16 * NB2) is column h * half_cols + cl % (16 * NB2);
  // rows without a column hold a copy of the last one and are never looked at
  const int rsub = lane >> 4;
  const uint8_t* xcol[W::kXInstr];
#pragma unroll
  for (int k = 0; k < W::kXInstr; ++k) {
    const int cl = 4 * (8 * k + wave) + rsub;
    const int h = cl / (16 * NB2);
    int col = h * p.half_cols + (cl - h * 16 * NB2);
    col = col < p.n_cols ? col : p.n_cols - 1;
    const int xb = col / p.gamma;
    const int xi = col - xb * p.gamma;
    xcol[k] = p.x + (int64_t)xb * p.x_sb + (int64_t)xi * p.x_sg + ((n16 ^ (cl & 15)) << 4);
  }
  // stage kc of a task reads chunk (kc + first 64-row block) mod n_chunks
  auto chunk_of = [&](int task, int kc) {
    const int c = kc + (task * MB) % n_chunks;
    return c >= n_chunks ? c - n_chunks : c;
  };
  int ia_task = blockIdx.x, ia_kc = 0;     // next A stage to issue
  int ix_task = blockIdx.x, ix_kc = 0;     // next X stage to issue
  const uint8_t* arow[W::kAInstr];
  auto setup_a = [&] {
#pragma unroll
    for (int j = 0; j < W::kAInstr; ++j) {
      const int rl = wave * 8 * MB + 4 * j + rsub;
      int row = ia_task * W::kRowsWg + rl;
      row = row < p.n_rows ? row : p.n_rows - 1;
      arow[j] = p.a + (int64_t)row * p.a_sr + ((n16 ^ (rl & 15)) << 4);
    }
  };
  // the next A stage, if there is one; returns whether this wave has a share of it
  auto issue_a = [&](int slot) {
    if (ia_task >= p.n_tasks) return false;
    const bool mine = ia_kc >= copy_from && ia_kc < copy_from + n_chunks;
    if (mine) {
      const int64_t off = (int64_t)chunk_of(ia_task, ia_kc) * kRowBytes;
      const uint32_t dst = ring + slot * W::kASlot + wave * (8 * MB * kRowBytes);
#pragma unroll
      for (int j = 0; j < W::kAInstr; ++j) dma16(arow[j] + off, dst + j * 1024);
    }
    if (++ia_kc == n_stages) {
      ia_kc = 0;
      ia_task += gridDim.x;
      if (ia_task < p.n_tasks) setup_a();
    }
    return mine;
  };
  auto issue_x = [&](int slot) {
    const int64_t off = (int64_t)chunk_of(ix_task, ix_kc) * kRowBytes;
    const uint32_t dst = ring + W::kXOff + slot * W::kXSlot;
#pragma unroll
    for (int k = 0; k < W::kXInstr; ++k)
      dma16<kCopyDefault>(xcol[k] + off, dst + (8 * k + wave) * 1024);
    if (++ix_kc == n_stages) {
      ix_kc = 0;
      ix_task += gridDim.x;
    }
  };

  f32x4 acc[MB][NB2];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB2; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the wave serves LDS columns wave, wave + 8, ... of each epilogue tile (32 columns: column
  // block jj of either half)
  ColumnState cst[4 * NB2];
#pragma unroll
  for (int t = 0; t < 4 * NB2; ++t) column_init(cst[t]);
  auto column_at = [&](int jj, int t, bool& on) {
    const int lc = wave + 8 * t;
    const int h = lc >> 4;
    const int within = jj * 16 + (lc & 15);
    const int width = h == 0 ? (p.half_cols < p.n_cols ? p.half_cols : p.n_cols)
                             : p.n_cols - p.half_cols;
    on = within < width;
    return h * p.half_cols + within;
  };

  int task = blockIdx.x, kc = 0;           // stage being consumed
  setup_a();
  wait_copies<0>();
  issue_x(0);
  issue_a(0);
  bool a_ahead = issue_a(1);               // this wave's share of the next A stage is on its way
  int sa = 0, sx = 0;                      // slots of the stage being consumed
  while (task < p.n_tasks) {
    if (a_ahead) wait_copies<W::kAInstr>(); else wait_copies<0>();
    __builtin_amdgcn_s_barrier();          // all shares landed; the slots of the last stage are free
    if (ix_task < p.n_tasks) issue_x(sx ^ 1);
    a_ahead = issue_a(sa == 0 ? 2 : sa - 1);
    const uint32_t aslot = ring + sa * W::kASlot;
    if (kc >= comp_from && kc < comp_from + n_chunks) {
      uint32_t a[4], x[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        a[ks] = aslot + wr * (16 * MB * kRowBytes) + oaddr[ks];
        x[ks] = ring + W::kXOff + sx * W::kXSlot + wc * (16 * NB2 * kRowBytes) + oaddr[ks];
      }
      u32x4 aop[MB][4];
      if constexpr (MB == 2) {
        u32x4 r[8];
        lds_read8_after<63, 16 * kRowBytes>(r, a);
#pragma unroll
        for (int i = 0; i < 8; ++i) aop[i >> 2][i & 3] = r[i];
      } else {
        lds_read4(aop[0], a);
      }
#pragma unroll
      for (int nb = 0; nb < NB2; ++nb) {
        u32x4 xop[4];
        uint32_t xa[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) xa[ks] = x[ks] + nb * 16 * kRowBytes;
        lds_read4(xop, xa);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[mb][nb] = mfma16(aop[mb][ks], xop[ks], acc[mb][nb]);
      }
    }
    if (kc == n_stages - 1) {
      // ---- end of a task: 32 columns at a time through the A slot just consumed
      const int row0 = task * W::kRowsWg;
      float* zt = reinterpret_cast<float*>(smem + sa * W::kASlot);
#pragma unroll
      for (int jj = 0; jj < NB2; ++jj) {
        __builtin_amdgcn_s_barrier();      // operand reads, or reads of the previous tile, are done
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          *reinterpret_cast<f32x4*>(zt + (wc * 16 + n16) * W::kZtStride + wr * 16 * MB + 16 * mb +
                                    4 * g4) = acc[mb][jj];
          acc[mb][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        barrier_after_lds_writes();
        uint32_t a[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
          a[t] = aslot + (uint32_t)lane * 4u + (wave + 8 * t) * (W::kZtStride * 4);
        float v[4][MB];
        read_columns4<MB>(v, a);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          bool on;
          const int col = column_at(jj, t, on);
          if (on) {
            if (p.logits != nullptr) {
#pragma unroll
              for (int j = 0; j < MB; ++j)
                if (row0 + lane + 64 * j < p.n_rows)
                  p.logits[(int64_t)col * p.n_rows + row0 + lane + 64 * j] = v[t][j];
            }
            column_fold<MB, SORT>(cst[4 * jj + t], v[t], row0 + lane, p.n_rows, p.topk,
                            p.stats_z != nullptr, lane);
          }
        }
      }
    }
    if (++kc == n_stages) {
      kc = 0;
      task += gridDim.x;
    }
    sa = sa == 2 ? 0 : sa + 1;
    sx ^= 1;
  }
#pragma unroll
  for (int jj = 0; jj < NB2; ++jj)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      bool on;
      const int col = column_at(jj, t, on);
      if (on) column_emit(cst[4 * jj + t], p, col, lane);
    }
}

// As many workgroups as fit at once, then trimmed so that every workgroup walks the same number
// of tasks (1188 tasks on 512 slots: 396 workgroups x 3 instead of 164 doing a third task while
// 348 sit idle).  The kernels are bandwidth-bound, so a few idle CUs cost nothing.
int stream_grid(int n_tasks, int slots) {
  int grid = n_tasks < slots ? n_tasks : slots;
  if (grid < 1) grid = 1;
  const int rounds = (n_tasks + grid - 1) / grid;
  if (rounds > 0) grid = (n_tasks + rounds - 1) / rounds;
  return grid < 1 ? 1 : grid;
}

template <int MODE, int MB, int NBX, int RB>
hipError_t launch_gemm(const GemmKernelArgs& a, int num_cu, hipStream_t stream) {
  using G = Geo<MB, NBX, RB>;
  static_assert(G::kZt <= G::kStage, "epilogue tile must fit in one ring slot");
  static_assert(G::kStages >= 2, "ring too small");
  static_assert(G::kInstrPerStage * (G::kStages - 2) <= 63, "copy counter range");
  const size_t lds = (size_t)G::kRing;
  static LdsLimitOnce lds_limit;
  hipError_t e = lds_limit.ensure(
      reinterpret_cast<const void*>(&gemm_stream_kernel<MODE, MB, NBX, RB>), lds);
  if (e != hipSuccess) return e;
  // (lm_head: one record per workgroup, the number the planner sized the records by)
  const int grid = !is_rel(MODE) ? a.n_rec : stream_grid(a.n_tasks, num_cu * G::kWgPerCu);
  hipLaunchKernelGGL((gemm_stream_kernel<MODE, MB, NBX, RB>), dim3(grid), dim3(256), lds, stream,
                     a);
  return hipGetLastError();
}

template <int MB, int NB2, bool SORT>
hipError_t launch_wide(const GemmKernelArgs& a, hipStream_t stream) {
  using W = Wide<MB, NB2>;
  static LdsLimitOnce lds_limit;
  hipError_t e = lds_limit.ensure(
      reinterpret_cast<const void*>(&lm_head_wide_kernel<MB, NB2, SORT>), W::kLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((lm_head_wide_kernel<MB, NB2, SORT>), dim3(a.n_rec), dim3(512), W::kLds, stream,
                     a);
  return hipGetLastError();
}

}  // namespace

int rel_rows_per_block(int big) { return big ? Geo<2, 1, 256>::kRowsWg : Geo<1, 1, 256>::kRowsWg; }
constexpr int kWideCols = 33;   // from here on lm_head_wide_kernel

int lmh_records(int n_cols, int n_tasks, int num_cu) {
  const int slots = n_cols >= kWideCols ? num_cu : num_cu * Geo<1, 1, 256>::kWgPerCu;
  return stream_grid(n_tasks, slots < kAcceptMaxRecords ? slots : kAcceptMaxRecords);
}

// Rows of a stage.  Up to 32 columns: 64-row stages with a three- or four-slot ring stream 2-4 %
// faster than 128-row stages with two slots (d = 2048 .. 7168), except at row pitches that are
// multiples of 8 KiB (d = 4096, 8192), where the 64 segments of a stage fall into too few HBM
// channels (d = 4096, five columns: 5.6 against 6.4 TB/s).  More columns: 128 rows (half the X
// traffic per lm_head byte), unless 64-row tasks give every CU one at most and 128-row tasks would
// leave half of them idle.  d = 5120, 96 columns, 64 and 128 rows: V = 8192 54.0 and 68.6 us, 16384
// 59.7 and 71.2; 24000 101 and 75, 36000 144 and 132 (although 128 rows leave the busiest CU a third
// more), 152064 427 and 326; d = 1024, 36 columns: 16384 20.9 and 22.1, 24000 31.0 and 25.2.
int lmh_block_rows(int n_cols, int64_t row_pitch_bytes, int n_rows, int num_cu) {
  if (n_cols >= kWideCols) return n_rows <= 64 * num_cu ? 64 : 128;
  return row_pitch_bytes % 8192 == 0 ? Geo<2, 1, 256>::kRowsWg : Geo<1, 1, 256>::kRowsWg;
}

// Part of the results: another block is another order of a logit's 32-bit sum (6e-6 apart, enough to
// swap tokens that nearly tie).  These are the blocks that the logits have had since the first
// release, when a block was also a task: 64 rows, but 128 for up to 32 hidden rows of a call where the
// row pitch asked for larger tasks, or where 64-row tasks would have left more candidates than a
// merge of that time could hold (20480).  So a row's logits are the same in every call of up to 32
// hidden rows with the same k, and in every call of more; between the two they may differ at
// d = 4096 and 8192 and, with V = 152064, at k above 8.
int lmh_order_rows(int n_cols, int64_t row_pitch_bytes, int n_rows, int topk) {
  if (n_cols >= kWideCols) return 64;
  const int64_t blocks64 = ((int64_t)n_rows + 63) / 64;
  return blocks64 * topk > 20480 || row_pitch_bytes % 8192 == 0 ? 128 : 64;
}

template <int MODE>
static hipError_t launch_rel_mode(const GemmKernelArgs& a, int num_cu, hipStream_t stream) {
  if (a.row_bytes == 512) return launch_gemm<MODE, 1, 1, 512>(a, num_cu, stream);
  const bool big = a.rows_per_block == Geo<2, 1, 256>::kRowsWg;
  if (a.n_cols <= 16)
    return big ? launch_gemm<MODE, 2, 1, 256>(a, num_cu, stream)
               : launch_gemm<MODE, 1, 1, 256>(a, num_cu, stream);
  return big ? launch_gemm<MODE, 2, 2, 256>(a, num_cu, stream)
             : launch_gemm<MODE, 1, 2, 256>(a, num_cu, stream);
}

// nv2 == nullptr: the caller prepared the rows' inverse norms, the pass takes dot products only
hipError_t launch_rel_gemm(const GemmKernelArgs& a, int num_cu, hipStream_t stream) {
  return a.nv2 != nullptr ? launch_rel_mode<MODE_REL>(a, num_cu, stream)
                          : launch_rel_mode<MODE_RELP>(a, num_cu, stream);
}

template <bool SORT>
static hipError_t launch_lmh(const GemmKernelArgs& a, int num_cu, hipStream_t stream) {
  constexpr int MODE = SORT ? MODE_LMHS : MODE_LMH;
  const bool rows64 = a.rows_per_block == 64;
  if (!rows64 && a.rows_per_block != 128) return hipErrorInvalidValue;
  if (a.n_cols >= kWideCols) {
    const int widest = a.half_cols > a.n_cols - a.half_cols ? a.half_cols : a.n_cols - a.half_cols;
    if (a.half_cols > a.n_cols || widest > 64) return hipErrorInvalidValue;
    if (widest <= 32)
      return rows64 ? launch_wide<1, 2, SORT>(a, stream) : launch_wide<2, 2, SORT>(a, stream);
    if (widest <= 48)
      return rows64 ? launch_wide<1, 3, SORT>(a, stream) : launch_wide<2, 3, SORT>(a, stream);
    return rows64 ? launch_wide<1, 4, SORT>(a, stream) : launch_wide<2, 4, SORT>(a, stream);
  }
  if (a.n_cols <= 16)
    return rows64 ? launch_gemm<MODE, 1, 1, 256>(a, num_cu, stream)
                  : launch_gemm<MODE, 2, 1, 256>(a, num_cu, stream);
  return rows64 ? launch_gemm<MODE, 1, 2, 256>(a, num_cu, stream)
                : launch_gemm<MODE, 2, 2, 256>(a, num_cu, stream);
}

hipError_t launch_lmh_gemm(const GemmKernelArgs& a, int num_cu, hipStream_t stream) {
  return a.topk > kSortTopk ? launch_lmh<true>(a, num_cu, stream) : launch_lmh<false>(a, num_cu, stream);
}

}  // namespace lvspec
