// Host side of the C ABI: argument checks, the workspace plans and the launch
// sequences of grkv_compress, the key step (grkv_compress_kv), ragged budgets
// and the budget rules, and the carrier diagnostics.  Everything is enqueued
// on the caller's stream; the only host-to-device transfer is the ragged
// call's copy of its per-unit table.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "grkv_internal.h"

namespace grkv {

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Split a key range of length len over at most `want` blocks of >= min_len keys,
// each a whole number of key tiles.
static void split_range(int64_t len, int64_t want, int64_t min_len, int* S, int* chunk) {
  int64_t s = want < 1 ? 1 : want;
  int64_t cap = ceil_div(len, min_len);
  if (s > cap) s = cap;
  if (s < 1) s = 1;
  int64_t ch = ceil_div(len, s);
  ch = ceil_div(ch, kKeyTile) * kKeyTile;
  if (ch < kKeyTile) ch = kKeyTile;
  *chunk = (int)ch;
  *S = (int)(len > 0 ? ceil_div(len, ch) : 1);
}

// The split count with which `units` such ranges finish first when `slots`
// blocks run at a time: rounds of blocks, each as long as its tiles plus
// kBlockTiles tiles' worth of prologue and epilogue.  Looked for from ranges of
// min_len keys, with `fine` half as many (at most `want` ranges), up to 8/5 of split_range's length
// for min_len, in steps of a tile or 1/32 of the length.  A last round that is
// nearly empty costs a whole one: 24 units of 32k tokens in 43 splits each
// (1032 blocks, 512 at a time) took pass B 107 us where 32 units (1024 blocks)
// took 123, and 8 units of 20011 tokens with 160 rows ran 40 splits each (320
// blocks, 256 at a time) as two rounds.  Ranges shorter than min_len pay where
// they still fit one round: 8 units of 8192 tokens in 32 splits 122 us a call, in
// 16 129 us; of 32k tokens in 128 (two rounds) 181 us, in 64 162 us.
static void split_rounds(int64_t len, int64_t want, int64_t min_len, bool fine, int64_t units,
                         int64_t slots, int* S, int* chunk) {
  constexpr uint32_t kBlockTiles = 10;
  split_range(len, want, min_len, S, chunk);
  const uint32_t usual = (uint32_t)*S, n = (uint32_t)len;
  if (fine) split_range(len, want, min_len / 2, S, chunk);
  auto cost = [&](uint32_t s, uint32_t c) {
    return (uint64_t)(((uint32_t)units * s + (uint32_t)slots - 1) / (uint32_t)slots) *
           (c / kKeyTile + kBlockTiles);
  };
  uint64_t best = cost(*S, *chunk);
  const uint32_t step = std::max<uint32_t>(1, (uint32_t)*chunk / (32 * kKeyTile)) * kKeyTile;
  for (uint32_t c = (uint32_t)*chunk + step;; c += step) {
    const uint32_t s = (n + c - 1) / c;
    if (s < 1 || 8 * s < 5 * usual) break;
    // (a change has to be worth 3%)
    if (100 * cost(s, c) < 97 * best) {
      best = cost(s, c);
      *S = (int)s;
      *chunk = (int)c;
    }
    if (s == 1) break;
  }
}

static void layout_plan(Plan* p, size_t slots, size_t splits2, size_t splits3, size_t tab);

int make_plan(const grkv_problem* prob, int64_t n, int32_t window, int32_t budget,
              int32_t pool_kernel, float lambda, const grkv_options* opt, Plan* p, bool ragged) {
  if (!prob) return GRKV_ERR_INVALID;
  if (prob->units < 1 || prob->group < 1) return GRKV_ERR_INVALID;
  if (prob->dtype != GRKV_BF16 && prob->dtype != GRKV_F32) return GRKV_ERR_INVALID;
  if (window < 1 || budget < window || (int64_t)budget > n || n > (int64_t(1) << 30))
    return GRKV_ERR_INVALID;
  if (pool_kernel < 1 || pool_kernel % 2 == 0) return GRKV_ERR_INVALID;
  if (!(lambda >= 0.f) || !isfinite(lambda)) return GRKV_ERR_INVALID;
  grkv_options o;
  grkv_default_options(&o);
  if (opt) o = *opt;
  if (o.n_sink < 0 || !(o.beta >= 0.f && o.beta <= 1.f)) return GRKV_ERR_INVALID;
  if (prob->head_dim != 64 && prob->head_dim != 128) return GRKV_ERR_UNSUPPORTED;
  int64_t m = (int64_t)prob->group * window;
  if (m > 256) return GRKV_ERR_UNSUPPORTED;

  memset(p, 0, sizeof(*p));
  p->U = prob->units;
  p->G = prob->group;
  p->w = window;
  p->m = (int)m;
  // one wave per 32 rows, a power of two of them (1, 2, 4 or 8)
  int waves = 1;
  while (waves * kRowsPerWave < m) waves *= 2;
  p->waves = waves;
  p->mp = waves * kRowsPerWave;
  p->d = prob->head_dim;
  p->dtype = prob->dtype;
  p->n = n;
  p->c = budget;
  p->s_sel = budget - window;
  p->prefix = (int)(n - window);
  p->k_pool = pool_kernel;
  int64_t top = (int64_t)floor((double)o.beta * (double)budget);
  p->n_top_fixed = (int)(top < p->s_sel ? top : p->s_sel);
  p->lam = lambda;
  p->opt = o;

  // Target about 1024 blocks per launch (four per CU) for the full-cache
  // streaming passes, and about one block per CU for the bf16 retained pass
  // (which holds one block per CU): fewer splits mean fewer partials for the
  // solve to combine.
  int64_t target = 1024, target_ret = 256;
  if (const char* e = getenv("GRKV_TARGET_BLOCKS")) target = atoll(e);       // tuning experiments
  if (const char* e = getenv("GRKV_TARGET_RET_BLOCKS")) target_ret = atoll(e);
  const int64_t want = ceil_div(target, p->U);
  p->fast_merge = merge_fast_supported(*p);
  // calls with few units split the solve's right-hand-side columns over up
  // to d / 16 blocks per unit (one per compute unit at most)
  p->csplit = 1;
  if ((p->fast_merge || solve_big_supported(*p)) && (size_t)p->U * (p->d / 16) <= 256)
    p->csplit = p->d / 16;
  // fine: the finer splits of small calls; in fp32 the blocks that they make (0
  // and -1: the coarse splits; -2: 512 blocks, fewer than the coarse ones with
  // many units)
  auto splits = [&](int fine) {
    if (p->dtype == GRKV_F32) {
      // The fp32 kernels hold one to eight waves per block and little else, and
      // their key tiles are a serial chain, so a call with few units is split
      // down to two tiles per block, to `fine` blocks over the units at most
      // (2 units of 1024 tokens, 32 rows: with the blocked solve 287 -> 95 us),
      // and never into fewer splits than the coarse ones, whose blocks keep the
      // compute units busy in calls with many units (131 units of 10976 tokens,
      // 32 rows: 3 splits 2.40 ms, 8 splits 1.98)
      auto finest = [&](int64_t len, int64_t want_c, int64_t min_c, int* S, int* chunk) {
        split_range(len, want_c, min_c, S, chunk);
        int Sf, ch;
        split_range(len, std::max(fine, 1) / p->U, 64, &Sf, &ch);
        if (Sf > *S) {
          *S = Sf;
          *chunk = ch;
        }
      };
      finest(n, fine < -1 ? 512 / p->U : want, fine < -1 ? 64 : 512, &p->S1, &p->chunk1);
      finest(budget, fine < -1 ? 512 / p->U : fine < 0 ? ceil_div(256, p->U) : want,
             fine < -1 ? 64 : fine < 0 ? 256 : 128, &p->S2, &p->chunk2);
      if (p->chunk2 > 8192) split_range(budget, ceil_div(budget, 8192), 128, &p->S2, &p->chunk2);
      if (fine < -1 && solve_supported(*p)) {
        p->S3 = p->S2;
        p->chunk3 = p->chunk2;
      } else {
        finest(budget, ceil_div(256, p->U), 256, &p->S3, &p->chunk3);
      }
      layout_plan(p, (size_t)p->U * budget, (size_t)p->U * p->S2, (size_t)p->U * p->S3, 0);
      return;
    }
    // blocks that run at a time: pass B holds two blocks of up to four waves per
    // compute unit or one of eight, the retained pass one
    // (shorter ranges only from where the partials are combined by a launch of
    // their own: 50 units of 3280 tokens in 10 splits 167 us a call, in 7 158 us;
    // 64 of 2500 175 / 171 us)
    split_rounds(n, want, 512, fine, p->U, p->waves == 8 ? 256 : 512, &p->S1, &p->chunk1);
    if (p->S1 < kPrecombineSplits)
      split_rounds(n, want, 512, false, p->U, p->waves == 8 ? 256 : 512, &p->S1, &p->chunk1);
    if (p->fast_merge) {
      // (from 16 splits on, more of them cost the combine more than the pass
      // gains: 2048 retained keys in 32 splits 164 us a call, in 16 162 us; 512
      // in 8 124 us, in 4 129 us)
      // (here too: 50 units with 434 retained keys in 5 splits 169 us, in 4 167 us;
      // a ragged call has no such launch, its solve sums the partials: 8 units of
      // 1024 retained keys on average in 16 splits 150 us, in 8 141; 23 of 655 in 10
      // 153, in 6 144)
      const int64_t want_ret = std::min(ceil_div(target_ret, p->U),
                                        std::max<int64_t>(16, ceil_div(budget, 128)));
      split_rounds(budget, want_ret, 128, fine && !ragged, p->U, 256, &p->S2, &p->chunk2);
      if (p->S2 < kPrecombineRetSplits)
        split_rounds(budget, want_ret, 128, false, p->U, 256, &p->S2, &p->chunk2);
      if (p->chunk2 > 4096) split_range(budget, ceil_div(budget, 4096), 128, &p->S2, &p->chunk2);
      p->S3 = p->S2;
      p->chunk3 = p->chunk2;
    } else {
      split_range(budget, want, 128, &p->S2, &p->chunk2);
      if (p->chunk2 > 8192) split_range(budget, ceil_div(budget, 8192), 128, &p->S2, &p->chunk2);
      split_range(budget, ceil_div(256, p->U), fine ? 128 : 256, &p->S3, &p->chunk3);
    }
    layout_plan(p, (size_t)p->U * budget, (size_t)p->U * p->S2, (size_t)p->U * p->S3, 0);
  };
  // The finer splits, in fp32 the finest, that keep the call inside the fixed
  // scratch of the non-allocating entry point; a call that no splits keep inside
  // it takes the finest.  fp32: 512 blocks of up to four waves, 256 of eight (8
  // units of 8192 tokens, 128 rows, 2048 retained: coarse 363 us, 256 blocks 267,
  // 512 265; 124 units of 580 tokens, 256 rows: coarse 525 us, 256 blocks 523, 512
  // 618; 16 units of 4096 544, 392, 429)
  const int finest = p->dtype == GRKV_BF16 ? 1 : p->waves == 8 ? 256 : 512;
  const int coarsest = p->dtype == GRKV_BF16 ? 0 : -2;
  for (int fine = finest;; fine = fine > 0 ? fine * 3 / 4 : fine - 1) {
    splits(fine);
    if (p->total <= GRKV_NOALLOC_SCRATCH_BYTES) break;
    if (fine == coarsest) {
      splits(finest);
      break;
    }
  }
  return GRKV_OK;
}

// Workspace offsets: `slots` retained slots and `splits2` / `splits3`
// retained-pass and Gram partial blocks over all units, then `tab` bytes of
// ragged tables.
static void layout_plan(Plan* p, size_t slots, size_t splits2, size_t splits3, size_t tab) {
  const size_t U = p->U, mp = p->mp, d = p->d, P = p->prefix;
  const size_t esz = p->dtype == GRKV_BF16 ? 2 : 4;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o2 = off; off = align256(off + bytes); return o2; };
  p->pmax1 = take(U * p->S1 * mp * sizeof(float));
  p->psum1 = take(U * p->S1 * mp * sizeof(double));
  p->lse1 = take(U * mp * sizeof(double));
  p->lse1_log2 = take(U * mp * sizeof(float));
  p->ypart = take(U * p->S1 * mp * d * sizeof(float));
  p->y = take(U * mp * d * sizeof(float));
  p->colsum = take(U * (P > 0 ? P : 1) * sizeof(float));
  p->pooled = take(U * (P > 0 ? P : 1) * sizeof(float));
  p->fixed = take(slots);
  // the compact V0 copy serves the generic retained passes only; the fast
  // path reads V0 rows through idx
  const bool fast_path = stream_supported(*p) && merge_fast_supported(*p);
  p->v0c = take(fast_path ? 0 : slots * d * esz);
  p->pmax2 = take(splits2 * mp * sizeof(float));
  p->psum2 = take(splits2 * mp * sizeof(double));
  p->lse2 = take(U * mp * sizeof(double));
  p->lse2_log2 = take(U * mp * sizeof(float));
  p->xvpart = take(splits2 * mp * d * sizeof(float));
  p->x = take(p->fast_merge ? 0 : mp * slots * sizeof(float));   // generic path only
  p->resid = take(U * mp * d * sizeof(float));
  p->npart = take(splits3 * mp * mp * sizeof(float));
  p->mpart = take(fast_path ? splits2 * mp * sizeof(float) : 0);
  const size_t comb = fast_path && p->S2 >= kPrecombineRetSplits ? U : 0;
  p->xvcomb = take(comb * mp * d * sizeof(float));
  p->ncomb = take(comb * mp * mp * sizeof(float));
  p->mcomb = take(comb * mp * sizeof(float));
  p->gram = take(U * mp * mp * sizeof(float));
  p->z = take(U * d * mp * sizeof(float));
  p->zhi = take(U * d * mp * 2);
  p->zlo = take(U * d * mp * 2);
  p->stats_ws = take(U * 4 * sizeof(float));
  p->zpart = take(U * kZParts * sizeof(double));
  p->rag_tab = take(tab);
  p->total = off;
}

// Workspace of the key step, after the compress workspace.  A key-pass block
// holds all m rows of a unit and a split of its retained keys.
void make_key_plan(const Plan& p, int steps, KeyPlan* kp) {
  // While every unit is iterating: about one block per compute unit, the count
  // rounded down where a block fills one (128 rows: 48 units of 2000 keys in 5
  // splits 1.95 ms a call, in 6 2.19) and up where two fit: 32 rows; 64 with more
  // than 64 units (155 units of 3000 keys in one split 5.6 ms, in two 4.0), and
  // long units in fewer (52 of 5000 keys in 4 splits 2.40 ms, in 5 2.17; of 3000
  // 1.74 / 1.70; 60 of 2500 1.62 / 1.64, 40 of 2000 1.40 / 1.43).
  // Past 128 units of 128 rows one split leaves compute units idle, and two take
  // a second round of 2 U - 256 blocks, which is gone once U - 128 units have
  // converged: long units take two, from a length that rises with the units (one
  // split / two: 130 units of 1000 keys 3.27 / 3.15 ms; 150 of 1500 4.06 / 4.09, of
  // 1900 4.22 / 4.11; 170 of 1900 4.09 / 4.16, of 2100 3.96 / 3.88; 210 of 2100 4.63
  // / 4.64, of 3000 5.73 / 5.53; 250 of 1900 5.67 / 5.75, of 3000 6.22 / 6.00).
  // Later: about 2048 blocks, when a unit's iteration spanning several compute
  // units keeps it short once only a few units are still converging
  const bool up = p.mp == 32 || (p.mp == 64 && (p.U > 64 || p.c >= 2816)) ||
                  (p.mp == 128 && p.U > 128 && p.c >= std::min(2432, 1024 + 24 * (p.U - 130)));
  split_range(p.c, up ? ceil_div(256, p.U) : 256 / p.U, 64, &kp->S_full, &kp->chunk_full);
  split_range(p.c, ceil_div(2048, p.U), 64, &kp->S4, &kp->chunk4);
  // the ring passes' later iterations: about 1024 blocks (fewer partials for
  // the separate CG update to combine, measured faster than 2048), at most 16
  // per unit unless the first iterations have more (their blocks already fill
  // the compute units)
  const int64_t tail = std::min<int64_t>(ceil_div(1024, p.U), 16);
  split_range(p.c, std::max<int64_t>(tail, kp->S_full), 64, &kp->S4r, &kp->chunk4r);
  const int Smax = kp->S4 > kp->S_full ? kp->S4 : kp->S_full;
  const size_t U = p.U, mp = p.mp, d = p.d;
  size_t off = p.total;
  auto take = [&](size_t bytes) { size_t o2 = off; off = align256(off + bytes); return o2; };
  kp->Fm = take(U * mp * d * sizeof(float));
  kp->alpha = take(U * mp * d * sizeof(float));
  kp->r = take(U * mp * d * sizeof(float));
  kp->p = take(U * mp * d * sizeof(float));
  kp->sdot = take(U * mp * sizeof(float));
  kp->W = take(U * mp * mp * sizeof(float));
  kp->opart = take(U * Smax * mp * d * sizeof(float));
  kp->hpart = take(U * Smax * mp * sizeof(float));
  kp->cg = take(U * 4 * sizeof(double));
  kp->cgpart = take(U * kCgBlocks * sizeof(double));
  kp->cgcount = take(U * sizeof(int));
  const size_t later = steps > 1 ? 1 : 0;
  kp->q32 = take(later * U * p.m * d * sizeof(float));
  kp->v0f = take(later * U * p.c * d * sizeof(float));
  kp->v0c = take(later * U * p.c * d * sizeof(uint16_t));
  kp->x = take(later * U * mp * p.c * sizeof(float));
  kp->kcur = take(later * U * p.c * d * sizeof(float));
  kp->ring = key_ring_supported(p);
  kp->vsplit = take(kp->ring ? 2 * U * p.c * d * sizeof(uint16_t) : 0);
  kp->xs = take(kp->ring ? key_x_bytes(p) : 0);
  kp->total = off;
}

}  // namespace grkv

using namespace grkv;

extern "C" {

void grkv_default_options(grkv_options* opt) {
  if (!opt) return;
  opt->n_sink = 4;
  opt->beta = 0.10f;
  opt->fix_window = 1;
  opt->causal_window = 1;
}

const char* grkv_status_string(int status) {
  switch (status) {
    case GRKV_OK: return "ok";
    case GRKV_ERR_INVALID: return "invalid argument";
    case GRKV_ERR_WORKSPACE: return "workspace too small";
    case GRKV_ERR_UNSUPPORTED: return "unsupported shape (head_dim must be 64 or 128, group*window <= 256)";
    case GRKV_ERR_HIP: return "HIP launch failed";
  }
  return "unknown status";
}

size_t grkv_workspace_bytes(const grkv_problem* prob, int64_t n, int32_t window, int32_t budget) {
  Plan p;
  if (make_plan(prob, n, window, budget, 1, 0.f, nullptr, &p) != GRKV_OK) return 0;
  return p.total;
}

int grkv_workspace_layout(const grkv_problem* prob, int64_t n, int32_t window, int32_t budget,
                          grkv_layout* layout) {
  if (!layout) return GRKV_ERR_INVALID;
  Plan p;
  int st = make_plan(prob, n, window, budget, 1, 0.f, nullptr, &p);
  if (st != GRKV_OK) return st;
  layout->lse = p.lse1;
  layout->y = p.y;
  layout->score = p.colsum;
  layout->pooled = p.pooled;
  layout->fixed = p.fixed;
  layout->resid = p.resid;
  layout->gram = p.gram;
  layout->z = p.z;
  layout->total = p.total;
  return GRKV_OK;
}

}  // extern "C"

namespace {

// Pointer checks shared by the entry points.
int check_pointers(const void* q_obs, const void* K, const void* V, const grkv_problem* prob,
                   const grkv_outputs* out) {
  if (!q_obs || !K || !V || !prob || !out) return GRKV_ERR_INVALID;
  if (!out->idx || !out->k_out || !out->v_out || !out->workspace) return GRKV_ERR_INVALID;
  if (((uintptr_t)out->workspace & 255) != 0) return GRKV_ERR_INVALID;
  return GRKV_OK;
}

// The solve of up to 128 rows outside the fast path: Y combined already, X V0
// and Gram partials of the normalised X (no masses to divide by).  Several
// splits, or different counts of the two, are summed first by one launch over
// all units (generic_sums) into resid and gram, which the solve then reads
// element by element before it writes them.
bool generic_presum(const Plan& p) { return p.S2 > 2 || p.S3 != p.S2; }

hipError_t generic_sums(const Plan& p, char* ws, hipStream_t s) {
  if (!generic_presum(p)) return hipSuccess;
  auto F = [&](size_t o) { return (float*)(ws + o); };
  const float* part[kCombineSegs] = {F(p.xvpart), F(p.npart), nullptr, nullptr};
  float* const outs[kCombineSegs] = {F(p.resid), F(p.gram), nullptr, nullptr};
  const size_t per[kCombineSegs] = {(size_t)p.mp * p.d, (size_t)p.mp * p.mp, 0, 0};
  const int S[kCombineSegs] = {p.S2, p.S3, 0, 0};
  return launch_combine_parts(p.U, S, part, outs, per, s);
}

hipError_t generic_solve(const Plan& p, char* ws, float* y, float* stats, hipStream_t s) {
  auto F = [&](size_t o) { return (float*)(ws + o); };
  Plan q = p;
  q.csplit = 1;
  q.rag = nullptr;
  const bool pre = generic_presum(p);
  return launch_solve(q, y, 1, pre ? 1 : p.S2, pre ? F(p.resid) : F(p.xvpart),
                      pre ? F(p.gram) : F(p.npart), nullptr, nullptr, 0.f, nullptr, y, F(p.resid),
                      F(p.gram), F(p.z), (uint16_t*)(ws + p.zhi), (uint16_t*)(ws + p.zlo),
                      F(p.stats_ws), stats, (double*)(ws + p.zpart), nullptr, nullptr, nullptr,
                      nullptr, nullptr, s);
}

// The launch sequence of one call (arguments already checked).
int run_compress(const Plan& p, const void* q_obs, const void* K, const void* V, int64_t n,
                 hipStream_t s, const grkv_outputs* out, const float* ext_scores = nullptr) {
  char* ws = (char*)out->workspace;
  auto F = [&](size_t o) { return (float*)(ws + o); };
  auto Dd = [&](size_t o) { return (double*)(ws + o); };

#define GRKV_TRY(x) do { if ((x) != hipSuccess) return GRKV_ERR_HIP; } while (0)
  void** ev = out->stage_events;
  auto mark = [&](int stage, int end) -> hipError_t {
    if (!ev || !ev[2 * stage] || !ev[2 * stage + 1]) return hipSuccess;
    return hipEventRecord((hipEvent_t)ev[2 * stage + end], s);
  };
#define GRKV_STAGE(id, call) do { GRKV_TRY(mark(id, 0)); GRKV_TRY(call); GRKV_TRY(mark(id, 1)); } while (0)
  // 1. window attention over the full cache: LSE, then Y and the SnapKV scores
  AttnPass full = {};
  full.q = q_obs; full.k = K; full.v = V; full.kpos = nullptr; full.nk = (int)n;
  full.S = p.S1; full.chunk = p.chunk1;
  full.pmax = F(p.pmax1); full.psum = Dd(p.psum1);
  full.lse = Dd(p.lse1); full.lse_log2 = F(p.lse1_log2);
  // (with caller-supplied selection scores the window's column sums are not formed)
  full.ypart = F(p.ypart); full.colsum = p.prefix > 0 && !ext_scores ? F(p.colsum) : nullptr;
  full.prefix = p.prefix; full.xout = nullptr; full.split_p = true;
  const bool fast = stream_supported(p);
  auto pass_a = [&](const AttnPass& a) { return fast ? launch_stream(p, a, 0, s) : launch_lse_pass(p, a, s); };
  auto pass_b = [&](const AttnPass& a) { return fast ? launch_stream(p, a, 1, s) : launch_prob_pass(p, a, s); };
  GRKV_STAGE(GRKV_STAGE_FULL_LSE, pass_a(full));
  // (the bf16 streaming pass B combines the split partials itself, unless a
  // unit has so many splits that a kernel of its own does it faster: with 256
  // rows too, where every block's own loop over 32 to 40 splits took most of
  // pass B; with this and the split counts one layer of 8 units, 20011 tokens
  // and 160 rows went from 458 to 340 us, 32 units of 128k tokens from 1841 to
  // 1639 us)
  const bool pre = fast && p.fast_merge && p.S1 >= kPrecombineSplits;
  full.lse_ready = fast && p.S1 >= kPrecombineSplits;
  if (!fast || full.lse_ready)
    GRKV_STAGE(GRKV_STAGE_FULL_LSE_COMBINE,
               launch_lse_combine(p, full.pmax, full.psum, p.S1, Dd(p.lse1), F(p.lse1_log2), s));
  GRKV_STAGE(GRKV_STAGE_FULL_PROB, pass_b(full));
  // (the fast value step combines the Y partials inside its solve, again
  // unless there are many)
  // (with many retained splits too, the Y partials join the retained
  // partials' combine below: one launch for both)
  const bool pre2 = fast && p.fast_merge && !p.rag && p.S2 >= kPrecombineRetSplits;
  if (!p.fast_merge || (pre && !pre2))
    GRKV_STAGE(GRKV_STAGE_FULL_Y, launch_combine_rows(p, F(p.ypart), p.S1, nullptr, F(p.y), s));
  // 2. pooled top-k retention and the fixed set; gather K0, V0
  uint8_t* fixed = (uint8_t*)(ws + p.fixed);
  GRKV_STAGE(GRKV_STAGE_SELECT, launch_select(p, ext_scores ? ext_scores : F(p.colsum), F(p.pooled),
                                              out->idx, fixed, s));
  const bool fast_merge = p.fast_merge;
  // fast path: the retained pass A reads the K rows through idx and copies
  // them to k_out; V0 rows are read through idx where needed
  const bool direct = fast && fast_merge;
  if (!direct)
    GRKV_STAGE(GRKV_STAGE_GATHER, launch_gather(p, K, V, out->idx, out->k_out, ws + p.v0c,
                                                nullptr, s));
  // 3. window attention over the retained cache: X and X V0, then R = Y - X V0
  AttnPass ret = {};
  ret.q = q_obs; ret.k = out->k_out; ret.v = ws + p.v0c; ret.kpos = out->idx; ret.nk = p.c;
  ret.S = p.S2; ret.chunk = p.chunk2;
  ret.pmax = F(p.pmax2); ret.psum = Dd(p.psum2);
  ret.lse = Dd(p.lse2); ret.lse_log2 = F(p.lse2_log2);
  ret.ypart = F(p.xvpart); ret.colsum = nullptr; ret.prefix = 0;
  ret.xout = fast_merge ? nullptr : F(p.x);
  ret.split_p = true;
  ret.fixed = fixed; ret.npart = F(p.npart);
  if (direct) {
    // one pass over the retained set: K and V rows through idx (K tiles also
    // copied to k_out), P against the full-cache LSE; the solve normalises by
    // the retained row sums, so no retained log-sum-exp pass is needed
    ret.k = K; ret.gather_k = true; ret.kcopy = out->k_out;
    ret.v = V; ret.gather_v = true; ret.src_rows = n;
    ret.lse_log2 = F(p.lse1_log2); ret.lse_bias = kRetainedBias; ret.mpart = F(p.mpart);
  } else {
    GRKV_STAGE(GRKV_STAGE_RET_LSE, pass_a(ret));
    GRKV_STAGE(GRKV_STAGE_RET_LSE_COMBINE,
               launch_lse_combine(p, ret.pmax, ret.psum, p.S2, Dd(p.lse2), F(p.lse2_log2), s));
  }
  // the generic value step needs X itself, which only the generic pass writes
  GRKV_STAGE(GRKV_STAGE_RET_PROB,
             fast_merge ? launch_stream(p, ret, 2, s) : launch_prob_pass(p, ret, s));
  if (!fast_merge && solve_big_supported(p))
    GRKV_STAGE(GRKV_STAGE_RESID,
               launch_combine_rows(p, F(p.xvpart), p.S2, F(p.y), F(p.resid), s));
  // 4. value step: N, Cholesky solve for Z, V* = V0 + X_G^T Z
  if (!fast_merge) GRKV_STAGE(GRKV_STAGE_GRAM, launch_gram(p, F(p.x), fixed, F(p.npart), s));
  if (fast_merge) {
    // many retained splits per unit (small uniform calls): their partials are
    // summed by one launch over all units first
    if (pre2) {
      const float* part[kCombineSegs] = {F(p.xvpart), F(p.npart), F(p.mpart), F(p.ypart)};
      float* const outs[kCombineSegs] = {F(p.xvcomb), F(p.ncomb), F(p.mcomb), F(p.y)};
      const size_t per[kCombineSegs] = {(size_t)p.mp * p.d, (size_t)p.mp * p.mp, (size_t)p.mp,
                                        pre ? (size_t)p.mp * p.d : 0};
      const int S[kCombineSegs] = {p.S2, p.S2, p.S2, p.S1};
      GRKV_STAGE(GRKV_STAGE_RESID, launch_combine_parts(p.U, S, part, outs, per, s));
    }
    GRKV_TRY(mark(GRKV_STAGE_SOLVE, 0));
    GRKV_TRY(launch_solve(p, pre ? F(p.y) : F(p.ypart), pre ? 1 : p.S1, pre2 ? 1 : p.S2,
                          pre2 ? F(p.xvcomb) : F(p.xvpart), pre2 ? F(p.ncomb) : F(p.npart),
                          direct ? (pre2 ? F(p.mcomb) : F(p.mpart)) : nullptr, F(p.lse1_log2),
                          kRetainedBias, F(p.lse2_log2), F(p.y), F(p.resid), F(p.gram), F(p.z),
                          (uint16_t*)(ws + p.zhi), (uint16_t*)(ws + p.zlo), F(p.stats_ws),
                          out->stats, Dd(p.zpart), q_obs, out->k_out, V, out->idx, fixed, s));
    GRKV_TRY(mark(GRKV_STAGE_SOLVE, 1));
    GRKV_STAGE(GRKV_STAGE_UPDATE,
               launch_update(p, q_obs, out->k_out, F(p.lse2_log2), fixed,
                             (const uint16_t*)(ws + p.zhi),
                             (const uint16_t*)(ws + p.zlo), F(p.stats_ws),
                             V, out->idx, out->v_out, Dd(p.zpart), out->stats, s));
  } else {
    // 256 stacked rows: blocked factorisation, block-packed in LDS; up to 128
    // the solve of the fast path (on combined Y, plain X V0 and Gram partials)
    if (solve_big_supported(p)) {
      GRKV_STAGE(GRKV_STAGE_SOLVE,
                 launch_solve_big(p, F(p.npart), p.S3, F(p.y), F(p.resid), F(p.gram), F(p.z),
                                  F(p.stats_ws), out->stats, Dd(p.zpart), s));
    } else {
      GRKV_STAGE(GRKV_STAGE_RESID, generic_sums(p, ws, s));
      GRKV_STAGE(GRKV_STAGE_SOLVE, generic_solve(p, ws, F(p.y), out->stats, s));
    }
    GRKV_STAGE(GRKV_STAGE_UPDATE,
               launch_update_gen(p, F(p.x), fixed, F(p.z), F(p.stats_ws), ws + p.v0c,
                                 out->v_out, Dd(p.zpart), out->stats, s));
  }
#undef GRKV_STAGE
#undef GRKV_TRY
  return GRKV_OK;
}

}  // namespace

extern "C" {

int grkv_compress(const void* q_obs, const void* K, const void* V, int64_t n, int32_t window,
                  int32_t budget, int32_t pool_kernel, float lambda, void* stream,
                  const grkv_problem* prob, const grkv_options* opt, const grkv_outputs* out) {
  int st = check_pointers(q_obs, K, V, prob, out);
  if (st != GRKV_OK) return st;
  Plan p;
  st = make_plan(prob, n, window, budget, pool_kernel, lambda, opt, &p);
  if (st != GRKV_OK) return st;
  if (out->workspace_bytes < p.total) return GRKV_ERR_WORKSPACE;
  return run_compress(p, q_obs, K, V, n, (hipStream_t)stream, out);
}

int grkv_compress_scored(const void* q_obs, const void* K, const void* V, int64_t n,
                         int32_t window, int32_t budget, int32_t pool_kernel, float lambda,
                         void* stream, const grkv_problem* prob, const grkv_options* opt,
                         const float* scores, const grkv_outputs* out) {
  int st = check_pointers(q_obs, K, V, prob, out);
  if (st != GRKV_OK) return st;
  if (!scores && n > window) return GRKV_ERR_INVALID;
  Plan p;
  st = make_plan(prob, n, window, budget, pool_kernel, lambda, opt, &p);
  if (st != GRKV_OK) return st;
  if (out->workspace_bytes < p.total) return GRKV_ERR_WORKSPACE;
  return run_compress(p, q_obs, K, V, n, (hipStream_t)stream, out, scores);
}

size_t grkv_h2o_workspace_bytes(const grkv_problem* prob, int64_t n) {
  if (!prob || prob->units < 1 || prob->group < 1 || n < 1 || n > (int64_t(1) << 30)) return 0;
  if (!h2o_supported(prob->dtype, prob->head_dim, prob->group)) return 0;
  return (size_t)prob->units * prob->group * (size_t)n * sizeof(float);
}

int grkv_h2o_scores(const void* q_all, const void* K, int64_t n, int32_t window, void* stream,
                    const grkv_problem* prob, float* scores, void* workspace,
                    size_t workspace_bytes) {
  if (!q_all || !K || !prob || !workspace || (!scores && n > window)) return GRKV_ERR_INVALID;
  if (prob->units < 1 || prob->group < 1) return GRKV_ERR_INVALID;
  if (prob->dtype != GRKV_BF16 && prob->dtype != GRKV_F32) return GRKV_ERR_INVALID;
  if (window < 1 || (int64_t)window > n || n > (int64_t(1) << 30)) return GRKV_ERR_INVALID;
  if (((uintptr_t)workspace & 255) != 0) return GRKV_ERR_INVALID;
  if (!h2o_supported(prob->dtype, prob->head_dim, prob->group)) return GRKV_ERR_UNSUPPORTED;
  if (workspace_bytes < grkv_h2o_workspace_bytes(prob, n)) return GRKV_ERR_WORKSPACE;
  if (launch_h2o(q_all, K, prob->units, prob->group, prob->head_dim, n, (int)(n - window),
                 (float*)workspace, scores, (hipStream_t)stream) != hipSuccess)
    return GRKV_ERR_HIP;
  return GRKV_OK;
}

void grkv_default_key_options(grkv_key_options* kopt, float lambda) {
  if (!kopt) return;
  kopt->lambda_k = lambda;
  kopt->max_iter = 64;
  kopt->tol = 1e-5f;
  kopt->steps = 1;
}

size_t grkv_workspace_bytes_kv(const grkv_problem* prob, int64_t n, int32_t window,
                               int32_t budget, int32_t steps) {
  Plan p;
  if (steps < 1 || steps > 16) return 0;
  if (make_plan(prob, n, window, budget, 1, 0.f, nullptr, &p) != GRKV_OK) return 0;
  if (!key_supported(p)) return 0;
  KeyPlan kp;
  make_key_plan(p, steps, &kp);
  return kp.total;
}

int grkv_compress_kv(const void* q_obs, const void* K, const void* V, int64_t n, int32_t window,
                     int32_t budget, int32_t pool_kernel, float lambda, void* stream,
                     const grkv_problem* prob, const grkv_options* opt, const grkv_outputs* out,
                     const grkv_key_options* kopt, float* k_star, float* cg_info) {
  int st = check_pointers(q_obs, K, V, prob, out);
  if (st != GRKV_OK) return st;
  if (!k_star) return GRKV_ERR_INVALID;
  grkv_key_options ko;
  grkv_default_key_options(&ko, lambda);
  if (kopt) ko = *kopt;
  if (!(ko.lambda_k >= 0.f) || !isfinite(ko.lambda_k)) return GRKV_ERR_INVALID;
  if (ko.max_iter < 0 || ko.max_iter > 4096 || !(ko.tol >= 0.f) || !isfinite(ko.tol))
    return GRKV_ERR_INVALID;
  if (ko.steps < 1 || ko.steps > 16) return GRKV_ERR_INVALID;
  Plan p;
  st = make_plan(prob, n, window, budget, pool_kernel, lambda, opt, &p);
  if (st != GRKV_OK) return st;
  if (!key_supported(p)) return GRKV_ERR_UNSUPPORTED;
  KeyPlan kp;
  make_key_plan(p, ko.steps, &kp);
  if (out->workspace_bytes < kp.total) return GRKV_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  st = run_compress(p, q_obs, K, V, n, s, out);
  if (st != GRKV_OK) return st;

  char* ws = (char*)out->workspace;
  auto F = [&](size_t o) { return (float*)(ws + o); };
  KeyArgs a = {};
  a.q = (const uint16_t*)q_obs;
  a.k0 = (const uint16_t*)out->k_out;
  a.vs = out->v_out;
  if (kp.ring) {
    a.vh = (uint16_t*)(ws + kp.vsplit);
    a.vl = a.vh + (size_t)p.U * p.c * p.d;
    a.xs = F(kp.xs);
  }
  a.lse2 = F(p.lse2_log2);
  a.fixed = (const uint8_t*)(ws + p.fixed);
  a.idx = out->idx;
  a.y = F(p.y);
  a.zt = F(p.z);
  a.stats_ws = F(p.stats_ws);
  a.Fm = F(kp.Fm);
  a.alpha = F(kp.alpha);
  a.r = F(kp.r);
  a.p = F(kp.p);
  a.sdot = F(kp.sdot);
  a.W = F(kp.W);
  a.opart = F(kp.opart);
  a.hpart = F(kp.hpart);
  a.cg = (double*)(ws + kp.cg);
  a.cgpart = (double*)(ws + kp.cgpart);
  a.cgcount = (int*)(ws + kp.cgcount);
  a.kstar = k_star;
  a.cg_info = cg_info;
  a.lam_k = ko.lambda_k;
  a.tol = ko.tol;
  a.max_iter = ko.max_iter;
  void** ev = out->stage_events;
  const bool timed = ev && ev[2 * GRKV_STAGE_KEY] && ev[2 * GRKV_STAGE_KEY + 1];
  if (timed && hipEventRecord((hipEvent_t)ev[2 * GRKV_STAGE_KEY], s) != hipSuccess)
    return GRKV_ERR_HIP;
  if (launch_key(p, kp, a, s) != hipSuccess) return GRKV_ERR_HIP;

  // Later alternating steps (Algorithm 1, S > 1): the value step at the
  // current fp32 keys K^(t) (still anchored at V0) on the generic fp32
  // kernels, then the key step linearized at K^(t).
  if (ko.steps > 1) {
    Plan p32 = p;
    p32.dtype = GRKV_F32;
    float* q32 = F(kp.q32);
    float* v0f = F(kp.v0f);
    float* kcur = F(kp.kcur);
    float* x = F(kp.x);
    const size_t vbytes = (size_t)p.U * p.c * p.d * sizeof(float);
    if (launch_to_f32((const uint16_t*)q_obs, q32, (size_t)p.U * p.m * p.d, s) != hipSuccess)
      return GRKV_ERR_HIP;
    if (launch_gather(p, K, V, out->idx, out->k_out, ws + kp.v0c, v0f, s) != hipSuccess)
      return GRKV_ERR_HIP;
    a.kcur = kcur;
    for (int t = 1; t < ko.steps; ++t) {
      if (hipMemcpyAsync(kcur, k_star, vbytes, hipMemcpyDeviceToDevice, s) != hipSuccess)
        return GRKV_ERR_HIP;
      AttnPass r = {};
      r.q = q32; r.k = kcur; r.v = v0f; r.kpos = out->idx; r.nk = p.c;
      r.S = p.S2; r.chunk = p.chunk2;
      r.pmax = F(p.pmax2); r.psum = (double*)(ws + p.psum2);
      r.lse = (double*)(ws + p.lse2); r.lse_log2 = F(p.lse2_log2);
      r.ypart = F(p.xvpart); r.colsum = nullptr; r.prefix = 0; r.xout = x; r.split_p = true;
      uint8_t* fixed = (uint8_t*)(ws + p.fixed);
      if (launch_lse_pass(p32, r, s) != hipSuccess ||
          launch_lse_combine(p32, r.pmax, r.psum, p.S2, (double*)(ws + p.lse2), F(p.lse2_log2),
                             s) != hipSuccess ||
          launch_prob_pass(p32, r, s) != hipSuccess ||
          launch_gram(p32, x, fixed, F(p.npart), s) != hipSuccess ||
          generic_sums(p32, ws, s) != hipSuccess ||
          generic_solve(p32, ws, F(p.y), out->stats, s) != hipSuccess ||
          hipMemcpyAsync(out->v_out, v0f, vbytes, hipMemcpyDeviceToDevice, s) != hipSuccess ||
          launch_update_add(p32, x, fixed, F(p.z), F(p.stats_ws), out->v_out, s) != hipSuccess)
        return GRKV_ERR_HIP;
      if (launch_key(p, kp, a, s) != hipSuccess) return GRKV_ERR_HIP;
    }
  }
  if (timed && hipEventRecord((hipEvent_t)ev[2 * GRKV_STAGE_KEY + 1], s) != hipSuccess)
    return GRKV_ERR_HIP;
  return GRKV_OK;
}

int grkv_pyramid_budgets(int32_t layers, int32_t kv_heads, int32_t mean_budget, int32_t window,
                         int64_t n, float ratio, int32_t* budgets) {
  if (layers < 1 || kv_heads < 1 || !budgets || window < 1 || mean_budget < window ||
      (int64_t)mean_budget > n || !(ratio >= 0.f && ratio <= 1.f))
    return GRKV_ERR_INVALID;
  const int L = layers;
  int64_t* per = (int64_t*)malloc(sizeof(int64_t) * L);   // host scratch of the schedule
  if (!per) return GRKV_ERR_INVALID;
  if (L == 1) {
    per[0] = mean_budget;
  } else {
    const double top = (double)ratio * mean_budget, bot = (2.0 - (double)ratio) * mean_budget;
    int64_t sum = 0;
    for (int l = 0; l < L; ++l) {
      const double raw = bot + (top - bot) * (double)l / (double)(L - 1);
      int64_t b = (int64_t)floor(raw + 0.5);
      b = b < window ? window : b > n ? n : b;
      per[l] = b;
      sum += b;
    }
    // rounding remainder to the lowest layers, one token each, within [w, n]
    int64_t diff = (int64_t)L * mean_budget - sum;
    for (int i = 0; diff != 0 && i < 4 * L; ++i) {
      const int j = i % L;
      const int64_t step = diff > 0 ? 1 : -1;
      if (per[j] + step >= window && per[j] + step <= n) {
        per[j] += step;
        diff -= step;
      }
    }
  }
  for (int l = 0; l < L; ++l)
    for (int h = 0; h < kv_heads; ++h) budgets[(size_t)l * kv_heads + h] = (int32_t)per[l];
  free(per);
  return GRKV_OK;
}

int grkv_adaptive_budgets(const float* pooled, int32_t layers, int32_t kv_heads, int64_t n,
                          int32_t window, int32_t budget, void* stream, int32_t* budgets) {
  if (!pooled || !budgets || layers < 1 || kv_heads < 1 || window < 1 || budget < window ||
      (int64_t)budget > n)
    return GRKV_ERR_INVALID;
  if (kv_heads > 128) return GRKV_ERR_UNSUPPORTED;
  const int64_t P = n - window;
  if (P < 1 || (int64_t)kv_heads * P > (int64_t(1) << 31)) return GRKV_ERR_UNSUPPORTED;
  const int64_t kk = (int64_t)kv_heads * (budget - window);
  if (launch_adaptive_budgets(pooled, layers, kv_heads, (int)P, kk, window, budgets,
                              (hipStream_t)stream) != hipSuccess)
    return GRKV_ERR_HIP;
  return GRKV_OK;
}

// Native ragged plan (bf16 fast path): the budget-independent passes as for
// one budget; the retained pass in splits of one length over each unit's own
// budget, the update in blocks of one slot count, both as flat grids whose
// blocks find their unit in device tables.  `tab` receives the tables
// (RagUnit [U], the unit of every retained-pass split, the unit of every
// update block, then the two launch orders) for the caller to copy into the
// workspace.  *native is false
// when the shape or equal budgets take the generic path (one call per run of equal
// budgets).
static int make_ragged_plan(const grkv_problem* prob, int64_t n, int32_t window,
                            const int32_t* budgets, int32_t pool_kernel, float lambda,
                            const grkv_options* opt, Plan* p, std::vector<int32_t>* tab,
                            bool* native) {
  *native = false;
  if (!prob || !budgets || prob->units < 1) return GRKV_ERR_INVALID;
  const int U = prob->units;
  int64_t sum = 0;
  int cmax = 0;
  bool differ = false;
  for (int u = 0; u < U; ++u) {
    differ |= budgets[u] != budgets[0];
    if (budgets[u] < window || (int64_t)budgets[u] > n || window < 1) return GRKV_ERR_INVALID;
    sum += budgets[u];
    cmax = budgets[u] > cmax ? budgets[u] : cmax;
  }
  if (sum > INT32_MAX) return GRKV_ERR_UNSUPPORTED;   // packed slot offsets are int32
  int cmean = (int)((sum + U / 2) / U);
  if (cmean < window) cmean = window;
  if (cmean > n) cmean = (int)n;
  const int st = make_plan(prob, n, window, cmean, pool_kernel, lambda, opt, p, true);
  if (st != GRKV_OK) return st;
  // (equal budgets are the plain call, which combines its partials in launches of
  // their own: 8 units of 8192 tokens, 512 retained each, 141 -> 116 us)
  if (!differ || !(stream_supported(*p) && p->fast_merge)) return GRKV_OK;
  // slots per retained-pass split and per update block: the mean budget's, or up
  // to half as many more where the units' own block counts then take fewer
  // rounds of 256 (one block per compute unit at a time)
  auto block_len = [&](int len, int most) {
    constexpr int64_t kBlockTiles = 10;
    int best = len;
    int64_t best_cost = 0;
    for (int k = 0; k <= 4; ++k) {
      const int l = (int)(ceil_div((int64_t)len * (8 + k), 8 * kKeyTile) * kKeyTile);
      if (l > most) break;
      int64_t blocks = 0;
      for (int u = 0; u < U; ++u) blocks += (budgets[u] + l - 1) / l;
      const int64_t cost = ceil_div(blocks, 256) * (l / kKeyTile + kBlockTiles);
      if (k == 0 || 100 * cost < 97 * best_cost) {
        best = l;
        best_cost = cost;
      }
    }
    return best;
  };
  const int chunk = p->chunk2 = p->chunk3 = block_len(p->chunk2, 4096);
  const int spb = block_len(update_slots_per_block(*p, cmean), 4096);
  std::vector<int32_t> split_unit, upd_unit;
  tab->assign((size_t)8 * U, 0);
  int64_t off = 0;
  for (int u = 0; u < U; ++u) {
    const int c = budgets[u];
    RagUnit r;
    r.off = (int32_t)off;
    r.c = c;
    r.s0 = (int32_t)split_unit.size();
    r.ns = (c + chunk - 1) / chunk;
    const int64_t top = (int64_t)floor((double)p->opt.beta * (double)c);
    r.ntop = (int32_t)(top < c - window ? top : c - window);
    r.ub0 = (int32_t)upd_unit.size();
    r.nub = (c + spb - 1) / spb;
    r.pad = 0;
    split_unit.insert(split_unit.end(), r.ns, u);
    upd_unit.insert(upd_unit.end(), r.nub, u);
    memcpy(tab->data() + (size_t)8 * u, &r, sizeof(r));
    off += c;
  }
  p->rag_splits = (int)split_unit.size();
  p->rag_upd_blocks = (int)upd_unit.size();
  p->upd_spb = spb;
  // launch orders: splits (update blocks) by decreasing slot count, ties in
  // split order (a stable sort)
  auto order = [&](const std::vector<int32_t>& unit_of, int len, int first_of_unit) {
    std::vector<int32_t> o(unit_of.size()), size(unit_of.size());
    for (size_t f = 0; f < unit_of.size(); ++f) {
      const RagUnit* r = reinterpret_cast<const RagUnit*>(tab->data()) + unit_of[f];
      const int first = first_of_unit == 0 ? r->s0 : r->ub0;
      const int k = (int)f - first;
      const int rest = r->c - k * len;
      size[f] = rest < len ? rest : len;
      o[f] = (int32_t)f;
    }
    std::stable_sort(o.begin(), o.end(), [&](int32_t a, int32_t b) { return size[a] > size[b]; });
    return o;
  };
  const std::vector<int32_t> split_order = order(split_unit, chunk, 0);
  const std::vector<int32_t> upd_order = order(upd_unit, spb, 1);
  tab->insert(tab->end(), split_unit.begin(), split_unit.end());
  tab->insert(tab->end(), upd_unit.begin(), upd_unit.end());
  tab->insert(tab->end(), split_order.begin(), split_order.end());
  tab->insert(tab->end(), upd_order.begin(), upd_order.end());
  p->c = cmax;
  p->s_sel = cmax - window;
  layout_plan(p, (size_t)sum, split_unit.size(), split_unit.size(), tab->size() * sizeof(int32_t));
  *native = true;
  return GRKV_OK;
}

// Runs of consecutive units with one budget (generic path); the largest plan.
static int ragged_runs(const grkv_problem* prob, int64_t n, int32_t window,
                       const int32_t* budgets, int32_t pool_kernel, float lambda,
                       const grkv_options* opt, size_t* ws_max) {
  if (!prob || !budgets || prob->units < 1) return GRKV_ERR_INVALID;
  size_t mx = 0;
  for (int u0 = 0; u0 < prob->units;) {
    int u1 = u0 + 1;
    while (u1 < prob->units && budgets[u1] == budgets[u0]) ++u1;
    grkv_problem pr = *prob;
    pr.units = u1 - u0;
    Plan p;
    const int st = make_plan(&pr, n, window, budgets[u0], pool_kernel, lambda, opt, &p);
    if (st != GRKV_OK) return st;
    mx = p.total > mx ? p.total : mx;
    u0 = u1;
  }
  *ws_max = mx;
  return GRKV_OK;
}

size_t grkv_workspace_bytes_ragged(const grkv_problem* prob, int64_t n, int32_t window,
                                   const int32_t* budgets) {
  Plan p;
  std::vector<int32_t> tab;
  bool native = false;
  if (make_ragged_plan(prob, n, window, budgets, 1, 0.f, nullptr, &p, &tab, &native) != GRKV_OK)
    return 0;
  if (native) return p.total;
  size_t mx = 0;
  if (ragged_runs(prob, n, window, budgets, 1, 0.f, nullptr, &mx) != GRKV_OK) return 0;
  return mx;
}

int grkv_compress_ragged(const void* q_obs, const void* K, const void* V, int64_t n,
                         int32_t window, const int32_t* budgets, int32_t pool_kernel,
                         float lambda, void* stream, const grkv_problem* prob,
                         const grkv_options* opt, const grkv_outputs* out) {
  int st = check_pointers(q_obs, K, V, prob, out);
  if (st != GRKV_OK) return st;
  Plan rp;
  std::vector<int32_t> tab;
  bool native = false;
  st = make_ragged_plan(prob, n, window, budgets, pool_kernel, lambda, opt, &rp, &tab, &native);
  if (st != GRKV_OK) return st;
  if (native) {
    // one launch per stage over every unit; the tables go into the workspace
    // first (a pageable-memory copy: the host array is consumed on return)
    if (out->workspace_bytes < rp.total) return GRKV_ERR_WORKSPACE;
    char* ws = (char*)out->workspace;
    int32_t* dt = (int32_t*)(ws + rp.rag_tab);
    if (hipMemcpyAsync(dt, tab.data(), tab.size() * sizeof(int32_t), hipMemcpyHostToDevice,
                       (hipStream_t)stream) != hipSuccess)
      return GRKV_ERR_HIP;
    rp.rag = (const RagUnit*)dt;
    rp.rag_split_unit = dt + (size_t)8 * rp.U;
    rp.rag_upd_unit = rp.rag_split_unit + rp.rag_splits;
    rp.rag_split_order = rp.rag_upd_unit + rp.rag_upd_blocks;
    rp.rag_upd_order = rp.rag_split_order + rp.rag_splits;
    return run_compress(rp, q_obs, K, V, n, (hipStream_t)stream, out);
  }
  size_t need = 0;
  st = ragged_runs(prob, n, window, budgets, pool_kernel, lambda, opt, &need);
  if (st != GRKV_OK) return st;
  if (out->workspace_bytes < need) return GRKV_ERR_WORKSPACE;
  const size_t esz = prob->dtype == GRKV_BF16 ? 2 : 4;
  const size_t m = (size_t)prob->group * window, d = prob->head_dim;
  size_t off = 0;   // packed slot offset of unit u0
  for (int u0 = 0; u0 < prob->units;) {
    int u1 = u0 + 1;
    while (u1 < prob->units && budgets[u1] == budgets[u0]) ++u1;
    grkv_problem pr = *prob;
    pr.units = u1 - u0;
    Plan p;
    st = make_plan(&pr, n, window, budgets[u0], pool_kernel, lambda, opt, &p);
    if (st != GRKV_OK) return st;
    grkv_outputs o = *out;
    o.idx = out->idx + off;
    o.k_out = (char*)out->k_out + off * d * esz;
    o.v_out = out->v_out + off * d;
    o.stats = out->stats ? out->stats + (size_t)4 * u0 : nullptr;
    if (u0 > 0 || u1 < prob->units) o.stage_events = nullptr;   // (one run: its stages)
    st = run_compress(p, (const char*)q_obs + (size_t)u0 * m * d * esz,
                      (const char*)K + (size_t)u0 * n * d * esz,
                      (const char*)V + (size_t)u0 * n * d * esz, n, (hipStream_t)stream, &o);
    if (st != GRKV_OK) return st;
    off += (size_t)(u1 - u0) * budgets[u0];
    u0 = u1;
  }
  return GRKV_OK;
}

int grkv_carrier_stats(const void* K, int64_t n, int32_t budget, const grkv_problem* prob,
                       const int32_t* idx, const float* stats, void* stream, int32_t* assign,
                       int32_t* counts, float* metrics, float* l_common) {
  if (!K || !prob || !idx || !assign || !metrics) return GRKV_ERR_INVALID;
  if (prob->units < 1 || prob->group < 1) return GRKV_ERR_INVALID;
  if (prob->dtype != GRKV_BF16 && prob->dtype != GRKV_F32) return GRKV_ERR_INVALID;
  if (budget < 1 || (int64_t)budget > n || n > (int64_t(1) << 30)) return GRKV_ERR_INVALID;
  if (!carrier_supported(prob->dtype, prob->head_dim, budget)) return GRKV_ERR_UNSUPPORTED;
  if (launch_carrier(K, idx, prob->units, n, budget, prob->head_dim, stats, assign, counts,
                     metrics, l_common, (hipStream_t)stream) != hipSuccess)
    return GRKV_ERR_HIP;
  return GRKV_OK;
}

}  // extern "C"
