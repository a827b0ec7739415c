// The host plans of libgrkv.so as plain numbers, for tests/test_host_plan.py
// (no GPU work).
#include "grkv_internal.h"

using namespace grkv;

// out: S1, chunk1, S2, chunk2, S3, chunk3, csplit, mp, update slots per block,
// total bytes, then S_full, S4, S4r of the key step (0 where it does not apply)
extern "C" int plan_probe(const grkv_problem* prob, int64_t n, int32_t window, int32_t budget,
                          int32_t ragged, int64_t* out) {
  Plan p;
  const int st = make_plan(prob, n, window, budget, 7, 0.01f, nullptr, &p, ragged != 0);
  if (st != GRKV_OK) return st;
  const int64_t v[10] = {p.S1, p.chunk1, p.S2, p.chunk2, p.S3, p.chunk3, p.csplit, p.mp,
                         update_slots_per_block(p, p.c), (int64_t)p.total};
  for (int i = 0; i < 10; ++i) out[i] = v[i];
  out[10] = out[11] = out[12] = 0;
  if (key_supported(p)) {
    KeyPlan k;
    make_key_plan(p, 1, &k);
    out[10] = k.S_full;
    out[11] = k.S4;
    out[12] = k.S4r;
  }
  return st;
}
