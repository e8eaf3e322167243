// Drives the host layer of libkvs (kvs_api.hip, linked with launch_stubs.cpp) through its C ABI on the CPU: argument
// errors, workspace sizing and carve-up, alias checks, and whole calls on problems of many ragged units whose
// "launches" are stubs.  Built with -fsanitize=address,undefined by tests/test_host_sanitizers.py: any out-of-bounds
// access, overflow or misaligned access in make_plan / carve / check_ranges / for_each_group ends the run.
// Device pointers are fake addresses that nothing dereferences.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "kvs.h"
#include "kvs_debug.h"

namespace kvs { int stub_launches(); bool stub_values_rode(); int stub_most_parts(); int stub_chunks(); int stub_pieces(); extern bool stub_asks_for_fused; }

static int g_failed = 0;
#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED %s (line %d)\n", #cond, __LINE__); ++g_failed; } } while (0)

struct Problem {
  std::vector<int32_t> len, budget;
  std::vector<int64_t> in_row, out_row;
  kvs_problem p{};
  long long rows_in = 0, rows_out = 0;
  Problem(std::vector<int32_t> l, std::vector<int32_t> b, int group, int window, int D, kvs_dtype dt) : len(l), budget(b) {
    for (size_t i = 0; i < len.size(); ++i) {
      in_row.push_back(rows_in);
      out_row.push_back(rows_out);
      rows_in += len[i];
      rows_out += std::min(len[i], budget[i]);
    }
    p.n_units = (int)len.size(); p.group = group; p.window = window; p.head_dim = D; p.n_sink = 4; p.n_recent = 0;
    p.io_dtype = dt; p.scale = 0.f; p.len = len.data(); p.budget = budget.data(); p.in_row = in_row.data();
    p.out_row = out_row.data(); p.key_rule = KVS_RULE_HESSIAN; p.causal = 0;
  }
};

// fake, non-overlapping, 256-byte aligned device ranges
struct Arena {
  uintptr_t next = (uintptr_t)1 << 40;
  void* take(size_t bytes) { void* r = (void*)next; next += (bytes + 4095) / 4096 * 4096 + 4096; return r; }
};

static void whole_calls(std::mt19937& rng, kvs_dtype dt, int group, int window, int D) {
  const size_t elt = dt == KVS_F32 ? 4 : 2;
  for (int rep = 0; rep < 20; ++rep) {
    const int nu = 1 + (int)(rng() % 150);                      // up to three launch groups
    std::vector<int32_t> len(nu), budget(nu);
    for (int u = 0; u < nu; ++u) {
      len[u] = 32 + (int)(rng() % (rep % 4 == 0 ? 200000 : 9000));
      budget[u] = std::max(8, (int)(len[u] / (2 + rng() % 6)));
      if (rng() % 11 == 0) budget[u] = len[u] + 3;               // pass-through
    }
    Problem pr(len, budget, group, window, D, dt);
    const int R = group * window;
    size_t ws_bytes = 0, pq_bytes = 0, dec_bytes = 0;
    EXPECT(kvs_workspace_size(&pr.p, &ws_bytes) == KVS_OK);
    EXPECT(ws_bytes % 256 == 0 && ws_bytes >= (size_t)pr.rows_in * 9);
    Arena a;
    void* Q = a.take((size_t)nu * R * D * elt);
    void* K = a.take((size_t)pr.rows_in * D * elt);
    void* V = a.take((size_t)pr.rows_in * D * elt);
    void* Ko = a.take((size_t)pr.rows_out * D * elt);
    void* Vo = a.take((size_t)pr.rows_out * D * elt);
    int32_t* cnt = (int32_t*)a.take((size_t)pr.rows_out * 4);
    float* alpha = (float*)a.take((size_t)pr.rows_in * 4);
    float* obar = (float*)a.take((size_t)nu * D * 4);
    uint8_t* mask = (uint8_t*)a.take((size_t)pr.rows_in);
    int32_t* slot = (int32_t*)a.take((size_t)pr.rows_in * 4);
    int32_t* cin = (int32_t*)a.take((size_t)pr.rows_in * 4);
    void* ws = a.take(ws_bytes);
    const int before = kvs::stub_launches();
    EXPECT(kvs_step(&pr.p, Q, K, V, Ko, Vo, cnt, slot, mask, ws, ws_bytes, nullptr) == KVS_OK);
    EXPECT(kvs_step_counts(&pr.p, Q, K, V, cin, Ko, Vo, cnt, nullptr, nullptr, ws, ws_bytes, nullptr) == KVS_OK);
    EXPECT(kvs_score(&pr.p, Q, K, V, alpha, obar, ws, ws_bytes, nullptr) == KVS_OK);
    EXPECT(kvs_select(&pr.p, alpha, mask, slot, nullptr, 0, nullptr) == KVS_OK);
    EXPECT(kvs_select(&pr.p, alpha, mask, slot, ws, ws_bytes, nullptr) == KVS_OK);          // several workgroups per unit
    EXPECT(kvs_select(&pr.p, alpha, mask, slot, ws, ws_bytes - 256, nullptr) == KVS_OK);    // too small: not used
    EXPECT(kvs_select(&pr.p, alpha, (uint8_t*)ws, slot, ws, ws_bytes, nullptr) == KVS_ERR_ALIAS);
    EXPECT(kvs_merge_compact(&pr.p, K, V, alpha, obar, mask, slot, Ko, Vo, cnt, nullptr, 0, nullptr) == KVS_OK);
    EXPECT(kvs_merge_compact(&pr.p, K, V, alpha, obar, mask, slot, Ko, Vo, cnt, ws, ws_bytes, nullptr) == KVS_OK);   // optional
    EXPECT(kvs_merge_compact(&pr.p, K, V, alpha, obar, mask, slot, Ko, Vo, cnt, ws, ws_bytes - 256, nullptr) == KVS_OK);
    EXPECT(kvs_merge_compact(&pr.p, K, V, alpha, obar, (uint8_t*)ws, slot, Ko, Vo, cnt, ws, ws_bytes, nullptr) == KVS_ERR_ALIAS);
    EXPECT(kvs::stub_launches() >= before + 5 * ((nu + 63) / 64));
    EXPECT(kvs_step(&pr.p, Q, K, V, Ko, Vo, cnt, slot, mask, ws, ws_bytes - 1, nullptr) == KVS_ERR_WORKSPACE);
    EXPECT(kvs_step(&pr.p, Q, K, V, Ko, Ko, cnt, slot, mask, ws, ws_bytes, nullptr) == KVS_ERR_ALIAS);
    EXPECT(kvs_step(&pr.p, Q, K, V, Ko, Vo, cnt, slot, (uint8_t*)ws + 256, ws, ws_bytes, nullptr) == KVS_ERR_ALIAS);
    {                                          // per-query aggregation: both dtypes
      EXPECT(kvs_per_query_workspace_size(&pr.p, &pq_bytes) == KVS_OK && pq_bytes > ws_bytes);
      void* pws = a.take(pq_bytes);
      float* a_tok = (float*)a.take((size_t)pr.rows_in * 4);
      float* c_edge = (float*)a.take((size_t)pr.rows_in * 4);
      EXPECT(kvs_sensitivity(&pr.p, Q, K, V, alpha, a_tok, c_edge, pws, pq_bytes, nullptr) == KVS_OK);
      EXPECT(kvs_step_per_query(&pr.p, Q, K, V, Ko, Vo, cnt, nullptr, nullptr, pws, pq_bytes, nullptr) == KVS_OK);
      EXPECT(kvs_merge_compact_norms(&pr.p, K, V, a_tok, c_edge, mask, slot, Ko, Vo, cnt, nullptr, 0, nullptr) == KVS_OK);
      EXPECT(kvs_merge_compact_norms(&pr.p, K, V, a_tok, c_edge, mask, slot, Ko, Vo, cnt, ws, ws_bytes, nullptr) == KVS_OK);
      EXPECT(kvs_sensitivity_counts(&pr.p, Q, K, V, cin, alpha, a_tok, c_edge, pws, pq_bytes, nullptr) == KVS_OK);
      EXPECT(kvs_step_per_query_counts(&pr.p, Q, K, V, cin, Ko, Vo, cnt, nullptr, nullptr, pws, pq_bytes, nullptr) == KVS_OK);
      EXPECT(kvs_merge_compact_norms_counts(&pr.p, K, V, cin, a_tok, c_edge, mask, slot, Ko, Vo, cnt, nullptr, 0, nullptr) == KVS_OK);
      EXPECT(kvs_sensitivity_counts(&pr.p, Q, K, V, (const int32_t*)a_tok, alpha, a_tok, c_edge, pws, pq_bytes, nullptr) == KVS_ERR_ALIAS);
    }
    if (R <= KVS_MAX_DECODE_ROWS) {
      EXPECT(kvs_decode_workspace_size(&pr.p, &dec_bytes) == KVS_OK);
      float* out = (float*)a.take((size_t)nu * R * D * 4);
      void* dws = a.take(dec_bytes);
      EXPECT(kvs_decode_attention(&pr.p, Q, K, V, cin, out, dws, dec_bytes, nullptr) == KVS_OK);
    }
    // the static entry refuses what its array cannot hold, before any device call
    if (ws_bytes > KVS_STATIC_SCRATCH_BYTES) {
      EXPECT(kvs_step_static(&pr.p, Q, K, V, nullptr, Ko, Vo, cnt, nullptr, nullptr, nullptr) == KVS_ERR_WORKSPACE);
    }
  }
}

// Equal units in several launch groups, some with chunks of another length than the others (65 to 128 bf16 rows), and
// launches that cut the groups elsewhere: every table has to stand for itself.
static void equal_units(int nu, int len, int window) {
  Problem pr(std::vector<int32_t>(nu, len), std::vector<int32_t>(nu, len / 4), 4, window, 128, KVS_BF16);
  size_t ws_bytes = 0, pq_bytes = 0;
  EXPECT(kvs_workspace_size(&pr.p, &ws_bytes) == KVS_OK);
  EXPECT(kvs_per_query_workspace_size(&pr.p, &pq_bytes) == KVS_OK);
  Arena a;
  void* Q = a.take((size_t)nu * 4 * window * 128 * 2);
  void* K = a.take((size_t)pr.rows_in * 128 * 2);
  void* V = a.take((size_t)pr.rows_in * 128 * 2);
  void* Ko = a.take((size_t)pr.rows_out * 128 * 2);
  void* Vo = a.take((size_t)pr.rows_out * 128 * 2);
  int32_t* cnt = (int32_t*)a.take((size_t)pr.rows_out * 4);
  void* ws = a.take(pq_bytes);
  EXPECT(kvs_step(&pr.p, Q, K, V, Ko, Vo, cnt, nullptr, nullptr, ws, ws_bytes, nullptr) == KVS_OK);
  EXPECT(kvs_step_per_query(&pr.p, Q, K, V, Ko, Vo, cnt, nullptr, nullptr, ws, pq_bytes, nullptr) == KVS_OK);
}

// One step over nu equal units (one launch, more than the caches hold): whether sweep 1 carries the pass over V, and the
// select workgroups per unit.  A unit of more than 32768 tokens whose selection is not shared out by parts that meet keeps V
// apart: that selection is then hidden beside the pass.
static void values_ride(int nu, int len, int budget, bool rode, int parts, int window = 32, int D = 128, bool counts = false,
                        int more = 0) {
  std::vector<int32_t> lens(nu, len);
  lens[0] += more;                              // units of unequal lengths
  Problem pr(lens, std::vector<int32_t>(nu, budget), 4, window, D, KVS_BF16);
  pr.p.n_sink = 32;
  size_t ws_bytes = 0;
  EXPECT(kvs_workspace_size(&pr.p, &ws_bytes) == KVS_OK);
  Arena a;
  void* Q = a.take((size_t)nu * 128 * 128 * 2);
  void* K = a.take((size_t)pr.rows_in * 128 * 2);
  void* V = a.take((size_t)pr.rows_in * 128 * 2);
  void* Ko = a.take((size_t)pr.rows_out * 128 * 2);
  void* Vo = a.take((size_t)pr.rows_out * 128 * 2);
  int32_t* cnt = (int32_t*)a.take((size_t)pr.rows_out * 4);
  void* ws = a.take(ws_bytes);
  int32_t* cin = counts ? (int32_t*)a.take((size_t)pr.rows_in * 4) : nullptr;
  EXPECT(kvs_step_counts(&pr.p, Q, K, V, cin, Ko, Vo, cnt, nullptr, nullptr, ws, ws_bytes, nullptr) == KVS_OK);
  if (kvs::stub_values_rode() != rode || kvs::stub_most_parts() != parts) {
    std::printf("%d x %d: V %s, %d select workgroups per unit\n", nu, len, kvs::stub_values_rode() ? "rode" : "apart",
                kvs::stub_most_parts());
    EXPECT(!"the rule above");
  }
}

// How many score chunks a call on the given units (one launch) is cut into.
static void chunks_of(std::vector<int32_t> len, int group, int window, int D, kvs_dtype dt, bool per_query, int chunks,
                      bool counts = false) {
  std::vector<int32_t> budget(len);
  for (int32_t& b : budget) b /= 3;
  Problem pr(len, budget, group, window, D, dt);
  const size_t elt = dt == KVS_F32 ? 4 : 2;
  size_t ws_bytes = 0;
  EXPECT((per_query ? kvs_per_query_workspace_size(&pr.p, &ws_bytes) : kvs_workspace_size(&pr.p, &ws_bytes)) == KVS_OK);
  Arena a;
  void* Q = a.take(len.size() * group * window * D * elt);
  void* K = a.take((size_t)pr.rows_in * D * elt);
  void* V = a.take((size_t)pr.rows_in * D * elt);
  void* Ko = a.take((size_t)pr.rows_out * D * elt);
  void* Vo = a.take((size_t)pr.rows_out * D * elt);
  int32_t* cnt = (int32_t*)a.take((size_t)pr.rows_out * 4);
  int32_t* cin = counts ? (int32_t*)a.take((size_t)pr.rows_in * 4) : nullptr;
  void* ws = a.take(ws_bytes);
  EXPECT((per_query ? kvs_step_per_query_counts(&pr.p, Q, K, V, cin, Ko, Vo, cnt, nullptr, nullptr, ws, ws_bytes, nullptr)
                    : kvs_step_counts(&pr.p, Q, K, V, cin, Ko, Vo, cnt, nullptr, nullptr, ws, ws_bytes, nullptr)) == KVS_OK);
  if (chunks >= 0 && kvs::stub_chunks() != chunks) {
    std::printf("%zu units, the first of %d tokens, %d rows, head dim %d%s%s: %d chunks instead of %d\n", len.size(), len[0],
                group * window, D, dt == KVS_F32 ? ", fp32" : "", per_query ? ", per query" : "", kvs::stub_chunks(), chunks);
    EXPECT(!"the launch's chunks");
  }
}

// The pieces that the bf16 per-query kernels cut the chunks into.
static void pieces_of(int nu, int len, int rows, int D, int pieces) {
  chunks_of(std::vector<int32_t>(nu, len), 1, rows, D, KVS_BF16, true, -1);
  if (kvs::stub_pieces() != pieces) {
    std::printf("%d units of %d tokens, %d rows, head dim %d: %d pieces instead of %d\n", nu, len, rows, D, kvs::stub_pieces(), pieces);
    EXPECT(!"the launch's pieces");
  }
}

// Whole rounds of workgroups: fewer rounds than chunks of the ordinary length would take, or as many with shorter chunks, and
// never longer ones in as many rounds (512 workgroups at a time here, 256 above 256 rows).
static void whole_rounds() {
  auto equal = [](int nu, int len) { return std::vector<int32_t>(nu, len); };
  chunks_of(equal(48, 16384), 7, 32, 128, KVS_BF16, true, 480);     // 528 would be two rounds
  chunks_of(equal(48, 16384), 7, 32, 128, KVS_BF16, false, 480);
  chunks_of(equal(64, 32768), 4, 32, 128, KVS_BF16, false, 512);    // 1024
  chunks_of(equal(8, 131072), 8, 64, 128, KVS_BF16, false, 256);    // 512, 256 at a time
  chunks_of(equal(16, 10000), 4, 32, 128, KVS_BF16, true, 512);     // one round of 320 tokens each, not of 384
  chunks_of(equal(16, 10000), 7, 32, 128, KVS_BF16, true, 512);
  chunks_of(equal(12, 50000), 7, 32, 128, KVS_BF16, true, 504);
  chunks_of(equal(24, 6500), 4, 16, 128, KVS_BF16, true, 504);
  chunks_of(equal(64, 3277), 4, 32, 128, KVS_BF16, true, 512);
  chunks_of(equal(100, 21000), 4, 32, 128, KVS_BF16, true, 1000);   // two rounds either way, of 2112 tokens each
  for (int window : {17, 32}) {
    chunks_of(equal(100, 11000), 4, window, 128, KVS_BF16, false, 500);
    chunks_of(equal(100, 11000), 4, window, 128, KVS_BF16, true, 500);
    chunks_of(equal(100, 21000), 4, window, 128, KVS_BF16, false, 1000);
    chunks_of(equal(64, 21000), 4, window, 128, KVS_BF16, false, 512);
  }
  chunks_of(equal(40, 32768), 4, 16, 128, KVS_BF16, true, 480);     // pieces of whole tiles of 32 that all wavefronts share
  chunks_of(equal(8, 16431), 4, 64, 64, KVS_BF16, false, 416);
  chunks_of(equal(34, 4481), 4, 32, 128, KVS_BF16, false, 408);     // a tile for each of four wavefronts: 384 tokens take no longer than 320
  chunks_of(equal(16, 10000), 4, 32, 128, KVS_BF16, false, 432);
  chunks_of(equal(24, 10721), 8, 64, 64, KVS_BF16, false, 216);     // two rounds of 512 and one of 1280, and what a workgroup does once
  chunks_of(equal(16, 8402), 1, 64, 128, KVS_F32, false, 432);
  std::vector<int32_t> ragged;
  for (int i = 0; i < 16; ++i) ragged.push_back(4000 + 2400 * i);
  chunks_of(ragged, 7, 32, 128, KVS_BF16, false, 507);
  chunks_of(ragged, 7, 32, 128, KVS_BF16, true, 507);
  // 768 at a time: one to three rows, and up to 64 rows of 64 channels with cardinalities; 1024 without
  for (kvs_dtype dt : {KVS_F32, KVS_BF16}) {
    chunks_of(equal(150, 4000), 1, 1, 128, dt, false, 750);
    chunks_of(equal(100, 11000), 3, 1, 64, dt, false, 700);
    chunks_of(ragged, 1, 1, 128, dt, false, 649);
  }
  chunks_of(equal(64, 32768), 4, 4, 64, KVS_BF16, false, 1024);
  chunks_of(equal(64, 32768), 4, 4, 64, KVS_BF16, false, 768, true);
  chunks_of(equal(64, 32768), 4, 4, 64, KVS_F32, false, 512);
  chunks_of(equal(16, 25759), 4, 2, 64, KVS_BF16, false, 464);      // 512 at a time with fewer tokens than 512 for each of the 1024
  chunks_of(equal(30, 10000), 4, 16, 64, KVS_BF16, false, 480);
  chunks_of(equal(149, 2777), 1, 64, 64, KVS_BF16, false, 447);
  chunks_of(equal(100, 5300), 4, 8, 64, KVS_BF16, false, 900);
  // 256 at a time: 129 to 192 rows without cardinalities, of 64 channels or read past the caches
  chunks_of(equal(48, 16384), 5, 32, 128, KVS_BF16, false, 240);
  chunks_of(equal(48, 16384), 5, 32, 128, KVS_BF16, false, 480, true);
  chunks_of(equal(48, 16384), 5, 32, 128, KVS_BF16, true, 480);
  chunks_of(equal(32, 9000), 5, 32, 64, KVS_BF16, false, 256);
  chunks_of(equal(32, 9000), 7, 32, 64, KVS_BF16, false, 512);
  // ragged launches a little above one round, or two: chunks as much longer as it takes, of a tile for each of four wavefronts
  std::vector<int32_t> some;
  for (int i = 0; i < 20; ++i) some.push_back(20000 + 640 * i);
  for (int group : {1, 2, 4}) chunks_of(some, group, 32, 128, KVS_BF16, false, 463);
  chunks_of(some, 4, 32, 128, KVS_BF16, true, 489);
  std::vector<int32_t> many;
  for (int i = 0; i < 100; ++i) many.push_back(8000 + 222 * i);
  for (int group : {1, 2, 4}) chunks_of(many, group, 32, 128, KVS_BF16, false, 978);
  chunks_of(many, 4, 32, 128, KVS_BF16, true, 1006);
}

int main() {
  std::mt19937 rng(12345);
  size_t bytes = 0;
  EXPECT(kvs_workspace_size(nullptr, &bytes) == KVS_ERR_INVALID_ARG);
  {
    Problem pr({1024, 500}, {512, 600}, 2, 4, 64, KVS_F32);
    EXPECT(kvs_workspace_size(&pr.p, nullptr) == KVS_ERR_INVALID_ARG);
    EXPECT(kvs_workspace_size(&pr.p, &bytes) == KVS_OK && bytes % 256 == 0);
    kvs_problem q = pr.p;
    q.head_dim = 96; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_INVALID_ARG);
    q = pr.p; q.group = 64; q.window = 32; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_INVALID_ARG);
    q = pr.p; q.io_dtype = (kvs_dtype)7; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_DTYPE);
    q = pr.p; q.len = nullptr; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_INVALID_ARG);
    q = pr.p; q.n_units = 0; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_INVALID_ARG);
    q = pr.p; q.causal = 2; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_INVALID_ARG);
    q = pr.p; q.key_rule = (kvs_key_rule)5; EXPECT(kvs_workspace_size(&q, &bytes) == KVS_ERR_INVALID_ARG);
  }
  {
    Problem pr({KVS_MAX_LEN, 5}, {KVS_MAX_LEN / 2, 5}, 4, 32, 128, KVS_BF16);       // the longest unit, 32-bit offsets
    EXPECT(kvs_workspace_size(&pr.p, &bytes) == KVS_OK);
    Problem bad({KVS_MAX_LEN + 1, 5}, {KVS_MAX_LEN / 2, 5}, 4, 32, 128, KVS_BF16);
    EXPECT(kvs_workspace_size(&bad.p, &bytes) == KVS_ERR_INVALID_ARG);
    Problem small({1024, 500}, {3, 600}, 2, 4, 64, KVS_F32);                        // budget below n_sink + 1
    EXPECT(kvs_workspace_size(&small.p, &bytes) == KVS_ERR_BUDGET);
    Problem overlap({1024, 500}, {512, 600}, 2, 4, 64, KVS_F32);
    overlap.in_row[1] = 1000;
    EXPECT(kvs_workspace_size(&overlap.p, &bytes) == KVS_ERR_INVALID_ARG);
  }
  whole_calls(rng, KVS_F32, 1, 8, 64);
  whole_calls(rng, KVS_BF16, 4, 32, 128);       // the one-pass score kernel's tables are part of the workspace
  whole_calls(rng, KVS_BF16, 8, 64, 128);       // 512 query rows
  whole_calls(rng, KVS_BF16, 1, 3, 64);
  kvs_debug_set(KVS_DEBUG_SCORE_FUSED, 2);
  whole_calls(rng, KVS_BF16, 4, 32, 128);
  kvs_debug_set(KVS_DEBUG_SCORE_FUSED, 0);
  kvs_debug_set(KVS_DEBUG_SELECT_SPLIT, 2);     // as many select workgroups per unit as the units can have
  whole_calls(rng, KVS_BF16, 4, 32, 128);
  for (int mode : {0, 2, 3}) {                  // (2 and 3: launches of at most 64 units)
    kvs_debug_set(KVS_DEBUG_SELECT_SPLIT, mode);
    for (int window : {17, 32}) {
      equal_units(164, 21000, window);
      equal_units(256, 20000, window);
      equal_units(300, 2560, window);
    }
  }
  kvs_debug_set(KVS_DEBUG_SELECT_SPLIT, 1);     // never more than one
  whole_calls(rng, KVS_F32, 1, 8, 64);
  kvs_debug_set(KVS_DEBUG_SELECT_SPLIT, 0);
  for (int cap : {7, 64, 100}) {                // launch groups held to a few units, to the inline descriptors, beyond them
    kvs_debug_set(KVS_DEBUG_GROUP_UNITS, cap);
    whole_calls(rng, KVS_BF16, 4, 32, 128);
  }
  kvs_debug_set(KVS_DEBUG_GROUP_UNITS, 0);
  values_ride(64, 32768, 8192, true, 4);        // (256 compute units, also where there is no GPU)
  values_ride(16, 32790, 8192, false, 8);       // eight slices, by as many workgroups that do not meet
  values_ride(8, 131072, 8192, true, 32);       // by parts that meet
  values_ride(8, 262000, 8192, true, 32);       // the longest that 32 parts can hold
  values_ride(32, 65500, 8192, true, 8);
  values_ride(33, 65500, 8192, false, 1);       // a launch of many units
  values_ride(32, 131072, 8192, false, 1);      // too long for the parts that the unit may have
  values_ride(20, 131072, 8192, false, 1);
  values_ride(24, 100000, 8192, false, 1);
  values_ride(8, 300000, 8192, false, 1);
  values_ride(8, 524288, 8192, false, 1);
  values_ride(64, 32768, 8192, true, 4, 8);     // 32 rows: with 64 channels where two workgroups run on a compute unit, or
  values_ride(64, 32768, 8192, false, 1, 8, 64);                  // three of equal units with cardinalities
  values_ride(8, 131072, 8192, true, 32, 8, 64);
  values_ride(64, 32768, 8192, true, 4, 8, 64, true);
  values_ride(64, 32700, 8192, false, 1, 8, 64, true, 60);
  values_ride(64, 32700, 8192, true, 4, 8, 128, true, 60);
  values_ride(60, 9000, 2000, false, 1, 8);                       // with 128 channels in the larger launches, or cardinalities
  values_ride(60, 9000, 2000, true, 3, 8, 128, true);
  values_ride(60, 9000, 2000, true, 3);
  values_ride(8, 60000, 9000, true, 30, 8);                       // and with long units whose selection is shared out
  values_ride(64, 32768, 8192, true, 4, 17, 64);
  values_ride(8, 131072, 131072, false, 1);     // nothing to select: as before the selection was shared out
  kvs::stub_asks_for_fused = true;              // the switch for the one-pass kernel changes inside a call on a large group
  equal_units(100, 2560, 32);
  kvs::stub_asks_for_fused = false;
  kvs_debug_set(KVS_DEBUG_SCORE_FUSED, 0);
  whole_rounds();
  // small launches of 9 to 32 rows of 128 channels: pieces down to a tile of 32 tokens, else of 64 at least
  pieces_of(1, 800, 32, 128, 28);
  pieces_of(4, 1000, 16, 128, 128);
  pieces_of(8, 1000, 32, 128, 256);
  pieces_of(1, 6000, 32, 128, 94);
  pieces_of(1, 800, 8, 128, 14);
  pieces_of(1, 800, 32, 64, 14);
  pieces_of(8, 1900, 32, 128, 240);
  EXPECT(kvs_debug_set(99, 1) == -1);
  std::printf(g_failed ? "host layer: %d checks failed\n" : "host layer: all checks passed (%d stub launches)\n",
              g_failed ? g_failed : kvs::stub_launches());
  return g_failed ? 1 : 0;
}
