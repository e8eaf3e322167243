// Host-only stand-ins for the kernel launchers of libkvs: every launch "succeeds" without touching a GPU, so that
// the host layer (argument validation, workspace carve-up, unit tables, launch sequencing in kvs_api.hip) can run
// to the end of a call on the CPU, under AddressSanitizer and UndefinedBehaviorSanitizer.  Test infrastructure.
#include "kvs_device.h"

namespace kvs {

static int g_launches = 0;
int stub_launches() { return g_launches; }
static bool g_values_rode = false;      // the last score launch carried the pass over V
static int g_most_parts = 0;            // select workgroups of the unit that had most of them in the last selection
bool stub_asks_for_fused = false;       // launch_unit_table sets KVS_DEBUG_SCORE_FUSED, as another thread may at any time
bool stub_values_rode() { return g_values_rode; }
int stub_most_parts() { return g_most_parts; }
static int g_chunks = 0;                // score chunks of the last launch
int stub_chunks() { return g_chunks; }
static int g_pieces = 0;                // pieces of the last launch of the bf16 per-query kernels
int stub_pieces() { return g_pieces; }

static hipError_t ok() { ++g_launches; return hipSuccess; }

// what a launcher may assume about its table: checked here so that a wrong table fails the sanitizer run
static const Unit* g_written = nullptr;   // where the last launch_unit_table put its descriptors, and how many
static int g_written_n = 0;

static void check_table(const UnitTable& tab) {
  g_chunks = tab.total_chunks;
  if (tab.n_units < 1 || tab.n_units > kMaxGroupUnits) __builtin_trap();
  // a group beyond the inline descriptors must have had its descriptors written, to where the kernels will look
  if (tab.n_units > kInlineUnits) {
    if (tab.ext == nullptr || tab.host == nullptr || tab.ext != g_written || tab.n_units != g_written_n) __builtin_trap();
  } else if (tab.ext != nullptr || tab.host != nullptr) {
    __builtin_trap();
  }
  long long tokens = 0;
  for (int i = 0; i + 1 < tab.n_units; ++i) tokens += tab.unit(i).len;
  if (tab.n_units > kInlineUnits && tokens >= kGroupTokens) __builtin_trap();   // the group was full before its last unit
  int chunks = 0, mblocks = 0, ochunks = 0;
  for (int i = 0; i < tab.n_units; ++i) {
    const Unit u = tab.unit(i);
    if (u.len < 1 || u.n_out < 1 || u.n_out > u.len) __builtin_trap();
    if (u.chunk_len % kWave != 0 || u.n_chunks < 1 || u.n_chunks > kMaxChunks) __builtin_trap();
    if ((long long)u.chunk_len * u.n_chunks < u.len) __builtin_trap();
    if (u.chunk_base != chunks || u.m_base != mblocks || u.o_base != ochunks) __builtin_trap();
    chunks += u.n_chunks;
    mblocks += (u.len + kMergeTokens - 1) / kMergeTokens;
    ochunks += obar_chunks(u.len);
  }
  if (tab.total_chunks != chunks || tab.total_mblocks != mblocks || tab.total_ochunks != ochunks) __builtin_trap();
  // what the kernels find by a division (`even`) and form from the first two descriptors (`regular`)
  for (int i = 0; i < tab.n_units; ++i) {
    const Unit u = tab.unit(i);
    if (tab.even && (u.chunk_base != i * (chunks / tab.n_units) || u.m_base != i * (mblocks / tab.n_units) ||
                     u.o_base != i * (ochunks / tab.n_units) || u.f_base != i * (tab.total_fitems / tab.n_units) ||
                     u.s_base != i * (tab.total_sparts / tab.n_units))) {
      __builtin_trap();
    }
    if (tab.regular) {
      const Unit &a = tab.u[0], &b = tab.u[1];
      if (!tab.even || u.len != a.len || u.n_out != a.n_out || u.chunk_len != a.chunk_len || u.n_chunks != a.n_chunks ||
          u.index != a.index + i || u.in_row != a.in_row + i * (b.in_row - a.in_row) ||
          u.out_row != a.out_row + i * (b.out_row - a.out_row)) {
        __builtin_trap();
      }
    }
  }
  for (int i = 0; i < tab.n_units; ++i) {          // select workgroups: one or several per unit, in unit order
    const int next = i + 1 < tab.n_units ? tab.unit(i + 1).s_base : tab.total_sparts;
    const int parts = next - tab.unit(i).s_base;
    if (tab.unit(i).s_base < i || parts < 1 || parts > kSelMaxParts) __builtin_trap();
    if (parts > 1 && tab.n_units > kInlineUnits) __builtin_trap();   // the exchange area has kInlineUnits entries
  }
}

hipError_t launch_unit_table(const Unit* units, int n_units, Unit* dst, hipStream_t) {
  if (units == nullptr || dst == nullptr || n_units <= kInlineUnits || n_units > kMaxGroupUnits) __builtin_trap();
  volatile long long touch = 0;
  for (int i = 0; i < n_units; ++i) touch = touch + units[i].len;   // (readable to its end, for the sanitizer)
  g_written = dst;
  g_written_n = n_units;
  if (stub_asks_for_fused) kvs_debug_set(KVS_DEBUG_SCORE_FUSED, 2);
  return ok();
}
hipError_t launch_score_finalize(const UnitTable& tab, const Shape&, const Workspace&, hipStream_t) { check_table(tab); return ok(); }
hipError_t launch_score_valu(const UnitTable& tab, const Shape&, kvs_dtype, const void*, const void*, const int32_t*,
                             float*, const Workspace&, hipStream_t) { check_table(tab); return ok(); }
hipError_t launch_score_mfma(const UnitTable& tab, const Shape&, kvs_dtype, const void*, const void*, const int32_t*,
                             float*, const Workspace&, const void* V, hipStream_t) {
  check_table(tab);
  g_values_rode = V != nullptr;
  return ok();
}
bool score_mfma_supported(const UnitTable& tab, const Shape& sh, kvs_dtype) {
  if (sh.R < 4) return false;
  for (int i = 0; i < tab.n_units; ++i) if (tab.unit(i).len < 32) return false;
  return true;
}
bool score_mfma_takes_values(const Shape& sh, kvs_dtype dt) { return dt == KVS_BF16 && sh.R >= 4; }
bool score_fused_supported(const UnitTable&, const Shape& sh, kvs_dtype dt) { return dt == KVS_BF16 && sh.R > 64 && sh.R <= 128; }
hipError_t launch_score_fused(const UnitTable& tab, const Shape&, const void*, const void*, const void*, const int32_t*,
                              float*, const Workspace& ws, hipStream_t) {
  check_table(tab);
  if (ws.fstats == nullptr || ws.fo_part == nullptr || ws.fsync == nullptr) __builtin_trap();
  if (tab.n_units > kInlineUnits) __builtin_trap();          // its counters are for that many, and its table
  return ok();
}
hipError_t launch_select_obar(const UnitTable& tab, const Shape&, kvs_dtype, bool, const float*, uint8_t*, int32_t*,
                              const void*, const int32_t*, float*, hipStream_t, const float*, float*, unsigned int* sel_shared) {
  check_table(tab);
  if (tab.total_sparts != tab.n_units && sel_shared == nullptr) __builtin_trap();
  g_most_parts = 0;
  for (int i = 0; i < tab.n_units; ++i) {
    const int parts = (i + 1 < tab.n_units ? tab.unit(i + 1).s_base : tab.total_sparts) - tab.unit(i).s_base;
    if (parts > g_most_parts) g_most_parts = parts;
  }
  return ok();
}
hipError_t launch_select_clear(const UnitTable& tab, unsigned int* sel_shared, hipStream_t) {
  check_table(tab);
  if (sel_shared == nullptr) __builtin_trap();
  return ok();
}
hipError_t launch_obar_reduce(const UnitTable& tab, const Shape&, const float*, float*, hipStream_t) { check_table(tab); return ok(); }
hipError_t launch_merge(const UnitTable& tab, const Shape&, kvs_dtype, const void*, const void*, const int32_t*, const float*,
                        const float*, const float*, const uint8_t*, const int32_t*, void*, void*, int32_t*, hipStream_t) { check_table(tab); return ok(); }
hipError_t launch_merge_norms(const UnitTable& tab, const Shape&, kvs_dtype, const void*, const void*, const int32_t*, const float*,
                              const float*, const uint8_t*, const int32_t*, void*, void*, int32_t*, hipStream_t) { check_table(tab); return ok(); }
hipError_t launch_per_query_norms(const UnitTable& tab, const Shape& sh, const void*, const void*, const void*, const int32_t*,
                                  const float*, float* o_part, uint16_t* o_hi, uint16_t*, float*, float*, float*, hipStream_t) {
  check_table(tab);
  long long rows = 0, longest = 1;
  for (int i = 0; i < tab.n_units; ++i) {
    const Unit u = tab.unit(i);
    rows += u.len;
    if (u.len < u.chunk_len ? u.len > longest : u.chunk_len > longest) longest = u.len < u.chunk_len ? u.len : u.chunk_len;
  }
  g_pieces = tab.total_chunks << pq_split(tab.n_units, tab.total_chunks, rows, longest, sh.R, sh.D);
  // the pieces' outputs, references, sums and weights' sums lie before what follows them in the workspace
  if ((long long)((char*)o_hi - (char*)o_part) < (long long)g_pieces * sh.R * (sh.D + 3) * (long long)sizeof(float)) __builtin_trap();
  return ok();
}
hipError_t launch_per_query_norms_f32(const UnitTable& tab, const Shape&, const void*, const void*, const void*, const int32_t*,
                                      const float*, float*, float*, float*, float*, hipStream_t) { check_table(tab); return ok(); }
hipError_t launch_decode(const UnitTable& tab, const Shape&, kvs_dtype, const void*, const void*, const void*, const int32_t*,
                         float*, float*, hipStream_t) { check_table(tab); return ok(); }

}  // namespace kvs
