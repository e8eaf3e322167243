// Internal declarations shared by the host layer and the gfx950 kernels of libkvs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kvs.h"
#include "kvs_debug.h"

namespace kvs {

// Current value of a testing switch (kvs_debug.h): one relaxed atomic load, no environment lookup.
int debug_switch(kvs_debug_switch which);

// Units of one launch ("group").  Up to kInlineUnits unit descriptors travel by value in the kernel arguments; a
// larger group (many short units: the streaming regime's caches of 2.5 K rows) hands its kernels the first two, where the
// others follow from them (units_regular), or has its descriptors written to the
// workspace first, by small kernels that carry them in THEIR arguments, kInlineUnits at a time.  A group takes
// kInlineUnits units whatever their lengths, and more as long as it has fewer than kGroupTokens tokens (64 units of
// 32 K tokens: longer launches gain nothing), up to kMaxGroupUnits units.
constexpr int kInlineUnits = 64;
constexpr int kMaxGroupUnits = 1024;
#ifndef KVS_GROUP_TOKENS
#define KVS_GROUP_TOKENS (64ll * 32768)
#endif
constexpr long long kGroupTokens = KVS_GROUP_TOKENS;
constexpr int kMaxChunks = 64;           // token chunks (= score workgroups) per unit
constexpr int kMinChunkLen = 256;        // tokens, but for launches of fewer workgroups than compute units
constexpr long long kTinyWorkgroups = 256;
constexpr int kMaxChunkLen = 2048;       // tokens that chunks aim for at most.  A chunk is up to a quarter longer to save a launch
                                         // a round of workgroups, and longer still where a unit has kMaxChunks of them: nothing
                                         // may be sized by this
constexpr int kMaxRoundChunkLen = 4096;  // tokens that chunks cut for whole rounds of workgroups are at most
constexpr int kScoreWorkgroups = 1024;   // score workgroups a launch aims for (4 per CU)
constexpr int kObarMinChunk = 1024;      // tokens per workgroup of the o_bar pass (at most kMaxChunks per unit)
#ifndef KVS_MERGE_TOKENS
#define KVS_MERGE_TOKENS 256
#endif
constexpr int kMergeTokens = KVS_MERGE_TOKENS;   // tokens per merge workgroup
constexpr int kWave = 64;
// K plus V bytes of one launch above which rows are streamed past the caches (256 MB of memory-side
// cache: below that, a sweep finds the rows its predecessor left there)
constexpr long long kStreamBytes = 192ll << 20;
// One-pass score kernel: bytes of K (bf16 rows) that one of its work items keeps in LDS between the statistics
// phase and the alpha_bar phase (one workgroup per CU: 128 KB of K + 16 KB of Q + tables of 160 KB)
constexpr int kFusedChunkBytes = 128 * 1024;

// One (sequence, KV head).  Rows are in elements of D, not bytes.
struct Unit {
  long long in_row;     // first row in K, V, alpha_bar, edge_mask, slot_of_token
  long long out_row;    // first row in K_out, V_out, counts_out
  int len;              // cached tokens
  int n_out;            // output rows: min(len, budget)
  int chunk_len;        // tokens per score chunk (multiple of 64)
  int n_chunks;         // ceil(len / chunk_len), <= kMaxChunks
  int chunk_base;       // chunks of the launch's earlier units
  int m_base;           // merge workgroups (kMergeTokens tokens each) of the launch's earlier units
  int index;            // position of the unit in the caller's problem (indexes Q, o_bar, partials)
  int o_base;           // o_bar-pass workgroups of the launch's earlier units
  int f_base;           // work items of the one-pass score kernel that belong to the launch's earlier units
  int s_base;           // select workgroups of the launch's earlier units (a unit has one, or several parts)
};

// Whether the descriptors of a group follow from the first two by equal steps: units of one length, budget and chunk length
// whose rows lie at equal distances (the heads of all layers of a model).  A group of more than kInlineUnits such units needs no
// launches that write descriptors: 256 caches of 2560 rows 224 -> 221 us per step, a decode step over 256 caches of 4096
// rows 112 -> 105.  (Smaller groups keep a table, see RegularTable: forming the descriptors is code to fetch and costs a
// per-layer step 2 us.)
inline bool units_regular(const Unit* u, int n) {
  if (n < 2) return false;
  const long long di = u[1].in_row - u[0].in_row, dout = u[1].out_row - u[0].out_row;
  for (int i = 1; i < n; ++i) {
    if (u[i].len != u[0].len || u[i].n_out != u[0].n_out || u[i].chunk_len != u[0].chunk_len ||
        u[i].in_row - u[i - 1].in_row != di || u[i].out_row - u[i - 1].out_row != dout) {
      return false;
    }
  }
  return true;
}

// Work items of the one-pass score kernel: chunks of kFusedChunkBytes of K rows (a function of D and the length).
__host__ __device__ inline int fused_chunk_len(int D) { return kFusedChunkBytes / (D * 2); }
__host__ __device__ inline int fused_chunks(int len, int D) {
  const int cl = fused_chunk_len(D);
  return (len + cl - 1) / cl;
}

// Chunking of the o_bar pass over V: a function of the unit's length only.
__host__ __device__ inline int obar_chunk_len(int len) {
  const int per = (len + kMaxChunks - 1) / kMaxChunks;
  const int rounded = (per + kWave - 1) / kWave * kWave;
  return rounded > kObarMinChunk ? rounded : kObarMinChunk;
}
__host__ __device__ inline int obar_chunks(int len) {
  const int cl = obar_chunk_len(len);
  return (len + cl - 1) / cl;
}

// Selection over several workgroups ("parts") per unit.  A part keeps at most kSelPartKeys edge scores in LDS; what
// the parts of a unit exchange goes through kSelSharedInts unsigned ints of device memory per unit of the launch,
// which must be zero when the select kernel starts (the score kernels of the same call clear them, sh.sel_exchange):
//   [kSelNotMin] ~(smallest key), [kSelMax] largest key, [kSelNCand] candidates listed so far,
//   [kSelArrive + phase] parts that finished a phase (bit kSelGaveUp: a part ran out of time there),
//   [kSelPartLow + part] keys of a part in the bins below the threshold's,
//   [kSelHist + bin] histogram of the first digit, [kSelCand + i] keys of the threshold's bin and
//   [kSelCandPart + i] the parts they came from.
constexpr int kSelThreads = 1024;         // threads of a select workgroup
constexpr int kSelRegSlices = 8;          // slices of 4096 keys that a select workgroup keeps in registers when two of them
constexpr int kSelMaxSlices = 16;         // share a CU, and at most
constexpr int kSelMaxParts = 32;
constexpr int kSelPartKeys = 8192;
constexpr int kSelMinPartKeys = 2048;     // parts are not made smaller than this unless a test asks for it
constexpr int kSelNotMin = 0, kSelMax = 1, kSelNCand = 2, kSelArrive = 4, kSelPhases = 3;
constexpr unsigned int kSelGaveUp = 1u << 16;
constexpr int kSelPartLow = 16;
constexpr int kSelHist = 64, kSelHistBins = 2048;
constexpr int kSelCand = kSelHist + kSelHistBins, kSelCandMax = 2048;
constexpr int kSelCandPart = kSelCand + kSelCandMax;
constexpr int kSelSharedInts = kSelCandPart + kSelCandMax;
static_assert(kSelPartLow + kSelMaxParts <= kSelHist && kSelSharedInts % 4 == 0, "layout of the exchange area");

template <int CAP>
struct UnitTableT {
  const Unit* ext;      // DEVICE: the descriptors of a group of more than kInlineUnits units, else null
                        // (first, beside n_units: a kernel's first scalar load then brings both)
  int n_units;
  int total_chunks;
  int total_mblocks;
  int total_ochunks;
  int total_fitems;     // work items of the one-pass score kernel
  int total_sparts;     // select workgroups
  int even;             // 1: every unit has the same number of chunks, merge workgroups, ... (see find_unit_by)
  int regular;          // HOST: more than kInlineUnits units, and regular ones (units_regular): kernels get a RegularTable
  const Unit* host;     // HOST: the same descriptors for the launchers (meaningless on the device), else null
  Unit u[CAP];          // the descriptors of a smaller group

  // Descriptor i, on either side.  On the device the external table is read through the constant address space:
  // the index is wavefront-uniform, so these are scalar loads like those of the kernel arguments.
  __host__ __device__ __forceinline__ Unit unit(int i) const {
#if defined(__HIP_DEVICE_COMPILE__)
    if (CAP == kInlineUnits && ext != nullptr) return ((const __attribute__((address_space(4))) Unit*)ext)[i];
    return u[i];
#else
    return host != nullptr ? host[i] : u[i];
#endif
  }
};
typedef UnitTableT<kInlineUnits> UnitTable;
// The table of a launch of few units.  64 descriptors are 3.6 KB of kernel arguments, which the host copies to where
// the GPU reads them at every launch: a launch of an empty kernel takes 4.0 to 6.7 us with them and 3.5 to 3.8 with
// 64 bytes, and a call on one layer is five such launches.  So kernels exist for the tables below (the table's type is
// a template argument), and launch_with_table picks the one a launch needs.
constexpr int kFewUnits = 8;
typedef UnitTableT<kFewUnits> FewUnitTable;
// The table of a group of more than kInlineUnits regular units: the first two descriptors stand for all.  A type of its own,
// since the arithmetic in the kernels for up to 64 units was code to fetch there (steps on 36 ragged units of 1000 to 2300
// tokens, 128 query rows 39.3 us with it and 37.7 without; 36 of 1500, 32 rows, head dim 64 28.0 and 27.2; 64 of 2000, 32
// rows 44.2 and 43.1) and the other 62 descriptors are arguments to copy here (per-query step on 100 units of 1100 130.3
// and 126.2).
struct RegularTable {
  static constexpr int even = 1;
  int n_units, total_chunks, total_mblocks, total_ochunks, total_fitems, total_sparts;
  Unit u[2];
  __device__ __forceinline__ Unit unit(int i) const {
    i = __builtin_amdgcn_readfirstlane(i);          // (uniform, but it may come from a vector register: scalar arithmetic)
    Unit x = u[0];
    x.in_row += i * (u[1].in_row - u[0].in_row);
    x.out_row += i * (u[1].out_row - u[0].out_row);
    x.chunk_base += i * (u[1].chunk_base - u[0].chunk_base);
    x.m_base += i * (u[1].m_base - u[0].m_base);
    x.index += i;
    x.o_base += i * (u[1].o_base - u[0].o_base);
    x.f_base += i * (u[1].f_base - u[0].f_base);
    x.s_base += i * (u[1].s_base - u[0].s_base);
    return x;
  }
};
template <typename T> struct TableTypeOf;
template <typename T> struct TableTypeOf<const T&> { typedef T type; };
// f(table): f launches a kernel with the table it is handed.
template <typename F>
inline void launch_with_table(const UnitTable& tab, F&& f) {
  if (tab.regular) {
    const RegularTable r = {tab.n_units, tab.total_chunks, tab.total_mblocks, tab.total_ochunks, tab.total_fitems,
                            tab.total_sparts, {tab.u[0], tab.u[1]}};
    f(r);
    return;
  }
  if (tab.n_units > kFewUnits) {
    f(tab);
    return;
  }
  FewUnitTable few;
  few.ext = nullptr;
  few.host = nullptr;
  few.n_units = tab.n_units;
  few.total_chunks = tab.total_chunks;
  few.total_mblocks = tab.total_mblocks;
  few.total_ochunks = tab.total_ochunks;
  few.total_fitems = tab.total_fitems;
  few.total_sparts = tab.total_sparts;
  few.even = tab.even;
  few.regular = 0;
  for (int i = 0; i < kFewUnits; ++i) few.u[i] = tab.u[i];
  f(few);
}
#define KVS_TABLE_TYPE(t) typename TableTypeOf<decltype(t)>::type

struct Shape {
  int R;            // query rows per unit (G*W)
  int D;            // head dim
  int n_sink;
  int n_recent;
  float scale_log2; // logit scale * log2(e): logits are kept in the base-2 domain
  int stream;       // 1: the launch's K and V exceed the last-level cache, rows are read non-temporally
  int ride;         // 1: the pass over V rides along in score sweep 1 where the kernel can carry it
  int rule;         // kvs_key_rule of the merged Key
  int sel_slices;   // the parts of units of more slices than this meet through the exchange area, see select_parts
  int sel_exchange; // 1: the launch has such a unit: the area must be zero when the select kernel starts
  int causal;       // 0, or the window W when query row q only sees the rows up to its own position n - W + q % W
  int keep_rows;    // 1: the caller reads the rows' normalisers (c_row) after the score phase
  int fold;         // 1: sweep 1 reduces the chunks' statistics itself (load_row_consts), no finalize kernel has run
  unsigned int* sel_clear;  // with fold: the exchange area of the selection that follows, which sweep 1 zeroes (per-query
                            // aggregation, with c_row_out: its kernels do)
  float* alpha_out; // per-query aggregation (bf16): where its kernels leave alpha_bar, or null where the score phase has left it
  float* c_row_out; // per-query aggregation (bf16): where its kernels leave the rows' normalisers, or null where the
                    // score phase has left them
  int dec_chunk;    // decode attention: rows per workgroup, at least (chosen per launch, see launch_decode)
  int o_from_score; // where the partial sums of o_bar are: 0: o_part, one per chunk of the o_bar pass; 1: o_part, one
                    // per SCORE chunk (written by sweep 1); 2: fo_part, one per work item of the one-pass score kernel
};

// Slices of 4 * kSelThreads keys of a unit with E eligible edges (with the padding to aligned groups of four).
__host__ __device__ inline int select_slices(int E) { return ((E + 6) / 4 + kSelThreads - 1) / kSelThreads; }
// Whether the parts of a unit's selection meet through the exchange area (or each goes over all its keys by itself).
__host__ __device__ inline bool select_exchanges(const Unit& un, const Shape& sh) {
  return select_slices((un.len - 2 - sh.n_recent) - sh.n_sink + 1) > sh.sel_slices;
}

// How many partials of o_bar a unit has, and where its partial c starts (index of its first float).
__host__ __device__ inline int obar_partials(const Shape& sh, const Unit& un) {
  return sh.o_from_score == 2 ? fused_chunks(un.len, sh.D) : sh.o_from_score == 1 ? un.n_chunks : obar_chunks(un.len);
}
__host__ __device__ inline size_t obar_partial_at(const Shape& sh, const Unit& un, int c) {
  return sh.o_from_score == 2 ? ((size_t)un.f_base + c) * sh.D : ((size_t)un.index * kMaxChunks + c) * sh.D;
}

// Workspace carve-up (all offsets multiples of 256 bytes).
struct Workspace {
  float2* stats_part;   // [n_units][kMaxChunks][R]  (running max, sum) of every chunk, base-2 domain
  float* c_row;         // [n_units][R]  unit-wide normaliser of every query row, see score_finalize_kernel
  float* o_part;        // [n_units][kMaxChunks][D]  partial o_bar of every chunk of the o_bar pass
  float* alpha_bar;     // [rows]    (kvs_step only)
  float* o_bar;         // [n_units][D] (kvs_step only)
  uint8_t* edge_mask;   // [rows]    (kvs_step only, when the caller keeps it internal)
  int32_t* slot;        // [rows]
  // one-pass score kernel (bf16, 65..128 query rows); sized for the largest launch group, null otherwise
  float* fstats;        // [work items][R]  log2 of the sum of 2^logit over the item's tokens, for every query row
  float* fo_part;       // [work items][D]  partial o_bar of every item
  unsigned int* fsync;  // kFusedSyncInts counters and flags, then one entry per work item (items given up on)
  unsigned int* sel_shared;  // [kInlineUnits][kSelSharedInts]  exchange area of the split selection (only groups of
                             // at most kInlineUnits units spread a unit's selection over workgroups)
  Unit* unit_tab;            // [kMaxGroupUnits]  descriptors of a group of more than kInlineUnits units
  size_t bytes;
};

// Layout of Workspace::fsync (unsigned ints).
constexpr int kFusedTicket = 0;                       // next work item
constexpr int kFusedDeferred = 32;                    // number of items handed to the second kernel
constexpr int kFusedDone = 64;                        // [kInlineUnits] items of the unit whose statistics are out
constexpr int kFusedSyncInts = 64 + kInlineUnits;     // the list of deferred items starts here
                                                      // (the one-pass kernel's groups have at most kInlineUnits units)
// A normaliser c_row[unit][q] that the one-pass kernel has not produced yet holds this bit pattern (a NaN that no
// arithmetic yields): the kernel's workgroups poll the words themselves, so no separate flag has to travel.
constexpr unsigned int kFusedNotYet = 0xffffffffu;

// Device helpers --------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// float -> bf16 bits, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return f32_to_bf16(lo) | (f32_to_bf16(hi) << 16);
}

// 16-byte row piece -> floats.  T = float: 4 values; T = bf16 (uint16_t): 8 values.
template <typename T> struct Piece;
template <> struct Piece<float> {
  static constexpr int N = 4;
  __device__ __forceinline__ static void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  __device__ __forceinline__ static uint4 pack(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
  }
};
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// two floats -> packed bf16 pair with the hardware converter (v_cvt_pk_bf16_f32, round to nearest even)
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  const f32x2_t f = {lo, hi};
  const bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
  return *reinterpret_cast<const uint32_t*>(&b);
}

template <> struct Piece<uint16_t> {
  static constexpr int N = 8;
  __device__ __forceinline__ static void unpack(const uint4& r, float* f) {
    f[0] = bf16_lo(r.x); f[1] = bf16_hi(r.x); f[2] = bf16_lo(r.y); f[3] = bf16_hi(r.y);
    f[4] = bf16_lo(r.z); f[5] = bf16_hi(r.z); f[6] = bf16_lo(r.w); f[7] = bf16_hi(r.w);
  }
  __device__ __forceinline__ static uint4 pack(const float* f) {
    return make_uint4(cvt_pk_bf16(f[0], f[1]), cvt_pk_bf16(f[2], f[3]), cvt_pk_bf16(f[4], f[5]), cvt_pk_bf16(f[6], f[7]));
  }
};

// Sum over the LPR (8, 16 or 32) adjacent lanes that share a row; every lane gets the total.
// gfx950 has no xor-by-4/8 DPP pattern, but once the four lanes of a quad agree, mirroring a
// half-row and then a row swaps exactly the partners a butterfly would.
template <int LPR>
__device__ __forceinline__ float row_group_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));  // row_half_mirror
  if (LPR >= 16)
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true));  // row_mirror
  if (LPR >= 32) x += __shfl_xor(x, 16, kWave);
  return x;
}

// Causal window: the last row that query row `qrow` of a unit with n rows attends to.
__device__ __forceinline__ int last_seen_row(int causal_w, int n, int qrow) {
  return causal_w > 0 ? n - causal_w + qrow % causal_w : 0x7fffffff;
}

// The launch's total of a running count.
template <int Unit::*BASE, typename Tab>
__host__ __device__ __forceinline__ int total_of(const Tab& tab) {
  if constexpr (BASE == &Unit::chunk_base) return tab.total_chunks;
  else if constexpr (BASE == &Unit::m_base) return tab.total_mblocks;
  else if constexpr (BASE == &Unit::o_base) return tab.total_ochunks;
  else if constexpr (BASE == &Unit::f_base) return tab.total_fitems;
  else return tab.total_sparts;
}

// The last unit whose running count BASE (chunks, merge workgroups, ... of the launch's earlier units) is at most x:
// the unit that work item x of the launch belongs to.  A division where all units have the same count (the heads of
// one layer); otherwise a binary search, because the table lives in the kernel arguments and every probe is a scalar
// load that the next one depends on (about a quarter of a microsecond when it misses the scalar cache: walking the
// table unit by unit cost a 64-unit select launch 15 of its 37 us).
template <int Unit::*BASE, typename Tab>
__device__ __forceinline__ int find_unit_by(const Tab& tab, int x) {
  if (tab.even) return x / (total_of<BASE>(tab) / tab.n_units);
  int lo = 0, hi = tab.n_units - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tab.unit(mid).*BASE <= x) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
// Which unit a workgroup of a chunk-indexed launch works on.
template <typename Tab>
__device__ __forceinline__ int find_unit(const Tab& tab, int chunk) {
  return find_unit_by<&Unit::chunk_base>(tab, chunk);
}

// log2 of a positive normal number, by way of its mantissa: the instruction rounds in proportion to its result, and not
// evenly, so that what it takes from a large logarithm doesn't cancel over the terms of a sum.
__device__ __forceinline__ float even_log2(float x) {
  return (float)__builtin_amdgcn_frexp_expf(x) + __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(x));
}
// A row's normaliser M + log2(s), rounded once: what the sum of M and the exponent loses joins the logarithm of the
// mantissa.  (With the instruction alone, 14 units of 20000 tokens and 224 rows: alpha_bar summed up to 1 + 3.2e-7 to
// 1 + 6.1e-7.)
__device__ __forceinline__ float plus_log2(float M, float s) {
  const float e = (float)__builtin_amdgcn_frexp_expf(s);
  const float hi = M + e, part = hi - M;
  const float lost = (M - (hi - part)) + (e - part);
  return hi + (lost + __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(s)));
}

// The sweep-1 kernels for up to 128 query rows (and the 256-row form of small launches) reduce the statistics of their
// unit themselves: a workgroup fetches them in one round trip of its prologue, which costs it less than a finalize
// kernel between the sweeps costs the call (one fp32 unit of 1024 tokens: 27.6 against 30.1 us per step; 8 units of 8192:
// 44.0 against 45.5; 8 of 32768, 64 chunks each: 85.0 against 86.6; 256 of 32768: 2069 against 2080).

// The normalisers c[q] of the unit's query rows q0 .. q0 + n - 1 -> sm_c (infinity for rows that do not exist:
// exp2(-inf) = 0), read from c_row or, with sh.fold, formed from the chunks' (max, sum) pairs: M_q + log2(Z_q * R), see
// score_finalize_kernel.  Two threads share a row, the chunks of each in flight together; fixed order.  Called by all
// THREADS threads of the workgroup; a barrier is inside, and another one has to follow before sm_c is read.
template <int THREADS>
__device__ __forceinline__ void load_row_consts(const Shape& sh, const Unit& un, int unit_pos, bool first_chunk,
                                                const float* __restrict__ c_row,
                                                const float2* __restrict__ stats_part, int q0, int n, float* sm_c) {
  const int R = sh.R;
  if (!sh.fold) {
    for (int i = threadIdx.x; i < n; i += THREADS)
      sm_c[i] = q0 + i < R ? c_row[(size_t)un.index * R + q0 + i] : INFINITY;
    return;
  }
  if (first_chunk && sh.sel_clear != nullptr && unit_pos < kInlineUnits) {
    uint4* z = reinterpret_cast<uint4*>(sh.sel_clear + (size_t)unit_pos * kSelSharedInts);
    for (int i = threadIdx.x; i < kSelSharedInts / 4; i += THREADS) z[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  constexpr int HALF = THREADS / 2, PER = kMaxChunks / 2;
  static_assert(PER % 8 == 0, "batches of eight loads");
  __shared__ float2 sm_second[HALF];
  const int h = (int)threadIdx.x / HALF, r = (int)threadIdx.x % HALF;
  for (int i0 = 0; i0 < n; i0 += HALF) {
    const int i = i0 + r, q = q0 + i;
    const bool ok = i < n && q < R;
    const float2* src = stats_part + (size_t)un.index * kMaxChunks * R + q;
    float2 v[PER];
#pragma unroll
    for (int k0 = 0; k0 < PER; k0 += 8) {                    // (uniform: a unit of few chunks is spared the rest)
#pragma unroll
      for (int k = k0; k < k0 + 8; ++k) v[k] = make_float2(-INFINITY, 0.f);
      if (2 * k0 < un.n_chunks) {
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k) {
          if (ok && 2 * k + h < un.n_chunks) v[k] = src[(size_t)(2 * k + h) * R];
        }
      }
    }
    float M = -INFINITY, Z = 0.f;
#pragma unroll
    for (int k = 0; k < PER; ++k) M = fmaxf(M, v[k].x);
#pragma unroll
    for (int k0 = 0; k0 < PER; k0 += 8) {
      if (2 * k0 < un.n_chunks) {
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k) {
          if (v[k].y > 0.f) Z += v[k].y * __builtin_amdgcn_exp2f(v[k].x - M);
        }
      }
    }
    if (h == 1) sm_second[r] = make_float2(M, Z);
    __syncthreads();
    if (h == 0 && i < n) {
      const float2 b = sm_second[r];
      const float Mq = fmaxf(M, b.x);
      float Zq = Z * __builtin_amdgcn_exp2f(M - Mq);
      if (b.y > 0.f) Zq += b.y * __builtin_amdgcn_exp2f(b.x - Mq);
      sm_c[i] = ok ? plus_log2(Mq, Zq * (float)R) : INFINITY;
    }
    if (i0 + HALF < n) __syncthreads();
  }
}

// bf16 launches of 129 to 192 rows whose two score sweeps are the wide kernel's form with eight wavefronts, one workgroup per
// compute unit, whatever their number (the reasons stand where the kernel is chosen).
inline bool score_rows_in_one_workgroup(int R, int D, bool stream, bool counts) {
  return R > 128 && R <= 192 && !counts && (D == 64 || stream);
}

// Launchers (defined next to their kernels).  All enqueue on `stream` and return the launch status.
// The descriptors of a group of more than kInlineUnits units (host memory) into the workspace, by kernels that
// carry them in their arguments; nothing where they are regular (UnitTableT::regular: nobody reads them there).
hipError_t launch_unit_table(const Unit* units, int n_units, Unit* dst, hipStream_t stream);
// Unit-wide softmax statistics from the chunks' partial ones (one small workgroup per unit).
// (it also zeroes ws.sel_shared for the selection that follows, when there is one)
hipError_t launch_score_finalize(const UnitTable& tab, const Shape& sh, const Workspace& ws, hipStream_t stream);
// Between the sweeps of a launcher whose sweep-1 kernel calls load_row_consts: nothing, sweep 1 does the finalize kernel's
// work (sh.fold), or that kernel, for callers that read the normalisers themselves.
inline hipError_t between_sweeps(const UnitTable& tab, Shape& sh, const Workspace& ws, const float* alpha_bar,
                                 hipStream_t stream) {
  if (alpha_bar == nullptr || sh.keep_rows) return launch_score_finalize(tab, sh, ws, stream);
  sh.fold = 1;
  sh.sel_clear = sh.sel_exchange ? ws.sel_shared : nullptr;
  return hipSuccess;
}
// Both score sweeps: chunk statistics, the finalize kernel where sweep 1 does not do its work, then alpha_bar (null: the
// first sweep and the finalize kernel only).
// counts_in (here and below): cardinalities of the input rows when the cache is already a merged one, or null.
// V non-null: the caller also needs o_bar; where the score kernel can carry the pass over V along, it does,
// leaves the partial sums in the workspace and sets *o_layout to where they are (a value for Shape::o_from_score
// other than 0: the caller then skips the separate pass and tells the consumers).
hipError_t launch_score(const UnitTable& tab, const Shape& sh, kvs_dtype dt, const void* Q, const void* K,
                        const int32_t* counts_in, float* alpha_bar, const Workspace& ws, hipStream_t stream,
                        const void* V = nullptr, int* o_layout = nullptr);
// One launch, several kinds of workgroups: the first `with_select ? tab.total_sparts : 0` select edges (one workgroup
// per unit, or several parts per unit that meet through sel_shared), the others stream one chunk of V each into
// o_part (skipped when V is null).
// A third kind (o_bar_out non-null, one workgroup per unit) adds up the partial sums that a score kernel left
// (sh.o_from_score says where) into o_bar_out[unit][D].
// sel_shared: the zeroed exchange area (see kSelSharedInts), needed when any unit has more than one part.
hipError_t launch_select_obar(const UnitTable& tab, const Shape& sh, kvs_dtype dt, bool with_select,
                              const float* alpha_bar, uint8_t* edge_mask, int32_t* slot, const void* V,
                              const int32_t* counts_in, float* o_part, hipStream_t stream,
                              const float* parts_in = nullptr, float* o_bar_out = nullptr,
                              unsigned int* sel_shared = nullptr);
// Zeroes the exchange area of the launch's units (callers that did not run the score kernels before the selection).
hipError_t launch_select_clear(const UnitTable& tab, unsigned int* sel_shared, hipStream_t stream);
// How many select workgroups a unit gets in a launch of n_units units on a chip of n_cus compute units
// (mode: the KVS_DEBUG_SELECT_SPLIT switch; sh.sel_slices is set; beside_values: beside a pass over V).
int select_parts(const Unit& un, const Shape& sh, int n_units, int n_cus, int mode, bool beside_values);
// o_bar[u] = sum of the unit's partial sums, in chunk order (only when o_bar itself is an output).
hipError_t launch_obar_reduce(const UnitTable& tab, const Shape& sh, const float* parts, float* o_bar,
                              hipStream_t stream);
// The two sweeps (and the finalize kernel) for bf16 windows of more than 128 rows (kvs_score_shared.hip).
hipError_t launch_score_shared(const UnitTable& tab, const Shape& sh, const void* Q, const void* K,
                               const int32_t* counts_in, float* alpha_bar, const Workspace& ws, const void* V,
                               hipStream_t stream);
// The same for fp32 windows of more than 64 rows (kvs_score_split.hip).
hipError_t launch_score_split(const UnitTable& tab, const Shape& sh, const void* Q, const void* K,
                              const int32_t* counts_in, float* alpha_bar, const Workspace& ws, hipStream_t stream);
// One-pass score for bf16 windows of 65..128 rows (kvs_score_fused.hip): K is read once and kept in LDS between
// the statistics and the alpha_bar phase; the pass over V rides along (partials in ws.fo_part).
bool score_fused_supported(const UnitTable& tab, const Shape& sh, kvs_dtype dt);
hipError_t launch_score_fused(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                              const int32_t* counts_in, float* alpha_bar, const Workspace& ws, hipStream_t stream);
// Exactly one of o_bar (final values) and o_part (chunk sums, added up by every workgroup) is non-null.
hipError_t launch_merge(const UnitTable& tab, const Shape& sh, kvs_dtype dt, const void* K, const void* V,
                        const int32_t* counts_in, const float* alpha_bar, const float* o_bar, const float* o_part,
                        const uint8_t* edge_mask,
                        const int32_t* slot, void* K_out, void* V_out, int32_t* counts, hipStream_t stream);

// The same pass with A_t and C_t read from arrays instead of formed from alpha_bar and o_bar (per-query aggregation).
hipError_t launch_merge_norms(const UnitTable& tab, const Shape& sh, kvs_dtype dt, const void* K, const void* V,
                              const int32_t* counts_in, const float* a_tok, const float* c_edge,
                              const uint8_t* edge_mask, const int32_t* slot, void* K_out, void* V_out, int32_t* counts,
                              hipStream_t stream);
// Workgroups per score chunk of the per-query kernels (bf16) are 2^pq_split (a workgroup of pq_out leaves one partial
// output, so the workspace is sized by this too).  rows, longest: rows of the launch and of its longest chunk.
//
// A launch of few chunks cuts them, as long as all pieces still run at once: two workgroups on each of the 256 CUs, or
// one where more than 64 rows of 128 channels keep a workgroup busy enough and what it does once for its piece costs
// more (14 ragged units, 60000 rows, 256 query rows, 241 chunks: 136 us uncut, 173 in four; 8 units of 8192, 256 chunks,
// 128 query rows, head dim 64: 69.2 in two, 71.6 uncut).  And a launch whose chunks are of different lengths, or too few,
// because a unit has at most 64, cuts them as long as the longest piece is a larger share of the rows than that (3 ragged
// units, 255000 rows, 128 query rows, 188 chunks: 187 us in two, 250 uncut; 14 units, where all chunks are as long: 191
// against 175): not below 128 rows, and into at most kMaxPqPieces.
// No second workgroup for pieces below 64 rows (8 of 2048, 64 query rows: 256 pieces of 64 46.8 us, 512 of 32 50.6; 4 of 4000 44.2
// and 48.8; head dim 64, 128 rows, 8 of 2048 45.8 and 49.5).
// Up to 32 rows the four wavefronts take tiles of their own, and a piece costs its combination of their sums: no second
// workgroup on a CU (8 units of 8192, 256 chunks: 50.4 us uncut, 59.0 in two, with pq_out_kernel 61.2; 2 of 30000, 118 chunks:
// 58.5 in two, 65.4 in four) and no pieces below 64 rows (8 of 2048, 128 chunks of 128: 39.3 in two, 41.0 uncut, 47.7 in four).
constexpr int kMaxPqPieces = 1024;
constexpr int kMaxPqSplit = 3;
// Small launches of 9 to 32 rows of 128 channels keep pq_out_kernel, whose workgroups have no sums of four wavefronts to add up,
// and its pieces down to a tile (with pq_out_narrow_kernel and pieces of 64, us: 32 rows, one unit of 800 35.7, so 34.1, 4 of 1000
// 38.1 and 36.7, 8 of 1000 40.9 and 40.2; 16 rows, one of 800 32.1 and 31.2; one of 6000 40.3 and 40.8, 8 of 1900 40.5 and 40.2
// with pieces of 64, so neither longer units nor larger launches).
constexpr int kPqNarrowRows = 32;         // up to here a tile takes one wavefront of the per-query kernels (bf16)
inline bool pq_small(long long units, long long rows, int R, int D) {
  return D == 128 && R > 8 && R <= kPqNarrowRows && rows <= 8192 && rows <= 3500 * units;
}
inline int pq_split(long long units, long long chunks, long long rows, long long longest, int R, int D) {
  const bool narrow = R <= kPqNarrowRows && !pq_small(units, rows, R, D), light = !narrow && (R <= 64 || D == 64);
  int split = 0;
  while (split < kMaxPqSplit) {
    const long long pieces = chunks << (split + 1);
    const bool few = pieces <= (light && (longest >> (split + 1)) >= 64 ? 512 : 256);
    const bool uneven = (longest >> split) * (light || narrow ? 320 : 240) > rows && (longest >> split) > 256;
    if ((longest >> (split + 1)) < (narrow ? 64 : 32)) break;               // (a tile's rows)
    if (!few && !(uneven && pieces <= kMaxPqPieces)) break;
    ++split;
  }
  return split;
}
// Per-query aggregation (bf16, every unit at least 32 rows): a_tok, c_edge and alpha_bar (sh.alpha_out, if set) from Q, K, V
// and, unless they leave them in sh.c_row_out (the same array) themselves, the rows' normalisers c_row.  o_part: [pieces of
// the launch's chunks][R][D] fp32, then references and sums [pieces][R] float2, then weights' sums [pieces][R]; o_hi, o_lo: [n_units][R][D] bf16; oo: [n_units][R].
hipError_t launch_per_query_norms(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                                  const int32_t* counts_in, const float* c_row, float* o_part, uint16_t* o_hi,
                                  uint16_t* o_lo, float* oo, float* a_tok, float* c_edge, hipStream_t stream);
// The same for fp32 inputs (any unit length, vector ALU).  o: [n_units][R][D] fp32.
hipError_t launch_per_query_norms_f32(const UnitTable& tab, const Shape& sh, const void* Q, const void* K,
                                      const void* V, const int32_t* counts_in, const float* c_row, float* o_part,
                                      float* o, float* a_tok, float* c_edge, hipStream_t stream);

// Decode attention over a (merged) cache: chunk partials into `part`, then out[n_units, R, D].
hipError_t launch_decode(const UnitTable& tab, const Shape& sh, kvs_dtype dt, const void* Q, const void* K,
                         const void* V, const int32_t* counts, float* part, float* out, hipStream_t stream);

}  // namespace kvs
