// Per-query aggregation of the sensitivity norms (bf16 inputs).
//
// Sec. 4 derives the forward-only vectors c_tt = alpha_t (1 - 2 alpha_t)(v_t - o) and
// c_{t,t+1} = -alpha_t alpha_{t+1} (v_t + v_{t+1} - 2o) (Eqs. c11_def-c12_def) for ONE query.  Here every
// query row q of the window keeps its own attention alpha^{(q)} and its own output o^{(q)} (Eq.
// attn_def_vec), and the NORMS are averaged over the R rows:
//   A_t = (1/R) sum_q alpha_t^{(q)} |1 - 2 alpha_t^{(q)}| ||v_t - o^{(q)}||
//   C_t = (1/R) sum_q alpha_t^{(q)} alpha_{t+1}^{(q)} ||v_t + v_{t+1} - 2 o^{(q)}||
// The merge kernel then uses A and C in the weight form of Eq. kstar_final.
//
// Three kernels, without a score sweep before them.  (With cardinalities the first sweep runs and leaves the rows' normalisers:
// those are then numbers from 20 to 40, whose rounding is most of the error of alpha_bar, and the kernels' own would
// round differently from kvs_score's: 3.4e-7 in the root mean square for cardinalities up to 1e7.  Windows of one to three
// rows run both sweeps and have alpha_bar from them.)
//   pq_out_kernel         O^T[d, q] = sum_t V[t, d] P[t, q], P = 2^(logit - reference) from K Q^T tile by tile, every piece
//                         of a chunk with a reference of its own for every row (see kSumLimit), which rises now and then.
//                         Both products run on v_mfma_f32_32x32x16_bf16.  The contraction over tokens needs
//                         V with the token index along the MFMA k dimension; a 32x32 block of the V tile is
//                         turned by one more MFMA against an identity operand (exact in bf16), which leaves it
//                         in the accumulator layout that IS the k-major operand layout of the next product
//                         (one block per wavefront, shared through LDS).
//                         P enters as a bf16 pair hi + lo, so that the rounding of P to bf16 does not limit
//                         the accuracy of o; the sum of the weights, as the pairs carry them, is kept beside it.
//                         The pieces' partials go to memory, with the references and the sums of the terms.
//   pq_out_reduce_kernel  the rows' normalisers, and o^{(q)} = (sum of the partials) / (sum of their weights), each
//                         brought to a common reference and added in the order of the chunks: a convex combination of the
//                         Values with the weights as they were rounded, so that where a row puts nearly all its
//                         weight on one token, o - v_t is as accurate as the small weights of the others (dividing
//                         by the nominal sum 1 / R would leave the weights' rounding times ||v_t||).
//                         -2 o^{(q)} stored as a bf16 pair hi + lo, and ||o^{(q)}||^2.
//   pq_norms_kernel       per tile of 32 tokens: S' = Q K^T (logits), X' = (-2 O) V^T (hi and lo, accumulated on top of
//                         ||o||^2), then per (t, q)
//                         ||v_t - o||^2 = ||v_t||^2 + X',
//                         ||v_t + v_{t+1} - 2o||^2 = ||v_t + v_{t+1}||^2 + 2 (X'_t + X'_{t+1}),
//                         two square roots, and the sums over q.  Tiles overlap by one row (stride 31), so
//                         the next token of every output row is in the same tile.  Tokens where the expansions
//                         cancel (o^{(q)} close to v_t for some q) are marked, and done once more at the end, every
//                         squared norm as a sum of squared differences (redo_marked).  The sum of alpha^{(q)}_t over q is
//                         alpha_bar: one addition per (t, q) here instead of a sweep of its own (16.6 us for 8 units
//                         of 32768 tokens and 128 rows).
// COUNTS: the rows are slots of an already merged cache (Sec. 3.1, streaming regime), row t standing for c_t tokens
// whose Values add up to V[t]: every query row sees it as one token with logit e + ln c_t and value V[t] / c_t.  The
// products still run on the stored rows; c_t multiplies the term in the sums over a row (a logarithm in the exponent would
// round with its size), the weight of the Value SUM is the term of ONE token, and 1 / c_t scales
// the product V_t . o and the squared norms afterwards.
// A workgroup has four wavefronts; but for the narrow kernels' few query rows wavefront w owns query rows 32w .. 32w+31 of a pass of 128
// rows and keeps their operands in registers; all four walk the same K and V tiles, staged through LDS (XOR-swizzled
// 16-byte pieces, as in the score kernels).  Results do not depend on timing: no atomics, fixed orders.
#include <algorithm>
#include <type_traits>

#include "kvs_mfma_tile.h"

namespace kvs {
namespace {

using namespace mfma;                     // bf16x8, f32x16, kTile, ex2, kHeadroom, kSumLimit, add_compensated

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kPassRows = 32 * kWaves;    // query rows per pass over the chunk
constexpr int kRedoSpan = 1024;           // redo_marked: tokens of a call
constexpr float kCancel = 1.f / 16.f;     // pq_norms: a squared norm below this share of its leading term is formed again

// (one instruction; written out because the compiler forms it from nested fminf only now and then)
__device__ __forceinline__ float min3(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// c + a.lo * b.lo + a.hi * b.hi for two packed bf16 pairs (v_dot2c_f32_bf16)
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& u) { return __builtin_bit_cast(bf16x8, u); }

// eight floats -> bf16 operand (round to nearest even)
__device__ __forceinline__ bf16x8 pack8(const float* f) {
  return as_bf16x8(make_uint4(cvt_pk_bf16(f[0], f[1]), cvt_pk_bf16(f[2], f[3]), cvt_pk_bf16(f[4], f[5]),
                              cvt_pk_bf16(f[6], f[7])));
}
// eight floats -> hi + lo: hi = bf16(f), lo = bf16(f - hi)
__device__ __forceinline__ void split8(const float* f, bf16x8& hi, bf16x8& lo) {
  uint32_t h[4];
  float r[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = cvt_pk_bf16(f[2 * i], f[2 * i + 1]);
    r[2 * i] = f[2 * i] - bf16_lo(h[i]);
    r[2 * i + 1] = f[2 * i + 1] - bf16_hi(h[i]);
  }
  hi = as_bf16x8(make_uint4(h[0], h[1], h[2], h[3]));
  lo = pack8(r);
}

// The same, and w[i] = the value the pair stands for (hi + lo as floats).
__device__ __forceinline__ void split8w(const float* f, bf16x8& hi, bf16x8& lo, float* w) {
  uint32_t h[4], l[4];
  float r[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = cvt_pk_bf16(f[2 * i], f[2 * i + 1]);
    r[2 * i] = f[2 * i] - bf16_lo(h[i]);
    r[2 * i + 1] = f[2 * i + 1] - bf16_hi(h[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    l[i] = cvt_pk_bf16(r[2 * i], r[2 * i + 1]);
    w[2 * i] = bf16_lo(h[i]) + bf16_lo(l[i]);
    w[2 * i + 1] = bf16_hi(h[i]) + bf16_hi(l[i]);
  }
  hi = as_bf16x8(make_uint4(h[0], h[1], h[2], h[3]));
  lo = as_bf16x8(make_uint4(l[0], l[1], l[2], l[3]));
}

// The tokens of workgroup b: piece b % 2^split of its chunk, a multiple of 32 tokens long (the last one: what is left).
__device__ __forceinline__ void piece_range(const Unit& un, int b, int split, int& t0, int& t1) {
  const int c0 = ((b >> split) - un.chunk_base) * un.chunk_len;
  const int c1 = min(un.len, c0 + un.chunk_len);
  const int per = ((un.chunk_len >> split) + kTile - 1) / kTile * kTile;
  t0 = min(c1, c0 + (b & ((1 << split) - 1)) * per);
  t1 = min(c1, t0 + per);
}

// A 32-row tile of K or V: global -> registers -> LDS.  Piece p of row r lands in slot p ^ (r % LPR).
template <int D>
struct Tile {
  static constexpr int LPR = D / 8;                       // 16-byte pieces per row
  static constexpr int ROWB = D * 2;
  static constexpr int BYTES = kTile * ROWB;
  static constexpr int NP = kTile * LPR / kThreads;       // pieces per thread: 1 or 2
  // (two named registers instead of an array: an array handed on by reference across the loop stayed in
  // scratch memory, with a wait after every load)
  struct Regs { uint4 a, b; };
  __device__ __forceinline__ static Regs load(const unsigned char* tile_base, int tid) {
    Regs r;
    r.a = *reinterpret_cast<const uint4*>(tile_base + (size_t)tid * 16);
    r.b = (NP > 1) ? *reinterpret_cast<const uint4*>(tile_base + (size_t)(tid + kThreads) * 16) : make_uint4(0, 0, 0, 0);
    return r;
  }
  __device__ __forceinline__ static void store_piece(unsigned char* sm, const uint4& x, int pi) {
    const int row = pi / LPR, piece = pi % LPR;
    *reinterpret_cast<uint4*>(sm + row * ROWB + ((piece ^ (row % LPR)) * 16)) = x;
  }
  __device__ __forceinline__ static void store(unsigned char* sm, const Regs& r, int tid) {
    store_piece(sm, r.a, tid);
    if (NP > 1) store_piece(sm, r.b, tid + kThreads);
  }
  // MFMA operand of k-step kk for this lane: row `row`, elements 16 kk + 8 half .. + 7
  __device__ __forceinline__ static bf16x8 operand(const unsigned char* sm, int row, int kk, int half) {
    const int piece = 2 * kk + half;
    return *reinterpret_cast<const bf16x8*>(sm + row * ROWB + ((piece ^ (row % LPR)) * 16));
  }
  __device__ __forceinline__ static uint4 piece_at(const unsigned char* sm, int row, int piece) {
    return *reinterpret_cast<const uint4*>(sm + row * ROWB + ((piece ^ (row % LPR)) * 16));
  }
};

// Operand of k-step kk from a row-major [rows, D] bf16 matrix in memory (zero for a row that does not exist).
template <int D>
__device__ __forceinline__ bf16x8 row_operand(const uint16_t* __restrict__ m, int row, bool ok, int kk, int half) {
  uint4 raw = make_uint4(0, 0, 0, 0);
  if (ok) raw = *reinterpret_cast<const uint4*>(m + (size_t)row * D + kk * 16 + 8 * half);
  return as_bf16x8(raw);
}

// ------------------------------------------------------------------------------------------------
// o_part[(piece of the launch), q, :] = sum over the piece's tokens of 2^(logit - reference) V[t], p_part the sum of those
// weights.  The reference: the row's normaliser where c_row is given (the weights are then alpha^{(q)}_t / R, with
// cardinalities that of one of the c tokens); else the piece's own, which goes to stat_part with the sum of the terms.
// Two workgroups per CU: the 64 accumulator registers of O^T and the 32 of the Q operands leave no room for a
// third wavefront per SIMD (at 168 registers the compiler spills inside the tile loop).
#ifndef KVS_PQ_OUT_OCC
#define KVS_PQ_OUT_OCC 2
#endif
template <int D, bool COUNTS, typename Tab>
__global__ __launch_bounds__(kThreads, KVS_PQ_OUT_OCC) void pq_out_kernel(
    const Tab tab, const Shape sh, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const int32_t* __restrict__ counts_in, const float* __restrict__ c_row,
    float* __restrict__ o_part, float* __restrict__ p_part, float2* __restrict__ stat_part, const int split) {
  typedef Tile<D> TL;
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;                // 32-wide blocks of the value dimension
  __shared__ __attribute__((aligned(16))) unsigned char sm_k[2][TL::BYTES];
  __shared__ __attribute__((aligned(16))) unsigned char sm_v[2][TL::BYTES];
  __shared__ __attribute__((aligned(16))) float sm_cc[2][kTile];                    // COUNTS: the rows' cardinalities
  __shared__ uint4 sm_vt[2][DB][2][kWave];   // the V tile's blocks turned token-major: two operands per lane and block

  const int ui = find_unit(tab, (int)blockIdx.x >> split);
  const Unit un = tab.unit(ui);
  int t0, t1;
  piece_range(un, blockIdx.x, split, t0, t1);
  const int ntiles = (t1 - t0 + kTile - 1) / kTile;          // (a piece may be empty: it leaves zeros)
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int R = sh.R;
  const float sl2 = sh.scale_log2;
  const unsigned char* Kg = reinterpret_cast<const unsigned char*>(K + (size_t)un.in_row * D);
  const unsigned char* Vg = reinterpret_cast<const unsigned char*>(V + (size_t)un.in_row * D);
  const uint16_t* Qu = Q + (size_t)un.index * R * D;
  const int32_t* cnt = COUNTS ? counts_in + un.in_row : nullptr;

  // identity operand: element i of k-step kk is 1 where 16 kk + 8 half + i is this lane's column
  bf16x8 ident[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k0 = 16 * kk + 8 * half + 2 * i;
      w[i] = (k0 == col ? 0x3F80u : 0u) | (k0 + 1 == col ? 0x3F800000u : 0u);
    }
    ident[kk] = as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
  }
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // a tile always holds 32 whole rows: the ragged last one is moved back to end at the chunk's end and the
  // rows it shares with the tile before are skipped (every unit on this path has at least 32 rows)
  // (t1 is at least 32, also that of an empty piece)
  auto tile_base = [&](int j) { return min(t0 + j * kTile, t1 - kTile); };

  for (int qp = 0; qp < R; qp += kPassRows) {
    const int qrow = qp + 32 * wave + col;
    const bool ok = qrow < R;
    bf16x8 bq[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) bq[kk] = row_operand<D>(Qu, qrow, ok, kk, half);
    // reference of the row's exponents: its normaliser (always with cardinalities), or one of this piece's own
    // (exp2(-inf) = 0: no such row)
    float m_run = !ok ? INFINITY : c_row != nullptr ? c_row[(size_t)un.index * R + qrow] : -INFINITY;
    float z = 0.f, z_lost = 0.f;            // sum of the row's terms (only against a reference of its own)
    const int lim = last_seen_row(sh.causal, un.len, qrow);               // causal window: last row attended to
    f32x16 accO[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) accO[db] = zero;
    float wsum = 0.f;                       // the same sum over this lane's token rows, as the pairs hi + lo carry it

    typename TL::Regs rk = TL::load(Kg + (size_t)tile_base(0) * TL::ROWB, tid);
    typename TL::Regs rv = TL::load(Vg + (size_t)tile_base(0) * TL::ROWB, tid);
    for (int j = 0; j < ntiles; ++j) {
      const int buf = j & 1;
      TL::store(sm_k[buf], rk, tid);
      TL::store(sm_v[buf], rv, tid);
      if (COUNTS && tid < kTile) {
        sm_cc[buf][tid] = (float)cnt[tile_base(j) + tid];
      }
      __syncthreads();
      const int shift = t0 + j * kTile - tile_base(j);       // leading rows that belong to the tile before
      {                                     // the next tile flies during this one (the last one is fetched twice)
        const int jn = min(j + 1, ntiles - 1);
        rk = TL::load(Kg + (size_t)tile_base(jn) * TL::ROWB, tid);
        rv = TL::load(Vg + (size_t)tile_base(jn) * TL::ROWB, tid);
        asm volatile("" ::: "memory");        // issue them here: sunk below the products they would be waited for at once
      }
      // The block V[tile rows, 32 w .. 32 w + 31] into the token-major operand layout, by wavefront w for all four
      // (every wavefront turning all blocks itself costs six more MFMAs and 48 conversions per tile and wavefront):
      // one product against the identity (exact: the values are bf16 numbers) leaves it in the accumulator layout,
      // which is the k-major operand layout of the product with P below.
      if (wave < DB) {
        f32x16 y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::operand(sm_v[buf], col, 2 * wave, half), ident[0], zero, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::operand(sm_v[buf], col, 2 * wave + 1, half), ident[1], y, 0, 0, 0);
        float yf[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) yf[v] = y[v];
        sm_vt[buf][wave][0][lane] = __builtin_bit_cast(uint4, pack8(yf));
        sm_vt[buf][wave][1][lane] = __builtin_bit_cast(uint4, pack8(yf + 8));
      }
      // logits of the tile against this wavefront's 32 query rows
      f32x16 acc = zero;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::operand(sm_k[buf], col, kk, half), bq[kk], acc, 0, 0, 0);
      // accumulator element v: token row 8 (v / 4) + 4 half + v % 4, query column `col`.  The weight of a row's Values is
      // 2^(logit - reference), also where they are the sum over c tokens (c equal terms, each of V / c).
      float p[16];
      // rows of the tile before (a moved-back last tile) and rows behind the causal window's limit drop out;
      // both are rare and uniform per tile, so the common tile carries no per-element test
      const bool masked = shift > 0 || (sh.causal > 0 && tile_base(j) + kTile > un.len - sh.causal + 1);
      auto seen = [&](int v) {
        const int row = 8 * (v / 4) + 4 * half + (v % 4);
        return row >= shift && tile_base(j) + row <= lim;
      };
      auto terms = [&](float m) {           // the tile's terms against reference m; returns their sum
#pragma unroll
        for (int v = 0; v < 16; ++v) p[v] = ex2(fmaf(acc[v], sl2, -m));
        if (masked) {
#pragma unroll
          for (int v = 0; v < 16; ++v) p[v] = seen(v) ? p[v] : 0.f;
        }
        float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 16; ++v) s4[v % 4] += p[v];
        return (s4[0] + s4[1]) + (s4[2] + s4[3]);
      };
      float ts = terms(m_run);
      // A sum that is not below the limit (the first tile's, whose reference is minus infinity, among them): the
      // reference rises to the tile's largest logit and the headroom, in both halves of the wavefront alike, and what
      // has been added up is brought to it (see kSumLimit).  Never against a finished normaliser.
      if (!COUNTS && c_row == nullptr && __any(!(ts < kSumLimit))) {
        float tm = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) tm = fmaxf(tm, !masked || seen(v) ? acc[v] : -INFINITY);
        tm = fmaxf(tm, __shfl_xor(tm, 32, kWave));
        const float m_new = fmaxf(m_run, fmaf(tm, sl2, kHeadroom));
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;
        const float down = m_run == m_new ? 1.f : ex2(m_run - m_safe);
#pragma unroll
        for (int db = 0; db < DB; ++db) accO[db] *= down;
        wsum *= down;
        z *= down;
        z_lost *= down;
        m_run = m_new;
        ts = terms(m_safe);
      }
      add_compensated(z, z_lost, ts);
      // as the operand of the next product, element i of k-step s is accumulator element 8 s + i
      bf16x8 ph[2], pl[2];
      float pw[16];
      split8w(p, ph[0], pl[0], pw);
      split8w(p + 8, ph[1], pl[1], pw + 8);
      if (COUNTS) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 cc = *reinterpret_cast<const float4*>(&sm_cc[buf][8 * g + 4 * half]);
          wsum = fmaf(pw[4 * g], cc.x, wsum);
          wsum = fmaf(pw[4 * g + 1], cc.y, wsum);
          wsum = fmaf(pw[4 * g + 2], cc.z, wsum);
          wsum = fmaf(pw[4 * g + 3], cc.w, wsum);
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) wsum += pw[v];
      }
      __syncthreads();                      // the turned blocks are in place
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 vt0 = as_bf16x8(sm_vt[buf][db][0][lane]), vt1 = as_bf16x8(sm_vt[buf][db][1][lane]);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt0, ph[0], accO[db], 0, 0, 0);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt1, ph[1], accO[db], 0, 0, 0);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt0, pl[0], accO[db], 0, 0, 0);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt1, pl[1], accO[db], 0, 0, 0);
      }
    }
    __syncthreads();                        // the next pass starts with buffer 0 again
    wsum += __shfl_xor(wsum, 32, kWave);    // the other half's token rows
    z -= z_lost;
    z += __shfl_xor(z, 32, kWave);
    if (ok && half == 0) {
      p_part[(size_t)blockIdx.x * R + qrow] = wsum;
      if (c_row == nullptr) stat_part[(size_t)blockIdx.x * R + qrow] = make_float2(m_run, z);
    }
    if (ok) {
      float* dst = o_part + ((size_t)blockIdx.x * R + qrow) * D;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 o4 = make_float4(accO[db][4 * g], accO[db][4 * g + 1], accO[db][4 * g + 2], accO[db][4 * g + 3]);
          *reinterpret_cast<float4*>(dst + 32 * db + 8 * g + 4 * half) = o4;
        }
      }
    }
  }
}

// The same for few query rows: the kernel above gives every wavefront 32 rows of its own, so with up to 32 three of four would
// multiply rows that don't exist.  Here a tile takes RB wavefronts, one per block of 32 rows, and the workgroup's 4 / RB teams
// take the piece's tiles in turn, every wavefront with its operands straight from memory (nothing is shared, so nothing goes through LDS and nothing waits for a barrier), and
// add their sums up at the end, in wavefront order, each brought to the largest of their references.
// The registers of the K and V operands are refilled for the wavefront's next tile as soon as they have been multiplied.
// Bound by memory where there are many pieces, else by the wavefronts' chains.  Steps, before -> with both narrow kernels (us):
// 32 rows, 100 units of 21000 tokens 902 -> 749 (two passes over K and V and the merge of it at 5 TB/s: 680), 8 of 32768
// 127 -> 108, 8 of 8192 61 -> 50 (see pq_split); head dim 64, 12 of 29384 130 -> 88; 16 rows and cardinalities, 40 of 20000 510 -> 343;
// 7 rows, 128 ragged ones of 700 to 1500 110 -> 90.  One unit of 1000 tokens: 29.3 -> 27.5.
template <int D, bool COUNTS, int RB, typename Tab>
__global__ __launch_bounds__(kThreads, 2) void pq_out_narrow_kernel(
    const Tab tab, const Shape sh, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const int32_t* __restrict__ counts_in, const float* __restrict__ c_row,
    float* __restrict__ o_part, float* __restrict__ p_part, float2* __restrict__ stat_part, const int split) {
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int ROWB = D * 2;
  constexpr int TEAMS = kWaves / RB;
  __shared__ __attribute__((aligned(16))) float sm_o[kWaves][32][D + 4];
  __shared__ float sm_m[kWaves][32], sm_z[kWaves][32], sm_w[kWaves][32];

  const int ui = find_unit(tab, (int)blockIdx.x >> split);
  const Unit un = tab.unit(ui);
  int t0, t1;
  piece_range(un, blockIdx.x, split, t0, t1);
  const int ntiles = (t1 - t0 + kTile - 1) / kTile;          // (a piece may be empty: it leaves zeros)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int team = wave / RB, qrow = 32 * (wave % RB) + col;
  const int R = sh.R;
  const float sl2 = sh.scale_log2;
  const unsigned char* Kg = reinterpret_cast<const unsigned char*>(K + (size_t)un.in_row * D);
  const unsigned char* Vg = reinterpret_cast<const unsigned char*>(V + (size_t)un.in_row * D);
  const int32_t* cnt = COUNTS ? counts_in + un.in_row : nullptr;
  const uint32_t lane_at = (uint32_t)col * ROWB + (uint32_t)half * 16;     // this lane's first piece in a tile

  bf16x8 ident[2];                          // identity operand, as above
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k0 = 16 * kk + 8 * half + 2 * i;
      w[i] = (k0 == col ? 0x3F80u : 0u) | (k0 + 1 == col ? 0x3F800000u : 0u);
    }
    ident[kk] = as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
  }
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // a tile always holds 32 whole rows, see above (a wavefront without a tile loads the last one and uses nothing of it)
  auto tile_base = [&](int j) { return min(t0 + min(j, max(ntiles - 1, 0)) * kTile, t1 - kTile); };
  auto load = [&](const unsigned char* base, int j, uint4* r) {
    const unsigned char* src = base + (size_t)tile_base(j) * ROWB;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) r[kk] = *reinterpret_cast<const uint4*>(src + (lane_at + 32u * kk));
    asm volatile("" ::: "memory");          // issue them here: sunk to their use they would be waited for at once
  };

  const bool ok = qrow < R;
  bf16x8 bq[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) bq[kk] = row_operand<D>(Q + (size_t)un.index * R * D, qrow, ok, kk, half);
  float m_run = !ok ? INFINITY : c_row != nullptr ? c_row[(size_t)un.index * R + qrow] : -INFINITY;
  float z = 0.f, z_lost = 0.f, wsum = 0.f;
  const int lim = last_seen_row(sh.causal, un.len, qrow);
  f32x16 accO[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) accO[db] = zero;

  uint4 rk[KS], rv[KS];
  load(Kg, team, rk);
  load(Vg, team, rv);
  for (int j = team; j < ntiles; j += TEAMS) {
    const int base = tile_base(j);
    const int shift = t0 + j * kTile - base;                 // leading rows that belong to the tile before
    float cc[16];
    if (COUNTS) {
#pragma unroll
      for (int v = 0; v < 16; ++v) cc[v] = (float)cnt[base + 8 * (v / 4) + 4 * half + (v % 4)];
    }
    f32x16 acc = zero;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(rk[kk]), bq[kk], acc, 0, 0, 0);
    load(Kg, j + TEAMS, rk);
    float p[16];
    const bool masked = shift > 0 || (sh.causal > 0 && base + kTile > un.len - sh.causal + 1);
    auto seen = [&](int v) {
      const int row = 8 * (v / 4) + 4 * half + (v % 4);
      return row >= shift && base + row <= lim;
    };
    auto terms = [&](float m) {             // the tile's terms against reference m; returns their sum
#pragma unroll
      for (int v = 0; v < 16; ++v) p[v] = ex2(fmaf(acc[v], sl2, -m));
      if (masked) {
#pragma unroll
        for (int v = 0; v < 16; ++v) p[v] = seen(v) ? p[v] : 0.f;
      }
      float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 16; ++v) s4[v % 4] += p[v];
      return (s4[0] + s4[1]) + (s4[2] + s4[3]);
    };
    float ts = terms(m_run);
    if (!COUNTS && c_row == nullptr && __any(!(ts < kSumLimit))) {         // the reference rises, as above
      float tm = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) tm = fmaxf(tm, !masked || seen(v) ? acc[v] : -INFINITY);
      tm = fmaxf(tm, __shfl_xor(tm, 32, kWave));
      const float m_new = fmaxf(m_run, fmaf(tm, sl2, kHeadroom));
      const float m_safe = m_new == -INFINITY ? 0.f : m_new;
      const float down = m_run == m_new ? 1.f : ex2(m_run - m_safe);
#pragma unroll
      for (int db = 0; db < DB; ++db) accO[db] *= down;
      wsum *= down;
      z *= down;
      z_lost *= down;
      m_run = m_new;
      ts = terms(m_safe);
    }
    add_compensated(z, z_lost, ts);
    bf16x8 ph[2], pl[2];
    float pw[16];
    split8w(p, ph[0], pl[0], pw);
    split8w(p + 8, ph[1], pl[1], pw + 8);
#pragma unroll
    for (int v = 0; v < 16; ++v) wsum = COUNTS ? fmaf(pw[v], cc[v], wsum) : wsum + pw[v];
#pragma unroll
    for (int db = 0; db < DB; ++db) {       // a block of V turned token-major (see above) and multiplied
      f32x16 y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(rv[2 * db]), ident[0], zero, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(rv[2 * db + 1]), ident[1], y, 0, 0, 0);
      float yf[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) yf[v] = y[v];
      const bf16x8 vt0 = pack8(yf), vt1 = pack8(yf + 8);
      accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt0, ph[0], accO[db], 0, 0, 0);
      accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt1, ph[1], accO[db], 0, 0, 0);
      accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt0, pl[0], accO[db], 0, 0, 0);
      accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt1, pl[1], accO[db], 0, 0, 0);
    }
    load(Vg, j + TEAMS, rv);
  }

  wsum += __shfl_xor(wsum, 32, kWave);      // the other half's token rows
  z -= z_lost;
  z += __shfl_xor(z, 32, kWave);
  if (half == 0) {
    sm_m[wave][col] = m_run;
    sm_z[wave][col] = z;
    sm_w[wave][col] = wsum;
  }
#pragma unroll
  for (int db = 0; db < DB; ++db) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(&sm_o[wave][col][32 * db + 8 * g + 4 * half]) =
          make_float4(accO[db][4 * g], accO[db][4 * g + 1], accO[db][4 * g + 2], accO[db][4 * g + 3]);
  }
  __syncthreads();
  // thread: four dimensions of a query row
  for (int x = tid; x < R * (D / 4); x += kThreads) {
    const int q = x / (D / 4), d = x % (D / 4) * 4;
    const int first = q / 32, qw = q % 32;  // the first wavefront with this row, and its row there
    float m = sm_m[first][qw];
#pragma unroll
    for (int w = RB; w < kWaves; w += RB) m = fmaxf(m, sm_m[first + w][qw]);
    const float m_safe = m == -INFINITY ? 0.f : m;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    float zs = 0.f, ws = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; w += RB) {
      const float mw = sm_m[first + w][qw];
      const float f = mw == m ? 1.f : ex2(mw - m_safe);
      const float4 ow = *reinterpret_cast<const float4*>(&sm_o[first + w][qw][d]);
      o.x = fmaf(f, ow.x, o.x);
      o.y = fmaf(f, ow.y, o.y);
      o.z = fmaf(f, ow.z, o.z);
      o.w = fmaf(f, ow.w, o.w);
      zs = fmaf(f, sm_z[first + w][qw], zs);
      ws = fmaf(f, sm_w[first + w][qw], ws);
    }
    *reinterpret_cast<float4*>(o_part + ((size_t)blockIdx.x * R + q) * D + d) = o;
    if (d == 0) {
      p_part[(size_t)blockIdx.x * R + q] = ws;
      if (c_row == nullptr) stat_part[(size_t)blockIdx.x * R + q] = make_float2(m, zs);
    }
  }
}

// o^{(q)} from the pieces' partials and the sums of their weights, as a bf16 pair hi + lo, and its squared norm; and, where
// the pieces had references of their own (stat_part: reference and sum of the terms), the row's normaliser
// M + log2(Z * R) from them.  One workgroup per (unit, query row): the pieces' factors 2^(reference - M) first, a
// thread per piece, while the partials travel; then thread (g, d) adds the pieces of the g-th quarter up in order and the
// quarters are added in order.  (Bound by the latency of the loads: with all pieces in one thread's loop, eight in flight,
// the kernel took 13.9 us for 8 units of 64 pieces and 128 rows, and takes 8.2 with the quarters.)
constexpr int kReduceParts = 4;
template <int D, typename Tab>
__global__ __launch_bounds__(D * kReduceParts) void pq_out_reduce_kernel(const Tab tab, const Shape sh,
                                                          const float* __restrict__ o_part,
                                                          const float* __restrict__ p_part,
                                                          const float2* __restrict__ stat_part,
                                                          uint16_t* __restrict__ o_hi, uint16_t* __restrict__ o_lo,
                                                          float* __restrict__ oo, const int split) {
  constexpr int NT = D * kReduceParts, NW = NT / kWave;
  constexpr int MAXP = kMaxChunks << kMaxPqSplit, PPT = MAXP / NT;      // most pieces of a unit, per thread
  constexpr int UN = 16;                    // partials in flight per thread
  __shared__ float sm_ss[D / kWave];
  __shared__ float sm_s[kReduceParts][D];
  __shared__ float sm_f[MAXP];              // the pieces' factors
  __shared__ float sm_m[NW], sm_w[NW], sm_z[NW];
  const int R = sh.R;
  const int ui = blockIdx.x / R;
  const Unit un = tab.unit(ui);
  const int q = blockIdx.x % R;
  const int tid = threadIdx.x, d = tid % D, g = tid / D;
  const int base = un.chunk_base << split, n = un.n_chunks << split;
  if (q == 0 && sh.sel_clear != nullptr && ui < kInlineUnits) {          // the exchange area of the selection that follows
    uint4* zero = reinterpret_cast<uint4*>(sh.sel_clear + (size_t)ui * kSelSharedInts);
    for (int i = tid; i < kSelSharedInts / 4; i += NT) zero[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  const int per = (n + kReduceParts - 1) / kReduceParts;
  const int c0 = g * per, c1 = min(n, c0 + per);
  float v[UN];
  auto load = [&](int c) {
#pragma unroll
    for (int u = 0; u < UN; ++u) v[u] = c + u < c1 ? o_part[((size_t)(base + c + u) * R + q) * D + d] : 0.f;
  };
  load(c0);
  float2 st[PPT];
  float pw[PPT];
  float M = -INFINITY;
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int c = tid + i * NT;
    st[i] = make_float2(-INFINITY, 0.f);
    pw[i] = 0.f;
    if (c < n) {
      pw[i] = p_part[(size_t)(base + c) * R + q];
      if (stat_part != nullptr) st[i] = stat_part[(size_t)(base + c) * R + q];
    }
    M = fmaxf(M, st[i].x);
  }
  if (stat_part != nullptr) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) M = fmaxf(M, __shfl_xor(M, m, kWave));
    if (tid % kWave == 0) sm_m[tid / kWave] = M;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) M = fmaxf(M, sm_m[i]);
  }
  float w = 0.f, z = 0.f;
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const float f = stat_part == nullptr ? 1.f : st[i].x == -INFINITY ? 0.f : ex2(st[i].x - M);
    sm_f[tid + i * NT] = f;
    w = fmaf(pw[i], f, w);
    z = fmaf(st[i].y, f, z);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    w += __shfl_xor(w, m, kWave);
    z += __shfl_xor(z, m, kWave);
  }
  if (tid % kWave == 0) {
    sm_w[tid / kWave] = w;
    sm_z[tid / kWave] = z;
  }
  __syncthreads();
  float s = 0.f;
  for (int c = c0; c < c1; c += UN) {
    if (c != c0) load(c);
#pragma unroll
    for (int u = 0; u < UN; ++u) s = fmaf(v[u], sm_f[min(c + u, MAXP - 1)], s);
  }
  sm_s[g][d] = s;
  __syncthreads();
  if (g == 0) {                             // (whole wavefronts)
    s = sm_s[0][d];
    w = sm_w[0];
    z = sm_z[0];
#pragma unroll
    for (int i = 1; i < kReduceParts; ++i) s += sm_s[i][d];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
      w += sm_w[i];
      z += sm_z[i];
    }
    if (tid == 0 && stat_part != nullptr) sh.c_row_out[(size_t)un.index * R + q] = plus_log2(M, z * (float)R);
    const float m2o = -2.f * (s / w);                      // stored with the factor of ||v - o||^2 = ||v||^2 - 2 v.o + ||o||^2
    const uint32_t hi = f32_to_bf16(m2o);
    const uint32_t lo = f32_to_bf16(m2o - bf16_lo(hi));
    const size_t idx = ((size_t)un.index * R + q) * D + d;
    o_hi[idx] = (uint16_t)hi;
    o_lo[idx] = (uint16_t)lo;
    const float oe = -0.5f * (bf16_lo(hi) + bf16_lo(lo));  // the o the products below see
    float ss = oe * oe;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, kWave);
    if (d % kWave == 0) sm_ss[d / kWave] = ss;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = sm_ss[0];
#pragma unroll
    for (int i = 1; i < D / kWave; ++i) t += sm_ss[i];
    oo[(size_t)un.index * R + q] = t;
  }
}

// ------------------------------------------------------------------------------------------------
// Tokens of [t0, t1) (at most kRedoSpan) that pq_norms_kernel has marked (sign bit of A_t): A_t and C_t over all query rows
// once more, every squared norm as a sum of squared differences: ||v_t - o||^2 from v_t and the stored pair -2 o = hi + lo,
// likewise ||v_t + v_{t+1} - 2 o||^2.  The marked tokens are listed and
// taken in turn: D / 8 adjacent lanes share a query row, eight dimensions each (one round of coalesced loads per row), the
// rows' terms are added per lane group in row order and the groups in a fixed butterfly order.  Every marked token leaves
// with a non-negative A_t, so no mark outlives pq_norms_kernel.
template <int D>
struct RedoSmem {
  int list[kRedoSpan];
  int n;
  float row[4][D];                          // k_t, k_{t+1}, v_t, v_{t+1} (the Values divided by their cardinalities)
  float sum[2][kWaves];
};
template <int D, bool COUNTS>
__device__ __forceinline__ void redo_marked(
    const Shape& sh, const Unit& un, const int t0, const int t1, const uint16_t* __restrict__ Q,
    const uint16_t* __restrict__ K, const uint16_t* __restrict__ V, const int32_t* __restrict__ counts_in,
    const float* __restrict__ c_row, const uint16_t* __restrict__ o_hi, const uint16_t* __restrict__ o_lo, float* a_tok,
    float* c_edge, RedoSmem<D>& sm) {
  constexpr int LPR = D / 8;                // lanes per query row
  constexpr int RPP = kThreads / LPR;       // query rows per pass of the workgroup
  int (&sm_list)[kRedoSpan] = sm.list;
  int& sm_n = sm.n;
  float (&sm_row)[4][D] = sm.row;
  float (&sm_sum)[2][kWaves] = sm.sum;
  static_assert(kRedoSpan / kThreads <= 32, "one bit per token and thread");

  const int tid = threadIdx.x, part = tid % LPR;
  float* At = a_tok + un.in_row;
  float* Ce = c_edge + un.in_row;
  // the span's marks: bit k is token t0 + tid + 256 k
  uint32_t marks = 0;
#pragma unroll
  for (int k = 0; k < kRedoSpan / kThreads; ++k) {
    const int t = t0 + tid + k * kThreads;
    if (t < t1) marks |= (__float_as_uint(At[t]) >> 31) << k;
  }
  if (!__syncthreads_or((int)marks)) return;
  if (tid == 0) sm_n = 0;
  __syncthreads();
  for (int k = 0; k < kRedoSpan / kThreads; ++k) {           // (any order: tokens are independent)
    if ((marks >> k) & 1) sm_list[atomicAdd(&sm_n, 1)] = t0 + tid + k * kThreads;
  }
  __syncthreads();
  const int n_marked = sm_n;
  const int R = sh.R;
  const float Rf = (float)R;
  const uint16_t* Kg = K + (size_t)un.in_row * D;
  const uint16_t* Vg = V + (size_t)un.in_row * D;
  const uint16_t* Qu = Q + (size_t)un.index * R * D + 8 * part;
  const uint16_t* Oh = o_hi + (size_t)un.index * R * D + 8 * part;
  const uint16_t* Ol = o_lo + (size_t)un.index * R * D + 8 * part;
  const float* cr = c_row + (size_t)un.index * R;

  {
    for (int m = 0; m < n_marked; ++m) {
      const int t = sm_list[m];
      const bool has_next = t + 1 < un.len;
      float lc = 0.f, lcn = 0.f;
      {
        float ic = 1.f, icn = 1.f;
        if (COUNTS) {
          const float c = (float)counts_in[un.in_row + t];
          const float cn = has_next ? (float)counts_in[un.in_row + t + 1] : 1.f;
          lc = even_log2(c);
          lcn = even_log2(cn);
          ic = __builtin_amdgcn_rcpf(c);
          icn = __builtin_amdgcn_rcpf(cn);
        }
        if (tid < 4 * LPR) {                  // one 16-byte piece per thread
          const int which = tid / LPR, pc = tid % LPR;
          float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          if (!(which & 1) || has_next) {
            const uint16_t* src = (which < 2 ? Kg : Vg) + (size_t)(t + (which & 1)) * D + 8 * pc;
            Piece<uint16_t>::unpack(*reinterpret_cast<const uint4*>(src), x);
          }
          const float f = which < 2 ? 1.f : ((which & 1) ? icn : ic);
#pragma unroll
          for (int i = 0; i < 8; ++i) sm_row[which][8 * pc + i] = x[i] * f;
        }
      }
      __syncthreads();
      float kt[8], kn[8], vt[8], vn[8];     // this lane's eight dimensions of the four rows
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        kt[i] = sm_row[0][8 * part + i];
        kn[i] = sm_row[1][8 * part + i];
        vt[i] = sm_row[2][8 * part + i];
        vn[i] = sm_row[3][8 * part + i];
      }
      float sumA = 0.f, sumC = 0.f;
      // (four passes of rows per trip, so that their loads are in flight together: the kernel's time is the latency
      // of these rounds; rows beyond R are computed on row 0's data and dropped)
      for (int q00 = 0; q00 < R; q00 += 4 * RPP) {
        uint4 rq[4], rh[4], rl[4];
        float rc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q00 + u * RPP + tid / LPR;
          const int qc = q < R ? q : 0;
          rq[u] = *reinterpret_cast<const uint4*>(Qu + (size_t)qc * D);
          rh[u] = *reinterpret_cast<const uint4*>(Oh + (size_t)qc * D);
          rl[u] = *reinterpret_cast<const uint4*>(Ol + (size_t)qc * D);
          rc[u] = cr[qc];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q00 + u * RPP + tid / LPR;
          const bool ok = q < R;              // (uniform over the lanes of a row, not over the wavefront: no branch around the sums)
          const int qc = ok ? q : 0;
          float qv[8], h[8], l[8];
          Piece<uint16_t>::unpack(rq[u], qv);
          Piece<uint16_t>::unpack(rh[u], h);
          Piece<uint16_t>::unpack(rl[u], l);
          float e = 0.f, en = 0.f, sA = 0.f, sC = 0.f;
  #pragma unroll
          for (int i = 0; i < 8; ++i) {
            e = fmaf(qv[i], kt[i], e);
            en = fmaf(qv[i], kn[i], en);
            const float m2o = h[i] + l[i];                                 // -2 o
            const float da = fmaf(0.5f, m2o, vt[i]);                       // v_t - o
            const float dc = vt[i] + vn[i] + m2o;                          // v_t + v_{t+1} - 2 o
            sA = fmaf(da, da, sA);
            sC = fmaf(dc, dc, sC);
          }
          e = row_group_sum<LPR>(e);
          en = row_group_sum<LPR>(en);
          sA = row_group_sum<LPR>(sA);
          sC = row_group_sum<LPR>(sC);
          const int lim = last_seen_row(sh.causal, un.len, qc);
          float a = ex2(fmaf(e, sh.scale_log2, lc - rc[u]));               // alpha / R
          float a_n = ex2(fmaf(en, sh.scale_log2, lcn - rc[u]));
          if (!ok || (sh.causal > 0 && t > lim)) a = 0.f;
          if (!has_next || (sh.causal > 0 && t + 1 > lim)) a_n = 0.f;
          sumA = fmaf(a * fabsf(fmaf(-2.f * Rf, a, 1.f)), __builtin_amdgcn_sqrtf(sA), sumA);
          sumC = fmaf(a * a_n, __builtin_amdgcn_sqrtf(sC), sumC);
        }
      }
      if (part != 0) sumA = sumC = 0.f;     // (all lanes of a row hold the same sums: one of them counts)
#pragma unroll
      for (int m2 = 32; m2 >= 1; m2 >>= 1) {
        sumA += __shfl_xor(sumA, m2, kWave);
        sumC += __shfl_xor(sumC, m2, kWave);
      }
      if (tid % kWave == 0) {
        sm_sum[0][tid / kWave] = sumA;
        sm_sum[1][tid / kWave] = sumC;
      }
      __syncthreads();
      if (tid == 0) {
        float a = sm_sum[0][0], c = sm_sum[1][0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) { a += sm_sum[0][w]; c += sm_sum[1][w]; }
        At[t] = a;
        Ce[t] = has_next ? c * Rf : 0.f;
      }
      __syncthreads();                      // sm_row and sm_sum are reused by the next token
    }
  }
}

// ------------------------------------------------------------------------------------------------
// A_t and C_t of every token of the chunk.
//
// Both products are taken with the query rows as the accumulator ROWS: S'[q, t] = Q K^T, X'[q, t] = (-2 O) V^T.
// A lane then holds ONE token (column t = lane % 32) and 16 query rows, so the sums over q are plain
// register additions (plus one exchange between the wavefront's halves), and token t + 1 is the next lane
// (one DPP wavefront shift).  Per (t, q): one exp2, two square roots, eleven other instructions.
template <int D, bool COUNTS, typename Tab>
__global__ __launch_bounds__(kThreads, 2) void pq_norms_kernel(
    const Tab tab, const Shape sh, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const int32_t* __restrict__ counts_in, const float* __restrict__ c_row,
    const uint16_t* __restrict__ o_hi,
    const uint16_t* __restrict__ o_lo, const float* __restrict__ oo, float* a_tok, float* c_edge, const int split) {
  typedef Tile<D> TL;
  constexpr int KS = D / 16;
  constexpr int STRIDE = kTile - 1;         // output rows per tile: the last row only serves as "next token"
  constexpr int PPT = TL::LPR / 8;          // pieces per thread when 8 threads share a row
  __shared__ __attribute__((aligned(16))) unsigned char sm_k[2][TL::BYTES];
  __shared__ __attribute__((aligned(16))) unsigned char sm_v[2][TL::BYTES];
  __shared__ int sm_marked;                                          // a token of the piece has been marked
  __shared__ float sm_vv[2][kTile + 1];                              // ||v_r||^2 (one spare entry: the last row's "next")
  __shared__ float sm_vd[2][kTile];                                  // v_r . v_{r+1}
  __shared__ float2 sm_out[2][kWaves][kTile];                        // (sum_q A, sum_q C) of every wavefront
  __shared__ float sm_al[2][kWaves][kTile];                          // sum_q alpha / R: the wavefront's share of alpha_bar
  __shared__ __attribute__((aligned(16))) float sm_negc[kPassRows];  // per query row of the pass: -c[q]
  __shared__ __attribute__((aligned(16))) int sm_lim[kPassRows];     // causal window: last row attended to
  __shared__ float sm_cc[2][kTile + 1], sm_ic[2][kTile + 1];         // COUNTS: c and 1 / c of the tile's rows

  const int ui = find_unit(tab, (int)blockIdx.x >> split);
  const Unit un = tab.unit(ui);
  int t0, t1;
  piece_range(un, blockIdx.x, split, t0, t1);
  if (t0 >= t1) return;                     // nothing left of the chunk for this piece
  const int ntiles = (t1 - t0 + STRIDE - 1) / STRIDE;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  if (tid == 0) sm_marked = 0;              // (the first tile's barriers come before the first mark)
  const int col = lane % 32, half = lane / 32;
  const int R = sh.R;
  const float Rf = (float)R;
  const float sl2 = sh.scale_log2;
  const unsigned char* Kg = reinterpret_cast<const unsigned char*>(K + (size_t)un.in_row * D);
  const unsigned char* Vg = reinterpret_cast<const unsigned char*>(V + (size_t)un.in_row * D);
  const uint16_t* Qu = Q + (size_t)un.index * R * D;
  const uint16_t* Oh = o_hi + (size_t)un.index * R * D;
  const uint16_t* Ol = o_lo + (size_t)un.index * R * D;
  float* At = a_tok + un.in_row;
  float* Ce = c_edge + un.in_row;
  float* Al = sh.alpha_out != nullptr ? sh.alpha_out + un.in_row : nullptr;
  const int32_t* cnt = COUNTS ? counts_in + un.in_row : nullptr;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // Tile j puts out tokens t0 + 31 j .. + 30 and reads one row more.  Near the unit's end it is moved back
  // to hold 32 existing rows; the `shift` leading rows then belong to earlier tiles.
  auto tile_first = [&](int j) { return t0 + j * STRIDE; };
  auto tile_base = [&](int j) { return min(tile_first(j), un.len - kTile); };

  for (int qp = 0; qp < R; qp += kPassRows) {
    const int qrow = qp + 32 * wave + col;
    const bool ok = qrow < R;
    bf16x8 bq[KS], boh[KS], bol[KS];        // this wavefront's 32 query rows: Q, and -2 o as hi + lo
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      bq[kk] = row_operand<D>(Qu, qrow, ok, kk, half);
      boh[kk] = row_operand<D>(Oh, qrow, ok, kk, half);
      bol[kk] = row_operand<D>(Ol, qrow, ok, kk, half);
    }
    if (tid < kPassRows) {                  // (read after the first tile's barriers)
      const int q = qp + tid;
      sm_negc[tid] = (q < R) ? -c_row[(size_t)un.index * R + q] : -INFINITY;   // exp2(-inf) = 0: no such row
      sm_lim[tid] = last_seen_row(sh.causal, un.len, q);
    }
    // ||o^{(q)}||^2 of this lane's 16 accumulator rows: the value the X' accumulator starts from
    f32x16 oo_init;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int q = qp + 32 * wave + 8 * (v / 4) + 4 * half + (v % 4);
      oo_init[v] = (q < R) ? oo[(size_t)un.index * R + q] : 0.f;
    }

    // sums of the tile before -> memory (threads 0..31, one row each; the wavefronts in a fixed order)
    auto flush = [&](int j) {
      if (tid < kTile) {
        const int buf = j & 1;
        const int base = tile_base(j), shift = tile_first(j) - base;
        const int r = tid, t = base + r;
        if (r >= shift && r <= shift + STRIDE - 1 && t < t1) {
          float a = 0.f, c = 0.f, al = 0.f;
          uint32_t mark = 0;                               // sign bit: some wavefront, or an earlier pass, marked the token
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            const float2 o = sm_out[buf][w][r];
            mark |= __float_as_uint(o.x);
            a += fabsf(o.x);
            c += o.y;
            al += sm_al[buf][w][r];
          }
          if (r == kTile - 1) c = 0.f;                     // only the unit's last token: it has no next one
          if (COUNTS) al *= sm_cc[buf][r];
          if (qp > 0) {                                    // later passes add their query rows
            const float before = At[t];
            mark |= __float_as_uint(before);
            a += fabsf(before);
            c += Ce[t];
            if (Al != nullptr) al += Al[t];
          }
          if (mark & 0x80000000u) sm_marked = 1;
          At[t] = __uint_as_float(__float_as_uint(a) | (mark & 0x80000000u));
          Ce[t] = c;
          if (Al != nullptr) Al[t] = al;
        }
      }
    };

    typename TL::Regs rk = TL::load(Kg + (size_t)tile_base(0) * TL::ROWB, tid);
    typename TL::Regs rv = TL::load(Vg + (size_t)tile_base(0) * TL::ROWB, tid);
    for (int j = 0; j < ntiles; ++j) {
      const int buf = j & 1;
      TL::store(sm_k[buf], rk, tid);
      TL::store(sm_v[buf], rv, tid);
      if (COUNTS && tid <= kTile) {           // (the spare entry stands for the last row's "next", which is never used)
        const float c = tid < kTile ? (float)cnt[tile_base(j) + tid] : 1.f;
        sm_cc[buf][tid] = c;
        sm_ic[buf][tid] = __builtin_amdgcn_rcpf(c);
      }
      __syncthreads();
      {                                     // the next tile flies during this one (the last one is fetched twice)
        const int jn = min(j + 1, ntiles - 1);
        rk = TL::load(Kg + (size_t)tile_base(jn) * TL::ROWB, tid);
        rv = TL::load(Vg + (size_t)tile_base(jn) * TL::ROWB, tid);
        asm volatile("" ::: "memory");        // issue them here: sunk below the products they would be waited for at once
      }
      if (j > 0) flush(j - 1);
      // squared norms of the rows and of the sums of adjacent rows: eight threads per row
      {
        const int r = tid / 8, part = tid % 8;
        const int rn = min(r + 1, kTile - 1);
        float s_rr = 0.f, s_rn = 0.f;
#pragma unroll
        for (int x = 0; x < PPT; ++x) {           // (two bf16 products per instruction, added in fp32)
          const uint4 a = TL::piece_at(sm_v[buf], r, part * PPT + x);
          const uint4 b = TL::piece_at(sm_v[buf], rn, part * PPT + x);
          s_rr = dot2(a.x, a.x, s_rr); s_rn = dot2(a.x, b.x, s_rn);
          s_rr = dot2(a.y, a.y, s_rr); s_rn = dot2(a.y, b.y, s_rn);
          s_rr = dot2(a.z, a.z, s_rr); s_rn = dot2(a.z, b.z, s_rn);
          s_rr = dot2(a.w, a.w, s_rr); s_rn = dot2(a.w, b.w, s_rn);
        }
        s_rr = row_group_sum<8>(s_rr);
        s_rn = row_group_sum<8>(s_rn);
        if (part == 0) {
          sm_vv[buf][r] = s_rr;
          sm_vd[buf][r] = s_rn;
          if (r == kTile - 1) sm_vv[buf][kTile] = 0.f;       // read by the last column, whose edge is never used
        }
      }
      // S' = Q K^T and X' = (-2 O) V^T for this wavefront's 32 query rows
      f32x16 accS = zero, accX = COUNTS ? zero : oo_init;     // X'' = ||o||^2 - 2 v.o (COUNTS: -2 V.o, scaled below)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        accS = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[kk], TL::operand(sm_k[buf], col, kk, half), accS, 0, 0, 0);
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const bf16x8 bv = TL::operand(sm_v[buf], col, kk, half);
        accX = __builtin_amdgcn_mfma_f32_32x32x16_bf16(boh[kk], bv, accX, 0, 0, 0);
        accX = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bol[kk], bv, accX, 0, 0, 0);
      }
      __syncthreads();                      // sm_vv / sm_vd of this tile are complete
      // accumulator element v: query row 32 wave + 8 (v / 4) + 4 half + v % 4 of the pass, token column `col`
      float vv = sm_vv[buf][col];
      float vp = fmaf(2.f, sm_vd[buf][col], vv + sm_vv[buf][col + 1]);         // ||v_t + v_{t+1}||^2
      float cc = 1.f, ic = 1.f;               // COUNTS: this lane's token stands for c tokens, v = V / c
      if (COUNTS) {
        cc = sm_cc[buf][col];
        ic = sm_ic[buf][col];
        const float icn = sm_ic[buf][col + 1];
        const float vvn = sm_vv[buf][col + 1] * icn * icn;
        vv = vv * ic * ic;
        vp = fmaf(2.f * ic * icn, sm_vd[buf][col], vv + vvn);
      }
      const int t_abs = tile_base(j) + col;
      float sumA = 0.f, sumC = 0.f, sumP = 0.f;
      float leastA = INFINITY, leastC = INFINITY;   // smallest squared norms this lane forms in the tile (see below)
      // TAIL: the tile reaches into the causal window's masked rows (a uniform condition)
      auto rows = [&](auto tail_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int q0 = 32 * wave + 8 * g + 4 * half;
          const float4 nc4 = *reinterpret_cast<const float4*>(&sm_negc[q0]);
          const float nc[4] = {nc4.x, nc4.y, nc4.z, nc4.w};
          int lim[4] = {0, 0, 0, 0};
          if (TAIL) {
            const int4 l4 = *reinterpret_cast<const int4*>(&sm_lim[q0]);
            lim[0] = l4.x; lim[1] = l4.y; lim[2] = l4.z; lim[3] = l4.w;
          }
          float d2s[4], p2s[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int v = 4 * g + i;
            // alpha / R (COUNTS: first of one of the c tokens; log2 c in the exponent would round with c's size)
            float a = ex2(fmaf(accS[v], sl2, nc[i]));
            if (TAIL && t_abs > lim[i]) a = 0.f;
            sumP += a;
            if (COUNTS) a *= cc;
            const float x = COUNTS ? fmaf(accX[v], ic, oo_init[v]) : accX[v]; // ||o||^2 - 2 v_t . o
            // the same quantities of token t + 1: the next lane (the last column's are not used)
            const float a_n = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0x130, 0xF, 0xF, true));
            const float x_n = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x130, 0xF, 0xF, true));
            const float d2 = vv + x;                                       // ||v_t - o||^2
            const float p2 = fmaf(2.f, x + x_n, vp);                       // ||v_t + v_{t+1} - 2o||^2
            // (a rounding-size negative value stands for zero: the square roots take the magnitude)
            sumA = fmaf(a * fabsf(fmaf(-2.f * Rf, a, 1.f)), __builtin_amdgcn_sqrtf(fabsf(d2)), sumA);
            sumC = fmaf(a * a_n, __builtin_amdgcn_sqrtf(fabsf(p2)), sumC);
            d2s[i] = d2;
            p2s[i] = p2;
          }
          leastA = min3(min3(leastA, d2s[0], d2s[1]), d2s[2], d2s[3]);
          leastC = min3(min3(leastC, p2s[0], p2s[1]), p2s[2], p2s[3]);
          __builtin_amdgcn_sched_barrier(0);  // four rows at a time: interleaving all sixteen runs out of registers
        }
      };
      if (sh.causal > 0 && tile_base(j) + kTile > un.len - sh.causal + 1) rows(std::true_type{});
      else rows(std::false_type{});
      // Cancellation.  Where o^{(q)} comes close to v_t (a query row that puts nearly all its weight on one token) the
      // expansion above loses what is left of ||v_t - o||^2 to the rounding of its terms of size ||v_t||^2.  A token
      // one of whose squared norms falls below kCancel of its leading term is marked (the sign bit of its A_t, which
      // is never negative) and formed again by redo_marked, from differences.  The test costs one three-way
      // minimum per (t, q).
      int redo = (leastA < kCancel * vv || leastC < kCancel * vp) ? 1 : 0;
      redo |= __shfl_xor(redo, 32, kWave);
      sumA += __shfl_xor(sumA, 32, kWave);    // the other half's 16 query rows
      sumC += __shfl_xor(sumC, 32, kWave);
      sumP += __shfl_xor(sumP, 32, kWave);
      if (half == 0) {
        sm_out[buf][wave][col] = make_float2(redo ? -sumA : sumA, sumC * Rf);                // (sumA >= 0; -0 counts)
        sm_al[buf][wave][col] = sumP;
      }
    }
    __syncthreads();
    flush(ntiles - 1);
    __syncthreads();                        // the next pass reuses the buffers
  }
  // The marked tokens, nearly always none (one in 30000 on the generated inputs), by the workgroup that has marked them:
  // a launch of its own for them was 12 us behind the 55 of this kernel (8 units of 32768 tokens, 128 rows).
  if (sm_marked) {
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this workgroup's A_t and C_t are out
    __syncthreads();
    static_assert(sizeof(RedoSmem<D>) <= sizeof(sm_k), "the K tiles' buffers are free now");
    RedoSmem<D>& sm = *reinterpret_cast<RedoSmem<D>*>(&sm_k[0][0]);
    for (int t = t0; t < t1; t += kRedoSpan) {
      redo_marked<D, COUNTS>(sh, un, t, min(t1, t + kRedoSpan), Q, K, V, counts_in, c_row, o_hi, o_lo, a_tok, c_edge, sm);
      __syncthreads();
    }
  }
}

// The same for few query rows: RB wavefronts to a tile, and their operands straight from memory, as in pq_out_narrow_kernel.
// With one a tile's sums are whole in its wavefront and nothing waits.
template <int D, bool COUNTS, int RB, typename Tab>
__global__ __launch_bounds__(kThreads, 2) void pq_norms_narrow_kernel(
    const Tab tab, const Shape sh, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const int32_t* __restrict__ counts_in, const float* __restrict__ c_row,
    const uint16_t* __restrict__ o_hi,
    const uint16_t* __restrict__ o_lo, const float* __restrict__ oo, float* a_tok, float* c_edge, const int split) {
  constexpr int KS = D / 16;
  constexpr int ROWB = D * 2;
  constexpr int STRIDE = kTile - 1;         // output rows per tile: the last row only serves as "next token"
  constexpr int TEAMS = kWaves / RB, ROWS = 32 * RB;
  __shared__ int sm_marked;
  __shared__ __attribute__((aligned(16))) float sm_negc[ROWS], sm_oo[ROWS];
  __shared__ __attribute__((aligned(16))) int sm_lim[ROWS];
  __shared__ float sm_out[RB > 1 ? 2 : 1][RB > 1 ? kWaves : 1][3][kTile];    // sums of A, C and alpha / R over a wavefront's rows
  __shared__ RedoSmem<D> sm_redo;

  const int ui = find_unit(tab, (int)blockIdx.x >> split);
  const Unit un = tab.unit(ui);
  int t0, t1;
  piece_range(un, blockIdx.x, split, t0, t1);
  if (t0 >= t1) return;                     // nothing left of the chunk for this piece
  const int ntiles = (t1 - t0 + STRIDE - 1) / STRIDE;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int team = wave / RB, rb = wave % RB, qrow = 32 * rb + col;
  const int R = sh.R;
  const float Rf = (float)R;
  const float sl2 = sh.scale_log2;
  const unsigned char* Kg = reinterpret_cast<const unsigned char*>(K + (size_t)un.in_row * D);
  const unsigned char* Vg = reinterpret_cast<const unsigned char*>(V + (size_t)un.in_row * D);
  float* At = a_tok + un.in_row;
  float* Ce = c_edge + un.in_row;
  float* Al = sh.alpha_out != nullptr ? sh.alpha_out + un.in_row : nullptr;
  const int32_t* cnt = COUNTS ? counts_in + un.in_row : nullptr;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const uint32_t lane_at = (uint32_t)col * ROWB + (uint32_t)half * 16;

  auto tile_first = [&](int j) { return t0 + j * STRIDE; };
  auto tile_base = [&](int j) { return min(tile_first(min(j, ntiles - 1)), un.len - kTile); };
  auto load = [&](const unsigned char* base, int j, uint4* r) {
    const unsigned char* src = base + (size_t)tile_base(j) * ROWB;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) r[kk] = *reinterpret_cast<const uint4*>(src + (lane_at + 32u * kk));
    asm volatile("" ::: "memory");
  };
  uint4 rk[KS], rv[KS];
  load(Kg, team, rk);
  load(Vg, team, rv);

  bf16x8 bq[KS], boh[KS], bol[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    bq[kk] = row_operand<D>(Q + (size_t)un.index * R * D, qrow, qrow < R, kk, half);
    boh[kk] = row_operand<D>(o_hi + (size_t)un.index * R * D, qrow, qrow < R, kk, half);
    bol[kk] = row_operand<D>(o_lo + (size_t)un.index * R * D, qrow, qrow < R, kk, half);
  }
  if (tid == 0) sm_marked = 0;
  if (tid < ROWS) {
    sm_negc[tid] = (tid < R) ? -c_row[(size_t)un.index * R + tid] : -INFINITY;   // exp2(-inf) = 0: no such row
    sm_oo[tid] = (tid < R) ? oo[(size_t)un.index * R + tid] : 0.f;
    sm_lim[tid] = last_seen_row(sh.causal, un.len, tid);
  }
  __syncthreads();

  // the value of the next lane (the next token's; the last column's is not used)
  auto next_f = [](float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x130, 0xF, 0xF, true));
  };
  auto next_u = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xF, 0xF, true); };
  // (as many rounds for every wavefront, since those of a team meet in each; one without a tile does the last one again and
  // leaves it)
  for (int j = team, round = 0; j - team < ntiles; j += TEAMS, ++round) {
    if (RB == 1 && j >= ntiles) break;
    const int base = tile_base(j), shift = tile_first(j) - base;
    float cc = 1.f, ic = 1.f;               // COUNTS: this lane's token stands for c tokens, v = V / c
    if (COUNTS) {
      cc = (float)cnt[base + col];
      ic = __builtin_amdgcn_rcpf(cc);
    }
    f32x16 accS = zero;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      accS = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[kk], as_bf16x8(rk[kk]), accS, 0, 0, 0);
    load(Kg, j + TEAMS, rk);
    f32x16 accX;                            // ||o||^2 - 2 v.o (COUNTS: -2 V.o, scaled below)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 o4 = *reinterpret_cast<const float4*>(&sm_oo[32 * rb + 8 * g + 4 * half]);
      accX[4 * g] = COUNTS ? 0.f : o4.x;
      accX[4 * g + 1] = COUNTS ? 0.f : o4.y;
      accX[4 * g + 2] = COUNTS ? 0.f : o4.z;
      accX[4 * g + 3] = COUNTS ? 0.f : o4.w;
    }
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      accX = __builtin_amdgcn_mfma_f32_32x32x16_bf16(boh[kk], as_bf16x8(rv[kk]), accX, 0, 0, 0);
      accX = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bol[kk], as_bf16x8(rv[kk]), accX, 0, 0, 0);
    }
    // squared norm of the row and its product with the next one: this lane's half of the dimensions, then both
    float vv = 0.f, vd = 0.f;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const uint4 a = rv[kk];
      vv = dot2(a.x, a.x, vv); vd = dot2(a.x, next_u(a.x), vd);
      vv = dot2(a.y, a.y, vv); vd = dot2(a.y, next_u(a.y), vd);
      vv = dot2(a.z, a.z, vv); vd = dot2(a.z, next_u(a.z), vd);
      vv = dot2(a.w, a.w, vv); vd = dot2(a.w, next_u(a.w), vd);
    }
    load(Vg, j + TEAMS, rv);
    vv += __shfl_xor(vv, 32, kWave);
    vd += __shfl_xor(vd, 32, kWave);
    if (COUNTS) {
      vv = vv * ic * ic;
      vd = vd * ic * next_f(ic);
    }
    const float vp = fmaf(2.f, vd, vv + next_f(vv));                       // ||v_t + v_{t+1}||^2
    const int t_abs = base + col;
    float sumA = 0.f, sumC = 0.f, sumP = 0.f;
    float leastA = INFINITY, leastC = INFINITY;
    auto rows = [&](auto tail_tag) {        // the terms of pq_norms_kernel
      constexpr bool TAIL = decltype(tail_tag)::value;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int q0 = 32 * rb + 8 * g + 4 * half;
        const float4 nc4 = *reinterpret_cast<const float4*>(&sm_negc[q0]);
        const float nc[4] = {nc4.x, nc4.y, nc4.z, nc4.w};
        float ov[4] = {0.f, 0.f, 0.f, 0.f};
        if (COUNTS) {
          const float4 o4 = *reinterpret_cast<const float4*>(&sm_oo[q0]);
          ov[0] = o4.x; ov[1] = o4.y; ov[2] = o4.z; ov[3] = o4.w;
        }
        int lim[4] = {0, 0, 0, 0};
        if (TAIL) {
          const int4 l4 = *reinterpret_cast<const int4*>(&sm_lim[q0]);
          lim[0] = l4.x; lim[1] = l4.y; lim[2] = l4.z; lim[3] = l4.w;
        }
        float d2s[4], p2s[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 4 * g + i;
          float a = ex2(fmaf(accS[v], sl2, nc[i]));
          if (TAIL && t_abs > lim[i]) a = 0.f;
          sumP += a;
          if (COUNTS) a *= cc;
          const float x = COUNTS ? fmaf(accX[v], ic, ov[i]) : accX[v];
          const float a_n = next_f(a), x_n = next_f(x);
          const float d2 = vv + x;
          const float p2 = fmaf(2.f, x + x_n, vp);
          sumA = fmaf(a * fabsf(fmaf(-2.f * Rf, a, 1.f)), __builtin_amdgcn_sqrtf(fabsf(d2)), sumA);
          sumC = fmaf(a * a_n, __builtin_amdgcn_sqrtf(fabsf(p2)), sumC);
          d2s[i] = d2;
          p2s[i] = p2;
        }
        leastA = min3(min3(leastA, d2s[0], d2s[1]), d2s[2], d2s[3]);
        leastC = min3(min3(leastC, p2s[0], p2s[1]), p2s[2], p2s[3]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (sh.causal > 0 && base + kTile > un.len - sh.causal + 1) rows(std::true_type{});
    else rows(std::false_type{});
    int redo = (leastA < kCancel * vv || leastC < kCancel * vp) ? 1 : 0;     // see pq_norms_kernel
    redo |= __shfl_xor(redo, 32, kWave);
    sumA += __shfl_xor(sumA, 32, kWave);    // the other half's 16 query rows
    sumC += __shfl_xor(sumC, 32, kWave);
    sumP += __shfl_xor(sumP, 32, kWave);
    if (RB > 1) {                           // the team's other rows (two buffers: one barrier per round)
      float (&out)[kWaves][3][kTile] = reinterpret_cast<float (&)[2][kWaves][3][kTile]>(sm_out)[round & 1];
      if (half == 0) {
        out[wave][0][col] = redo ? -sumA : sumA;
        out[wave][1][col] = sumC;
        out[wave][2][col] = sumP;
      }
      __syncthreads();
      sumA = sumC = sumP = 0.f;
      redo = 0;
#pragma unroll
      for (int w = 0; w < RB; ++w) {
        const float a = out[team * RB + w][0][col];
        redo |= (int)(__float_as_uint(a) >> 31);
        sumA += fabsf(a);
        sumC += out[team * RB + w][1][col];
        sumP += out[team * RB + w][2][col];
      }
      if (rb != 0 || j >= ntiles) continue;
    }
    if (half == 0 && col >= shift && col <= shift + STRIDE - 1 && t_abs < t1) {
      if (redo) sm_marked = 1;
      At[t_abs] = redo ? -sumA : sumA;      // (sumA >= 0; -0 counts)
      Ce[t_abs] = col == kTile - 1 ? 0.f : sumC * Rf;        // (only the unit's last token: it has no next one)
      if (Al != nullptr) Al[t_abs] = COUNTS ? sumP * cc : sumP;
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0): this wavefront's A_t and C_t are out
  __syncthreads();
  if (sm_marked) {
    for (int t = t0; t < t1; t += kRedoSpan) {
      redo_marked<D, COUNTS>(sh, un, t, min(t1, t + kRedoSpan), Q, K, V, counts_in, c_row, o_hi, o_lo, a_tok, c_edge, sm_redo);
      __syncthreads();
    }
  }
}

template <int D, bool COUNTS>
hipError_t launch_t(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                    const int32_t* counts_in, const float* c_row, float* o_part, uint16_t* o_hi, uint16_t* o_lo,
                    float* oo, float* a_tok, float* c_edge, hipStream_t stream) {
  long long rows = 0;
  int longest_chunk = 1;
  for (int u = 0; u < tab.n_units; ++u) {
    const Unit& un = tab.unit(u);
    rows += un.len;
    longest_chunk = std::max(longest_chunk, std::min(un.len, un.chunk_len));
  }
  const int split = pq_split(tab.n_units, tab.total_chunks, rows, longest_chunk, sh.R, D);
  const dim3 grid(tab.total_chunks << split), block(kThreads);
  float2* stat_part = reinterpret_cast<float2*>(o_part + (size_t)grid.x * sh.R * D);   // behind the launch's partials
  float* p_part = reinterpret_cast<float*>(stat_part + (size_t)grid.x * sh.R);
  const bool own_rows = sh.c_row_out != nullptr;            // the normalisers come from here
  // Up to 32 rows both narrow kernels (figures at pq_out_narrow_kernel), in small launches the norms' alone (see pq_small).  33 to 64 rows, two wavefronts to a tile, with 64
  // channels (12 units of 29384 135 -> 114 us, one of 1000 35.6 -> 34.8); with 128 channels the outputs' reads of every tile by
  // two wavefronts cost more than the idle rows (8 of 32768 131 -> 138), and the norms gain from some 256 K tokens on
  // (8 of 32768 131.3 -> 130.0, 4 of 100000 193 -> 186, 100 of 21000 892 -> 865, 40 of 20000 with cardinalities 446 -> 418;
  // 4 ragged ones, 150000 tokens, 90.1 -> 92.2, 32 of 3000 85.9 -> 87.8).
  const bool one = sh.R <= kPqNarrowRows, two = !one && sh.R <= 2 * kPqNarrowRows;
  const bool small = pq_small(tab.n_units, rows, sh.R, D);
  const bool narrow_norms = D == 64 || rows >= (1 << 18);
  launch_with_table(tab, [&](const auto& t) {
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, block, 0, stream, t, sh, (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)V, counts_in,
                         own_rows ? nullptr : c_row, o_part, p_part, stat_part, split);
    };
    if constexpr (D == 64) {
      if (two) return launch(pq_out_narrow_kernel<D, COUNTS, 2, KVS_TABLE_TYPE(t)>);
    }
    if (one && !small) return launch(pq_out_narrow_kernel<D, COUNTS, 1, KVS_TABLE_TYPE(t)>);
    launch(pq_out_kernel<D, COUNTS, KVS_TABLE_TYPE(t)>);
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_with_table(tab, [&](const auto& t) {
    hipLaunchKernelGGL((pq_out_reduce_kernel<D, KVS_TABLE_TYPE(t)>), dim3(tab.n_units * sh.R), dim3(D * kReduceParts), 0, stream, t, sh,
                       o_part, p_part, own_rows ? stat_part : nullptr, o_hi, o_lo, oo, split);
  });
  if ((e = hipGetLastError()) != hipSuccess) return e;
  launch_with_table(tab, [&](const auto& t) {
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, block, 0, stream, t, sh, (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)V, counts_in,
                         c_row, o_hi, o_lo, oo, a_tok, c_edge, split);
    };
    if (one) return launch(pq_norms_narrow_kernel<D, COUNTS, 1, KVS_TABLE_TYPE(t)>);
    if (two && narrow_norms) return launch(pq_norms_narrow_kernel<D, COUNTS, 2, KVS_TABLE_TYPE(t)>);
    launch(pq_norms_kernel<D, COUNTS, KVS_TABLE_TYPE(t)>);
  });
  return hipGetLastError();
}

}  // namespace

hipError_t launch_per_query_norms(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                                  const int32_t* counts_in, const float* c_row, float* o_part, uint16_t* o_hi,
                                  uint16_t* o_lo, float* oo, float* a_tok, float* c_edge, hipStream_t stream) {
#define KVS_PQ_ARGS tab, sh, Q, K, V, counts_in, c_row, o_part, o_hi, o_lo, oo, a_tok, c_edge, stream
  if (counts_in) return sh.D == 64 ? launch_t<64, true>(KVS_PQ_ARGS) : launch_t<128, true>(KVS_PQ_ARGS);
  return sh.D == 64 ? launch_t<64, false>(KVS_PQ_ARGS) : launch_t<128, false>(KVS_PQ_ARGS);
#undef KVS_PQ_ARGS
}

}  // namespace kvs
