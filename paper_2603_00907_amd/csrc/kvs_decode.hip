// Decode attention over a merged cache (the consumer of kvs_merge_compact's outputs).
//
// A row (k', V', c) of a merged cache stands for c tokens that all carry the Key k' and whose Values
// add up to V' (Sec. 3.1: the pair (k_m, k_{m+1}) is replaced by (k, k), the Values are summed, and the
// cardinality is carried along).  Attention of a query q over such a cache is
//   o = sum_S exp(e_S) V'_S / sum_S c_S exp(e_S),      e_S = scale * q . k'_S,
// i.e. ordinary attention over the c_S copies of every slot.  With c = 1 it is plain attention.
//
// Split over the rows of a unit (chunks whose length is chosen per launch, at most 64 per unit, one workgroup
// each; the grid is chunks x units): LPR adjacent lanes read one K row and one V row (16 bytes each), four query rows at a time
// sit in registers, every lane group keeps an online softmax (running maximum, denominator,
// D-wide numerator) for its rows, the groups of a workgroup are combined through LDS, and a second
// small kernel combines the chunks.  Everything is ordered: no atomics, results do not depend on
// timing.  The kernel is meant for decode-sized query blocks (at most KVS_MAX_DECODE_ROWS rows per
// unit); it reads the cache once per block of four query rows.
//
// From five query rows on, caches whose units have at least 32 rows take decode_mfma_kernel (bf16; fp32: its variant
// decode_mfma_f32_kernel) instead: both products on
// v_mfma_f32_32x32x16_bf16, 32 query rows per pass, the operands loaded from memory in the MFMA layout (a lane
// fetches the 16-byte pieces of ITS row), so nothing is staged in LDS and the wavefronts of a workgroup, which
// split the chunk's 32-row tiles, never wait for each other inside the loop.  The chunk partials have the same
// format and go through the same second kernel.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "kvs_device.h"

namespace kvs {
namespace {

#ifndef KVS_DEC_THREADS
#define KVS_DEC_THREADS 256
#endif
constexpr int kThreads = KVS_DEC_THREADS;
constexpr int kQB = 4;                    // query rows per block
constexpr int kFewRows = 2, kMoreRows = 4;   // cache rows per lane group in flight, see launch_t
#ifndef KVS_DEC_CHUNK
#define KVS_DEC_CHUNK 256
#endif
constexpr int kDecMinChunk = KVS_DEC_CHUNK;   // rows per workgroup, where the launch is large enough for it

// Chunking of a unit's rows: a function of its length and of the launch's least chunk length.
__host__ __device__ inline int dec_chunk_len(int len, int min_chunk) {
  const int per = (len + kMaxChunks - 1) / kMaxChunks;
  const int rounded = (per + kWave - 1) / kWave * kWave;
  return rounded > min_chunk ? rounded : min_chunk;
}
__host__ __device__ inline int dec_chunks(int len, int min_chunk) {
  const int cl = dec_chunk_len(len, min_chunk);
  return (len + cl - 1) / cl;
}

// Chunks of the unit that has most of them.
int most_chunks(const UnitTable& tab, int min_chunk) {
  int most = 1;
  for (int i = 0, before = 0; i < tab.n_units; ++i) {
    const int len = tab.unit(i).len;
    if (len != before) most = std::max(most, dec_chunks(len, min_chunk));
    before = len;
  }
  return most;
}

// partial result of one (unit, chunk, query row): numerator[D], running maximum, denominator
__device__ __forceinline__ size_t part_index(int unit_index, int chunk, int R, int row, int D) {
  return (((size_t)unit_index * kMaxChunks + chunk) * R + row) * (size_t)(D + 2);
}

template <typename T, int D, int kUnroll, typename Tab>
__global__ __launch_bounds__(kThreads) void decode_partial_kernel(
    const Tab tab, const Shape sh, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const int32_t* __restrict__ counts, float* __restrict__ part) {
  constexpr int EPL = Piece<T>::N;
  constexpr int LPR = D / EPL;
  constexpr int RPW = kWave / LPR;
  constexpr int GROUPS = RPW * (kThreads / kWave);       // lane groups (= rows in flight) per workgroup

  __shared__ float sm_acc[GROUPS][kQB][D];
  __shared__ float2 sm_ml[GROUPS][kQB];

  const Unit un = tab.unit(blockIdx.y);
  const int chunk = blockIdx.x;
  if (chunk >= dec_chunks(un.len, sh.dec_chunk)) return;               // the grid is as wide as the longest unit needs
  const int clen = dec_chunk_len(un.len, sh.dec_chunk);
  const int t0 = chunk * clen;
  const int t1 = min(un.len, t0 + clen);
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int grp = lane / LPR, piece = lane % LPR;
  const int group = wave * RPW + grp;
  const int R = sh.R;

  const uint4* Kp = reinterpret_cast<const uint4*>(K + (size_t)un.in_row * D) + piece;
  const uint4* Vp = reinterpret_cast<const uint4*>(V + (size_t)un.in_row * D) + piece;
  const uint4* Qp = reinterpret_cast<const uint4*>(Q + (size_t)un.index * R * D) + piece;
  const int32_t* cnt = counts ? counts + un.in_row : nullptr;

  for (int qb = 0; qb < R; qb += kQB) {
    float qf[kQB][EPL];
#pragma unroll
    for (int j = 0; j < kQB; ++j) {
      const uint4 raw = Qp[(size_t)min(qb + j, R - 1) * LPR];      // rows past R repeat the last one
      Piece<T>::unpack(raw, qf[j]);
    }
    float m[kQB], l[kQB], acc[kQB][EPL];
#pragma unroll
    for (int j = 0; j < kQB; ++j) {
      m[j] = -INFINITY;
      l[j] = 0.f;
#pragma unroll
      for (int i = 0; i < EPL; ++i) acc[j][i] = 0.f;
    }

    // kUnroll rows per lane group and trip, all their loads issued before the first use
    for (int tb = t0 + group; tb < t1; tb += GROUPS * kUnroll) {
      uint4 kraw[kUnroll], vraw[kUnroll];
      float cc[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int t = tb + u * GROUPS;
        const int tc = min(t, t1 - 1);
        kraw[u] = Kp[(size_t)tc * LPR];
        vraw[u] = Vp[(size_t)tc * LPR];
        cc[u] = cnt ? (float)cnt[tc] : 1.f;
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if (tb + u * GROUPS >= t1) break;                        // uniform per lane group
        float kf[EPL], vf[EPL];
        Piece<T>::unpack(kraw[u], kf);
        Piece<T>::unpack(vraw[u], vf);
        const float c = cc[u];
#pragma unroll
        for (int j = 0; j < kQB; ++j) {
          float d = 0.f;
#pragma unroll
          for (int i = 0; i < EPL; ++i) d = fmaf(qf[j][i], kf[i], d);
          const float s = row_group_sum<LPR>(d) * sh.scale_log2;
          // online softmax; the running maximum rises only a few times per lane group, so the rescale of
          // the numerator stays out of the common path (the first row meets m = -inf: corr = 0)
          if (s > m[j]) {
            const float corr = __builtin_amdgcn_exp2f(m[j] - s);
            l[j] *= corr;
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[j][i] *= corr;
            m[j] = s;
          }
          const float p = __builtin_amdgcn_exp2f(s - m[j]);
          l[j] = fmaf(c, p, l[j]);                               // c copies of the slot in the denominator
#pragma unroll
          for (int i = 0; i < EPL; ++i) acc[j][i] = fmaf(p, vf[i], acc[j][i]);
        }
      }
    }

    // the lane groups of the workgroup, in group order
#pragma unroll
    for (int j = 0; j < kQB; ++j) {
#pragma unroll
      for (int i = 0; i < EPL; ++i) sm_acc[group][j][piece * EPL + i] = acc[j][i];
      if (piece == 0) sm_ml[group][j] = make_float2(m[j], l[j]);
    }
    __syncthreads();
    for (int o = tid; o < kQB * D; o += kThreads) {
      const int j = o / D, dch = o % D;
      if (qb + j < R) {
        float M = -INFINITY;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) M = fmaxf(M, sm_ml[g][j].x);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
          const float2 ml = sm_ml[g][j];
          if (ml.y > 0.f) {                                      // a group that saw no row has m = -inf, l = 0
            const float w = __builtin_amdgcn_exp2f(ml.x - M);
            num = fmaf(sm_acc[g][j][dch], w, num);
            den = fmaf(ml.y, w, den);
          }
        }
        float* dst = part + part_index(un.index, chunk, R, qb + j, D);
        dst[dch] = num;
        if (dch == 0) { dst[D] = M; dst[D + 1] = den; }
      }
    }
    __syncthreads();
  }
}

// out[unit, row, :] from the unit's chunk partials, in chunk order.  One workgroup per (unit, row), PARTS * D threads:
// thread (g, d) adds up the g-th part of the chunks in order, eight at a time, and the parts are added in order.
// Bound by latency: everything a thread needs is requested at once, so that the partials cost one round trip (a workgroup of
// D threads that went over the chunks eight at a time, for the maximum and again for the sums, made eight of them: 5.7 us
// for 8 units of 32 chunks, 3.0 now).  Four parts, or one where no unit has more than eight chunks (256 units of four:
// 4.4 us, 5.1 with four parts).
template <int D, int PARTS, typename Tab>
__global__ __launch_bounds__(PARTS * D) void decode_reduce_kernel(const Tab tab, const Shape sh,
                                                          const float* __restrict__ part, float* __restrict__ out) {
  constexpr int PER = PARTS == 1 ? 8 : kMaxChunks / PARTS;   // most chunks of a part
  static_assert(kMaxChunks <= kWave && PER % 8 == 0, "a lane per chunk, eight chunks' sums at a time");
  __shared__ float sm_num[PARTS][D];
  const int R = sh.R;
  const Unit un = tab.unit(blockIdx.x / R);
  const int row = blockIdx.x % R;
  const int nc = dec_chunks(un.len, sh.dec_chunk);
  const int tid = threadIdx.x, d = tid % D, g = __builtin_amdgcn_readfirstlane(tid / D), lane = tid % kWave;
  // (of parts that have more than eight chunks, the rest in a second batch)
  const int per = (nc + PARTS - 1) / PARTS;
  const int c0 = g * per, c1 = min(nc, c0 + per);
  const float* src = part + part_index(un.index, 0, R, row, D);
  const uint32_t stride = (uint32_t)R * (D + 2);
  float x[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) x[i] = 0.f;
#pragma unroll
  for (int i0 = 0; i0 < PER; i0 += 8) {
    if (c0 + i0 < c1) {
#pragma unroll
      for (int i = i0; i < i0 + 8; ++i) x[i] = src[min(c0 + i, nc - 1) * stride + d];
    }
  }
  const float m = src[min(lane, nc - 1) * stride + D];
  const float l = lane < nc ? src[min(lane, nc - 1) * stride + D + 1] : 0.f;
  float M = lane < nc ? m : -INFINITY;
#pragma unroll
  for (int k = 32; k >= 1; k >>= 1) M = fmaxf(M, __shfl_xor(M, k, kWave));
  const uint64_t used = __ballot(l > 0.f);       // (a chunk without a term is left out, whatever its partial holds)
  const float w = __builtin_amdgcn_exp2f(m - M);
  float den = l > 0.f ? l * w : 0.f;
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) den += __shfl_xor(den, k, kWave);
  float num = 0.f;
#pragma unroll
  for (int i0 = 0; i0 < PER; i0 += 8) {
    float n8 = 0.f;
#pragma unroll
    for (int i = i0; i < i0 + 8; ++i) {
      const float wc = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), min(c0 + i, kWave - 1)));
      n8 = c0 + i < c1 && ((used >> (c0 + i)) & 1) ? fmaf(x[i], wc, n8) : n8;
    }
    num += n8;
  }
  sm_num[g][d] = num;
  __syncthreads();
  if (g == 0) {
    num = sm_num[0][d];
#pragma unroll
    for (int i = 1; i < PARTS; ++i) num += sm_num[i][d];
    out[((size_t)un.index * R + row) * D + d] = num / den;
  }
}

// ------------------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& u) { return __builtin_bit_cast(bf16x8, u); }
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

constexpr int kMfmaThreads = 256;
constexpr int kMfmaWaves = kMfmaThreads / kWave;
constexpr int kTile = 32;

// The wavefronts' numerators, maxima and denominators (in LDS) -> the chunk's partial result for query rows qb ..
template <int D>
__device__ __forceinline__ void combine_waves(const float (&sm_acc)[kMfmaWaves][kTile][D + 4], int unit_index,
                                              int chunk, int R, int qb, float* __restrict__ part) {
  for (int o = threadIdx.x; o < kTile * D; o += kMfmaThreads) {
    const int q = o / D, dch = o % D;
    if (qb + q < R) {
      float M = -INFINITY;
#pragma unroll
      for (int w = 0; w < kMfmaWaves; ++w) M = fmaxf(M, sm_acc[w][q][D]);
      float num = 0.f, den = 0.f;
#pragma unroll
      for (int w = 0; w < kMfmaWaves; ++w) {
        const float lw = sm_acc[w][q][D + 1];
        if (lw > 0.f) {                                      // a wavefront that had no tile has m = -inf, l = 0
          const float wgt = __builtin_amdgcn_exp2f(sm_acc[w][q][D] - M);
          num = fmaf(sm_acc[w][q][dch], wgt, num);
          den = fmaf(lw, wgt, den);
        }
      }
      float* dst = part + part_index(unit_index, chunk, R, qb + q, D);
      dst[dch] = num;
      if (dch == 0) { dst[D] = M; dst[D + 1] = den; }
    }
  }
}

// Per tile of 32 cache rows and block of 32 query rows (one per lane column):
//   S[t, q] = K_tile Q^T               8 (D = 128) products; a lane holds one query column and 16 rows
//   online softmax per column          the running maximum is lane-private (exchanged once between the halves of
//                                      the wavefront); the numerator is rescaled only when the maximum rises
//   Y = V_tile[:, 32 db ..] I          the V block in the accumulator layout, which is the token-major operand
//                                      layout the next product needs (exact: bf16 times one)
//   O^T[d, q] += Y^T P                 P as a bf16 pair hi + lo
template <int D, typename Tab>
__global__ __launch_bounds__(kMfmaThreads, 2) void decode_mfma_kernel(
    const Tab tab, const Shape sh, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const int32_t* __restrict__ counts, float* __restrict__ part) {
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int ROWB = D * 2;
  constexpr int ACCW = D + 4;               // numerator, maximum, denominator; rows stay 16-byte aligned
  __shared__ __attribute__((aligned(16))) float sm_acc[kMfmaWaves][kTile][ACCW];
  __shared__ __attribute__((aligned(16))) float sm_cnt[kMfmaWaves][kTile];

  const Unit un = tab.unit(blockIdx.y);
  const int chunk = blockIdx.x;
  if (chunk >= dec_chunks(un.len, sh.dec_chunk)) return;               // the grid is as wide as the longest unit needs
  const int clen = dec_chunk_len(un.len, sh.dec_chunk);
  const int t0 = chunk * clen;
  const int t1 = min(un.len, t0 + clen);
  const int ntiles = (t1 - t0 + kTile - 1) / kTile;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int R = sh.R;
  const float sl2 = sh.scale_log2;
  const unsigned char* Kg = reinterpret_cast<const unsigned char*>(K + (size_t)un.in_row * D);
  const unsigned char* Vg = reinterpret_cast<const unsigned char*>(V + (size_t)un.in_row * D);
  const uint16_t* Qu = Q + (size_t)un.index * R * D;
  const int32_t* cnt = counts ? counts + un.in_row : nullptr;

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

  for (int qb = 0; qb < R; qb += kTile) {
    const int qrow = qb + col;
    bf16x8 bq[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      uint4 raw = make_uint4(0, 0, 0, 0);
      if (qrow < R) raw = *reinterpret_cast<const uint4*>(Qu + (size_t)qrow * D + kk * 16 + 8 * half);
      bq[kk] = as_bf16x8(raw);
    }
    f32x16 accO[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) accO[db] = zero;
    float m_run = -INFINITY, l_run = 0.f;

    for (int j = wave; j < ntiles; j += kMfmaWaves) {
      // the ragged last tile is moved back to end at the chunk's end (every unit on this path has at least 32
      // rows); the `shift` rows it shares with the tile before drop out
      const int tile_t0 = t0 + j * kTile;
      const int base_t = min(tile_t0, t1 - kTile);
      const int shift = tile_t0 - base_t;
      // operands straight from memory: this lane's row of the tile, 16 bytes per k-step
      const unsigned char* krow = Kg + (size_t)(base_t + col) * ROWB + half * 16;
      const unsigned char* vrow = Vg + (size_t)(base_t + col) * ROWB + half * 16;
      bf16x8 ka[KS], va[KS];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) ka[kk] = as_bf16x8(*reinterpret_cast<const uint4*>(krow + kk * 32));
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) va[kk] = as_bf16x8(*reinterpret_cast<const uint4*>(vrow + kk * 32));
      if (cnt != nullptr && half == 0) sm_cnt[wave][col] = (float)cnt[base_t + col];

      f32x16 acc = zero;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk], bq[kk], acc, 0, 0, 0);
      // accumulator element v: cache row 8 (v / 4) + 4 half + v % 4 of the tile, query column `col`
      float sv[16];
      float tm = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = 8 * (v / 4) + 4 * half + (v % 4);
        sv[v] = (row >= shift) ? acc[v] * sl2 : -INFINITY;
        tm = fmaxf(tm, sv[v]);
      }
      tm = fmaxf(tm, __shfl_xor(tm, 32, kWave));           // both halves feed the same column of O^T
      if (tm > m_run) {                                    // rare after the first tiles
        const float corr = __builtin_amdgcn_exp2f(m_run - tm);     // the first tile meets -inf: corr = 0
        l_run *= corr;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
          for (int v = 0; v < 16; ++v) accO[db][v] *= corr;
        }
        m_run = tm;
      }
      float p[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) p[v] = __builtin_amdgcn_exp2f(sv[v] - m_run);
      // denominator: c copies of every slot (the tile's sum first: a chain over all tiles rounds sixteen times as often
      // at the size of the whole)
      float sum = 0.f;
      if (cnt != nullptr) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 c4 = *reinterpret_cast<const float4*>(&sm_cnt[wave][8 * g + 4 * half]);
          sum = fmaf(c4.x, p[4 * g], sum);
          sum = fmaf(c4.y, p[4 * g + 1], sum);
          sum = fmaf(c4.z, p[4 * g + 2], sum);
          sum = fmaf(c4.w, p[4 * g + 3], sum);
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) sum += p[v];
      }
      l_run += sum;
      // as the operand of the next product, element i of k-step s is accumulator element 8 s + i
      bf16x8 ph[2], pl[2];
      split8(p, ph[0], pl[0]);
      split8(p + 8, ph[1], pl[1]);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        f32x16 y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[2 * db], ident[0], zero, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[2 * db + 1], ident[1], y, 0, 0, 0);
        float yf[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) yf[v] = y[v];
        const bf16x8 vt0 = pack8(yf), vt1 = pack8(yf + 8);     // exact: the values are bf16 numbers
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt0, ph[0], accO[db], 0, 0, 0);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt1, ph[1], accO[db], 0, 0, 0);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt0, pl[0], accO[db], 0, 0, 0);
        accO[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt1, pl[1], accO[db], 0, 0, 0);
      }
    }

    // the wavefronts of the workgroup, in wavefront order.  O^T element v of block db: channel
    // 32 db + 8 (v / 4) + 4 half + v % 4 of query column `col`
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        *reinterpret_cast<float4*>(&sm_acc[wave][col][32 * db + 8 * g + 4 * half]) =
            make_float4(accO[db][4 * g], accO[db][4 * g + 1], accO[db][4 * g + 2], accO[db][4 * g + 3]);
      }
    }
    if (half == 0) { sm_acc[wave][col][D] = m_run; sm_acc[wave][col][D + 1] = l_tot; }
    __syncthreads();
    combine_waves<D>(sm_acc, un.index, chunk, R, qb, part);
    __syncthreads();
  }
}

// fp32 caches: the same scheme with v_mfma_f32_32x32x2_f32 (fp32 products and sums).  Both operands of both products
// come from memory as they lie: in S = K Q^T a lane holds one row of K, every second 16-byte piece of it (the
// contraction index may be split between the halves of the wavefront in any way that both operands share); in
// O^T += V^T P step v contracts the two rows 8 (v / 4) + 4 half + v % 4, for which the lane's accumulator element v of
// S IS the operand, and the other one is a piece of D / 32 neighbouring channels of that row of V, channel
// D / 32 * i + e being row i of accumulator e.  So nothing is turned and nothing staged but the Q block.
// What bounds it: 128 products of 64 cycles per 32 rows (D = 128) and 32 KB, about the same time at 2 wavefronts per
// SIMD; the vector-ALU kernel reads the cache once per four query rows instead (32 caches of 16384 rows, 32 query rows:
// 134 us here, 4.0 TB/s, and 731 there).
template <int D, typename Tab>
__global__ __launch_bounds__(kMfmaThreads, 2) void decode_mfma_f32_kernel(
    const Tab tab, const Shape sh, const float* __restrict__ Q, const float* __restrict__ K,
    const float* __restrict__ V, const int32_t* __restrict__ counts, float* __restrict__ part) {
  constexpr int NP = D / 8;                 // 16-byte pieces of a row per half of the wavefront
  constexpr int LPR = D / 4;                // 16-byte pieces per row
  constexpr int DB = D / 32;                // channels per lane of a V row = accumulators of O^T
  constexpr int ACCW = D + 4;
  typedef float vpiece __attribute__((ext_vector_type(DB)));
  // the Q block (piece s of row r in slot s ^ r % LPR) during the tiles, the wavefronts' results afterwards
  __shared__ __attribute__((aligned(16))) float sm_acc[kMfmaWaves][kTile][ACCW];
  __shared__ __attribute__((aligned(16))) float sm_cnt[kMfmaWaves][kTile];
  float4* sm_q = reinterpret_cast<float4*>(&sm_acc[0][0][0]);
  static_assert(kTile * LPR * 16 <= sizeof(sm_acc), "the Q block fits");

  const Unit un = tab.unit(blockIdx.y);
  const int chunk = blockIdx.x;
  if (chunk >= dec_chunks(un.len, sh.dec_chunk)) return;               // the grid is as wide as the longest unit needs
  const int clen = dec_chunk_len(un.len, sh.dec_chunk);
  const int t0 = chunk * clen;
  const int t1 = min(un.len, t0 + clen);
  const int ntiles = (t1 - t0 + kTile - 1) / kTile;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int R = sh.R;
  const float sl2 = sh.scale_log2;
  const float* Kg = K + (size_t)un.in_row * D;
  const float* Vg = V + (size_t)un.in_row * D;
  const float* Qu = Q + (size_t)un.index * R * D;
  const int32_t* cnt = counts ? counts + un.in_row : nullptr;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // the ragged last tile is moved back to end at the chunk's end (every unit on this path has at least 32 rows)
  auto tile_base = [&](int j) { return min(t0 + j * kTile, t1 - kTile); };
  auto load_keys = [&](int j, float4 (&a)[NP]) {
    const float4* src = reinterpret_cast<const float4*>(Kg + (size_t)(tile_base(j) + col) * D) + half;
#pragma unroll
    for (int i = 0; i < NP; ++i) a[i] = src[2 * i];
  };

  for (int qb = 0; qb < R; qb += kTile) {
    float4 a[NP];
    asm volatile("" ::: "memory");            // (not hoisted out of the loop over the query rows: it would be spilled)
    load_keys(min(wave, ntiles - 1), a);
    for (int i = tid; i < kTile * LPR; i += kMfmaThreads) {
      const int r = i / LPR, s = i % LPR;
      const int qrow = min(qb + r, R - 1);                   // rows past R repeat the last one
      sm_q[r * LPR + (s ^ (r % LPR))] = reinterpret_cast<const float4*>(Qu + (size_t)qrow * D)[s];
    }
    __syncthreads();
    f32x16 accO[DB];
#pragma unroll
    for (int e = 0; e < DB; ++e) accO[e] = zero;
    float m_run = -INFINITY, l_run = 0.f;

    for (int j = wave; j < ntiles; j += kMfmaWaves) {
      const int base_t = tile_base(j);
      const int shift = t0 + j * kTile - base_t;             // leading rows that belong to the tile before
      // the rows of V in two halves, and the next tile's Keys between them: all at once does not fit the registers (the
      // marks keep the compiler from issuing them earlier)
      vpiece vv[16];
      auto load_values = [&](auto half_c) {
#pragma unroll
        for (int v = 8 * decltype(half_c)::value; v < 8 * decltype(half_c)::value + 8; ++v) {
          const int row = 8 * (v / 4) + 4 * half + (v % 4);
          vv[v] = reinterpret_cast<const vpiece*>(Vg + (size_t)(base_t + row) * D)[col];
        }
        asm volatile("" ::: "memory");
      };
      if (cnt != nullptr && half == 0) sm_cnt[wave][col] = (float)cnt[base_t + col];
      // Four products of each logit from zero, then added up in pairs, and eight rows of V from zero below: this
      // instruction rounds at every product, and one chain through all of them had an error against 64 bits of 1.6 to
      // 3.3 times the vector-ALU kernel's.  This way it is 0.97 to 1.04 times that (means over 6 inputs each of 6 shapes
      // from 1000 to 30000 rows and 7 to 64 query rows, 0.99 over all) for 5 % of the time at 32 query rows.
      f32x16 acc, pair[5];
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const float4 q4 = sm_q[col * LPR + ((2 * i + half) ^ (col % LPR))];
        const float qv[4] = {q4.x, q4.y, q4.z, q4.w};
        const float kv[4] = {a[i].x, a[i].y, a[i].z, a[i].w};
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          f32x16 s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[2 * g], qv[2 * g], zero, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[2 * g + 1], qv[2 * g + 1], s, 0, 0, 0);
          // (a binary counter of finished sums: level l holds one of 2^l groups)
          int level = 0;
#pragma unroll
          for (int l = 0; l < 5; ++l) {
            if (((2 * i + g) >> l) % 2 == 1 && level == l) {
#pragma unroll
              for (int v = 0; v < 16; ++v) s[v] += pair[l][v];
              level = l + 1;
            }
          }
          if (2 * i + g == 2 * NP - 1) acc = s;
          else pair[level] = s;
        }
        if (i == NP / 2 - 1) load_values(std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
      load_values(std::integral_constant<int, 1>{});
      // accumulator element v: cache row 8 (v / 4) + 4 half + v % 4 of the tile, query column `col`
      float p[16];
      float tm = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = 8 * (v / 4) + 4 * half + (v % 4);
        p[v] = (row >= shift) ? acc[v] * sl2 : -INFINITY;
        tm = fmaxf(tm, p[v]);
      }
      tm = fmaxf(tm, __shfl_xor(tm, 32, kWave));             // both halves feed the same column of O^T
      if (tm > m_run) {                                      // rare after the first tiles
        const float corr = __builtin_amdgcn_exp2f(m_run - tm);       // the first tile meets -inf: corr = 0
        l_run *= corr;
#pragma unroll
        for (int e = 0; e < DB; ++e) {
#pragma unroll
          for (int v = 0; v < 16; ++v) accO[e][v] *= corr;
        }
        m_run = tm;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) p[v] = __builtin_amdgcn_exp2f(p[v] - m_run);
      if (shift > 0) {                        // a row that dropped out counts for nothing whatever its Value is
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          if (8 * (v / 4) + 4 * half + (v % 4) < shift) vv[v] = vpiece{};
        }
      }
      // denominator: c copies of every slot
      float sum = 0.f;                        // (the tile's first, as above)
      if (cnt != nullptr) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 c4 = *reinterpret_cast<const float4*>(&sm_cnt[wave][8 * g + 4 * half]);
          sum = fmaf(c4.x, p[4 * g], sum);
          sum = fmaf(c4.y, p[4 * g + 1], sum);
          sum = fmaf(c4.z, p[4 * g + 2], sum);
          sum = fmaf(c4.w, p[4 * g + 3], sum);
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) sum += p[v];
      }
      l_run += sum;
      // (eight rows from zero, like the logits' four products)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_keys(min(j + kMfmaWaves, ntiles - 1), a);     // flies during the rest (the last tile is fetched twice)
          asm volatile("" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < DB; ++e) {
          f32x16 s = zero;
#pragma unroll
          for (int v = 8 * h; v < 8 * h + 8; ++v) s = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[v][e], p[v], s, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 16; ++v) accO[e][v] += s[v];
        }
      }
    }

    // the wavefronts of the workgroup, in wavefront order.  O^T element v of accumulator e: channel
    // DB (8 (v / 4) + 4 half + v % 4) + e of query column `col`
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    __syncthreads();                          // the Q block has been read
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      vpiece o;
#pragma unroll
      for (int e = 0; e < DB; ++e) o[e] = accO[e][v];
      *reinterpret_cast<vpiece*>(&sm_acc[wave][col][DB * (8 * (v / 4) + 4 * half + (v % 4))]) = o;
    }
    if (half == 0) { sm_acc[wave][col][D] = m_run; sm_acc[wave][col][D + 1] = l_tot; }
    __syncthreads();
    combine_waves<D>(sm_acc, un.index, chunk, R, qb, part);
    __syncthreads();
  }
}

// most: chunks of the unit that has most of them
template <int D>
hipError_t launch_reduce(const UnitTable& tab, const Shape& sh, int most, const float* part, float* out, hipStream_t stream) {
  const dim3 grid(tab.n_units * sh.R);
  launch_with_table(tab, [&](const auto& t) {
    if (most <= 8)
      hipLaunchKernelGGL((decode_reduce_kernel<D, 1, KVS_TABLE_TYPE(t)>), grid, dim3(D), 0, stream, t, sh, part, out);
    else
      hipLaunchKernelGGL((decode_reduce_kernel<D, 4, KVS_TABLE_TYPE(t)>), grid, dim3(4 * D), 0, stream, t, sh, part, out);
  });
  return hipGetLastError();
}

template <int D>
hipError_t launch_mfma_f32(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                           const int32_t* counts, float* part, float* out, hipStream_t stream) {
  const int widest = most_chunks(tab, sh.dec_chunk);
  launch_with_table(tab, [&](const auto& t) {
    hipLaunchKernelGGL((decode_mfma_f32_kernel<D, KVS_TABLE_TYPE(t)>), dim3(widest, tab.n_units), dim3(kMfmaThreads), 0, stream, t, sh,
                       (const float*)Q, (const float*)K, (const float*)V, counts, part);
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce<D>(tab, sh, widest, part, out, stream);
}

template <int D>
hipError_t launch_mfma(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                       const int32_t* counts, float* part, float* out, hipStream_t stream) {
  const int widest = most_chunks(tab, sh.dec_chunk);
  launch_with_table(tab, [&](const auto& t) {
    hipLaunchKernelGGL((decode_mfma_kernel<D, KVS_TABLE_TYPE(t)>), dim3(widest, tab.n_units), dim3(kMfmaThreads), 0, stream, t, sh,
                       (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)V, counts, part);
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce<D>(tab, sh, widest, part, out, stream);
}

template <typename T, int D>
hipError_t launch_t(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const void* V,
                    const int32_t* counts, float* part, float* out, hipStream_t stream) {
  const int widest = most_chunks(tab, sh.dec_chunk);
  auto launch = [&](auto unroll) {
    launch_with_table(tab, [&](const auto& t) {
      hipLaunchKernelGGL((decode_partial_kernel<T, D, decltype(unroll)::value, KVS_TABLE_TYPE(t)>), dim3(widest, tab.n_units),
                         dim3(kThreads), 0, stream, t, sh, (const T*)Q, (const T*)K, (const T*)V, counts, part);
    });
  };
  // A launch with no more than a workgroup per compute unit is a chain of round trips, and four rows in flight per lane
  // group make fewer of them (one cache of 32768 rows 25.3 -> 23.6 us, 16 of 4096 18.8 -> 17.8); more workgroups have the
  // rows in flight between them (64 of 4096: 29.5 with two, 34.3 with four; 256: 112 and 126).
  if (widest * tab.n_units <= 256) launch(std::integral_constant<int, kMoreRows>{});
  else launch(std::integral_constant<int, kFewRows>{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce<D>(tab, sh, widest, part, out, stream);
}

// Rows per workgroup of a launch (n_units units, `rows` rows, `first` of them in the first unit), from the lengths alone:
// a call's results don't depend on its budgets.  Every workgroup has a fixed cost (the query block, the wavefronts'
// results combined, a partial result written), and the launch takes as long as its rounds of resident workgroups do, two
// per CU for the MFMA kernels and four for the vector-ALU ones.
// Equal lengths: the fewest rounds whose workgroups take up to 2048 rows (MFMA, up to 32 query rows) or 1024, at least 256,
// and for them the shortest pieces that fit.  32 caches of 22047 rows, 16 query rows: 78.2 us in one round, with twice to
// four times the workgroups 85 and 97; 64 of 4096, 32 query rows: 37.7 against 48.1; 64 of 17187, where one round would
// take more rows than that: 64 query rows 222 us with two rounds of 1088, 272 with 1024 rows, which don't fit two; 4 query
// rows (vector ALU) 115 with two rounds, 137 with 1024 rows.
// Different lengths leave the last workgroups of the long caches alone on the chip, and smaller pieces even that out:
// about 2048 workgroups on the vector ALU (100 caches of 2.7 K to 21 K rows, 4 query rows: 148 us against 164 at 1024),
// 768 for the MFMA kernels (64 caches, 500000 rows, 8 query rows: 56.4 us, 65.2 at 512), and from 786432 rows on, where
// 768 would be cut off at 1024 rows each, rounds of up to 1024 rows, two at least (256 caches, 1100000 rows, 64 query
// rows: 275 us, 320 with 1024 rows).
// The vector-ALU kernels go down to 64 rows in a launch that would leave compute units without a workgroup (8 caches
// of 4096 rows: 16.9 us with 128 against 20.9; 64 caches stay: 30.7 with 256 against 37.0); the MFMA kernels'
// wavefronts take 32 rows each (8 caches of 4096 rows, 32 query rows: 20.3 us with 256, 20.6 with 128, 26.7 with 64).
int rows_per_workgroup(int n_units, int first, bool even, long long rows, bool mfma, int R) {
  auto round_up = [](long long x) { return (x + kWave - 1) / kWave * kWave; };
  if (!mfma && rows < 256 * kDecMinChunk) return (int)std::max<long long>(kWave, round_up(rows / 256));
  const long long slots = mfma ? 512 : 1024;
  if (even) {
    const long long most = mfma && R <= kTile ? 2048 : 1024;
    for (long long rounds = std::max<long long>(1, rows / (slots * most));; ++rounds) {
      long long chunk = std::max<long long>(kDecMinChunk, round_up(rows / (slots * rounds)));
      while (chunk <= most && (long long)n_units * dec_chunks(first, (int)chunk) > slots * rounds) chunk += kWave;
      if (chunk <= most) return (int)chunk;
    }
  }
  if (!mfma || rows < 3 * 256 * 1024) {
    const long long chunk = round_up(rows / (mfma ? 768 : 2048));
    return (int)std::min<long long>(std::max<long long>(kDecMinChunk, chunk), 1024);
  }
  for (long long rounds = 2;; ++rounds) {
    const long long chunk = round_up(rows / (slots * rounds));
    if (chunk <= 1024) return (int)chunk;
  }
}

}  // namespace

hipError_t launch_decode(const UnitTable& tab, const Shape& sh_in, kvs_dtype dt, const void* Q, const void* K,
                         const void* V, const int32_t* counts, float* part, float* out, hipStream_t stream) {
  // The vector-ALU kernels read the cache once per four query rows, the MFMA kernels once per 32.  bf16: up to four
  // rows they are equally fast (both latency-bound on caches of a few thousand rows), above that the MFMA kernel wins
  // (64 caches of 4096 rows: 42 against 62 us at 8 rows, 55 against 200 us at 32 rows).  fp32, 32 caches: 43.5 against
  // 62 us at 8 rows and 4096 cache rows, 134 against 731 us at 32 rows and 16384 cache rows.
  // KVS_DEBUG_DECODE_PATH forces one of them (used by the tests to cover both).
  Shape sh = sh_in;
  const int force = debug_switch(KVS_DEBUG_DECODE_PATH);
  bool mfma = sh.R > kQB;
  if (force == 1) mfma = false;
  if (force == 2) mfma = true;
  const int first = tab.unit(0).len;
  int shortest = first;
  long long rows = 0;
  bool even = true;                                        // (the budgets don't matter here: tab.even is not it)
  for (int i = 0; i < tab.n_units; ++i) {
    const int len = tab.unit(i).len;
    rows += len;
    shortest = std::min(shortest, len);
    even = even && len == first;
  }
  if (shortest < kTile) mfma = false;                      // its tiles hold 32 whole rows
  sh.dec_chunk = rows_per_workgroup(tab.n_units, first, even, rows, mfma, sh.R);
  if (dt == KVS_F32) {
    if (mfma) {
      return sh.D == 64 ? launch_mfma_f32<64>(tab, sh, Q, K, V, counts, part, out, stream)
                        : launch_mfma_f32<128>(tab, sh, Q, K, V, counts, part, out, stream);
    }
    return sh.D == 64 ? launch_t<float, 64>(tab, sh, Q, K, V, counts, part, out, stream)
                      : launch_t<float, 128>(tab, sh, Q, K, V, counts, part, out, stream);
  }
  if (mfma) {
    return sh.D == 64 ? launch_mfma<64>(tab, sh, Q, K, V, counts, part, out, stream)
                      : launch_mfma<128>(tab, sh, Q, K, V, counts, part, out, stream);
  }
  return sh.D == 64 ? launch_t<uint16_t, 64>(tab, sh, Q, K, V, counts, part, out, stream)
                    : launch_t<uint16_t, 128>(tab, sh, Q, K, V, counts, part, out, stream);
}

}  // namespace kvs
