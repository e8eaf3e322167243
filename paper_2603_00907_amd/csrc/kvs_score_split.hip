// Score kernel for fp32 inputs and more than 64 query rows: the two sweeps of kvs_score_mfma.hip with every fp32 number
// taken as the sum of three bf16 numbers, so that the products run at the bf16 matrix rate (16 times the fp32 one).
//
// x = hi + mid + lo with hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid), each rounded to nearest: 24 bits and
// signs, so nothing is lost but what lies below 2^-27 of x, or below 2^-126, where bf16 has no normal numbers (see
// products_f32 for the rows where that counts).  Of the nine products six are formed (hi hi, hi mid, mid hi,
// mid mid, hi lo, lo hi; the others are below 2^-26 of the largest), each exact in the fp32 accumulator, in two chains
// from small to large.  48 MFMAs of 32 cycles per 32 x 32 logits (D = 128) against 64 of 64 cycles: the step over 8
// units of 32768 tokens with 128 rows takes 190 us against 241 with fp32 products, 64 units of 16384 683 against 875.
// The error of alpha_bar against 64 bits is smaller than with fp32 products and a running maximum (the products' sums take
// eight times as many rounding steps there): 23000 tokens, 96 to 320 rows, Queries of half, once and twice the usual size,
// 2-norm of the error 0.9e-7 to 1.2e-6 against 3.7e-7 to 2.0e-6, largest relative error 0.5e-6 to 0.7e-5 against 1.3e-6 to
// 1.5e-5.
//
// A workgroup's wavefronts own 32 query rows each (operands of all three parts in registers: 96 for D = 128) and walk
// the same tiles of 32 tokens: a tile is fetched, split once and left in LDS as three bf16 tiles (XOR-swizzled 16-byte
// pieces), one tile ahead of its use, the next one's loads in flight; one barrier per tile.  The split of the next tile
// sits between the products of this one (2 % faster than in front of them).  NW = 4 wavefronts: up to
// 128 rows, two workgroups per CU; NW = 8: one launch per 256 rows.  Accumulator layouts, statistics and the sum over
// the wavefronts in sweep 1 are those of kvs_score_shared.hip.
//
// Infinities and NaN (and numbers that round to infinity as bf16) have no such split: a tile whose sums come out not
// finite is done again with fp32 MFMAs, straight from memory, so that what it contributes is what it always did.  Nor have
// numbers below 2^-100, whose parts fall below 2^-126: a wavefront with such a query element, or with one so large that
// what a Key of that kind loses could count, takes fp32 MFMAs for all its tiles.
#include "kvs_mfma_tile.h"

namespace kvs {
namespace {

using namespace mfma;

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// eight floats -> three bf16 operands whose sum they are
__device__ __forceinline__ void split3(const float4& x, const float4& y, uint4& hi, uint4& mid, uint4& lo) {
  const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
  uint32_t h[4], m[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = f[2 * i], b = f[2 * i + 1];
    h[i] = cvt_pk_bf16(a, b);
    a -= bf16_lo(h[i]);
    b -= bf16_hi(h[i]);
    m[i] = cvt_pk_bf16(a, b);
    a -= bf16_lo(m[i]);
    b -= bf16_hi(m[i]);
    l[i] = cvt_pk_bf16(a, b);
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  mid = make_uint4(m[0], m[1], m[2], m[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

template <int D, int NW, int PHASE, typename Tab>
__global__ __launch_bounds__(NW * kWave, 2) void score_split_kernel(
    const Tab tab, const Shape sh, const float* __restrict__ Q, const float* __restrict__ K,
    const int32_t* __restrict__ counts_in, float* __restrict__ alpha_bar, float2* __restrict__ stats_part,
    const float* __restrict__ c_row, const int qp) {
  constexpr int KS = D / 16;                // MFMA k-steps
  constexpr int LPR = D / 8;                // 16-byte pieces per bf16 row
  constexpr int TILEB = kTile * D * 2;      // bytes of one part of a tile
  constexpr int PIECES = kTile * LPR;
  constexpr int THREADS = NW * kWave;
  constexpr int NP = (PIECES + THREADS - 1) / THREADS;       // pieces (8 floats) per thread and tile

  __shared__ __attribute__((aligned(1024))) unsigned char sm_k[2][3 * TILEB];
  __shared__ float sm_p[2][NW][kTile];      // sweep 1: the wavefronts' shares of alpha_bar, two tiles
  __shared__ __attribute__((aligned(16))) float sm_lc[2][kTile];   // sweep 0: log2 of the rows' cardinalities

  const int ui = find_unit(tab, blockIdx.x);
  const Unit un = tab.unit(ui);
  const int chunk = blockIdx.x - un.chunk_base;
  const int t0 = chunk * un.chunk_len;
  const int t1 = min(un.len, t0 + un.chunk_len);
  const int ntiles = (t1 - t0 + kTile - 1) / kTile;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int R = sh.R;
  const int rows_here = min(R - qp, NW * 32);
  const float sl2 = sh.scale_log2;
  const bool last_launch = qp + NW * 32 >= R;
  const int32_t* cnt = counts_in ? counts_in + un.in_row : nullptr;
  const float sc = cnt ? 1.f : sl2;         // sweep 0: the accumulators hold finished logits when cardinalities were added
  const float* Kg = K + (size_t)un.in_row * D;
  const float* Qu = Q + (size_t)un.index * R * D;
  const int q_first = 32 * wave;            // this wavefront's rows of the launch
  const bool idle = q_first >= rows_here;   // (it only fetches)

  // tile j: global memory -> registers (tokens past the chunk's end repeat its last one)
  float4 raw[NP][2];
  float raw_c = 1.f;
  auto fetch = [&](int j) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = tid + i * THREADS;
      const int t = min(t0 + j * kTile + p / LPR, t1 - 1);
      const float4* src = reinterpret_cast<const float4*>(Kg + (size_t)t * D + (p % LPR) * 8);
      if (PIECES % THREADS == 0 || p < PIECES) { raw[i][0] = src[0]; raw[i][1] = src[1]; }
    }
    if (PHASE == 0 && cnt != nullptr && tid < kTile) raw_c = (float)cnt[min(t0 + j * kTile + tid, t1 - 1)];
  };
  // ... -> three bf16 tiles in LDS (piece s of row r in slot s ^ r % LPR)
  auto put = [&](unsigned char* __restrict__ dst, int buf) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = tid + i * THREADS;
      const int row = p / LPR;
      const int at = row * (D * 2) + ((p % LPR) ^ (row % LPR)) * 16;
      uint4 hi, mid, lo;
      split3(raw[i][0], raw[i][1], hi, mid, lo);
      if (PIECES % THREADS == 0 || p < PIECES) {
        *reinterpret_cast<uint4*>(dst + at) = hi;
        *reinterpret_cast<uint4*>(dst + TILEB + at) = mid;
        *reinterpret_cast<uint4*>(dst + 2 * TILEB + at) = lo;
      }
    }
    if (PHASE == 0 && cnt != nullptr && tid < kTile) sm_lc[buf][tid] = even_log2(raw_c);
  };
  fetch(0);

  // this wavefront's query rows, split (rows past R repeat the last one).  plain: the split would lose what counts.  Below
  // 2^-100 an element's third part is no normal number, and a Key of up to 2^127 may meet what is lost (2^-127 or less of
  // the element); a Key's own loss, and a product of parts that is no normal number, count where they meet 2^90 or a scale
  // of 2^60.  Elsewhere either is below 2^-36 of the base-2 logit.
  bf16x8 bq[3][KS];
  u16x2 most = {0, 0}, least = {0xFFFF, 0xFFFF};             // of the elements' magnitudes, as bits of bf16 numbers
  {
    const float* qr = Qu + (size_t)min(qp + q_first + col, R - 1) * D + 8 * half;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const float4* src = reinterpret_cast<const float4*>(qr + 16 * kk);
      uint4 hi, mid, lo;
      split3(src[0], src[1], hi, mid, lo);
      for (const uint32_t w : {hi.x, hi.y, hi.z, hi.w}) {
        const u16x2 a = __builtin_bit_cast(u16x2, w & 0x7FFF7FFFu);
        most = __builtin_elementwise_max(most, a);
        least = __builtin_elementwise_min(least, a);
      }
      bq[0][kk] = __builtin_bit_cast(bf16x8, hi);
      bq[1][kk] = __builtin_bit_cast(bf16x8, mid);
      bq[2][kk] = __builtin_bit_cast(bf16x8, lo);
    }
  }
  bool plain = __any(sl2 >= 0x1p60f || __uint_as_float((uint32_t)max(most.x, most.y) << 16) * sl2 >= 0x1p90f);
  if (__any(min(least.x, least.y) < (__float_as_uint(0x1p-100f) >> 16))) {    // such an element, or a zero
    const float* qr = Qu + (size_t)min(qp + q_first + col, R - 1) * D + half * (D / 2);
    bool small = false;
#pragma unroll 1
    for (int i = 0; i < D / 2; ++i) small |= (qr[i] != 0.f) & (fabsf(qr[i]) < 0x1p-100f);
    plain |= __any(small);
  }
  // sweep 1: the normalisers of the lane's 16 accumulator rows (exp2(-inf) = 0: no such row)
  float cq[16];
  if (PHASE == 1) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int q = q_first + 8 * (v / 4) + 4 * half + (v % 4);
      cq[v] = q < rows_here ? c_row[(size_t)un.index * R + qp + q] : INFINITY;
    }
  }
  const int lim = last_seen_row(sh.causal, un.len, qp + q_first + col);    // sweep 0: of this lane's query column
  put(sm_k[0], 0);
  if (ntiles > 1) fetch(1);

  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint32_t a_ofs[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) a_ofs[kk] = col * (D * 2) + ((2 * kk + half) ^ (col % LPR)) * 16;
  auto mul = [&](const bf16x8& k, const bf16x8& q, const f32x16& c) {
    return PHASE == 0 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q, c, 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_bf16(q, k, c, 0, 0, 0);
  };
  // dot products of tile j (in `rd`): two chains of 3 KS products, small ones first.  The next tile is split and put
  // into `wr` between them (the two are different buffers, and saying so lets the compiler mix the two streams).
  auto products_and_put = [&](const unsigned char* __restrict__ rd, unsigned char* __restrict__ wr, int j) {
    f32x16 a = zero, b = zero;
    bf16x8 kh[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const bf16x8 kl = *reinterpret_cast<const bf16x8*>(rd + 2 * TILEB + a_ofs[kk]);
      kh[kk] = *reinterpret_cast<const bf16x8*>(rd + a_ofs[kk]);
      a = mul(kl, bq[0][kk], a);
      b = mul(kh[kk], bq[2][kk], b);
    }
    if (j + 1 < ntiles) {
      put(wr, (j + 1) & 1);
      if (j + 2 < ntiles) fetch(j + 2);
    }
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const bf16x8 km = *reinterpret_cast<const bf16x8*>(rd + TILEB + a_ofs[kk]);
      a = mul(km, bq[1][kk], a);
      b = mul(kh[kk], bq[1][kk], b);
      a = mul(km, bq[0][kk], a);
      b = mul(kh[kk], bq[0][kk], b);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) a[v] += b[v];
    return a;
  };
  // the same with fp32 products, from memory (numbers that have no split)
  auto products_f32 = [&](int j) {
    f32x16 a = zero;
    const float4* kr = reinterpret_cast<const float4*>(Kg + (size_t)min(t0 + j * kTile + col, t1 - 1) * D) + half * (D / 8);
    const float4* qr = reinterpret_cast<const float4*>(Qu + (size_t)min(qp + q_first + col, R - 1) * D) + half * (D / 8);
#pragma unroll 1
    for (int i = 0; i < D / 8; ++i) {
      const float4 k4 = kr[i], q4 = qr[i];
      const float kv[4] = {k4.x, k4.y, k4.z, k4.w}, qv[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        a = PHASE == 0 ? __builtin_amdgcn_mfma_f32_32x32x2f32(kv[e], qv[e], a, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x2f32(qv[e], kv[e], a, 0, 0, 0);
    }
    return a;
  };

  float m_run = -INFINITY, l_run = 0.f, l_lost = 0.f;       // (see add_compensated)
  // sweep 0, any tile: what is masked drops out, the reference rises with the maximum (see kSumLimit)
  auto add_terms_any = [&](f32x16 acc, int j) {
    const int tile_t0 = t0 + j * kTile;
    if (t1 - tile_t0 < kTile || (sh.causal > 0 && tile_t0 + kTile > un.len - sh.causal + 1)) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int t = tile_t0 + 8 * (v / 4) + 4 * half + (v % 4);
        if (t >= t1 || t > lim) acc[v] = -INFINITY;
      }
    }
    if (cnt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 lc = *reinterpret_cast<const float4*>(&sm_lc[j & 1][8 * g + 4 * half]);
        acc[4 * g] = fmaf(acc[4 * g], sl2, lc.x);
        acc[4 * g + 1] = fmaf(acc[4 * g + 1], sl2, lc.y);
        acc[4 * g + 2] = fmaf(acc[4 * g + 2], sl2, lc.z);
        acc[4 * g + 3] = fmaf(acc[4 * g + 3], sl2, lc.w);
      }
    }
    float tm = acc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) tm = fmaxf(tm, acc[v]);
    const float m_new = fmaxf(m_run, fmaf(tm, sc, kHeadroom));
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    float s = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) s += ex2(fmaf(acc[v], sc, -m_safe));
    const float down = ex2(m_run - m_safe);
    l_run *= down;
    l_lost *= down;
    add_compensated(l_run, l_lost, s);
    m_run = m_new;
  };
  // sweep 1: this lane's token summed over the wavefront's query rows
  auto share = [&](const f32x16& acc, int j) {
    const int tile_t0 = t0 + j * kTile;
    const bool masked = sh.causal > 0 && tile_t0 + kTile > un.len - sh.causal + 1;
    float p = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = ex2(fmaf(acc[4 * g + i], sl2, -cq[4 * g + i]));
      if (masked) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = q_first + 8 * g + 4 * half + i;
          if (tile_t0 + col > last_seen_row(sh.causal, un.len, qp + q)) e[i] = 0.f;
        }
      }
      p += (e[0] + e[1]) + (e[2] + e[3]);
    }
    return p + __shfl_xor(p, 32, kWave);
  };
  // sweep 1: tile j's tokens (threads 0 .. 31)
  auto finish = [&](int j) {
    const int t = t0 + j * kTile + tid;
    if (tid < kTile && t < t1) {
      float p = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) p += sm_p[j & 1][w][tid];
      if (qp > 0) p += alpha_bar[un.in_row + t];             // the rows of the launches before
      // a row that stands for c tokens has c equal terms in every softmax sum (2^(e + log2 c) = c 2^e)
      if (cnt && last_launch) p *= (float)cnt[t];
      alpha_bar[un.in_row + t] = p;
    }
  };

  for (int j = 0; j < ntiles; ++j) {
    __syncthreads();                          // tile j is in place, nobody reads tile j - 1 any more
    if (PHASE == 1 && j > 0) finish(j - 1);
    f32x16 acc = products_and_put(sm_k[j & 1], sm_k[(j + 1) & 1], j);
    if (idle) {
      if (PHASE == 1 && half == 0) sm_p[j & 1][wave][col] = 0.f;
      continue;
    }
    if (PHASE == 0) {
      const int tile_t0 = t0 + j * kTile;
      if (!plain && j > 0 && cnt == nullptr && tile_t0 + kTile <= t1 &&
          !(sh.causal > 0 && tile_t0 + kTile > un.len - sh.causal + 1)) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v % 4] += ex2(fmaf(acc[v], sl2, -m_run));
        const float sum = (s[0] + s[1]) + (s[2] + s[3]);
        if (!__any(!(sum < kSumLimit))) {      // (else the reference is too low, or the sum is not a number)
          add_compensated(l_run, l_lost, sum);
          continue;
        }
      }
      const float l_old = l_run, m_old = m_run, lost_old = l_lost;
      add_terms_any(acc, j);
      if (plain || __any(!(l_run < INFINITY))) {
        l_run = l_old;
        l_lost = lost_old;
        m_run = m_old;
        add_terms_any(products_f32(j), j);
      }
    } else {
      float p = share(acc, j);
      if (plain || __any(!(p < INFINITY))) p = share(products_f32(j), j);
      if (half == 0) sm_p[j & 1][wave][col] = p;
    }
  }

  if (PHASE == 0) {
    // the two halves of a wavefront hold the same query column for different token rows
    l_run -= l_lost;
    const float m_o = __shfl_xor(m_run, 32, kWave);
    const float l_o = __shfl_xor(l_run, 32, kWave);
    const float m_n = fmaxf(m_run, m_o);
    const float m_s = (m_n == -INFINITY) ? 0.f : m_n;
    const float l_n = l_run * ex2(m_run - m_s) + l_o * ex2(m_o - m_s);
    const int q = q_first + col;
    if (half == 0 && q < rows_here)
      stats_part[((size_t)un.index * kMaxChunks + chunk) * R + qp + q] = make_float2(m_n, l_n);
  } else {
    __syncthreads();
    finish(ntiles - 1);
  }
}

template <int D, int NW>
hipError_t launch_t(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const int32_t* counts_in,
                    float* alpha_bar, const Workspace& ws, hipStream_t stream) {
  const dim3 grid(tab.total_chunks), block(NW * kWave);
  hipError_t e;
  for (int qp = 0; qp < sh.R; qp += NW * 32) {
    launch_with_table(tab, [&](const auto& t) {
      hipLaunchKernelGGL((score_split_kernel<D, NW, 0, KVS_TABLE_TYPE(t)>), grid, block, 0, stream, t, sh, (const float*)Q,
                         (const float*)K, counts_in, alpha_bar, ws.stats_part, ws.c_row, qp);
    });
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = launch_score_finalize(tab, sh, ws, stream)) != hipSuccess || alpha_bar == nullptr) return e;
  for (int qp = 0; qp < sh.R; qp += NW * 32) {
    launch_with_table(tab, [&](const auto& t) {
      hipLaunchKernelGGL((score_split_kernel<D, NW, 1, KVS_TABLE_TYPE(t)>), grid, block, 0, stream, t, sh, (const float*)Q,
                         (const float*)K, counts_in, alpha_bar, ws.stats_part, ws.c_row, qp);
    });
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_score_split(const UnitTable& tab, const Shape& sh, const void* Q, const void* K,
                              const int32_t* counts_in, float* alpha_bar, const Workspace& ws, hipStream_t stream) {
  if (sh.R <= 128) {
    return sh.D == 64 ? launch_t<64, 4>(tab, sh, Q, K, counts_in, alpha_bar, ws, stream)
                      : launch_t<128, 4>(tab, sh, Q, K, counts_in, alpha_bar, ws, stream);
  }
  return sh.D == 64 ? launch_t<64, 8>(tab, sh, Q, K, counts_in, alpha_bar, ws, stream)
                    : launch_t<128, 8>(tab, sh, Q, K, counts_in, alpha_bar, ws, stream);
}

}  // namespace kvs
