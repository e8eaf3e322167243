// Score kernel for more than 128 query rows (bf16): the two sweeps of kvs_score_mfma.hip with the rows spread over
// the wavefronts and the K tiles shared.
//
// What bounds these windows is arithmetic, not memory: per 32 tokens x 64 query rows a wavefront issues 16 MFMAs and
// 32 x (fma, exp2, add).  A bare loop of exactly these instructions, two wavefronts per SIMD, takes 0.31 us per such
// block on zeros and 0.41 to 0.43 us on random data (the chip lowers its clock under matrix work), which makes 105 us
// per sweep over 8 units of 131072 tokens with 512 rows.  So the operands must cost next to nothing: every wavefront
// owns up to 64 query rows, whose operands stay in its registers for the whole chunk (64 registers), and all
// wavefronts of the workgroup walk the same K tiles, staged through LDS once for all of them.  Before, every
// wavefront had tiles of its own and re-read the Q block from LDS for each of them, waiting for those reads, in one
// launch per 256 rows: the step on those 8 units took 533 us, with this kernel 466; 112 units of 32768 tokens with 224
// rows 1140 and 1064.  NW = 4 wavefronts cover up to 256 rows (two workgroups per CU), NW = 8 up to 512 (one per CU);
// beyond that there is one launch per 512 rows.
//
// K streams into a ring of stages by global_load_lds, 16-byte pieces XOR-swizzled by the row number; one barrier per stage.
// A stage is NW * 32 tokens, the next one on its way (LONG), or NW * 16 tokens, two on their way, always so with the pass over
// V, whose rows take registers (with the rows of V of NW * 32 tokens in registers, or half of them at a time, the kernel
// spilled, and sweep 1 of 64 units of 32768 tokens took 236 to 310 us instead of 210).  Long stages fill and drain the pipeline
// of products and terms less often; short ones waste less where a chunk ends inside one, and have more loads on their way
// (both measured, see launch_t).  The steps are blocks of 32 rows, which leaves registers for a whole tile's operands (64 rows
// at a time and short stages: sweep 0 of 8 units of 131072 tokens, 512 rows, 178 us, now 167; 64 of 32768, 224 rows, 183 and
// 164, with V in sweep 1 210 and 212).
// Sweep 0 takes S^T = K Q^T (a lane holds one query column and 16 token rows: running statistics are lane-private and no
// wavefront needs another's).  Sweep 1 takes S = Q K^T (a lane holds one token and 16 query rows: the sum over the
// wavefront's rows is a sum over registers); the wavefronts' shares meet in LDS, and each of them finishes its 32 or 16 of
// the stage's tokens after the next barrier: alpha_bar, and with OBAR the same tokens' rows of V, requested one stage before.
//
// Running statistics without a running maximum: sum 2^(e - m) for a reference m that stays (see kSumLimit in
// kvs_mfma_tile.h).  The first stage of a chunk takes m from its maxima; a stage whose own sum is not below the limit in
// some lane is done again with the maxima taken into account, from the tiles that are still in LDS.  That leaves 3
// instead of 3.75 instructions per logit.
// Cardinalities enter the common stage as factors of its terms, four of them per LDS read.  (With log2 c added to every logit,
// in the stage that is kept for masked tokens, 48 units of 32768 tokens took 452 us with 160 rows and 455 with 224, now 311
// and 339; 8 units of 32768 with 520 rows 271, now 200.)
#include <type_traits>

#include "kvs_mfma_tile.h"

namespace kvs {
namespace {

using namespace mfma;

// s_waitcnt: at most N vector-memory operations outstanding, all LDS operations done
template <int N>
__device__ __forceinline__ void wait_loads_and_lds() {
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}

template <int D, int NW, int PHASE, bool STREAM, bool OBAR, bool LONG, typename Tab>
__global__ __launch_bounds__(NW * kWave, 2) void score_shared_kernel(
    const Tab tab, const Shape sh, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const int32_t* __restrict__ counts_in, float* __restrict__ alpha_bar, float2* __restrict__ stats_part,
    const float* __restrict__ c_row, const uint16_t* __restrict__ V, float* __restrict__ o_part, const int qp) {
  static_assert(!OBAR || (PHASE == 1 && !LONG), "the Value pass belongs to sweep 1 and to short stages");
  constexpr int KS = D / 16;                // MFMA k-steps
  constexpr int LPR = D / 8;                // 16-byte pieces per row
  constexpr int RPI = kWave / LPR;          // rows per load instruction
  constexpr int ROWB = D * 2;
  constexpr int TILEB = kTile * ROWB;
  constexpr int RW = LONG ? 32 : 16;        // rows of a stage that every wavefront fetches
  constexpr int AHEAD = LONG ? 1 : 2;       // stages of K on their way while one is read
  constexpr int kBuf = AHEAD + 1;
  constexpr int STAGE = RW * NW;            // tokens per stage
  constexpr int NT = STAGE / kTile;         // tiles per stage
  constexpr int NLD = RW / RPI;             // load instructions per wavefront and stage
  constexpr int STAGEB = STAGE * ROWB;

  __shared__ __attribute__((aligned(1024))) unsigned char sm_k[kBuf][STAGEB];
  __shared__ float sm_p[2][NW][STAGE];      // sweep 1: the wavefronts' shares of alpha_bar, two stages
  __shared__ float sm_o[NW][D];             // OBAR: the wavefronts' partial o_bar
  __shared__ int sm_lim[NW * 64 + 32];           // sweep 1, causal window: the last row each query row attends to
  __shared__ __attribute__((aligned(16))) float sm_c[2][STAGE];   // sweep 0: the cardinalities of two stages' rows

  const int ui = find_unit(tab, blockIdx.x);
  const Unit un = tab.unit(ui);
  const int chunk = blockIdx.x - un.chunk_base;
  const int t0 = chunk * un.chunk_len;
  const int t1 = min(un.len, t0 + un.chunk_len);
  const int nstages = (t1 - t0 + STAGE - 1) / STAGE;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int col = lane % 32, half = lane / 32;
  const int R = sh.R;
  const int rows_here = min(R - qp, NW * 64);
  const float sl2 = sh.scale_log2;
  const bool last_launch = qp + NW * 64 >= R;
  const int32_t* cnt = counts_in ? counts_in + un.in_row : nullptr;

  const unsigned char* Kg = reinterpret_cast<const unsigned char*>(K + (size_t)un.in_row * D);
  const uint16_t* Qu = Q + (size_t)un.index * R * D;
  const int st_row = lane / LPR, st_slot = lane % LPR;

  // The launch's blocks of 32 query rows: one or two per wavefront, the first wavefronts taking two.  (A launch with
  // fewer blocks than wavefronts leaves some without rows: their operands repeat the last row and count for nothing.)
  const int nb = (rows_here + 31) / 32;
  const int extra = max(nb - NW, 0);
  const int q_first = 32 * (wave + min(wave, extra));
  const bool two_blocks = wave < extra;

  // sweep 0, cardinalities of stage s: memory -> a register of the first STAGE threads (one stage later: -> LDS, as floats)
  int32_t raw_c = 1;
  const bool has_counts = PHASE == 0 && cnt != nullptr && wave < STAGE / kWave;
  auto fetch_counts = [&](int s) {
    if (has_counts) raw_c = cnt[min(t0 + s * STAGE + tid, t1 - 1)];
  };
  // K stage s -> ring buffer `dst`; tokens past the chunk's end repeat its last one
  auto issue_stage = [&](int s, unsigned char* dst) {
    const int s0 = t0 + s * STAGE;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int r0 = (i * NW + wave) * RPI;                  // first of the instruction's rows (uniform)
      const int row = r0 + st_row;
      const int t = min(s0 + row, t1 - 1);
      const unsigned char* src = Kg + (uint32_t)t * (uint32_t)ROWB + (st_slot ^ (row % LPR)) * 16;
      // (sweep 1 keeps the ordinary cache policy also in launches larger than the caches: the merge pass starts from
      // what it leaves of K in the memory-side cache)
      __builtin_amdgcn_global_load_lds(KVS_GLOBAL_PTR(src), KVS_LDS_PTR(dst + r0 * ROWB), 16, 0,
                                       STREAM && PHASE == 0 ? kNonTemporal : 0);
    }
  };
  fetch_counts(0);
  issue_stage(0, sm_k[0]);
  if (AHEAD == 2 && nstages > 1) issue_stage(1, sm_k[1]);
  if (has_counts) sm_c[0][tid] = (float)raw_c;
  fetch_counts(1);
  if (PHASE == 1) {                         // (read after the loop's barriers)
    sm_lim[tid] = last_seen_row(sh.causal, un.len, qp + tid);
    if (tid < 32) sm_lim[NW * 64 + tid] = 0;
  }
  // this wavefront's query rows: MFMA operands for the whole chunk (rows past R repeat the last one)
  bf16x8 bq[2][KS];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int qrow = min(qp + q_first + 32 * nt + col, R - 1);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      bq[nt][kk] = *reinterpret_cast<const bf16x8*>(Qu + (size_t)qrow * D + kk * 16 + 8 * half);
  }
  // sweep 1: the normalisers of the lane's 16 accumulator rows per block (exp2(-inf) = 0: no such row)
  float cq[2][16];
  if (PHASE == 1) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int q = q_first + 32 * nt + 8 * (v / 4) + 4 * half + (v % 4);
        cq[nt][v] = ((nt == 0 || two_blocks) && q < rows_here) ? c_row[(size_t)un.index * R + qp + q] : INFINITY;
      }
    }
  }
  // (all of it has to be there before the loop: the compiler would otherwise wait for EVERY load in flight in front of
  // the loop body's first product)
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(bq[nt][kk]));
    if (PHASE == 1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) asm volatile("" : "+v"(cq[nt][v]));
    }
  }

  uint32_t a_ofs[KS];                       // this lane's K operands within a tile
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) a_ofs[kk] = col * ROWB + ((2 * kk + half) ^ (col % LPR)) * 16;

  // sums against the reference m_run, and what their additions have lost so far (see add_compensated)
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f}, l_lost[2] = {0.f, 0.f};
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 vr[NLD];
  float o_acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o_acc[e] = 0.f;
  const unsigned char* Vg = OBAR ? reinterpret_cast<const unsigned char*>(V + (size_t)un.in_row * D) : nullptr;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // logits of the tile at `tile` (LDS) against this wavefront's rows
  auto products = [&](const unsigned char* tile, f32x16 (&acc)[2]) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(tile + a_ofs[kk]);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        acc[nt] = (PHASE == 0) ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bq[nt][kk], kk == 0 ? zero : acc[nt], 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[nt][kk], a, kk == 0 ? zero : acc[nt], 0, 0, 0);
      }
    }
  };
  // sweep 0, any tile: rows past the chunk's end or the causal limit drop out, cardinalities join, the reference rises
  auto add_terms_any = [&](f32x16 (&acc)[2], int tile_t0, const float* tile_c) {
    const int valid = t1 - tile_t0;
    if (valid < kTile) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if (8 * (v / 4) + 4 * half + (v % 4) >= valid) { acc[0][v] = -INFINITY; acc[1][v] = -INFINITY; }
      }
    }
    if (sh.causal > 0 && tile_t0 + kTile > un.len - sh.causal + 1) {
      const int q = qp + q_first + col;
      const int lim2[2] = {last_seen_row(sh.causal, un.len, q), last_seen_row(sh.causal, un.len, q + 32)};
      mask_causal<2>(acc, lim2, tile_t0, half);
    }
    if (cnt) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float lc = even_log2(tile_c[8 * (v / 4) + 4 * half + (v % 4)]);
        acc[0][v] = fmaf(acc[0][v], sl2, lc);
        acc[1][v] = fmaf(acc[1][v], sl2, lc);
      }
    }
    const float sc = cnt ? 1.f : sl2;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      float tm = acc[nt][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) tm = fmaxf(tm, acc[nt][v]);
      const float m_new = fmaxf(m_run[nt], fmaf(tm, sc, kHeadroom));
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      float s = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) s += ex2(fmaf(acc[nt][v], sc, -m_safe));
      const float down = ex2(m_run[nt] - m_safe);
      l_run[nt] *= down;
      l_lost[nt] *= down;
      add_compensated(l_run[nt], l_lost[nt], s);
      m_run[nt] = m_new;
    }
  };
  // sweep 1: this lane's token summed over the wavefront's query rows, into the stage's table
  auto put_share = [&](const f32x16 (&acc)[2], int buf, int tile, int tile_t0, bool masked) {
    float p = 0.f;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = ex2(fmaf(acc[nt][4 * g + i], sl2, -cq[nt][4 * g + i]));
        if (masked) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int q = q_first + 32 * nt + 8 * g + 4 * half + i;
            e[i] = (tile_t0 + col > sm_lim[q]) ? 0.f : e[i];
          }
        }
        p += (e[0] + e[1]) + (e[2] + e[3]);
      }
    }
    p += __shfl_xor(p, 32, kWave);
    if (half == 0) sm_p[buf][wave][tile * kTile + col] = p;
  };
  // sweep 1: the tokens of stage s that this wavefront finishes: rows (n * NW + wave) * RPI + r of the stage for
  // n < NLD, r < RPI, token (n, r) in lane n * RPI + r (the rows of V that its load n brings, too)
  auto finish_stage = [&](int s) {
    const int s0 = t0 + s * STAGE;
    const int lt = lane % RW;
    const int row = ((lt / RPI) * NW + wave) * RPI + lt % RPI;
    float p = 0.f;
    {
      const float* src = &sm_p[s & 1][0][row];
#pragma unroll
      for (int w = 0; w < NW; ++w) p += src[w * STAGE];
    }
    const int t = s0 + row;
    const bool ok = t < t1;
    if (qp > 0 && ok) p += alpha_bar[un.in_row + t];         // the rows of the launches before
    if (OBAR) {
      const float wt = ok ? p : 0.f;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const float w = __shfl(wt, i * RPI + st_row, kWave);
        float vf[8];
        Piece<uint16_t>::unpack(make_uint4(vr[i].x, vr[i].y, vr[i].z, vr[i].w), vf);
#pragma unroll
        for (int e = 0; e < 8; ++e) o_acc[e] = fmaf(w, vf[e], o_acc[e]);
      }
    }
    // (the store below stays behind the use of vr, in front of which it would be waited for)
    if (OBAR) asm volatile("" : "+v"(o_acc[0]), "+v"(o_acc[1]), "+v"(o_acc[2]), "+v"(o_acc[3]), "+v"(o_acc[4]),
                                "+v"(o_acc[5]), "+v"(o_acc[6]), "+v"(o_acc[7]) :: "memory");
    // a row that stands for c tokens has c equal terms in every softmax sum (2^(e + log2 c) = c 2^e)
    if (cnt && last_launch && ok) p *= (float)cnt[t];
    if (lane < RW && ok) alpha_bar[un.in_row + t] = p;
  };
  auto load_values = [&](int s) {
    const int s0 = t0 + s * STAGE;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int t = min(s0 + (i * NW + wave) * RPI + st_row, t1 - 1);
      const u32x4* src = reinterpret_cast<const u32x4*>(Vg + (uint32_t)t * (uint32_t)ROWB + st_slot * 16);
      vr[i] = STREAM ? __builtin_nontemporal_load(src) : *src;
    }
  };

  const int causal_from = sh.causal > 0 ? un.len - sh.causal + 1 : 0x7fffffff;   // first row that some query misses

  // One stage.  `rd` and `wr` are different buffers of the ring, and saying so (__restrict__ arguments) is what keeps
  // the compiler from waiting for the loads into `wr` in front of every read of `rd`.
  auto stage = [&](const int s, const unsigned char* __restrict__ rd, unsigned char* __restrict__ wr,
                   const float* __restrict__ rd_c) {
    if (has_counts) {
      sm_c[(s + 1) & 1][tid] = (float)raw_c;
      fetch_counts(s + 2);                                   // (before stage s + 2 of K, which the next wait may leave out)
    }
    if (s + AHEAD < nstages) issue_stage(s + AHEAD, wr);
    if (OBAR) load_values(s);
    const int s0 = t0 + s * STAGE;
    const bool plain = s0 + STAGE <= min(t1, causal_from - 1);   // no token of the stage is masked for anybody
    // The common stage, block after block (a tile against 32 of the wavefront's rows): k-step kk of block m issues one product
    // and forms a share of block m - 1's terms, and the order is pinned step by step: left to itself the compiler issues the
    // products in runs and the terms in runs, and the two wavefronts of a SIMD then fall into step and compete for one pipe
    // after the other.  A tile's operands stay in registers for its blocks; each is replaced by the next tile's when the last
    // block has used it.
    auto fast = [&](auto ntb_c, auto counts_c) {
      constexpr int NTB = decltype(ntb_c)::value;            // blocks of query rows
      constexpr bool COUNTS = decltype(counts_c)::value;     // sweep 0: a row that stands for c tokens has c equal terms
      asm volatile("; plain stage, %0 blocks" :: "n"(NTB));
      f32x16 acc[2];
      bf16x8 a[KS];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) a[kk] = *reinterpret_cast<const bf16x8*>(rd + a_ofs[kk]);
      constexpr int M = NT * NTB;                            // blocks of the stage
      constexpr int PER = 16 / KS;                           // terms per step
      float sum = 0.f, share = 0.f;
      // the cardinalities of the four rows that group g of a block's terms belongs to, read one group ahead
      float4 cc = make_float4(0.f, 0.f, 0.f, 0.f), cc_next = cc;
      auto group_counts = [&](int m, int g) {
        return *reinterpret_cast<const float4*>(rd_c + (m / NTB) * kTile + 8 * g + 4 * half);
      };
      if constexpr (COUNTS) cc_next = group_counts(0, 0);
      auto terms = [&](int m, int kk) {                      // share kk of block m's terms
        const int nt = m % NTB;
        float cf[PER];
        if constexpr (COUNTS) {
          constexpr int STEPS = 4 / PER;                     // steps per group of four rows
          if (kk % STEPS == 0) {
            cc = cc_next;
            const int g = 4 * m + kk / STEPS + 1;
            if (g < 4 * M) cc_next = group_counts(g / 4, g % 4);
          }
          const float c4[4] = {cc.x, cc.y, cc.z, cc.w};
#pragma unroll
          for (int j = 0; j < PER; ++j) cf[j] = c4[(kk % STEPS) * PER + j];
        }
        float e[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
          const int v = kk * PER + j;
          e[j] = ex2(fmaf(acc[m & 1][v], sl2, PHASE == 0 ? -m_run[nt] : -cq[nt][v]));
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) sum = COUNTS ? fmaf(cf[j], e[j], sum) : sum + e[j];
        if (kk == KS - 1) {
          if (PHASE == 0) {
            l_run[nt] += sum;
          } else if (nt == NTB - 1) {
            float p = NTB == 2 ? share + sum : sum;
            p += __shfl_xor(p, 32, kWave);
            if (half == 0) sm_p[s & 1][wave][(m / NTB) * kTile + col] = p;
          } else {
            share = sum;
          }
          sum = 0.f;
        }
      };
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int i = m / NTB, nt = m % NTB;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
          const f32x16 c = kk == 0 ? zero : acc[m & 1];
          acc[m & 1] = (PHASE == 0) ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], bq[nt][kk], c, 0, 0, 0)
                                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[nt][kk], a[kk], c, 0, 0, 0);
          if (nt == NTB - 1 && i + 1 < NT)
            a[kk] = *reinterpret_cast<const bf16x8*>(rd + (i + 1) * TILEB + a_ofs[kk]);
          if (m > 0) terms(m - 1, kk);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) terms(M - 1, kk);
      asm volatile("; plain stage ends, %0 blocks" :: "n"(NTB));
    };
    if (PHASE == 0) {
      const float l_old[2] = {l_run[0], l_run[1]};
      bool redo = true;
      if (s > 0 && plain) {
        l_run[0] = l_run[1] = 0.f;           // the stage's own sums
        auto run = [&](auto counts_c) {
          if (two_blocks) fast(std::integral_constant<int, 2>{}, counts_c);
          else fast(std::integral_constant<int, 1>{}, counts_c);
        };
        if (cnt != nullptr) run(std::true_type{});
        else run(std::false_type{});
        redo = __any(!(l_run[0] < kSumLimit) || !(l_run[1] < kSumLimit));
        if (!redo) {
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) {
            const float stage_sum = l_run[nt];
            l_run[nt] = l_old[nt];
            add_compensated(l_run[nt], l_lost[nt], stage_sum);
          }
        }
      }
      if (redo) {
        asm volatile("; any stage");
        l_run[0] = l_old[0];
        l_run[1] = l_old[1];
#pragma unroll 1
        for (int i = 0; i < NT; ++i) {
          if (s0 + i * kTile >= t1) break;
          f32x16 acc[2];
          products(rd + i * TILEB, acc);
          add_terms_any(acc, s0 + i * kTile, rd_c + i * kTile);
        }
      }
    } else if (plain) {
      if (two_blocks) fast(std::integral_constant<int, 2>{}, std::false_type{});
      else fast(std::integral_constant<int, 1>{}, std::false_type{});
    } else {
      // (the marks keep the branches' ends and beginnings apart: merged, their accesses lose what is known about them)
      asm volatile("; any stage");
#pragma unroll 1
      for (int i = 0; i < NT; ++i) {
        if (s0 + i * kTile >= t1) break;                     // (nobody reads the shares of tokens past the chunk's end)
        f32x16 acc[2];
        products(rd + i * TILEB, acc);
        put_share(acc, s & 1, i, s0 + i * kTile, s0 + i * kTile + kTile > causal_from);
      }
      asm volatile("; any stage ends");
    }
  };
  for (int s = 0; s < nstages; ++s) {
    // stage s has landed in every wavefront (with short stages those loads may be outstanding that are of stage s + 1), and
    // nobody reads the buffer of stage s - 1 any more
    if (AHEAD == 2 && s + 1 < nstages) wait_loads_and_lds<NLD>();
    else wait_loads_and_lds<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (PHASE == 1 && s > 0) finish_stage(s - 1);
    stage(s, sm_k[s % kBuf], sm_k[(s + AHEAD) % kBuf], sm_c[s & 1]);
  }

  if (PHASE == 0) {
    // the two halves of a wavefront hold the same query column for different token rows
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      l_run[nt] -= l_lost[nt];
      const float m_o = __shfl_xor(m_run[nt], 32, kWave);
      const float l_o = __shfl_xor(l_run[nt], 32, kWave);
      const float m_n = fmaxf(m_run[nt], m_o);
      const float m_s = (m_n == -INFINITY) ? 0.f : m_n;
      const float l_n = l_run[nt] * ex2(m_run[nt] - m_s) + l_o * ex2(m_o - m_s);
      const int q = q_first + 32 * nt + col;
      if (half == 0 && (nt == 0 || two_blocks) && q < rows_here)
        stats_part[((size_t)un.index * kMaxChunks + chunk) * R + qp + q] = make_float2(m_n, l_n);
    }
  } else {
    wait_loads_and_lds<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    finish_stage(nstages - 1);
    if (OBAR) {
      // lanes that hold the same piece of the row, then the wavefronts, in a fixed order
#pragma unroll
      for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) o_acc[e] += __shfl_xor(o_acc[e], off, kWave);
      }
      if (st_row == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sm_o[wave][st_slot * 8 + e] = o_acc[e];
      }
      __syncthreads();
      if (tid < D) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += sm_o[w][tid];
        o_part[((size_t)un.index * kMaxChunks + chunk) * D + tid] = sum;
      }
    }
  }
}

// Long stages in sweep 0 without cardinalities, but for 64 channels in workgroups of eight wavefronts, and with 64 channels where K
// is read past the caches, whatever the rest; never for chunks of no more than two of them in workgroups of four wavefronts.  And in
// a sweep 1 without V of 64 channels.  Steps with long -> short stages in sweep 0 (us): cardinalities, 48 units of 21845 tokens, 512
// rows 637 -> 618, 20 of 5000 to 30000, 224 rows 128 -> 126, 64 channels, 160 rows 96 -> 91; none, 64 channels, 512 rows, 24 of 10721
// 115 -> 112, 8 of 65536 190 -> 187; 72 of 383 to 3068, 256 rows, chunks of 256, 75.2 -> 74.6; but 104 of 5471 to 21885, 224 rows
// 509 -> 523, 48 of 3000 to 24000, 512 rows 313 -> 321, 64 channels, 256 rows, 32 of 10101 to 20203 135.5 -> 137.7, 16 of 40000 158 ->
// 160, 40 of 9000 98.4 either way, past the caches 152 of 6898, 512 rows 315 -> 325, 92 of 5698 to 22795, 256 rows 241 -> 248, with
// cardinalities 200 of 5000, 512 rows 361 -> 367, 64 of 32768, 256 rows 396 -> 401.  In sweep 1: 16 of 21000, 224 rows 129 -> 125,
// 160 rows 120 -> 117, 512 rows 176 -> 173; but 64 channels, 16 of 21000, 448 rows 130 -> 133.
template <int D, int NW, bool STREAM>
hipError_t launch_t(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const int32_t* counts_in,
                    float* alpha_bar, const Workspace& ws, const void* V, hipStream_t stream) {
  const dim3 grid(tab.total_chunks), block(NW * kWave);
  const bool long0 = (counts_in == nullptr || (D == 64 && STREAM)) && !(NW == 4 && tab.unit(0).chunk_len <= 2 * 32 * NW);
  constexpr bool LONG1 = D == 64;
  hipError_t e;
  for (int qp = 0; qp < sh.R; qp += NW * 64) {
    launch_with_table(tab, [&](const auto& t) {
      auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, t, sh, (const uint16_t*)Q, (const uint16_t*)K, counts_in, alpha_bar,
                           ws.stats_part, ws.c_row, (const uint16_t*)nullptr, (float*)nullptr, qp);
      };
      if constexpr (D == 128 || STREAM || NW == 4) {
        if (long0) return launch(score_shared_kernel<D, NW, 0, STREAM, false, true, KVS_TABLE_TYPE(t)>);
      }
      launch(score_shared_kernel<D, NW, 0, STREAM, false, false, KVS_TABLE_TYPE(t)>);
    });
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = launch_score_finalize(tab, sh, ws, stream)) != hipSuccess || alpha_bar == nullptr) return e;
  for (int qp = 0; qp < sh.R; qp += NW * 64) {
    if (V != nullptr && qp + NW * 64 >= sh.R) {              // the last launch alone knows the finished alpha_bar
      launch_with_table(tab, [&](const auto& t) {
        hipLaunchKernelGGL((score_shared_kernel<D, NW, 1, STREAM, true, false, KVS_TABLE_TYPE(t)>), grid, block, 0, stream, t, sh,
                           (const uint16_t*)Q, (const uint16_t*)K, counts_in, alpha_bar, ws.stats_part, ws.c_row,
                           (const uint16_t*)V, ws.o_part, qp);
      });
    } else {
      launch_with_table(tab, [&](const auto& t) {
        hipLaunchKernelGGL((score_shared_kernel<D, NW, 1, STREAM, false, LONG1, KVS_TABLE_TYPE(t)>), grid, block, 0, stream, t, sh,
                           (const uint16_t*)Q, (const uint16_t*)K, counts_in, alpha_bar, ws.stats_part, ws.c_row,
                           (const uint16_t*)nullptr, (float*)nullptr, qp);
      });
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D, int NW>
hipError_t launch_s(const UnitTable& tab, const Shape& sh, const void* Q, const void* K, const int32_t* counts_in,
                    float* alpha_bar, const Workspace& ws, const void* V, hipStream_t stream) {
  return sh.stream ? launch_t<D, NW, true>(tab, sh, Q, K, counts_in, alpha_bar, ws, V, stream)
                   : launch_t<D, NW, false>(tab, sh, Q, K, counts_in, alpha_bar, ws, V, stream);
}

}  // namespace

hipError_t launch_score_shared(const UnitTable& tab, const Shape& sh, const void* Q, const void* K,
                               const int32_t* counts_in, float* alpha_bar, const Workspace& ws, const void* V,
                               hipStream_t stream) {
  if (sh.R <= 256) {
    return sh.D == 64 ? launch_s<64, 4>(tab, sh, Q, K, counts_in, alpha_bar, ws, V, stream)
                      : launch_s<128, 4>(tab, sh, Q, K, counts_in, alpha_bar, ws, V, stream);
  }
  return sh.D == 64 ? launch_s<64, 8>(tab, sh, Q, K, counts_in, alpha_bar, ws, V, stream)
                    : launch_s<128, 8>(tab, sh, Q, K, counts_in, alpha_bar, ws, V, stream);
}

}  // namespace kvs
