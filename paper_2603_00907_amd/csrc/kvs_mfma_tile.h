// Pieces shared by the bf16 matrix-core score kernels: the 32-token tile, LDS operand reads with explicit waits,
// and the per-tile adjustments of the logits (cardinalities, causal window).
#pragma once

#include <type_traits>

#include "kvs_device.h"

namespace kvs {
namespace mfma {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTile = 32;                 // tokens per MFMA tile
constexpr int kNonTemporal = 2;           // cache-policy bit of K tile loads that no later sweep finds cached anyway

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// Sums of 2^(e - m) over a row's logits e against a reference m that stays where it is (sweep 0 of the bf16 kernels and of
// fp32 above 64 query rows): m is kHeadroom above the largest logit seen when it was last set, and a group of terms whose own
// sum is not below kSumLimit sets it again.  Any m would do for the sum, which is a floating-point number, but not for
// the exponent's argument, which is rounded in proportion to its size: the largest term's stays between -7.5 and 16,
// where that rounding is at most that of the finished normaliser.  (A row that puts its weight on one token 2^61 above
// its first ones: 0.24e-6 to 0.40e-6 for the normaliser's error, 0.31e-6 to 0.61e-6 with a running maximum, 2.6e-6 to
// 2.9e-6 with a limit of 2^64 and no headroom.)  Without headroom a limit this low is met in nearly every tile of a wide
// window (8 units of 131072 tokens, 512 rows, Queries three times as large: both sweeps 478 us, 431 with headroom; at
// their usual size 372 either way).
constexpr float kHeadroom = 7.5f;
constexpr float kSumLimit = 65536.f;
constexpr float kLeastUnit = 1.f / 4096.f;

// sum += x, where `lost` holds what the additions before have rounded away.  For a lane that meets all tiles of a chunk:
// a sum that is nearly all one term would round every later tile's share the same way (2048 tokens: 1e-6 of the sum).
__device__ __forceinline__ void add_compensated(float& sum, float& lost, float x) {
  const float y = x - lost;
  const float t = sum + y;
  lost = (t - sum) - y;
  sum = t;
}

// Four 16-byte LDS reads at byte addresses ad[0..3] + OFF, complete on return.  Written as inline
// assembly on purpose: the compiler treats every LDS read as dependent on ALL outstanding
// global->LDS loads and would wait for the tile that is still being prefetched into the other buffer;
// here the wait on the right tile is the explicit vmcnt above the call.
template <int OFF>
__device__ __forceinline__ void lds_read_4x16(bf16x8& a0, bf16x8& a1, bf16x8& a2, bf16x8& a3, const uint32_t* ad) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%8\n\t"
      "ds_read_b128 %1, %5 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%8\n\t"
      "ds_read_b128 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3)
      : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3]), "n"(OFF)
      : "memory");
}

// A float that all lanes hold, as a scalar.
__device__ __forceinline__ float uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// 2^-k, k the exponent of the largest cardinality that the wavefront's lanes hold (0 where none is above 1): a power of two,
// so that multiplying and dividing by it is exact.
__device__ __forceinline__ float unit_of_counts(float c) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) c = fmaxf(c, __shfl_xor(c, m, kWave));
  c = fmaxf(c, 1.f);
  return uniform(__uint_as_float((254u << 23) - (__float_as_uint(c) & 0x7f800000u)));
}

// The least of c over the wavefront's lower 32 lanes, in every lane (DPP moves: shifts inside a row of 16 lanes, then the last
// lane of row 0 into row 1).
__device__ __forceinline__ float least_of_tile(float c) {
  auto step = [&](auto ctrl) {
    const int x = __builtin_bit_cast(int, c);
    c = fminf(c, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, decltype(ctrl)::value, 0xF, 0xF, false)));
  };
  step(std::integral_constant<int, 0x111>{});     // row_shr:1
  step(std::integral_constant<int, 0x112>{});
  step(std::integral_constant<int, 0x114>{});
  step(std::integral_constant<int, 0x118>{});
  step(std::integral_constant<int, 0x142>{});     // row_bcast:15
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, c), 31));
}

// Four floats of LDS at byte address ad, complete on return (inline assembly for the same reason).
__device__ __forceinline__ void lds_read_four(float (&r)[4], uint32_t ad) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 x;
  asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x) : "v"(ad) : "memory");
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = x[i];
}

// Rows that stand for c tokens with one Key (an already merged cache) enter the softmax as c equal
// terms, i.e. with log2(c) added to the base-2 logit.  Turns the raw dot products of this lane's 16
// accumulator rows (tile at token base_t of the unit whose cardinalities start at cnt) into logits.
template <int NACC>
__device__ __forceinline__ void logits_with_counts(f32x16 (&acc)[NACC], const int32_t* __restrict__ cnt, int base_t,
                                                   int half, float sl2) {
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = 8 * (v / 4) + 4 * half + (v % 4);
    const float lc = even_log2((float)cnt[base_t + row]);
#pragma unroll
    for (int nt = 0; nt < NACC; ++nt) acc[nt][v] = fmaf(acc[nt][v], sl2, lc);
  }
}

// Causal window: accumulator rows past the last row a query column attends to leave the softmax
// (lim[i]: that row for the query column of accumulator i).
template <int NACC>
__device__ __forceinline__ void mask_causal(f32x16 (&acc)[NACC], const int (&lim)[NACC], int base_t, int half) {
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int t = base_t + 8 * (v / 4) + 4 * half + (v % 4);
#pragma unroll
    for (int i = 0; i < NACC; ++i) {
      if (t > lim[i]) acc[i][v] = -INFINITY;
    }
  }
}

#define KVS_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define KVS_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

// Two 16-byte LDS reads at each of two addresses (offsets OFF0 and OFF1), complete on return.
template <int OFF0, int OFF1>
__device__ __forceinline__ void lds_read_2x2(bf16x8& b00, bf16x8& b01, bf16x8& b10, bf16x8& b11, uint32_t ad0,
                                             uint32_t ad1) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%6\n\t"
      "ds_read_b128 %1, %4 offset:%7\n\t"
      "ds_read_b128 %2, %5 offset:%6\n\t"
      "ds_read_b128 %3, %5 offset:%7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(b00), "=&v"(b01), "=&v"(b10), "=&v"(b11)
      : "v"(ad0), "v"(ad1), "n"(OFF0), "n"(OFF1)
      : "memory");
}

// One 16-byte LDS read at each of two addresses (offset OFF), complete on return.
template <int OFF>
__device__ __forceinline__ void lds_read_2x1(bf16x8& b0, bf16x8& b1, uint32_t ad0, uint32_t ad1) {
  asm volatile(
      "ds_read_b128 %0, %2 offset:%4\n\t"
      "ds_read_b128 %1, %3 offset:%4\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(b0), "=&v"(b1)
      : "v"(ad0), "v"(ad1), "n"(OFF)
      : "memory");
}

}  // namespace mfma
}  // namespace kvs
