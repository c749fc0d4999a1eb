// Device helpers shared by the routing kernels.
#pragma once

#include "rr_internal.h"

namespace rr {

constexpr int kMaxRank = kMaxK + 1;

// Ranking key of a (score, expert) pair: the order-preserving image of the score, then the complement of the expert index
// (Eq. 1 argtopk, ties -> lower expert index).  A greater key is a better rank and the keys of different experts never
// tie.  The 38 bits sit in the bits of a positive double - 18 bits of the image behind an exponent that keeps it normal, the
// other 14 and the 6 of the expert in the low word - so the order is that of doubles, and a compare-exchange is one v_max_f64
// and one v_min_f64 (a comparison of 64-bit integers and four selects before; figures at topk_rank_kernel).
// 0.0 lies below every real key and decodes to expert -1.
typedef double rank_t;
__device__ inline rank_t rank_key(float v, int e) {
  const u32 image = score_key(v);
  const u32 hi = 0x40000000u | (image >> 14), lo = (image << 18) | ((u32)(kMaxE - 1 - e) << 12);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline u32 rank_key_score(rank_t key) {
  return (u32)(__builtin_bit_cast(unsigned long long, key) >> 18);
}
__device__ inline int rank_key_expert(rank_t key) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, key);
  return bits ? kMaxE - 1 - (int)((u32)bits >> 12 & (kMaxE - 1)) : -1;
}
static_assert(kMaxE == 64, "six bits of a ranking key hold the expert");
__device__ __forceinline__ rank_t rank_max(rank_t a, rank_t b) {
  rank_t r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ rank_t rank_min(rank_t a, rank_t b) {
  rank_t r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ inline rank_t rank_of_lane(rank_t key, int off) {  // the key of lane ^ off
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, key);
  const u32 lo = __shfl_xor((u32)bits, off), hi = __shfl_xor((u32)(bits >> 32), off);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// b[0] > b[1] > ... > b[N-1] are the N greatest keys seen so far: one compare-exchange per position.
template <int N>
__device__ inline void insert_key(rank_t (&b)[N], rank_t a) {
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const rank_t hi = rank_max(a, b[q]);
    if (q + 1 < N) a = rank_min(a, b[q]);
    b[q] = hi;
  }
}

// Eq. 1 argtopk over experts [e0, e1) of one row of scores held in LDS: the N best keys, best first
// (positions past the number of experts stay 0).
template <int N>
__device__ inline void top_keys_of_range(const float *row, int e0, int e1, rank_t (&b)[N]) {
#pragma unroll
  for (int q = 0; q < N; ++q) b[q] = 0.0;
  for (int e = e0; e < e1; ++e) insert_key(b, rank_key(row[e], e));
}

// Sec. 4.1: best expert among those of one group, ties -> lower expert index.
__device__ inline void best_in_group(const float *row, int e0, int e1, float &best, int &arg) {
  best = row[e0];
  arg = e0;
  for (int e = e0 + 1; e < e1; ++e) {
    float v = row[e];
    if (v > best) { best = v; arg = e; }
  }
}

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

// Workgroup -> token block for kernels whose neighbouring token blocks write neighbouring words of
// the same per-expert arrays.  Workgroups are dealt to the 8 XCDs round-robin and each XCD has its
// own L2: with block = workgroup, one cache line would be completed piecewise from 8 L2s.  Here XCD
// x walks its own contiguous eighth of the blocks, so the pieces of a line meet in one L2.
__device__ inline int xcd_block(int g, int NB) {
  const int per = NB >> 3, main = per << 3;
  return g < main ? (g & 7) * per + (g >> 3) : g;
}


}  // namespace rr
