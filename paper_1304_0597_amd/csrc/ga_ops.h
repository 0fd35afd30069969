// Pieces of the genetic operators shared by the generation kernels (ga.hip,
// resident.hip).
#pragma once

#include "philox.h"

namespace game {

__device__ __forceinline__ float clamp_unit(float v) {
  return v < -1.f ? -1.f : (v > 1.f ? 1.f : v);
}

__device__ __forceinline__ float rank_key_value(float f) {
  if (isnan(f)) return INFINITY;
  return f == 0.f ? 0.f : f;
}

// Order-preserving map of a canonical float to uint32.
__device__ __forceinline__ uint32_t ordered_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint64_t rank_key(float f, int i) {
  return ((uint64_t)ordered_bits(rank_key_value(f)) << 32) | (uint32_t)i;
}

// Linear ranking, pressure 2: rank r has weight P - r; the integer draw
// t = (u32 * P(P+1)/2) >> 32 falls in rank r's cumulative interval.
__device__ __forceinline__ int ranking_pick(const int32_t* order, int P, uint32_t u) {
  const int64_t W = (int64_t)P * (P + 1) / 2;
  const int64_t t = (int64_t)(((uint64_t)u * (uint64_t)W) >> 32);
  int lo = 0, hi = P - 1;                 // first r with cum_end(r) > t
  while (lo < hi) {
    const int r = (lo + hi) >> 1;
    const int64_t cum_end = (int64_t)(r + 1) * P - (int64_t)(r + 1) * r / 2;
    if (cum_end > t) hi = r;
    else lo = r + 1;
  }
  return order[lo];
}

// Roulette wheel: first index whose cumulative weight exceeds
// (u32 2^-32) * total; zero total draws uniformly.
__device__ __forceinline__ int roulette_pick(const double* cum, int P, uint32_t u) {
  const double total = cum[P - 1];
  if (!(total > 0.0)) return (int)(((uint64_t)u * (uint64_t)P) >> 32);
  const double target = ((double)u * 0x1p-32) * total;
  int lo = 0, hi = P;                      // first i with cum[i] > target
  while (lo < hi) {
    const int i = (lo + hi) >> 1;
    if (cum[i] > target) hi = i;
    else lo = i + 1;
  }
  return lo < P ? lo : P - 1;
}

// Pointer c ? x : y as integer arithmetic on already loaded values.  (A
// select between two fields of the argument structure is otherwise turned
// into a load through a selected field address, which keeps the whole
// structure in private memory.)
template <class T>
__device__ __forceinline__ T* pick(bool c, T* x, T* y) {
  const uintptr_t ux = (uintptr_t)x, uy = (uintptr_t)y;
  return (T*)(uy ^ ((ux ^ uy) & (uintptr_t)(-(intptr_t)c)));
}

// The 64-bit value of another lane of the 16-lane row (DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ uint64_t row_move(uint64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xF, 0xF, true);
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kHalfMirror = 0x141, kRowMirror = 0x140;
constexpr int kRowRor = 0x120;

// s + the same of lane l ^ N, where lanes 2 N apart hold equal values (N = 8:
// any): a rotation of the row by N.
template <int N>
__device__ __forceinline__ double row_add(double s) {
  return s + __longlong_as_double((long long)row_move<kRowRor + N>((uint64_t)__double_as_longlong(s)));
}

// The 64-bit value's two copies of v with the 32-lane halves (16-lane rows of
// each half) doubled.
template <bool ROWS>
__device__ __forceinline__ void spread(uint64_t v, uint64_t& first, uint64_t& second) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  if constexpr (ROWS) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto u = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    first = ((uint64_t)u[0] << 32) | l[0];
    second = ((uint64_t)u[1] << 32) | l[1];
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto u = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    first = ((uint64_t)u[0] << 32) | l[0];
    second = ((uint64_t)u[1] << 32) | l[1];
  }
}
// Smallest of the lanes l ^ 16, l ^ 32, l ^ 48 and l.
__device__ __forceinline__ uint64_t rows_min(uint64_t v) {
  uint64_t x, y;
  spread<true>(v, x, y);
  spread<false>(min(x, y), x, y);
  return min(x, y);
}

// Smallest key of each group of 8 lanes.
__device__ __forceinline__ uint64_t min8(uint64_t k) {
  k = min(k, row_move<kQuadXor1>(k));
  k = min(k, row_move<kQuadXor2>(k));
  return min(k, row_move<kHalfMirror>(k));
}

}  // namespace game
