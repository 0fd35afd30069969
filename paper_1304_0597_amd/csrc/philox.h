// Philox4x64-10 (Salmon et al., SC'11) and the values the genetic operators
// take from its blocks; see ga.hip for the streams and counters.
#pragma once

#include "common.h"

namespace game {

struct U64x4 {
  uint64_t o0, o1, o2, o3;
};

// Rounds R0 .. R1 - 1 of counter c under key (k0, k1).  The 128-bit products
// are formed once each (four 32-bit multiply-adds); a low product and a high
// product of their own take six.
template <int R0, int R1>
__device__ __forceinline__ U64x4 philox_rounds(U64x4 c, uint64_t k0, uint64_t k1) {
  constexpr uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  constexpr uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
  k0 += R0 * W0;
  k1 += R0 * W1;
#pragma unroll
  for (int r = R0; r < R1; ++r) {
    if (r > R0) {
      k0 += W0;
      k1 += W1;
    }
    const unsigned __int128 p0 = (unsigned __int128)M0 * c.o0, p1 = (unsigned __int128)M1 * c.o2;
    const uint64_t n0 = (uint64_t)(p1 >> 64) ^ c.o1 ^ k0, n2 = (uint64_t)(p0 >> 64) ^ c.o3 ^ k1;
    c = {n0, (uint64_t)p1, n2, (uint64_t)p0};
  }
  return c;
}

__device__ __forceinline__ U64x4 draw(uint64_t seed, uint64_t stream, uint64_t gen, uint64_t unit,
                                      uint64_t blk) {
  return philox_rounds<0, 10>({gen, unit, blk, 0}, seed, stream);
}

__device__ __forceinline__ float gauss12(const U64x4& b) {
  int32_t s = 0;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    s += (int32_t)((b.o1 >> (16 * f)) & 0xFFFF);
    s += (int32_t)((b.o2 >> (16 * f)) & 0xFFFF);
    s += (int32_t)((b.o3 >> (16 * f)) & 0xFFFF);
  }
  return (float)(s - 393210) * 0x1p-16f;  // both steps exact
}

// The draws of one genetic step that do not depend on the errors (DrawArgs):
// item i < n_pairs * blocks is the 8 selection words of block i % blocks of
// pair i / blocks; the items after them are the genes of the P slots, each the
// mutation to add (sigma z, rounded once; NaN for none, and for the elites'
// slots).  The gene items also copy the population pop being evaluated to
// a.cur.  gen is the generation to be built.
__device__ __forceinline__ void make_draw(const DrawArgs& a, const float* pop, int gen, int i) {
  const int n_words = a.n_pairs * a.blocks;
  if (i < n_words) {
    const int q = i / a.blocks;
    const U64x4 r = draw(a.seed, 1, (uint64_t)gen, (uint64_t)q, (uint64_t)(i - q * a.blocks));
    uint64_t* w = a.words + (int64_t)i * 4;
    w[0] = r.o0;
    w[1] = r.o1;
    w[2] = r.o2;
    w[3] = r.o3;
    return;
  }
  const int j = i - n_words;
  const float v = pop[j];
  const int s = j / a.K;
  float m = __uint_as_float(0x7FC00000u);
  if (s >= a.E) {
    const U64x4 r = draw(a.seed, 2, (uint64_t)gen, (uint64_t)s, (uint64_t)(j - s * a.K));
    if ((r.o0 & 0xFFFFFFFFull) < a.thr_mut) m = __fmul_rn(a.sigma, gauss12(r));
  }
  a.mut[j] = m;
  a.cur[j] = v;
}

}  // namespace game
