// Staging of pattern rows in LDS for the kernels that give each thread one
// pattern (predict.hip, rescore64.hip).
#pragma once

#include "common.h"

namespace game {

constexpr int kRows = 256;        // patterns per tile, one per thread

// Features staged at a time, so that four workgroups' rows share a CU's LDS.
constexpr int kChunk = 32;

// Whether a launch of so many workgroups stages its rows at all: fewer than
// one per CU leave each chunk's memory round trip uncovered, and each thread
// then reads its own row as it goes (300 features, 257 patterns, float64
// re-score: 17 us, 35 staged).
inline bool stages_rows(int64_t workgroups) { return workgroups >= 256; }

// LDS row stride for nf features: odd, so that threads reading their own
// rows hit different banks.
__host__ __device__ constexpr int row_stride(int nf) { return nf | 1; }

// Uniform values read through the constant address space are scalar loads.
using ConstGene = __attribute__((address_space(4))) const float;

// Copies features [f0, f0 + nf) of patterns [row0, row0 + n_rows) into LDS
// rows of stride S, the workgroup of THREADS reading consecutive addresses.
// Element e of the piece is row e / nf, column e % nf; a step of THREADS
// elements advances both without a division.
template <int THREADS = kRows>
__device__ __forceinline__ void stage_rows(float* rows, int S, const float* X, int64_t row0,
                                           int n_rows, int N, int f0, int nf) {
  const int q = THREADS / nf, rem = THREADS - q * nf;
  int row = threadIdx.x / nf, col = threadIdx.x - row * nf;
  const float* src = X + row0 * N + f0;
  while (row < n_rows) {
    constexpr int kU = 8;         // loads in flight per thread
    float v[kU];
    int at[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const bool in = row < n_rows;
      at[u] = in ? row * S + col : -1;
      v[u] = src[in ? (int64_t)row * N + col : 0];
      row += q;
      col += rem;
      if (col >= nf) {
        col -= nf;
        ++row;
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (at[u] >= 0) rows[at[u]] = v[u];
  }
}

}  // namespace game
