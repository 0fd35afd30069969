// Float64 re-score: the error of a few chromosomes (the elite at the end of
// a reduced-precision run, or an audit sample) computed in double precision
// on the vector ALUs, from the same X, t and genes (Eqs. 2-5, 10).
//
// Grid (pattern blocks, groups of R chromosomes): a thread takes one pattern
// of a 256-row tile at a time; the tile's rows (read in consecutive
// addresses) sit in LDS and the genes come in by scalar loads.  A block adds
// its threads' squared residuals in a fixed tree order, and a finish pass
// (one wave per chromosome) adds the blocks in a fixed order, so the result
// is deterministic.
//
// Bound by the float64 multiply-adds and the gene conversions, one of each
// per term next to the recurrence's, with the patterns' read under them.
// 250,000 x 32 patterns, Chebyshev 8, one chromosome: 15.6 us and 3.9 for
// the finish pass (37.5 in all with 256 blocks reading rows thread by thread
// and one thread adding their partials); 1,000,000 x 32: 54 us against 80
// (2.4 TB/s of patterns, 64 chromosomes 1.33 ms against 4.8).  Publishing
// the partials to a last block with device-scope atomics instead of a second
// launch was slower (24.4 us): its round trips are serial.
#include <algorithm>
#include <utility>

#include "basis.h"
#include "rows.h"

namespace game {

template <int BASIS, int D, int R, bool STAGE>
__global__ __launch_bounds__(kRows) void rescore64_kernel(Rescore64Args a) {
  constexpr int B = BASIS == 3 ? 2 : 1;
  extern __shared__ float rows[];
  __shared__ double red[R][kRows];
  const int N = a.N;
  const int FC = STAGE ? min(N, kChunk) : N;
  const int S = row_stride(FC);
  const int c0 = blockIdx.y * R;
  ConstGene* w[R];
  double acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    w[r] = (ConstGene*)a.genes + (int64_t)min(c0 + r, a.n - 1) * a.K;
    acc[r] = 0.0;
  }
  const int64_t n_tiles = (a.NP + kRows - 1) / kRows;
  for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int64_t row0 = tile * kRows;
    const int n_rows = (int)min((int64_t)kRows, a.NP - row0);
    const bool valid = (int)threadIdx.x < n_rows;
    const int64_t k = valid ? row0 + threadIdx.x : row0;
    const float* mine = STAGE ? rows + threadIdx.x * S : a.X + k * N;
    const float t = a.t[k];
    double out[R];
#pragma unroll
    for (int r = 0; r < R; ++r) out[r] = (double)w[r][0];
    for (int f0 = 0; f0 < N; f0 += FC) {
      const int nf = min(FC, N - f0);
      if constexpr (STAGE) {
        __syncthreads();                       // the rows staged before have been used
        stage_rows(rows, S, a.X, row0, n_rows, N, f0, nf);
        __syncthreads();
      }
      // Several features' scalar gene loads in flight (about 64 SGPRs).
      constexpr int kAhead = std::clamp(64 / (R * B * D), 1, 8);
#pragma unroll kAhead
      for (int fi = 0; fi < nf; ++fi) {
        const double x = (double)mine[fi];
        const int at = 1 + (f0 + fi) * B * D;
        double cx = 0.0, sx = 0.0;
        if constexpr (BASIS == 3) sincos(x, &sx, &cx);
#pragma unroll
        for (int b = 0; b < B; ++b) {
          Recur<BASIS, double> rc;
          if constexpr (BASIS == 3) rc.seed_cs(cx, sx, b);
          else rc.seed(x, 0);
          auto term = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int r = 0; r < R; ++r) out[r] = fma((double)w[r][at + b * D + j], rc.cur, out[r]);
            if constexpr (j + 1 < D) rc.template advance<j + 1>(x);
          };
          [&]<int... J>(std::integer_sequence<int, J...>) {
            (term(std::integral_constant<int, J>{}), ...);
          }(std::make_integer_sequence<int, D>{});
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double res = (double)t - out[r];
      double e = res * res;
      if (a.error_fn == 2) e = fabs(res) > a.R ? e : 0.0;
      else if (a.error_fn == 3) e = e > a.R ? e : 0.0;
      acc[r] += valid ? e : 0.0;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) red[r][threadIdx.x] = acc[r];
  __syncthreads();
  for (int s = kRows / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
#pragma unroll
      for (int r = 0; r < R; ++r) red[r][threadIdx.x] += red[r][threadIdx.x + s];
    }
    __syncthreads();
  }
  if ((int)threadIdx.x < R && c0 + (int)threadIdx.x < a.n)
    a.partial[(int64_t)blockIdx.x * a.n + c0 + threadIdx.x] = red[threadIdx.x][0];
}

// Sum of each chromosome's block partials, one wave per chromosome: lane l
// adds blocks l, l + 64, ... (at most 16 of them, all loaded before the first
// addition), then a butterfly.  One thread adding 256 partials in turn took
// longer than the re-score itself (19.5 us of 37).
__global__ __launch_bounds__(64) void rescore64_finish(const double* partial, int32_t blocks,
                                                       int32_t n, int64_t NP, int32_t error_fn,
                                                       double* out) {
  const int c = blockIdx.x;
  double v[kRescoreBlocks / 64], s = 0.0;
#pragma unroll
  for (int u = 0; u < kRescoreBlocks / 64; ++u) {
    const int b = threadIdx.x + 64 * u;
    v[u] = b < blocks ? partial[(int64_t)b * n + c] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kRescoreBlocks / 64; ++u) s += v[u];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) out[c] = error_from_sum(s, NP, error_fn);
}

template <int BASIS, int D, int R, bool STAGE>
static hipError_t launch_group(const Rescore64Args& a, hipStream_t s) {
  const size_t lds =
      STAGE ? (size_t)kRows * row_stride(std::min(a.N, kChunk)) * sizeof(float) : 0;
  hipLaunchKernelGGL((rescore64_kernel<BASIS, D, R, STAGE>), dim3(a.blocks, (a.n + R - 1) / R),
                     dim3(kRows), lds, s, a);
  return hipGetLastError();
}

// Chromosomes per thread: one when groups of 4 would leave most CUs without
// a workgroup, otherwise 1, 2 or 4 by their number.
template <int BASIS, int D>
static hipError_t launch_one(const Rescore64Args& a, hipStream_t s) {
  if (!stages_rows((int64_t)a.blocks * ((a.n + 3) / 4)))
    return launch_group<BASIS, D, 1, false>(a, s);
  if (a.n == 1) return launch_group<BASIS, D, 1, true>(a, s);
  return a.n == 2 ? launch_group<BASIS, D, 2, true>(a, s) : launch_group<BASIS, D, 4, true>(a, s);
}

template <int BASIS>
static hipError_t launch_basis(const Rescore64Args& a, int degree, hipStream_t s) {
  switch (degree) {
#define GAME_CASE(D) case D: return launch_one<BASIS, D>(a, s);
    GAME_CASE(1) GAME_CASE(2) GAME_CASE(3) GAME_CASE(4) GAME_CASE(5) GAME_CASE(6)
    GAME_CASE(7) GAME_CASE(8) GAME_CASE(9) GAME_CASE(10) GAME_CASE(11) GAME_CASE(12)
    GAME_CASE(13) GAME_CASE(14) GAME_CASE(15) GAME_CASE(16)
#undef GAME_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rescore64(const Rescore64Args& a, int basis, int degree, double* out,
                            hipStream_t s) {
  hipError_t e;
  switch (basis) {
    case 0: e = launch_basis<0>(a, degree, s); break;
    case 1: e = launch_basis<1>(a, degree, s); break;
    case 2: e = launch_basis<2>(a, degree, s); break;
    case 3: e = launch_basis<3>(a, degree, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(rescore64_finish, dim3(a.n), dim3(64), 0, s, a.partial, a.blocks, a.n, a.NP,
                     a.error_fn, out);
  return hipGetLastError();
}

}  // namespace game
