// Float64 re-score: the error of a few chromosomes (the elite at the end of
// a reduced-precision run, or an audit sample) computed in double precision
// on the vector ALUs, from the same X, t and genes (Eqs. 2-5, 10).
//
// Grid (pattern blocks, groups of R chromosomes): a thread takes T patterns
// of a 256-row tile at a time; the tile's rows (read in consecutive
// addresses) sit in LDS and the genes come in by scalar loads.  A block adds
// its threads' squared residuals in a fixed tree order, and a finish pass
// (one wave per chromosome) adds the blocks in a fixed order, so the result
// is deterministic.
//
// Bound by the float64 multiply-adds and the gene conversions, one of each
// per term next to the recurrence's, with the patterns' read under them.
// 250,000 x 32 patterns, Chebyshev 8, one chromosome: 15.7 us with the finish
// pass (37.5 with 256 blocks reading rows thread by thread and one thread
// adding their partials); 1,000,000 x 32: 54 us against 80 (2.4 TB/s of
// patterns, 64 chromosomes 1.33 ms against 4.8).  Publishing
// the partials to a last block with device-scope atomics instead of a second
// launch was slower (24.4 us): its round trips are serial.
#include <algorithm>
#include <utility>

#include "basis.h"
#include "rows.h"

namespace game {

template <int BASIS, int D, int R, int T, bool STAGE>
__global__ __launch_bounds__(kRows / T) void rescore64_kernel(Rescore64Args a) {
  constexpr int B = BASIS == 3 ? 2 : 1;
  constexpr int kThreads = kRows / T;
  extern __shared__ float rows[];
  __shared__ double red[R][kThreads];
  const int N = a.N;
  const int FC = STAGE ? min(N, kChunk) : N;
  const int S = row_stride(FC);
  const int c0 = blockIdx.y * R;
  ConstGene* w[R];
  double acc[T][R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    w[r] = (ConstGene*)a.genes + (int64_t)min(c0 + r, a.n - 1) * a.K;
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i][r] = 0.0;
  }
  const int64_t n_tiles = (a.NP + kRows - 1) / kRows;
  for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int64_t row0 = tile * kRows;
    const int n_rows = (int)min((int64_t)kRows, a.NP - row0);
    // Rows threadIdx.x + kThreads * i of the tile.
    bool valid[T];
    const float* mine[T];
    float t[T];
    double out[T][R];
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int row = (int)threadIdx.x + kThreads * i;
      valid[i] = row < n_rows;
      const int64_t k = valid[i] ? row0 + row : row0;
      mine[i] = STAGE ? rows + row * S : a.X + k * N;
      t[i] = a.t[k];
#pragma unroll
      for (int r = 0; r < R; ++r) out[i][r] = (double)w[r][0];
    }
    for (int f0 = 0; f0 < N; f0 += FC) {
      const int nf = min(FC, N - f0);
      if constexpr (STAGE) {
        __syncthreads();                       // the rows staged before have been used
        stage_rows<kThreads>(rows, S, a.X, row0, n_rows, N, f0, nf);
        __syncthreads();
      }
      // Several features' scalar gene loads in flight (about 64 SGPRs).
      constexpr int kAhead = std::clamp(64 / (R * B * D), 1, 8);
#pragma unroll kAhead
      for (int fi = 0; fi < nf; ++fi) {
        const int at = 1 + (f0 + fi) * B * D;
        double x[T], cx[T], sx[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
          x[i] = (double)mine[i][fi];
          if constexpr (BASIS == 3) sincos(x[i], &sx[i], &cx[i]);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
          Recur<BASIS, double> rc[T];
#pragma unroll
          for (int i = 0; i < T; ++i) {
            if constexpr (BASIS == 3) rc[i].seed_cs(cx[i], sx[i], b);
            else rc[i].seed(x[i], 0);
          }
          auto term = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const double g = (double)w[r][at + b * D + j];
#pragma unroll
              for (int i = 0; i < T; ++i) out[i][r] = fma(g, rc[i].cur, out[i][r]);
            }
            if constexpr (j + 1 < D) {
#pragma unroll
              for (int i = 0; i < T; ++i) rc[i].template advance<j + 1>(x[i]);
            }
          };
          [&]<int... J>(std::integer_sequence<int, J...>) {
            (term(std::integral_constant<int, J>{}), ...);
          }(std::make_integer_sequence<int, D>{});
        }
      }
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double res = (double)t[i] - out[i][r];
        double e = res * res;
        if (a.error_fn == 2) e = fabs(res) > a.R ? e : 0.0;
        else if (a.error_fn == 3) e = e > a.R ? e : 0.0;
        acc[i][r] += valid[i] ? e : 0.0;
      }
  }
  // The first steps of the tree over kRows sums are a thread's own.
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int h = T / 2; h > 0; h >>= 1)
#pragma unroll
      for (int i = 0; i < h; ++i) acc[i][r] += acc[i + h][r];
    red[r][threadIdx.x] = acc[0][r];
  }
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
#pragma unroll
      for (int r = 0; r < R; ++r) red[r][threadIdx.x] += red[r][threadIdx.x + s];
    }
    __syncthreads();
  }
  if ((int)threadIdx.x < R && c0 + (int)threadIdx.x < a.n)
    a.partial[(int64_t)blockIdx.x * a.n + c0 + threadIdx.x] = red[threadIdx.x][0];
}

// Fewer workgroups than CUs and many genes per feature (many_genes): block b takes
// the tiles b, b + blocks, ... of one chromosome, its genes widened once into LDS.
// The kernel above keeps 64 SGPRs of genes in flight, which is less the fewer
// features that is, and nothing else on the CU covers the rest.
template <int BASIS, int D>
__global__ __launch_bounds__(kRows) void rescore64_few_kernel(Rescore64Args a) {
  extern __shared__ double genes[];
  __shared__ double red[kRows];
  const int c = blockIdx.y;
  const float* g = a.genes + (int64_t)c * a.K;
  for (int i = threadIdx.x; i < a.K; i += blockDim.x) genes[i] = (double)g[i];
  __syncthreads();
  constexpr int B = BASIS == 3 ? 2 : 1;
  double acc = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < a.NP;
       k += (int64_t)gridDim.x * blockDim.x) {
    double out = genes[0];
    for (int f = 0; f < a.N; ++f) {
      const double x = (double)a.X[k * a.N + f];
      for (int b = 0; b < B; ++b) {
        Recur<BASIS, double> rc;
        rc.seed(x, b);
        const double* w = genes + 1 + (f * B + b) * D;
        auto term = [&](auto jc) {
          constexpr int j = decltype(jc)::value;
          out = fma(w[j], rc.cur, out);
          if constexpr (j + 1 < D) rc.template advance<j + 1>(x);
        };
        [&]<int... J>(std::integer_sequence<int, J...>) {
          (term(std::integral_constant<int, J>{}), ...);
        }(std::make_integer_sequence<int, D>{});
      }
    }
    const double r = (double)a.t[k] - out;
    double e = r * r;
    if (a.error_fn == 2) e = fabs(r) > a.R ? e : 0.0;
    else if (a.error_fn == 3) e = e > a.R ? e : 0.0;
    acc += e;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = kRows / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.partial[(int64_t)blockIdx.x * a.n + c] = red[0];
}

// Sum of each chromosome's block partials, one wave per chromosome: lane l
// adds blocks l, l + 64, ... (at most 16 of them, all loaded before the first
// addition), then a butterfly.  One thread adding 256 partials in turn took
// longer than the re-score itself (19.5 us of 37).
// U: loads per lane, 64 U >= blocks.
template <int U>
__global__ __launch_bounds__(64) void rescore64_finish(const double* partial, int32_t blocks,
                                                       int32_t n, int64_t NP, int32_t error_fn,
                                                       double* out) {
  const int c = blockIdx.x;
  double v[U], s = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = partial[(int64_t)min((int)threadIdx.x + 64 * u, blocks - 1) * n + c];
#pragma unroll
  for (int u = 0; u < U; ++u) s += (int)threadIdx.x + 64 * u < blocks ? v[u] : 0.0;
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) out[c] = error_from_sum(s, NP, error_fn);
}

// The same for up to kFewBlocks blocks, a thread per chromosome: no workgroup for
// each (255 x 7, Chebyshev 4, 16 chromosomes 5.3 us, 4.8 so).
constexpr int kFewBlocks = 4;
__global__ __launch_bounds__(256) void rescore64_finish_few(const double* partial, int32_t blocks,
                                                            int32_t n, int64_t NP,
                                                            int32_t error_fn, double* out) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= n) return;
  double s = 0.0;
  for (int b = 0; b < blocks; ++b) s += partial[(int64_t)b * n + c];
  out[c] = error_from_sum(s, NP, error_fn);
}

// Where the genes of an unstaged launch go through LDS: by what a term computes to
// cover its gene's load (a power least; sine and cosine have two genes a degree).
// 1,000 patterns, one to three chromosomes, LDS and scalar loads: trigonometric 16 x
// 8 features 9.0 and 10.0 us, 10 x 16 12.2 and 12.9, 4 x 30 17.0 and 16.8, 2 x 8 7.4
// and 6.7; power 12 x 17 and Legendre 16 x 20 lose 7 to 11 % to scalar loads, Chebyshev
// 10 x 32 and Legendre 8 x 32 gain 8 to 12.
constexpr bool many_genes(int basis, int d) {
  return d >= (basis == 3 ? 5 : basis == 2 ? 9 : 11);
}

template <int BASIS, int D, int R, int T, bool STAGE>
static hipError_t launch_group(const Rescore64Args& a, hipStream_t s) {
  const size_t lds =
      STAGE ? (size_t)kRows * row_stride(std::min(a.N, kChunk)) * sizeof(float) : 0;
  hipLaunchKernelGGL((rescore64_kernel<BASIS, D, R, T, STAGE>), dim3(a.blocks, (a.n + R - 1) / R),
                     dim3(kRows / T), lds, s, a);
  return hipGetLastError();
}

// Chromosomes per thread: one when groups of 4 would leave most CUs without
// a workgroup (their genes through LDS where many_genes says so), otherwise 1, 2
// or 4 by their number.  Patterns per thread: two for
// sine and cosine, whose long serial evaluations then overlap (200,000 x 13: degree
// 8, one chromosome 19.8 us, 26.5 with one; degree 3, five 31.4 and 43.5; four
// patterns 23.5 and 32.8); one otherwise, where the waves lost cost more than the
// gene conversions saved (1,000,000 x 32, Chebyshev 8: 50 us, 54 with two).
template <int BASIS, int D>
static hipError_t launch_one(const Rescore64Args& a, hipStream_t s) {
  constexpr int T = BASIS == 3 ? 2 : 1;
  if (!stages_rows((int64_t)a.blocks * ((a.n + 3) / 4))) {
    if constexpr (many_genes(BASIS, D)) {
      hipLaunchKernelGGL((rescore64_few_kernel<BASIS, D>), dim3(a.blocks, a.n), dim3(kRows),
                         (size_t)a.K * sizeof(double), s, a);
      return hipGetLastError();
    } else {
      return launch_group<BASIS, D, 1, 1, false>(a, s);
    }
  }
  if (a.n == 1) return launch_group<BASIS, D, 1, T, true>(a, s);
  return a.n == 2 ? launch_group<BASIS, D, 2, T, true>(a, s)
                  : launch_group<BASIS, D, 4, T, true>(a, s);
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
  auto finish = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(a.n), dim3(64), 0, s, a.partial, a.blocks, a.n, a.NP,
                       a.error_fn, out);
    return hipGetLastError();
  };
  static_assert(kRescoreBlocks == 64 * 16, "the widest finish");
  if (a.blocks <= kFewBlocks) {
    hipLaunchKernelGGL(rescore64_finish_few, dim3((a.n + 255) / 256), dim3(256), 0, s, a.partial,
                       a.blocks, a.n, a.NP, a.error_fn, out);
    return hipGetLastError();
  }
  if (a.blocks <= 64) return finish(rescore64_finish<1>);
  if (a.blocks <= 256) return finish(rescore64_finish<4>);
  return finish(rescore64_finish<16>);
}

}  // namespace game
