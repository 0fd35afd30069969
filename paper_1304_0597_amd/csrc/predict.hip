// The "run" and classification use cases (Sec. 2 use cases; Sec. 5 figures
// of merit): the model output Out (Eq. 2) of given chromosomes on a set of
// patterns, stored, or turned into class decisions and counted.
//
// Each output is one chain of float32 fused multiply-adds in the canonical
// gene order (feature, block, degree) on the vector ALUs.  Prediction and
// classification share the output routine, so a class decision equals the
// stored output compared with the threshold.
//
// A thread owns one pattern and R chromosomes at a time, so an expansion
// value feeds R chains.  The genes are uniform over a workgroup and come in
// by scalar loads, one SGPR operand per multiply-add; the degree is a
// template argument, so the recurrence's coefficients are constants.  The
// patterns' rows are read in consecutive addresses into LDS (odd row stride:
// conflict-free) and serve every chromosome group of the workgroup; narrow rows
// and those of few workgroups each thread reads for itself.  Bound
// by the vector multiply-adds for 8 chromosomes and by reading the patterns
// for one.  1,000,000 x 20 patterns, Legendre 8: 25 us for one chromosome
// (80 MB of patterns, 4 MB of outputs: 3.4 TB/s), 57 us for 8, 367 us for 64
// (56 TFLOP/s of multiply-adds); with one thread per (pattern, chromosome),
// a run-time degree and a row read per output they took 125, 728 and 5,580.
#include <algorithm>
#include <utility>

#include "basis.h"
#include "rows.h"

namespace game {

namespace {

// out[r] of this thread's pattern (row threadIdx.x of the tile) for the
// chromosomes of group grp (the last one repeated past n).  `staged` tells
// whether LDS holds the tile's whole rows already.
template <int BASIS, int D, int R, bool STAGE>
__device__ __forceinline__ void tile_outputs(const PredictArgs& a, float* rows, int grp,
                                             int64_t row0, int n_rows, bool& staged,
                                             float (&out)[R]) {
  constexpr int B = BASIS == 3 ? 2 : 1;
  const int N = a.N;
  const int FC = STAGE ? min(N, kChunk) : N;
  const int S = row_stride(FC);
  const float* mine = STAGE ? rows + threadIdx.x * S
                            : a.X + (row0 + min((int)threadIdx.x, n_rows - 1)) * N;
  ConstGene* w[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    w[r] = (ConstGene*)a.genes + (int64_t)min(grp * R + r, a.n - 1) * a.K;
    out[r] = w[r][0];
  }
  for (int f0 = 0; f0 < N; f0 += FC) {
    const int nf = min(FC, N - f0);
    if (STAGE && !staged) {
      __syncthreads();            // the rows staged before have been used
      stage_rows(rows, S, a.X, row0, n_rows, N, f0, nf);
      __syncthreads();
      staged = FC == N;
    }
    // Several features' scalar gene loads in flight (as many as about 64
    // SGPRs hold): a small set's few waves otherwise wait out each one.
    constexpr int kAhead = std::clamp(64 / (R * B * D), 1, 8);
#pragma unroll kAhead
    for (int fi = 0; fi < nf; ++fi) {
      const float x = mine[fi];
      const int at = 1 + (f0 + fi) * B * D;
      float c = 0.f, s = 0.f;
      if constexpr (BASIS == 3) sincosf(x, &s, &c);
#pragma unroll
      for (int b = 0; b < B; ++b) {
        Recur<BASIS> rc;
        if constexpr (BASIS == 3) rc.seed_cs(c, s, b);
        else rc.seed(x, 0);
        auto term = [&](auto jc) {
          constexpr int j = decltype(jc)::value;
#pragma unroll
          for (int r = 0; r < R; ++r) out[r] = fmaf(w[r][at + b * D + j], rc.cur, out[r]);
          if constexpr (j + 1 < D) rc.template advance<j + 1>(x);
        };
        [&]<int... J>(std::integer_sequence<int, J...>) {
          (term(std::integral_constant<int, J>{}), ...);
        }(std::make_integer_sequence<int, D>{});
      }
    }
  }
}

template <int BASIS, int D, int R, bool STAGE>
__global__ __launch_bounds__(kRows) void predict_kernel(PredictArgs a) {
  extern __shared__ float rows[];
  const int n_groups = (a.n + R - 1) / R;
  const int64_t n_tiles = (a.NP + kRows - 1) / kRows;
  for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int64_t row0 = tile * kRows;
    const int n_rows = (int)min((int64_t)kRows, a.NP - row0);
    bool staged = false;
    for (int grp = blockIdx.y; grp < n_groups; grp += gridDim.y) {
      float out[R];
      tile_outputs<BASIS, D, R, STAGE>(a, rows, grp, row0, n_rows, staged, out);
      if ((int)threadIdx.x < n_rows) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (grp * R + r < a.n) a.out[(int64_t)(grp * R + r) * a.NP + row0 + threadIdx.x] = out[r];
      }
    }
  }
}

// Outputs of one chromosome (blockIdx.y) on narrow rows (own_rows): a thread reads
// its own row and walks over the patterns, the genes in LDS once.  A tile is so
// little work there that staging its rows, and a workgroup for each tile, cost
// more than the outputs.  1,000,000 patterns: 1 feature, power degree 1, one
// chromosome 4.5 us, 8.7 in staged tiles; 4 features, power 4, two 10.6 and 11.8; 8
// features, power 1, two 7.6 and 12.8.
template <int BASIS, int D>
__global__ __launch_bounds__(kRows) void predict_rows_kernel(PredictArgs a) {
  constexpr int B = BASIS == 3 ? 2 : 1;
  extern __shared__ float w[];
  const int N = a.N;
  for (int i = threadIdx.x; i < a.K; i += kRows) w[i] = a.genes[(int64_t)blockIdx.y * a.K + i];
  __syncthreads();
  float* out_c = a.out + (int64_t)blockIdx.y * a.NP;
  for (int64_t k = (int64_t)blockIdx.x * kRows + threadIdx.x; k < a.NP;
       k += (int64_t)gridDim.x * kRows) {
    const float* row = a.X + k * N;
    float out = w[0];
    for (int f = 0; f < N; ++f) {
      const float x = row[f];
      const float* g = w + 1 + f * B * D;
      float c = 0.f, s = 0.f;
      if constexpr (BASIS == 3) sincosf(x, &s, &c);
#pragma unroll
      for (int b = 0; b < B; ++b) {
        Recur<BASIS> rc;
        if constexpr (BASIS == 3) rc.seed_cs(c, s, b);
        else rc.seed(x, 0);
        auto term = [&](auto jc) {
          constexpr int j = decltype(jc)::value;
          out = fmaf(g[b * D + j], rc.cur, out);
          if constexpr (j + 1 < D) rc.template advance<j + 1>(x);
        };
        [&]<int... J>(std::integer_sequence<int, J...>) {
          (term(std::integral_constant<int, J>{}), ...);
        }(std::make_integer_sequence<int, D>{});
      }
    }
    out_c[k] = out;
  }
}

// Counts per chromosome, integer sums: exact in any order.  A workgroup
// takes several tiles of its chromosome group and adds its counts once.  With
// a.tally set each addition also counts its workgroup in the word's top 16
// bits, so whoever adds last sees it in the value the addition returns, moves
// the sum to the output and leaves the word zero for the next launch: no
// launch clears the counts first, and nothing has to be fenced.  2,100 x 11
// patterns, 23 chromosomes, trigonometric degree 4: 6.1 us; 13.7 with a fence
// and a counter of finished workgroups, 11.9 in two launches before.
constexpr int kTallyShift = 48;
template <int BASIS, int D, int R, bool STAGE>
__global__ __launch_bounds__(kRows) void classify_kernel(PredictArgs a) {
  extern __shared__ float rows[];
  __shared__ unsigned int sums[R * 4];
  const int64_t n_tiles = (a.NP + kRows - 1) / kRows;
  const int n_groups = (a.n + R - 1) / R;
  for (int grp = blockIdx.y; grp < n_groups; grp += gridDim.y) {
    if (threadIdx.x < R * 4) sums[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
      const int64_t row0 = tile * kRows;
      const int n_rows = (int)min((int64_t)kRows, a.NP - row0);
      const bool valid = (int)threadIdx.x < n_rows;
      const bool pos = valid && a.t[row0 + threadIdx.x] > 0.5f;
      bool staged = false;
      float out[R];
      tile_outputs<BASIS, D, R, STAGE>(a, rows, grp, row0, n_rows, staged, out);
      const int lane = threadIdx.x & 63;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool pred = out[r] >= a.threshold;
        const unsigned tp = __popcll(__ballot(valid && pred && pos));
        const unsigned fp = __popcll(__ballot(valid && pred && !pos));
        const unsigned tn = __popcll(__ballot(valid && !pred && !pos));
        const unsigned fn = __popcll(__ballot(valid && !pred && pos));
        if (lane < 4)
          atomicAdd(&sums[r * 4 + lane], lane == 0 ? tp : lane == 1 ? fp : lane == 2 ? tn : fn);
      }
    }
    __syncthreads();
    const int i = threadIdx.x;
    const int64_t at = (int64_t)grp * R * 4 + i;
    const bool mine = i < R * 4 && at < (int64_t)a.n * 4;
    if (gridDim.x == 1) {
      if (mine) a.counts[at] = sums[i];
    } else if (!a.tally) {
      if (mine) atomicAdd((unsigned long long*)a.counts + at, (unsigned long long)sums[i]);
    } else {
      if (mine) {
        const unsigned long long add = (1ull << kTallyShift) + sums[i];
        const unsigned long long sum = atomicAdd(a.tally + at, add) + add;
        if ((sum >> kTallyShift) == gridDim.x) {
          a.counts[at] = (int64_t)(sum & ((1ull << kTallyShift) - 1));
          a.tally[at] = 0;
        }
      }
    }
    __syncthreads();              // sums are free again
  }
}

__global__ void zero_counts_kernel(int64_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

template <int BASIS, int D, int R, bool STAGE>
hipError_t launch_variant(PredictArgs a, hipStream_t s) {
  const int64_t tiles = (a.NP + kRows - 1) / kRows;
  const int64_t groups = (a.n + R - 1) / R;
  const size_t lds =
      STAGE ? (size_t)kRows * row_stride(std::min(a.N, kChunk)) * sizeof(float) : 0;
  if (!a.counts) {
    // Once the pattern tiles alone fill the GPU a workgroup serves several
    // chromosome groups in turn with one read of its rows.  A launch dimension
    // holds less than 2^32 threads: beyond 2^28 patterns a workgroup takes
    // several tiles.
    constexpr int64_t kMostTiles = 1 << 20;
    static_assert(kMostTiles * kRows < (int64_t)1 << 32, "threads of a launch dimension");
    const int64_t gx = std::min(tiles, kMostTiles);
    const int64_t gy = std::min(groups, std::max<int64_t>(1, 2048 / gx));
    hipLaunchKernelGGL((predict_kernel<BASIS, D, R, STAGE>), dim3((unsigned)gx, (unsigned)gy),
                       dim3(kRows), lds, s, a);
    return hipGetLastError();
  }
  const int64_t gx = std::min<int64_t>(tiles, 1024);
  if (gx > 1 && a.n > kTallyChromosomes) {
    a.tally = nullptr;
    const int64_t n = (int64_t)a.n * 4;
    hipLaunchKernelGGL(zero_counts_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       a.counts, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((classify_kernel<BASIS, D, R, STAGE>), dim3((unsigned)gx, (unsigned)groups),
                     dim3(kRows), lds, s, a);
  return hipGetLastError();
}

// Rows that each thread reads for itself, one chromosome at a time: those narrow
// enough for their cache lines to be used while they are there, as far as reading
// them again for each chromosome stays below what staging costs.  1,000,000
// patterns, power 1: 8 features, one chromosome 5.5 us (9.1 staged), two 7.6 (12.6),
// four 11.5 (13.5, but other degrees up to 26 % slower so); 12, one 13.2 (12.6); 3,
// four 10.2 (11.9).  With a sine and cosine for every read, 8 features of one
// chromosome take up to 30 % longer, 3 features of four 6 to 24.  Up to one and a
// half tiles a CU staging covers less: 66,000 patterns, 12 features, one chromosome 3.4
// us (4.5), 5 of four 3.7 (4.3).  Classification has more to do per tile: 1,000,000
// patterns, 1 feature, one chromosome 17.0 us (20.5), two 26.3 (19.7).
bool own_rows(const PredictArgs& a, int64_t tiles, bool trig) {
  const bool few = tiles < 384;
  if (a.counts) return a.n == 1 && a.N <= (trig ? 4 : 16);
  if (trig) return a.n <= 2 ? a.N <= 4 : a.N <= 3 && a.n * a.N <= 8;
  if (a.n <= 2) return a.N <= (few ? 16 : 8);
  return few ? a.N <= 6 && a.n * a.N <= 36 : a.N <= 3 && a.n * a.N <= 12;
}

// Chromosomes per thread: one when groups of 8 would leave most CUs without
// a workgroup (2,100 x 11 patterns, 23 chromosomes: 6.1 us against 11.5),
// otherwise groups of 4 or 8 (1,000,000 x 20, 5 chromosomes: 59 us for two
// groups of 4 or one of 8, 125 for five of one).
template <int BASIS, int D>
hipError_t launch_degree(const PredictArgs& a, hipStream_t s) {
  const int64_t tiles = (a.NP + kRows - 1) / kRows;
  const bool own = own_rows(a, tiles, BASIS == 3);
  if (!stages_rows(tiles * ((a.n + 7) / 8)) || (own && a.counts))
    return launch_variant<BASIS, D, 1, false>(a, s);
  if (own) {
    hipLaunchKernelGGL((predict_rows_kernel<BASIS, D>),
                       dim3((unsigned)std::min<int64_t>(tiles, 1024), (unsigned)a.n), dim3(kRows),
                       (size_t)a.K * sizeof(float), s, a);
    return hipGetLastError();
  }
  if (a.n == 1) return launch_variant<BASIS, D, 1, true>(a, s);
  return a.n <= 4 ? launch_variant<BASIS, D, 4, true>(a, s)
                  : launch_variant<BASIS, D, 8, true>(a, s);
}

template <int BASIS>
hipError_t launch_basis(const PredictArgs& a, hipStream_t s) {
  switch (a.degree) {
#define GAME_CASE(D) case D: return launch_degree<BASIS, D>(a, s);
    GAME_CASE(1) GAME_CASE(2) GAME_CASE(3) GAME_CASE(4) GAME_CASE(5) GAME_CASE(6)
    GAME_CASE(7) GAME_CASE(8) GAME_CASE(9) GAME_CASE(10) GAME_CASE(11) GAME_CASE(12)
    GAME_CASE(13) GAME_CASE(14) GAME_CASE(15) GAME_CASE(16)
#undef GAME_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_predict(const PredictArgs& a, int basis, hipStream_t s) {
  switch (basis) {
    case 0: return launch_basis<0>(a, s);
    case 1: return launch_basis<1>(a, s);
    case 2: return launch_basis<2>(a, s);
    case 3: return launch_basis<3>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace game
