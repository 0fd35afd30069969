// Fused GAME fitness in float32 on MFMA (gfx950).
//
// For chromosome p and pattern k (Eq. 2 with per-feature genes):
//   Out[k,p] = a_0(p) + sum_{i,b,j} gene_p(i,b,j) * phi_{b,j}(x_{k,i})
// and the fitness is sum_k E_k / NP with E_k = (t_k - Out[k,p])^2 (Eqs. 3-4)
// or its thresholded form (Eq. 10).  The sum over (i,b,j) is a dense
// contraction: M = patterns, N = chromosomes, K = B*N*d expansion terms.
//
// Design:
//  * v_mfma_f32_32x32x2_f32.  The A operand (patterns x K) is never stored:
//    each lane owns one pattern row and one sub-feature u = (i, b) and
//    produces phi_1..phi_d of that sub-feature with the basis's three-term
//    recurrence, one value per K-step.  K is ordered so that the two lane
//    halves of a K-step carry sub-features 2q and 2q+1 at the same degree j,
//    so a lane's recurrence never crosses a feature boundary.
//  * The B operand (K x chromosomes) is copied once per workgroup into LDS,
//    one row per chromosome in the canonical gene order (odd row stride:
//    conflict-free ds_read_b32), by LDS DMA (global_load_lds_dword), so the
//    copy costs no registers and one memory round trip.  When K does not
//    fit, it passes through two buffers in chunks of whole feature pairs,
//    the next chunk's copy in flight while the current one is used.
//  * Accumulators start at zero.  A last K-step brings in the bias and the
//    target (lane half 0: 1 x a_0(p); half 1: -t_k x 1), so the accumulators
//    end at Out - t; the epilogue squares (or applies the error function)
//    and sums the lane's 32 rows in float32, then adds into a float64
//    running sum.
//    Partials per (chromosome, split) are combined in a fixed order: the
//    result does not depend on scheduling.
//  * The trigonometric expansion (Eq. 8) is seeded with cos x and sin x of
//    the lane's feature.  For the run's own data set they come from a table
//    computed once per data set (FitArgs::cs); otherwise sincosf in every
//    chromosome tile.
//  * Wave tile 64 patterns x 32*CB chromosomes: each generated A value feeds
//    CB MFMAs per row block.  CB = 4: a workgroup takes 128 chromosomes with
//    eight waves, waves 0-3 on the even pattern tiles of its split and 4-7 on
//    the odd ones (two waves per SIMD, one gene copy per CU, up to 159 K-steps
//    of genes before they are chunked).  CB = 2 or 1: 64 or 32 chromosomes with
//    four waves, several workgroups per CU (up to 128 K-steps).  Wider tiles
//    spread the recurrence and the feature loads over more MFMAs, narrower
//    ones fill the GPU when there are few tiles; plan_fitness chooses.
//  * At low degree a feature pair is little work next to its load's latency:
//    the features of several pairs, and the targets, are loaded a group (a
//    tile) ahead, and rows of whole 16-byte quads a quad per lane and load.
//    7,168,000 x 16 patterns, degree 1, 23 chromosomes (TMSE): 347 us before,
//    172 so, and 130 in the loop of its own that narrow rows have
//    (fitness_f32_narrow).
//  * Grid: (pattern split) x (chromosome tile); consecutive blocks of one
//    split are mapped onto one XCD so its L2 serves the split's rows to all
//    chromosome tiles.
#include <algorithm>

#include "fitness_f32_body.h"
#include "philox.h"

namespace game {

// ROWS: the general tile body, the one for narrow rows, single features or
// whole quads at a time, or the general one reading two quads at a time.
enum { kGeneralRows, kNarrowRows, kNarrowQuads, kQuadRows };
template <int BASIS, int D, int CB, int ROWS>
__global__ __launch_bounds__(64 * fit_waves(CB), (ROWS && CB == 1 ? 16 : 8) / fit_waves(CB)) void
fitness_f32_kernel(FitArgs a) {
  extern __shared__ float lds[];
  const int total = a.n_ctiles * a.n_splits;
  const int b = blockIdx.x;
  const float* __restrict__ genes = a.genes;
  if (a.genes_alt) {
    if (*a.gen_sel & 1) genes = a.genes_alt;
    // Kept a branch: a population at a fixed place is staged without waiting
    // for the generation counter.
    __asm__ __volatile__("" : "+s"(genes));
  }
  if (b >= total) {
    // The genetic step's draws, on CUs that a small launch leaves idle.
    const int i = (b - total) * (int)blockDim.x + (int)threadIdx.x;
    if (!*a.stop && i < a.draw.n_items) make_draw(a.draw, genes, *a.gen_sel + 1, i);
    return;
  }
  // Consecutive L on one XCD (workgroup b runs on XCD b % 8), the first
  // total % 8 XCDs taking one more.
  const int xcd = b & 7;
  const int L = xcd * (total >> 3) + min(xcd, total & 7) + (b >> 3);
  const int split = L / a.n_ctiles;
  const int ctile = L - split * a.n_ctiles;
  if constexpr (ROWS == kGeneralRows)
    fitness_f32_block<BASIS, D, CB>(a, genes, split, ctile, lds, a.stop);
  else if constexpr (ROWS == kQuadRows)
    fitness_f32_block<BASIS, D, CB, 2, 4>(a, genes, split, ctile, lds, a.stop);
  else
    fitness_f32_narrow<BASIS, D, CB, ROWS == kNarrowQuads>(a, genes, split, ctile, lds, a.stop);
  if (b == 0 && threadIdx.x == 0) {
    if (a.stop_seen) *a.stop_seen = *a.stop;
    if (a.gen_seen) *a.gen_seen = *a.gen_sel;
  }
}

template <int BASIS, int D, int CB, int ROWS>
static hipError_t launch_rows(const FitArgs& a, hipStream_t s) {
  const size_t lds = ROWS == kNarrowRows || ROWS == kNarrowQuads
                         ? fit_waves(CB) * 32 * CB * sizeof(double)
                         : fitness_lds_bytes(a, D);
  const int threads = 64 * fit_waves(CB);
  const int grid = a.n_ctiles * a.n_splits + (a.draw.n_items + threads - 1) / threads;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)fitness_f32_kernel<BASIS, D, CB, ROWS>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((fitness_f32_kernel<BASIS, D, CB, ROWS>), dim3(grid), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template <int BASIS, int D, int CB>
static hipError_t launch_cb(const FitArgs& a, hipStream_t s) {
  if constexpr (BASIS < 3 && narrow_degree(D) && CB <= 2) {
    if (a.Q <= pairs_ahead(D, CB))
      return a.N % 4 == 0 && reinterpret_cast<uintptr_t>(a.X) % 16 == 0
                 ? launch_rows<BASIS, D, CB, kNarrowQuads>(a, s)
                 : launch_rows<BASIS, D, CB, kNarrowRows>(a, s);
  }
  // Wide tiles of rows that are pairs of quads: 1,000,000 x 32, 2,048
  // chromosomes, degree 1 1,266 us (1,416 by pairs), degree 2 2,151 (2,193).
  if constexpr (BASIS < 3 && D <= 2 && CB == 4) {
    if (a.N % 8 == 0 && reinterpret_cast<uintptr_t>(a.X) % 16 == 0)
      return launch_rows<BASIS, D, CB, kQuadRows>(a, s);
  }
  return launch_rows<BASIS, D, CB, kGeneralRows>(a, s);
}

template <int BASIS, int D>
static hipError_t launch_one(const FitArgs& a, hipStream_t s) {
  if (a.tile_cols == 128) return launch_cb<BASIS, D, 4>(a, s);
  if (a.tile_cols == 32) return launch_cb<BASIS, D, 1>(a, s);
  return launch_cb<BASIS, D, 2>(a, s);
}

template <int BASIS>
static hipError_t launch_basis(const FitArgs& a, int degree, hipStream_t s) {
  switch (degree) {
#define GAME_CASE(D) case D: return launch_one<BASIS, D>(a, s);
    GAME_CASE(1) GAME_CASE(2) GAME_CASE(3) GAME_CASE(4) GAME_CASE(5) GAME_CASE(6)
    GAME_CASE(7) GAME_CASE(8) GAME_CASE(9) GAME_CASE(10) GAME_CASE(11) GAME_CASE(12)
    GAME_CASE(13) GAME_CASE(14) GAME_CASE(15) GAME_CASE(16)
#undef GAME_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fitness_f32(const FitArgs& a, int basis, int degree, hipStream_t s) {
  switch (basis) {
    case 0: return launch_basis<0>(a, degree, s);
    case 1: return launch_basis<1>(a, degree, s);
    case 2: return launch_basis<2>(a, degree, s);
    case 3: return a.cs ? launch_basis<kTrigTable>(a, degree, s) : launch_basis<3>(a, degree, s);
    default: return hipErrorInvalidValue;
  }
}

bool narrow_rows(const FitArgs& a) {
  const int cb = a.tile_cols / 32;
  return a.basis < 3 && narrow_degree(a.degree) && cb <= 2 && a.Q <= pairs_ahead(a.degree, cb);
}

size_t fitness_lds_bytes(const FitArgs& a, int degree) {
  const int cols = a.tile_cols;
  const size_t w = (size_t)(a.n_chunks > 1 ? 2 : 1) * cols *
                   (2 * a.pairs_per_chunk * degree + 1) * sizeof(float);
  const size_t red = (size_t)fit_waves(cols / 32) * cols * sizeof(double);
  return w > red ? w : red;
}

// K-steps (per lane half) of genes that stay in LDS for the whole launch:
// several narrow workgroups share a CU, a 128-chromosome one has it to itself;
// beyond that the genes pass through two buffers in chunks.
static int max_staged_steps(int cb) { return cb == 4 ? kMaxWideSteps : kMaxChunkSteps; }

// Estimated time of a step (64 rows x 32 cb chromosomes) of w waves per SIMD,
// in cycles of the SIMD per wave.  The MFMAs take m; the rest (recurrence,
// feature and gene reads, epilogue) costs v beyond them at two or more waves
// per SIMD and twice that when nothing runs beside it; genes that pass through
// LDS in chunks cost the more the narrower the tile.  Fitted to launches of 16
// to 320 expansion terms and 23 to 2,048 chromosomes (within 5 % of their
// times, for 64-chromosome tiles within 15).
static int64_t step_cost(int cb, int pairs, int degree, int w, bool trig) {
  const int ksteps = pairs * degree;
  const int64_t m = 128 * cb * (ksteps + 1);
  // per feature pair (its loads, its seed) and per degree.  Two MFMAs (degree 1 of
  // a narrow tile) do not cover the reads of a pair of (cos x, sin x): 6,199 x 28,
  // 777 chromosomes 19.5 us in 32s, which were taken at 60 a pair, 18.2 in 128s.
  int64_t v = cb == 1 ? 1800 + (trig && degree == 1 ? 120 : 60) * pairs + 9 * ksteps
                      : (cb == 4 ? 4200 : 3400) + 100 * pairs + 27 * ksteps;
  if (ksteps > max_staged_steps(cb)) v += m * (cb == 4 ? 13 : cb == 2 ? 40 : 55) / 100;
  return m + (w > 1 ? v : 2 * v);
}

void plan_fitness(FitArgs& a, int degree, int basis, bool wide) {
  a.U = (basis == 3 ? 2 : 1) * a.N;
  a.Q = (a.U + 1) / 2;
  a.n_tiles = (int32_t)((a.NP + kTileRows - 1) / kTileRows);
  // Tile width and splits of a single run: the combination of least estimated
  // time.  Wide tiles do the least work besides MFMAs, but a launch has few of
  // them: 4,000 x 20 patterns, Legendre 8, 100 chromosomes take 31 us in 16
  // workgroups of 128 chromosomes and 13 in 64 of 32; 200,000 x 20 with 2,048
  // take 980 in 128s, 1,046 in 64s and 1,091 in 32s.  All workgroups of a
  // launch are resident at once (one of eight waves per CU, two or four of four
  // waves; launches of few terms run two rounds of four): splits are rounded down
  // to that, since a few workgroups more run a round of their own (100,000 x 32,
  // Chebyshev 10, 1,500 chromosomes: 1,615 us in 264 workgroups, 850 in 252).
  int best_cb = 2, best_tps = 1;
  int64_t best = INT64_MAX;
  for (int cb = 4; cb >= 1; cb >>= 1) {
    if (!wide && cb != 2) continue;
    if (cb > 1 && 32 * (cb / 2) >= a.n_chrom && wide) continue;   // half the tile would be empty
    const int ctiles = (a.n_chrom + 32 * cb - 1) / (32 * cb);
    const int streams = cb == 4 ? 2 : 1;
    // As many workgroups per CU as fit (few terms need the most reads in
    // flight: 8 are two rounds of 4), or fewer when that saves more than 3 %.
    // Narrow rows keep their genes in registers, and one round reads them once:
    // 7,168,000 x 16 in 1,024 workgroups 136 us, in 2,048 147.
    const bool narrow = basis < 3 && narrow_degree(degree) && a.Q <= pairs_ahead(degree, cb);
    const int most = cb == 4 ? 1 : cb == 2 ? 2 : a.Q * degree <= 16 && !narrow ? 8 : 4;
    int64_t best_of_cb = INT64_MAX;
    int tps_of_cb = 1;
    int64_t start_of_cb = 0;       // start-up of a CU's workgroups
    for (int per_cu = most; per_cu >= 1; --per_cu) {
      int splits = 256 * per_cu / ctiles;
      splits = std::min({std::max(splits, 1), max_splits(ctiles * 32 * cb), a.n_tiles});
      const int tps = (a.n_tiles + splits - 1) / splits;
      const int64_t groups = (int64_t)ctiles * ((a.n_tiles + tps - 1) / tps);
      // An odd tile count leaves one of a wide workgroup's streams its last tile
      // alone.
      const int64_t per_cu_groups = (groups + 255) / 256;
      const int64_t w = per_cu_groups * std::min(streams, tps);
      const int64_t cost = per_cu_groups * (streams == 1
                               ? tps * step_cost(cb, a.Q, degree, (int)w, basis == 3)
                               : (tps & ~1) * step_cost(cb, a.Q, degree, 2, basis == 3) +
                                     (tps & 1) * step_cost(cb, a.Q, degree, 1, basis == 3));
      if (best_of_cb == INT64_MAX || cost + cost / 32 < best_of_cb) {
        best_of_cb = cost;
        tps_of_cb = tps;
        start_of_cb = per_cu_groups * 1500;
      }
    }
    best_of_cb += start_of_cb;
    // (narrower tiles only where they win clearly: the estimate is within 15 %)
    if (best == INT64_MAX || best_of_cb + best_of_cb / 8 < best) {
      best = best_of_cb;
      best_cb = cb;
      best_tps = tps_of_cb;
    }
  }
  a.tile_cols = 32 * best_cb;
  a.tiles_per_split = best_tps;
  a.n_splits = (a.n_tiles + best_tps - 1) / best_tps;
  a.n_ctiles = (a.n_chrom + a.tile_cols - 1) / a.tile_cols;
  a.ld_partial = a.n_ctiles * a.tile_cols;
  int ppc = a.Q * degree <= max_staged_steps(best_cb) ? a.Q : kChunkSteps / degree;
  if (ppc < 1) ppc = 1;
  a.pairs_per_chunk = ppc;
  a.n_chunks = (a.Q + ppc - 1) / ppc;
}

// fitness[i] = sum_s partial[s][i] / NP (wave_split_sum order), RMSE takes
// the root; NaN becomes +inf.  One wave per chromosome.
__global__ void finish_kernel(const double* __restrict__ partial, int32_t ld, int32_t n,
                              int32_t n_splits, int64_t NP, int32_t error_fn, float* f32,
                              double* f64) {
  const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (i >= n) return;
  const double v = error_from_sum(wave_split_sum(partial, ld, n_splits, i), NP, error_fn);
  if ((threadIdx.x & 63) == 0) {
    if (f32) f32[i] = (float)v;
    if (f64) f64[i] = v;
  }
}

hipError_t launch_finish(const double* partial, int32_t ld, int32_t n, int32_t n_splits,
                         int64_t NP, int32_t error_fn, float* f32, double* f64, hipStream_t s) {
  hipLaunchKernelGGL(finish_kernel, dim3((n + 3) / 4), dim3(256), 0, s, partial, ld, n,
                     n_splits, NP, error_fn, f32, f64);
  return hipGetLastError();
}

}  // namespace game
