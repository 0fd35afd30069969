// Whole runs of the smallest problems in one workgroup.
//
// A generation of a small run is a fitness launch and a tail launch
// (ga.hip), 4 to 5 us each whatever they compute.  When the expanded data
// set fits one CU's LDS and the products are a few microseconds of that CU,
// one workgroup runs generation after generation with barriers in place of
// launches:
//  * The A operands (the expansion of every pattern, degree by degree, and the
//    bias/target step) are written to LDS once per launch, 64 rows to a unit,
//    and the B operands with each population, both in the lanes' own order; the
//    populations, the draws and the errors live there too.  Global memory is
//    read at the start and written at the end.
//  * Each of the 16 waves takes units u, u + 16, ... through all K-steps of
//    the float32 MFMA and leaves its rows' error sum.  Matrix and vector
//    instructions of a SIMD take turns (32x32x2 float32 products run at the
//    vector rate), so this phase is their sum; draws made beside it, or units
//    handed out by a counter, were slower (6.8 us a generation for 6.3).
//  * A barrier, the errors, a barrier, then lp lanes to a pair of children:
//    selection in one DPP step per halving, both children's genes.  Waves
//    without errors or children make the draws a generation ahead, half of the
//    Philox rounds in either phase.
// Products, sums and operators are taken in the order of the fitness kernel
// and the two-launch generation, so a run has the same bits on either path.
//
// 2,100 patterns x 8 features, degree 1, 23 chromosomes, 1,000 generations: 8.2 ms
// with two launches a generation and 5.2 here with the mean square, 6.2 with the
// thresholded error (4.5 us of a generation in the products and their error terms).
#include <algorithm>

#include "basis.h"
#include "ga_ops.h"

namespace game {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kResThreads = 1024;
constexpr int kResWaves = kResThreads / 64;
constexpr int kResPopulation = 64;     // two 32-column tiles

struct ResidentArgs {
  const float* X;
  const float* t;
  const float* cs;
  int64_t NP;
  int32_t N, D, basis, U, S;           // S: K-steps, without the bias step
  int32_t units, nct, n_tiles;
  int32_t error_fn;
  float R;
  int32_t blocks, need_order, generations;
  int32_t b_at, red_at, e64_at, words_at, pop_at;  // byte offsets in LDS
  float* fit32;
  double* fit64;
  RunState* state;
  GAArgs ga;
};

// The expansion of one feature (one lane half of it) to degree D, one value
// every `stride` floats of dst; rows past the data get zeros.
__device__ void expand(const ResidentArgs& a, float x, float sx, int h, bool keep, float* dst,
                       int stride) {
  float prev = 1.f, cur = x, m2 = 2.f * x;
  if (a.basis == 3) {
    prev = h ? 0.f : 1.f;
    cur = h ? sx : x;
  }
  if (!keep) prev = cur = 0.f;
  for (int j = 0; j < a.D; ++j) {
    dst[j * stride] = cur;
    if (a.basis == 2) {
      cur *= x;
    } else if (a.basis == 1) {
      const float n1 = (float)(j + 2);
      const float ca = __fdiv_rn((float)(2 * j + 3), n1), cb = __fdiv_rn((float)(j + 1), n1);
      const float n = fmaf(ca * x, cur, -(cb * prev));
      prev = cur;
      cur = n;
    } else {
      const float n = fmaf(m2, cur, -prev);
      prev = cur;
      cur = n;
    }
  }
}

template <int MODE>
__device__ __forceinline__ float unit_error(const f32x16 (&acc)[2], float R) {
  float s = 0.f;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float v = acc[rb][i];
      if constexpr (MODE == 0) {
        s = __builtin_fmaf(v, v, s);
      } else {
        const float e = __fmul_rn(v, v);
        s = __fadd_rn(s, (MODE == 2 ? fabsf(v) > R : e > R) ? e : 0.f);
      }
    }
  return s;
}

__global__ __launch_bounds__(kResThreads) void resident_kernel(ResidentArgs a) {
  extern __shared__ double lds8[];
  const GAArgs& g = a.ga;
  RunState* st = a.state;
  if (st->stop) return;
  const int P = g.P, K = g.K, E = g.E, W = K | 1, S = a.S;
  const int n = P * K, n_pairs = (P - E + 1) >> 1, C = 32 * a.nct;
  char* base = reinterpret_cast<char*>(lds8);
  float* A = reinterpret_cast<float*>(base);                          // [units][S + 1][2][64]
  float* B = reinterpret_cast<float*>(base + a.b_at);                 // [nct][S + 1][64]
  double* red = reinterpret_cast<double*>(base + a.red_at);           // [4 n_tiles][C]
  double* e64 = reinterpret_cast<double*>(base + a.e64_at);           // [P]
  double* cum = e64 + P;                                              // [P] (roulette)
  uint64_t* keys = reinterpret_cast<uint64_t*>(cum + P);              // [P]
  uint64_t* words = reinterpret_cast<uint64_t*>(base + a.words_at);   // [2][n_pairs][blocks][4]
  float* pop = reinterpret_cast<float*>(base + a.pop_at);             // [2][P][W]
  float* mut = pop + 2 * P * W;                                       // [2][P][K]
  int* order = reinterpret_cast<int*>(mut + 2 * n);                       // [P]
  int* b_of = order + P;                                              // [K] a gene's place in B
  __shared__ int best_sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31, h = lane >> 5;
  const int max_gen = st->max_gen;
  const double target = st->target;
  int gen = st->gen;

  // Units past the data contribute zero sums (they are never computed).
  for (int i = tid; i < 4 * a.n_tiles * C; i += kResThreads) red[i] = 0.0;
  // Zeros stay where there is no gene (columns past P, the odd half of the
  // last pair); the bias step's other half multiplies by 1.
  for (int i = tid; i < a.nct * (S + 1) * 64; i += kResThreads)
    B[i] = (i >> 6) % (S + 1) == S && (i & 32) ? 1.f : 0.f;
  for (int i = tid; i < K; i += kResThreads) {
    const int f = max(i - 1, 0) / a.D, j = max(i - 1, 0) - f * a.D;
    b_of[i] = i ? ((f >> 1) * a.D + j) * 64 + (f & 1) * 32 : S * 64;
  }
  const int Q = (a.U + 1) >> 1;
  const int unit_ld = (S + 1) * 128;
  for (int i = wave; i < a.units * Q; i += kResWaves) {
    const int u = i / Q, q = i - u * Q;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int64_t r = (int64_t)u * 64 + rb * 32 + m;
      const bool ok = r < a.NP;
      float x = 0.f, sx = 0.f;
      if (a.basis == 3) {
        if (ok) {
          x = a.cs[2 * (r * a.N + q)];
          sx = a.cs[2 * (r * a.N + q) + 1];
        }
      } else if (ok && 2 * q + h < a.U) {
        x = a.X[r * a.N + 2 * q + h];
      }
      float* dst = A + u * unit_ld + rb * 64 + lane;
      expand(a, x, sx, h, ok, dst + q * a.D * 128, 128);
      // lane half 0: the bias's 1, half 1: minus the target
      if (q == 0) dst[S * 128] = ok ? (h ? -a.t[r] : 1.f) : 0.f;
    }
  }
  __syncthreads();
  const float* src = (gen & 1) ? g.pop_b : g.pop_a;
  for (int i = tid; i < n; i += kResThreads) {
    const int s = i / K, gi = i - s * K;
    const float x = src[i];
    pop[((gen & 1) * P + s) * W + gi] = x;
    B[(s >> 5) * (S + 1) * 64 + b_of[gi] + (s & 31)] = x;
  }

  // Draws are made a generation ahead, 64 to a wave and turn: blocks of
  // selection words first, then the mutations of the genes past the elites.
  const float inv_k = 1.f / (float)K;
  const int n_words = n_pairs * a.blocks;
  const int n_draws = n_words + n - E * K, draw_items = (n_draws + 63) >> 6;
  // Waves without errors and children first, the last one (elites) last.
  const int first_draw = wave == kResWaves - 1 ? wave : kResWaves - 2 - wave;
  auto key1 = [&](int d) { return d * 64 + lane < n_words ? 1ull : 2ull; };   // the stream
  auto counter = [&](int d, uint32_t to) -> U64x4 {
    const int i = d * 64 + lane;
    if (i < n_words) {
      const int q = a.blocks == 1 ? i : i >> 1;
      return {(uint64_t)to, (uint64_t)q, (uint64_t)(i - q * a.blocks), 0};
    }
    const int j = i - n_words + E * K, s = (int)(((float)j + 0.5f) * inv_k);
    return {(uint64_t)to, (uint64_t)s, (uint64_t)(j - s * K), 0};
  };
  auto put_draw = [&](int d, uint32_t to, const U64x4& r) {
    const int i = d * 64 + lane;
    if (i < n_words) {
      uint64_t* o = words + ((to & 1) * n_words + i) * 4;
      o[0] = r.o0;
      o[1] = r.o1;
      o[2] = r.o2;
      o[3] = r.o3;
    } else if (i < n_draws) {
      mut[(to & 1) * n + i - n_words + E * K] = (r.o0 & 0xFFFFFFFFull) < g.thr_mut
                                                   ? __fmul_rn(g.sigma, gauss12(r))
                                                   : __uint_as_float(0x7FC00000u);
    }
  };
  for (int d = first_draw; d < draw_items; d += kResWaves)
    put_draw(d, gen + 1u, philox_rounds<0, 10>(counter(d, gen + 1u), g.seed, key1(d)));
  const int w = a.n_tiles <= 16 ? 16 : 32;
  const int per = kResThreads / w, sub = tid / w, l = tid & (w - 1);
  // Lanes per pair of the selection and the genes.
  const int lp = n_pairs < kResWaves ? 64 : 32;
  __syncthreads();

  int built = 0;
  bool stopped = false;
  for (;;) {
    const float* cur = pop + (gen & 1) * P * W;
    float* next = pop + ((gen + 1) & 1) * P * W;
    for (int i = wave; i < a.units * a.nct; i += kResWaves) {
      const int u = a.nct == 1 ? i : i >> 1, ct = a.nct == 1 ? 0 : i & 1;
      const float* av = A + u * unit_ld + lane;
      const float* bv = B + ct * (S + 1) * 64 + lane;
      f32x16 acc[2];
      float a0 = av[0], a1 = av[64], b = bv[0];
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b, f32x16{}, 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b, f32x16{}, 0, 0, 0);
      a0 = av[128], a1 = av[192], b = bv[64];
      for (int s = 1; s <= S; ++s) {
        av += 128;
        bv += 64;
        // (the last step's reads ahead are not used)
        const float n0 = av[128], n1 = av[192], nb = bv[64];
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b, acc[1], 0, 0, 0);
        a0 = n0, a1 = n1, b = nb;
      }
      // A wave at its error terms goes first, so that the waves of a SIMD drift
      // apart (3 %).
      __builtin_amdgcn_s_setprio(1);
      const float s = a.error_fn == 2   ? unit_error<2>(acc, a.R)
                      : a.error_fn == 3 ? unit_error<3>(acc, a.R)
                                        : unit_error<0>(acc, a.R);
      __builtin_amdgcn_s_setprio(0);
      double v = (double)s;
      v += __shfl_xor(v, 32);
      if (h == 0) red[u * C + ct * 32 + m] = v;
    }
    __syncthreads();

    // The first half of this wave's draws for the generation after the next.
    U64x4 half{};
    if (first_draw < draw_items)
      half = philox_rounds<0, 5>(counter(first_draw, gen + 2u), g.seed, key1(first_draw));

    // Errors: a tile's four units in order, then wave_split_sum over the tiles
    // (its lanes past them would only add zeros).
    for (int i0 = 0; i0 < P; i0 += per) {
      if (i0 + wave * 64 / w >= P) break;
      const int i = i0 + sub;
      const bool ok = i < P;
      double s = 0.0;
      if (ok && l < a.n_tiles) {
        const double* p = red + 4 * l * C + i;
        s = 0.0 + (((p[0] + p[C]) + p[2 * C]) + p[3 * C]);
      }
      if (w == 32) s += __shfl_xor(s, 16);
      s = row_add<1>(row_add<2>(row_add<4>(row_add<8>(s))));
      if (l == 0 && ok) {
        const double e = error_from_sum(s, a.NP, a.error_fn);
        e64[i] = e;
        keys[i] = rank_key((float)e, i);
        if (g.selection == 2) cum[i] = 1.0 / ((double)rank_key_value((float)e) + 1e-12);
      }
    }
    __syncthreads();

    if (a.need_order) {
      for (int i = tid; i < P; i += kResThreads) {
        const uint64_t ke = keys[i];
        int r = 0;
        for (int j = 0; j < P; ++j) r += keys[j] < ke ? 1 : 0;
        order[r] = i;
      }
      __syncthreads();
    }
    if (g.selection == 2) {
      if (tid == 0) {                      // left to right, as roulette_cum_body
        double s = 0.0;
        for (int i = 0; i < P; ++i) {
          s += cum[i];
          cum[i] = s;
        }
      }
      __syncthreads();
    }
    // The last wave: best chromosome, stop test, elites.
    if (wave == kResWaves - 1) {
      uint64_t best = min8(lane < P ? keys[lane] : ~0ull);
      best = rows_min(min(best, row_move<kRowMirror>(best)));
      const int b = (int)(uint32_t)best;
      if (lane == 0) best_sh = e64[b] <= target || gen >= max_gen ? ~b : b;
      for (int e = lane; e < E * K; e += 64) {
        const int s = (int)(((float)e + 0.5f) * inv_k), gi = e - s * K;
        const int at_b = (s >> 5) * (S + 1) * 64 + b_of[gi] + (s & 31);
        const float x = cur[(g.elite_mode == 0 ? b : order[s]) * W + gi];
        next[s * W + gi] = x;
        B[at_b] = x;
      }
    }
    // Pairs of children, lp lanes each.  (A run that has stopped does not read
    // what is built here.)
    const int q = tid / lp;
    if (q < n_pairs) {
      const uint32_t* wq = reinterpret_cast<const uint32_t*>(
          words + (((gen + 1) & 1) * n_pairs + q) * a.blocks * 4);
      const int k = g.selection == 0 ? g.k : 1;
      const uint32_t coin = wq[2 * k], at = wq[2 * k + 1];
      int p1, p2;
      if (g.selection == 0) {
        // Lowest (fitness, index) of the draws: the smallest key; of each 16
        // lanes the first 8 hold one parent's draws, the others the other's.
        const uint32_t u = wq[(lane & 8 ? k : 0) + min(lane & 7, k - 1)];
        const uint64_t key = min8(keys[(int)(((uint64_t)u * (uint64_t)P) >> 32)]);
        const int mine = (int)(uint32_t)key, other = (int)(uint32_t)row_move<kRowMirror>(key);
        p1 = lane & 8 ? other : mine;
        p2 = lane & 8 ? mine : other;
      } else {
        p1 = g.selection == 1 ? ranking_pick(order, P, wq[0]) : roulette_pick(cum, P, wq[0]);
        p2 = g.selection == 1 ? ranking_pick(order, P, wq[1]) : roulette_pick(cum, P, wq[1]);
      }
      const int cut = (uint64_t)coin < g.thr_cross
                          ? 1 + (int)(((uint64_t)at * (uint64_t)(K - 1)) >> 32) : K;
      const int sa = E + 2 * q;
      const int genes = sa + 1 < P ? 2 * K : K;
      for (int e = tid & (lp - 1); e < genes; e += lp) {
        const bool second = e >= K;
        const int gi = second ? e - K : e, s = sa + second;
        const float mu = mut[((gen + 1) & 1) * n + s * K + gi];
        const int at_b = (s >> 5) * (S + 1) * 64 + b_of[gi] + (s & 31);
        const bool swapped = gi >= cut;
        float x = cur[(second != swapped ? p2 : p1) * W + gi];
        if (!isnan(mu)) x = clamp_unit(__fadd_rn(x, mu));
        next[s * W + gi] = x;
        B[at_b] = x;
      }
    }
    if (first_draw < draw_items)
      put_draw(first_draw, gen + 2u, philox_rounds<5, 10>(half, g.seed, key1(first_draw)));
    for (int d = first_draw + kResWaves; d < draw_items; d += kResWaves)
      put_draw(d, gen + 2u, philox_rounds<0, 10>(counter(d, gen + 2u), g.seed, key1(d)));
    __syncthreads();
    stopped = best_sh < 0;
    if (stopped) break;
    ++gen;
    if (++built == a.generations) break;
  }

  // The last evaluation's errors, the current population (unless it is the
  // one read above) and the state.
  for (int i = tid; i < P; i += kResThreads) {
    a.fit64[i] = e64[i];
    a.fit32[i] = (float)e64[i];
  }
  if (built) {
    float* out = pick((gen & 1) != 0, g.out_b, g.out_a);
    for (int i = tid; i < n; i += kResThreads) {
      const int s = i / K;
      out[i] = pop[((gen & 1) * P + s) * W + (i - s * K)];
    }
  }
  if (tid == 0) {
    const int b = stopped ? ~best_sh : best_sh;
    st->best = b;
    st->best_err = e64[b];
    st->evaluated = stopped ? gen : gen - 1;
    st->gen = gen;
    if (stopped) st->stop = 1;
  }
}

// LDS layout; the size in bytes.
static size_t resident_layout(ResidentArgs& a) {
  const GAArgs& g = a.ga;
  const size_t n_pairs = (size_t)(g.P - g.E + 1) / 2, W = g.K | 1;
  size_t off = (size_t)a.units * (a.S + 1) * 128 * sizeof(float);
  a.b_at = (int)off;
  off += (size_t)a.nct * (a.S + 1) * 64 * sizeof(float) + 512;   // reads ahead
  a.red_at = (int)off;
  off += (size_t)a.n_tiles * 4 * 32 * a.nct * sizeof(double);
  a.e64_at = (int)off;
  off += (size_t)g.P * 24;
  a.words_at = (int)off;
  off += 2 * n_pairs * a.blocks * 32;
  a.pop_at = (int)off;
  return off + 2 * ((size_t)g.P * W + (size_t)g.P * g.K) * sizeof(float) +
         ((size_t)g.P + g.K) * sizeof(int);
}

constexpr size_t kResLds = 159 * 1024;

static bool resident_args(const FitArgs& f, const GAArgs& g, ResidentArgs& a) {
  const int64_t units = (f.NP + 63) / 64, S = (int64_t)f.Q * f.degree;
  const int blocks = compact_blocks(g.k, g.selection);
  if (!compact_fits(g) || g.P > kResPopulation ||
      f.tiles_per_split != 1 || f.n_tiles > 32 || (f.basis == 3 && !f.cs))
    return false;
  const int nct = (g.P + 31) / 32;
  // Estimated cycles of a generation here and in two launches, fitted to 1,000 shapes
  // (within 0.4 us as a rule).  Here: the units of a SIMD (their products; 32 rows'
  // error terms of one or four instructions), draws and children (which wait for one
  // another once children take most of the waves), the serial parts of an order and
  // of a roulette wheel.  Two launches: what they take whatever they compute, one
  // unit's products, the genes of the tail.  This kernel runs where it is ahead by
  // 0.4 us at least; of 500 other shapes that it takes so one was slower, by 1.5 %.
  // 2,100 x 8, degree 1, 23 chromosomes 5.2 us and 8.2; 1,000 x 5, degree 3, 50
  // chromosomes 8.4 and 9.6; 2,000 x 8, degree 1, 64 chromosomes would take 9.1 for
  // 8.5, 1,024 x 16 with 64 (thresholded) 10.6 for 9.3.
  const int64_t PK = (int64_t)g.P * g.K;
  const bool thresholded = f.error_fn >= 2, ordered = reads_order(g), wheel = g.selection == 2;
  const int64_t here = 4000 + (units + 3) / 4 * nct * (105 * (S + 1) + (thresholded ? 570 : 300)) +
                       6 * PK + 40 * std::max(0, g.P - 24 * nct) +
                       g.P * ((ordered ? 145 : 0) + (wheel ? 110 : 0));
  const int64_t launches = 18600 + 200 * S + 9 * PK / 4 + (thresholded ? 800 : 0) +
                           (f.basis == 3 ? 1500 : 0) - (narrow_rows(f) ? 700 : 0) +
                           g.P * ((ordered ? 77 : 0) + (wheel ? 72 : 0));
  if (here + 1000 > launches) return false;
  a.X = f.X;
  a.t = f.t;
  a.cs = f.cs;
  a.NP = f.NP;
  a.N = f.N;
  a.D = f.degree;
  a.basis = f.basis;
  a.U = f.U;
  a.S = (int)S;
  a.units = (int)units;
  a.nct = nct;
  a.n_tiles = f.n_tiles;
  a.error_fn = f.error_fn;
  a.R = f.R;
  a.blocks = blocks;
  a.need_order = reads_order(g);
  a.ga = g;
  return resident_layout(a) <= kResLds;
}

bool resident_fits(const FitArgs& f, const GAArgs& g) {
  ResidentArgs a{};
  return resident_args(f, g, a);
}

hipError_t launch_resident(const FitArgs& f, const GAArgs& g, const RankArgs& r, int generations,
                           hipStream_t s) {
  ResidentArgs a{};
  if (!resident_args(f, g, a)) return hipErrorInvalidValue;
  a.fit32 = r.fit32;
  a.fit64 = r.fit64;
  a.state = r.state;
  a.generations = generations;
  const size_t lds = resident_layout(a);
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)resident_kernel,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(resident_kernel, dim3(1), dim3(kResThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace game
