// The float32 fitness of one chromosome tile over one pattern split: the
// body shared by the single-run kernel (fitness_f32.hip) and the batched
// persistent kernel (batch.hip).  See fitness_f32.hip for the design.
#pragma once

#include <utility>

#include "basis.h"
#include "common.h"

namespace game {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// s plus the squared residual v (MSE, RMSE: one fused multiply-add) or its
// thresholded form (TMSE, Eq. 10: mode 2 keeps it when |v| > R, mode 3 when
// v^2 > R; square and sum rounded separately).  Every rounding is spelled
// out, so each instance of the body (single-run and batched) sums the same
// bits whatever the compiler would contract.
template <int MODE>
__device__ __forceinline__ float add_error_term(float s, float v, float R) {
  if constexpr (MODE == 2 || MODE == 3) {
    const float e = __fmul_rn(v, v);
    const bool keep = MODE == 2 ? fabsf(v) > R : e > R;
    return __fadd_rn(s, keep ? e : 0.f);
  }
  return __builtin_fmaf(v, v, s);
}

// A recurrence chain that yields zero at every degree: for rows past the
// data, so that their accumulators end at exactly zero.
template <class R>
__device__ __forceinline__ void zero_chain(R& r, bool keep) {
  r.cur = keep ? r.cur : 0.f;
  if constexpr (requires { r.prev; }) r.prev = keep ? r.prev : 0.f;
}

// Wave-uniform copies (readfirstlane) of launch parameters.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ T* uniform(T* p) {
  return reinterpret_cast<T*>(uniform((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// A pointer to global memory as such: its loads are global_load rather than
// flat_load, whose completion an LDS wait would also have to cover.
typedef const float __attribute__((address_space(1)))* gptr_f32;
__device__ __forceinline__ gptr_f32 global_f32(const float* p) { return (gptr_f32)p; }

// Waves per workgroup of the body with CB 32-column blocks per wave: four
// for 32- and 64-chromosome tiles, eight for 128-chromosome tiles (waves 0-3
// take the even row tiles of the split and 4-7 the odd ones, two per SIMD).
__host__ __device__ constexpr int fit_waves(int cb) { return cb == 4 ? 8 : 4; }

// lo = (a's lower half, b's lower half), hi = (a's upper, b's upper).
__device__ __forceinline__ void swap_halves(float a, float b, float& lo, float& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  lo = __uint_as_float(r[0]);
  hi = __uint_as_float(r[1]);
}

// Feature pairs whose loads are issued together, a group ahead of their use.
// A pair of degree d is 2 d CB MFMAs of work; at low degree that is far less
// than a load's latency.  Eight waves of wide tiles cover it with one pair at a
// time (groups of 4 cost them 3-7 % where the last is not whole: 361,685 x 5,
// Legendre 2, 920 chromosomes 117 us for 110); only whole quads pay (kQuadRows),
// and two pairs of the trigonometric expansion at degree 4, whose (cos x, sin x)
// are twice the bytes (six shapes 0.6 to 2.4 % faster, 200,000 x 20 with 2,048
// chromosomes 996 us for 1,020; the polynomial bases on the same shapes from 1.8 %
// slower to 1.1 % faster, and at degrees 1 to 3 two pairs cost up to 2.8 %).
__host__ __device__ constexpr int pairs_ahead(int d, int cb, bool trig = false) {
  return cb == 4 ? (trig && d == 4 ? 2 : 1) : (d == 1 ? 8 : d <= 4 ? 4 : d <= 8 ? 2 : 1);
}

// Tile range [split's tiles] x chromosome tile ctile (32*CB chromosomes,
// the first one ctile * 32*CB) of the launch described by a_in; writes
// a.partial[split * ld_partial + chromosome].  Each wave takes RB/2 consecutive 256-row tiles at a time
// (its 64-row slice of each: RB 32-row blocks).  genes: the chromosomes
// being scored; lds: the workgroup's dynamic LDS; stop: when set and nonzero
// nothing is computed.  D is the degree.  BASIS
// is the expansion family, QP the feature pairs loaded at a time (kTrigTable: the trigonometric one seeded from
// the stored (cos x, sin x) table a_in.cs instead of sincosf in every tile).
template <int BASIS, int D, int CB = 2, int RB = 2,
          int QP = RB == 2 ? pairs_ahead(D, CB, BASIS >= 3) : 1>
__device__ __forceinline__ void fitness_f32_block(const FitArgs& a_in, const float* __restrict__ genes,
                                                  int split, int ctile, float* lds,
                                                  const int32_t* stop = nullptr) {
  // Read here, tested once the first copies are on their way.
  const int32_t stopped = stop ? *stop : 0;
  // The parameters the body uses, read once into scalar registers (so that
  // no store in the loops can be taken to alias them and force reloads).
  FitArgs a;
  a.X = uniform(a_in.X);
  a.t = uniform(a_in.t);
  a.partial = uniform(a_in.partial);
  a.NP = uniform(a_in.NP);
  a.N = uniform(a_in.N);
  a.K = uniform(a_in.K);
  a.n_chrom = uniform(a_in.n_chrom);
  a.U = uniform(a_in.U);
  a.Q = uniform(a_in.Q);
  a.pairs_per_chunk = uniform(a_in.pairs_per_chunk);
  a.n_chunks = uniform(a_in.n_chunks);
  a.ld_partial = uniform(a_in.ld_partial);
  a.tiles_per_split = uniform(a_in.tiles_per_split);
  a.n_tiles = uniform(a_in.n_tiles);
  a.error_fn = uniform(a_in.error_fn);
  a.R = uniform(a_in.R);
  constexpr bool kTable = BASIS == kTrigTable;
  constexpr int FAM = kTable ? 3 : BASIS;   // expansion family
  static_assert(FAM >= 0 && FAM <= 3, "compile-time expansion family");
  a.cs = kTable ? uniform(a_in.cs) : nullptr;
  static_assert(D >= 1 && D <= kMaxDegree, "compile-time degree");
  constexpr int Dv = D;
  constexpr bool trig = FAM == 3;
  genes = uniform(genes);
  split = uniform(split);
  ctile = uniform(ctile);
  lds = uniform(lds);
  static_assert(CB == 1 || CB == 2 || CB == 4, "32-, 64- or 128-chromosome tiles");
  constexpr int NW = fit_waves(CB);   // waves per workgroup
  constexpr int TS = NW / 4;          // tile streams (wave groups)
  static_assert(RB == 2 || RB == 4, "one or two 256-row tiles per wave");
  constexpr int TPW = RB / 2;         // consecutive row tiles per wave
  constexpr int STEP = TS * TPW;      // row tiles per step of the workgroup
  constexpr int kCols = 32 * CB;      // chromosomes per tile
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wq = wave & 3;            // 64-row slice of a tile
  const int wg = TS == 1 ? 0 : wave >> 2;  // tile stream
  const int m = lane & 31;
  const int h = lane >> 5;
  const int c0 = ctile * kCols;

  const int ppc = a.pairs_per_chunk;
  const int SC = ppc * Dv;         // K-steps per chunk
  const int WS = 2 * SC + 1;       // LDS row stride in floats (odd)
  const int BUF = kCols * WS;      // floats per gene buffer
  const int nk = (2 * SC + 63) >> 6;  // 64-gene pieces of a row
  const int K = a.K;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);

  float w0[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int n = c0 + cb * 32 + m;
    w0[cb] = n < a.n_chrom ? global_f32(genes)[(int64_t)n * K] : 0.f;
  }

  // Issue the copy of the chunk's genes (sub-features [u0, u0 + 2 ppc)) into
  // buffer buf: row c = genes 1 + u0*D ... of chromosome c0 + c, canonical
  // order.  Rows past the population repeat the last chromosome (their sums
  // are never read).  Gene slots of a sub-feature past U (the odd half of the
  // last pair) are zeroed: that lane's expansion of x = 0 is not zero.  The
  // copy has landed once this wave's vmcnt reaches zero.
  auto stage_issue = [&](int chunk, int buf) {
    const int u0 = chunk * ppc * 2;
    const int rem = a.U - u0;
    const int valid = min(2 * SC, rem * Dv);
    float* dst0 = lds + buf * BUF;
    const float* src0 = genes + 1 + u0 * Dv + lane;
    for (int i = wave_u; i < kCols * nk; i += NW) {
      const int c = i / nk;
      const int k = i - c * nk;
      const int n = min(c0 + c, a.n_chrom - 1);
      if (k * 64 + lane < valid)
        __builtin_amdgcn_global_load_lds(
            (const void*)(src0 + (int64_t)n * K + k * 64),
            (__attribute__((address_space(3))) void*)(dst0 + c * WS + k * 64), 4, 0, 0);
    }
    if ((rem & 1) && rem < 2 * ppc) {
      for (int idx = threadIdx.x; idx < kCols * Dv; idx += 64 * NW) {
        const int c = idx / Dv;
        dst0[c * WS + rem * Dv + (idx - c * Dv)] = 0.f;
      }
    }
  };

  double acc64[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc64[cb] = 0.0;
  const int64_t NP = a.NP;
  const int N = a.N;
  const int tile_begin = split * a.tiles_per_split;
  const int tile_end = min(tile_begin + a.tiles_per_split, a.n_tiles);

  // x of sub-feature pair q for this lane's two rows (0 outside the data);
  // from the stored trig table, cos x into xo and sin x into so instead.
  // Row of block rb of the wave whose first tile is `tile`: blocks 2i and
  // 2i+1 are the wave's 64-row slice of tile + i.
  auto row_of = [&](int tile, int rb) -> int64_t {
    return (int64_t)(tile + rb / 2) * kTileRows + wq * 64 + (rb & 1) * 32 + m;
  };
  // Rows of whole 16-byte quads are read a quad per lane and load (low degrees,
  // whose feature reads would otherwise outnumber the MFMAs): a load of single
  // features moves 8 bytes of each row's 64-byte line.
  constexpr bool kQuads = !trig && QP >= 4;
  const bool quads = kQuads && N % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0 &&
                     (a.n_chunks == 1 || ppc % 4 == 0);
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef const f32x4 __attribute__((address_space(1)))* gptr_f32x4;
  // Features of pairs q0 .. q0 + n - 1 (n <= QP) of the wave's rows.
  auto load_x = [&](int tile, int q0, int n, float (&xo)[QP][RB], float (&so)[QP][RB]) {
    if constexpr (kTable) {
      typedef float f32x2 __attribute__((ext_vector_type(2)));
      typedef const f32x2 __attribute__((address_space(1)))* gptr_f32x2;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int64_t r = row_of(tile, rb);
        gptr_f32x2 src = (gptr_f32x2)a.cs + r * N + q0;
#pragma unroll
        for (int i = 0; i < QP; ++i) {
          f32x2 v = {0.f, 0.f};
          if (r < NP && (i == 0 || i < n)) v = src[i];
          xo[i][rb] = v.x;
          so[i][rb] = v.y;
        }
      }
      return;
    }
    if constexpr (kQuads) {
      if (quads) {
        // Half h reads the quad 2 q0 + 8 k + 4 h .. + 3 of its row; the halves'
        // words are exchanged (swap_halves) where a tile's values are next used.
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const int64_t r = row_of(tile, rb);
          const int f = 2 * q0 + 4 * h;
          gptr_f32x4 src = (gptr_f32x4)(global_f32(a.X) + r * N + f);
#pragma unroll
          for (int k = 0; k < QP / 4; ++k) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (r < NP && 4 * k < n && f + 8 * k < N) v = src[2 * k];
            xo[4 * k][rb] = v.x;
            xo[4 * k + 1][rb] = v.y;
            xo[4 * k + 2][rb] = v.z;
            xo[4 * k + 3][rb] = v.w;
          }
        }
        return;
      }
    }
    const int f0 = trig ? q0 : 2 * q0 + h;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int64_t r = row_of(tile, rb);
      gptr_f32 src = global_f32(a.X) + r * N + f0;
#pragma unroll
      for (int i = 0; i < QP; ++i) {
        const int off = trig ? i : 2 * i;
        // the odd half of the last pair may lie past the sub-features
        const bool in = (i == 0 || i < n) && (trig || f0 + off < a.U);
        xo[i][rb] = (r < NP && in) ? src[off] : 0.f;
      }
    }
  };

  float xn[QP][RB], sn[QP][RB];
#pragma unroll
  for (int i = 0; i < QP; ++i)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) xn[i][rb] = sn[i][rb] = 0.f;
  // The targets of the wave's rows (0 past the data), negated at their use so
  // that nothing waits for them here; at low degree they are read a tile ahead
  // too.
  constexpr bool kTargetsAhead = QP >= 4;
  float tn[RB];
  auto load_t = [&](int tile, float (&to)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int64_t r = row_of(tile, rb);
      to[rb] = (RB == 2 || tile + rb / 2 < tile_end) && r < NP ? global_f32(a.t)[r] : 0.f;
    }
  };
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) tn[rb] = 0.f;
  if (kTargetsAhead && tile_begin + wg * TPW < tile_end) load_t(tile_begin + wg * TPW, tn);
  const int first_n = min(QP, min(ppc, a.Q));   // pairs of a tile's first group
  if (tile_begin + wg * TPW < tile_end) load_x(tile_begin + wg * TPW, 0, first_n, xn, sn);
  if (a.n_chunks == 1) {
    stage_issue(0, 0);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's copies landed
    __syncthreads();
  }
  if (stopped) return;

  // Chunked genes: stage index st runs over (tile, chunk) in loop order and
  // uses buffer st & 1.
  int st = 0;
  if (a.n_chunks > 1 && tile_begin < tile_end) stage_issue(0, 0);

  // Every wave takes the same number of steps of STEP tiles.  A wave whose
  // stream has no tile left in the last step leaves at once when the genes
  // are staged once, and otherwise still joins the staging barriers of each
  // chunk but computes nothing.
  const int n_steps = (tile_end - tile_begin + STEP - 1) / STEP;
  for (int step = 0; step < n_steps; ++step) {
    const int tile = tile_begin + step * STEP + wg * TPW;   // the wave's first tile
    const bool active = TS == 1 || tile < tile_end;   // one stream: every step has its tile
    if (!active && a.n_chunks == 1) break;
    // Rows past the data take a zero A operand in every K-step (bias step
    // included), so their residuals are exactly zero and the epilogue needs
    // no row mask.
    bool row_ok[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      row_ok[rb] = (RB == 2 || tile + rb / 2 < tile_end) && row_of(tile, rb) < NP;
    // The targets join with the bias in a last K-step, so their load's latency
    // hides behind the K loop.
    float nt[RB];
    if constexpr (kTargetsAhead) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) nt[rb] = tn[rb];
      if (tile + STEP < tile_end) load_t(tile + STEP, tn);
    } else {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) nt[rb] = 0.f;
      if (active) load_t(tile, nt);
    }
    // Accumulators start at zero (an inline constant, nothing to keep live
    // across tiles).
    f32x16 acc[RB][CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x16{};

    for (int chunk = 0; chunk < a.n_chunks; ++chunk) {
      const float* wbuf = lds;
      if (a.n_chunks > 1) {
        // Every wave's copy of this chunk has landed and every wave is done
        // with the other buffer: start the copy of the next stage into it.
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
        if (chunk + 1 < a.n_chunks) stage_issue(chunk + 1, (st + 1) & 1);
        else if (step + 1 < n_steps) stage_issue(0, (st + 1) & 1);
        wbuf = lds + (st & 1) * BUF;
        ++st;
      }
      if (!active) continue;
      const int q_begin = chunk * ppc;
      const int q_end = min(q_begin + ppc, a.Q);
      for (int q0 = q_begin; q0 < q_end; q0 += QP) {
        float x[QP][RB], sx[QP][RB];
#pragma unroll
        for (int i = 0; i < QP; ++i)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            x[i][rb] = xn[i][rb];
            sx[i][rb] = sn[i][rb];
          }
        if constexpr (kQuads) {
          if (quads) {
            // Words 0..3 of a quad pair are features 0..3 in half 0 and 4..7
            // in half 1; pair i wants features 2 i + h.
#pragma unroll
            for (int k = 0; k < QP; k += 4)
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) {
                swap_halves(xn[k][rb], xn[k + 1][rb], x[k][rb], x[k + 2][rb]);
                swap_halves(xn[k + 2][rb], xn[k + 3][rb], x[k + 1][rb], x[k + 3][rb]);
              }
          }
        }
        // prefetch the next group, or the first one of the next tile
        const int nq = min(q0 + QP, q_end);
        if (nq < a.Q) load_x(tile, nq, min(QP, (nq < q_end ? q_end : min(nq + ppc, a.Q)) - nq), xn, sn);
        else if (tile + STEP < tile_end) load_x(tile + STEP, 0, first_n, xn, sn);
#pragma unroll
        for (int i = 0; i < QP; ++i) {
          if (i > 0 && q0 + i >= q_end) break;
          Recur<FAM> rc[RB];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            if constexpr (kTable) {
              rc[rb].seed_cs(x[i][rb], sx[i][rb], h);
            } else {
              rc[rb].seed(x[i][rb], h);
            }
            zero_chain(rc[rb], row_ok[rb]);
          }
          const float* wl = wbuf + m * WS + (2 * (q0 + i - q_begin) + h) * Dv;
          // One K-step per degree: CB MFMA columns x RB row blocks, then the
          // recurrence moves every lane's A value to the next degree.
          auto kstep = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            float b[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) b[cb] = wl[cb * 32 * WS + j];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
              for (int cb = 0; cb < CB; ++cb)
                acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(rc[rb].cur, b[cb], acc[rb][cb], 0, 0, 0);
            if constexpr (j + 1 < D) {
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) {
                rc[rb].template advance<j + 1>(x[i][rb]);
              }
            }
          };
          [&]<int... J>(std::integer_sequence<int, J...>) {
            (kstep(std::integral_constant<int, J>{}), ...);
          }(std::make_integer_sequence<int, D>{});
        }
      }
    }

    if (!active) continue;
    // Bias and target K-step: lane half 0 multiplies 1 by a0 of its column,
    // half 1 multiplies -t of its row by 1, so the accumulators end at
    // Out - t (0 for rows past the data).
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float ab = h ? -nt[rb] : (row_ok[rb] ? 1.f : 0.f);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(ab, h ? 1.f : w0[cb], acc[rb][cb], 0, 0, 0);
    }

    // Epilogue: residual Out - t, squared (or thresholded), summed over the
    // lane's 32 rows (register order; accumulator register i of row block rb
    // holds row rb*32 + 8*(i/4) + 4*h + i%4 of the wave's 64 rows).  Rows
    // past the data add exactly zero.
    // One float32 sum per row tile (its two row blocks), added to the
    // float64 running sum tile by tile, so that a tile's sum does not
    // depend on how many tiles a wave takes at once.
    float s[TPW][CB];
#pragma unroll
    for (int tp = 0; tp < TPW; ++tp)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) s[tp][cb] = 0.f;
    auto epilogue = [&](auto mode_c) {
      constexpr int mode = decltype(mode_c)::value;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            s[rb / 2][cb] = add_error_term<mode>(s[rb / 2][cb], acc[rb][cb][i], a.R);
    };
    if (a.error_fn == 2) epilogue(std::integral_constant<int, 2>{});
    else if (a.error_fn == 3) epilogue(std::integral_constant<int, 3>{});
    else epilogue(std::integral_constant<int, 0>{});
#pragma unroll
    for (int tp = 0; tp < TPW; ++tp)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc64[cb] += (double)s[tp][cb];
  }

  // Combine the two lane halves (same chromosome, different rows), then the
  // waves, in a fixed order.
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc64[cb] += __shfl_xor(acc64[cb], 32);
  __syncthreads();
  double* red = reinterpret_cast<double*>(lds);
  if (h == 0) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) red[wave * kCols + cb * 32 + m] = acc64[cb];
  }
  __syncthreads();
  if (threadIdx.x < kCols) {
    const int c = threadIdx.x;
    double v = red[c];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w * kCols + c];
    a.partial[(int64_t)split * a.ld_partial + c0 + c] = v;
  }
}


// Whether rows of Q feature pairs at degree D are narrow: one group of pairs.
__host__ __device__ constexpr bool narrow_degree(int d) { return d <= 4; }

// The same tile for narrow rows (Q <= pairs_ahead(D, CB), degree <= 4, no sine and
// cosine): all features of a row are one group, read a tile ahead, and a lane's
// genes stay in registers, so the loop over tiles touches neither LDS nor
// launch parameters.  float32 products run at the vector rate, so every vector
// instruction beside them counts: the general loop issued 385 a tile of 64 rows
// (60 to keep its bounds and addresses in vector lanes, 63 to clear and move
// accumulators) besides 18 products, this one 191.  7,168,000 x 16,
// degree 1, 23 chromosomes (TMSE), a whole generation: 178 us before, 136 now (the
// data read at 3.8 TB/s).
// QUADS: rows are whole aligned 16-byte quads, read one per lane and load.
template <int BASIS, int D, int CB, bool QUADS>
__device__ __forceinline__ void fitness_f32_narrow(const FitArgs& a_in,
                                                   const float* __restrict__ genes, int split,
                                                   int ctile, float* lds, const int32_t* stop) {
  static_assert(BASIS >= 0 && BASIS <= 2 && narrow_degree(D) && CB <= 2, "narrow rows");
  const int32_t stopped = stop ? *stop : 0;
  constexpr int QP = pairs_ahead(D, CB);
  constexpr int RB = 2;
  constexpr int kCols = 32 * CB;
  const gptr_f32 X = global_f32(uniform(a_in.X)), t = global_f32(uniform(a_in.t));
  const gptr_f32 G = global_f32(uniform(genes));
  const int64_t NP = uniform(a_in.NP);
  const int N = uniform(a_in.N), K = uniform(a_in.K), Q = uniform(a_in.Q);
  const int n_chrom = uniform(a_in.n_chrom), error_fn = uniform(a_in.error_fn);
  const float R = uniform(a_in.R);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 31, h = lane >> 5;
  const int c0 = ctile * kCols;
  const int tile_begin = split * uniform(a_in.tiles_per_split);
  const int tile_end = min(tile_begin + uniform(a_in.tiles_per_split), uniform(a_in.n_tiles));

  // The features of the lane's rows of a tile (0 outside the data) and their
  // targets.
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef const f32x4 __attribute__((address_space(1)))* gptr_f32x4;
  float xn[QP][RB], tn[RB];
  auto load = [&](int tile) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int64_t r = (int64_t)tile * kTileRows + wave * 64 + rb * 32 + m;
      const bool ok = r < NP;
      if constexpr (QUADS) {
        // Half h reads quads 2 k + h; the halves' words are exchanged at their use.
        const gptr_f32x4 src = (gptr_f32x4)(X + r * N) + h;
#pragma unroll
        for (int k = 0; k < QP / 4; ++k) {
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
          if (ok && 8 * k + 4 * h < N) v = src[2 * k];
          xn[4 * k][rb] = v.x;
          xn[4 * k + 1][rb] = v.y;
          xn[4 * k + 2][rb] = v.z;
          xn[4 * k + 3][rb] = v.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < QP; ++i) xn[i][rb] = ok && 2 * i + h < N ? X[r * N + 2 * i + h] : 0.f;
      }
      tn[rb] = ok ? t[r] : 0.f;           // (negated at its use: no wait here)
    }
  };
  if (tile_begin < tile_end) load(tile_begin);
  // Genes of this lane's columns: pair i, degree j; zero past the features.
  float b[QP * D][CB], w0[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const gptr_f32 g = G + (int64_t)min(c0 + cb * 32 + m, n_chrom - 1) * K;
    w0[cb] = g[0];
#pragma unroll
    for (int i = 0; i < QP; ++i)
#pragma unroll
      for (int j = 0; j < D; ++j)
        b[i * D + j][cb] = 2 * i + h < N ? g[1 + (2 * i + h) * D + j] : 0.f;
  }
  if (stopped) return;

  double acc64[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc64[cb] = 0.0;
  // One loop per error function: its branch inside the loop took 6 %.
  auto tiles = [&](auto mode_c) {
    constexpr int mode = decltype(mode_c)::value;
    for (int tile = tile_begin; tile < tile_end; ++tile) {
      float x[QP][RB], nt[RB];
      bool row_ok[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        row_ok[rb] = (int64_t)tile * kTileRows + wave * 64 + rb * 32 + m < NP;
        nt[rb] = tn[rb];
        if constexpr (QUADS) {
#pragma unroll
          for (int k = 0; k < QP; k += 4) {
            swap_halves(xn[k][rb], xn[k + 1][rb], x[k][rb], x[k + 2][rb]);
            swap_halves(xn[k + 2][rb], xn[k + 3][rb], x[k + 1][rb], x[k + 3][rb]);
          }
        } else {
#pragma unroll
          for (int i = 0; i < QP; ++i) x[i][rb] = xn[i][rb];
        }
      }
      if (tile + 1 < tile_end) load(tile + 1);
      f32x16 acc[RB][CB];
      auto pair = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        Recur<BASIS> rc[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          rc[rb].seed(x[i][rb], h);
          // (a power of a zero is zero by itself)
          if constexpr (D > 1 && BASIS != 2) zero_chain(rc[rb], row_ok[rb]);
        }
        auto kstep = [&](auto jc) {
          constexpr int j = decltype(jc)::value;
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
              if constexpr (i == 0 && j == 0)
                acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(rc[rb].cur, b[0][cb], f32x16{}, 0, 0, 0);
              else
                acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(rc[rb].cur, b[i * D + j][cb],
                                                                   acc[rb][cb], 0, 0, 0);
            }
          if constexpr (j + 1 < D) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) rc[rb].template advance<j + 1>(x[i][rb]);
          }
        };
        [&]<int... J>(std::integer_sequence<int, J...>) {
          (kstep(std::integral_constant<int, J>{}), ...);
        }(std::make_integer_sequence<int, D>{});
      };
      pair(std::integral_constant<int, 0>{});
      [&]<int... I>(std::integer_sequence<int, I...>) {
        ((I + 1 < Q && (pair(std::integral_constant<int, I + 1>{}), true)) && ...);
      }(std::make_integer_sequence<int, QP - 1>{});
      // Bias and target step, error terms: as in fitness_f32_block.
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float ab = h ? -nt[rb] : (row_ok[rb] ? 1.f : 0.f);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(ab, h ? 1.f : w0[cb], acc[rb][cb], 0, 0, 0);
      }
      float s[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) s[cb] = 0.f;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) s[cb] = add_error_term<mode>(s[cb], acc[rb][cb][i], R);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc64[cb] += (double)s[cb];
    }
  };
  if (error_fn == 2) tiles(std::integral_constant<int, 2>{});
  else if (error_fn == 3) tiles(std::integral_constant<int, 3>{});
  else tiles(std::integral_constant<int, 0>{});

  // Lane halves, then the waves, in the order of fitness_f32_block.
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc64[cb] += __shfl_xor(acc64[cb], 32);
  double* red = reinterpret_cast<double*>(lds);
  if (h == 0) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) red[wave * kCols + cb * 32 + m] = acc64[cb];
  }
  __syncthreads();
  if (threadIdx.x < kCols) {
    const int c = threadIdx.x;
    double v = red[c];
#pragma unroll
    for (int w = 1; w < 4; ++w) v += red[w * kCols + c];
    a_in.partial[(int64_t)split * a_in.ld_partial + c0 + c] = v;
  }
}

}  // namespace game
