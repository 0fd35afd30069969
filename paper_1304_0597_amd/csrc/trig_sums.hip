// Per-pattern sums of the paper's own model (Eq. 9), in which every feature
// shares the genes a_j, b_j: Out = a_0 + sum_j a_j C_j + sum_j b_j S_j with
// C_j = sum_i cos(j f_i) and S_j = sum_i sin(j f_i).  The sums do not depend
// on the genes, so they are computed once per data set (the parallel version
// of Sec. 4.1 does the same) and the training loop then runs the degree-1
// power model over the 2d sums as features.
//
// One thread per pattern: cos/sin(j x) by the recurrence of Eq. 8 seeded
// with cos x and sin x, everything in float64, rounded to float32 once.  The
// per-degree sums live in registers (degree is a template argument); long rows
// of large inputs come in, and the sums of high degrees of large inputs go out,
// through LDS in consecutive addresses.
//
// Bound by issuing float64 operations: a seed takes 24, the recurrence and the
// sums 4 d.  1,792,000 x 11, degree 4: 48 us (136 MB, 2.8 TB/s; 61 with the
// library's sincos and strided stores), 200,000 x 64: 47 us (73).
//
// Also here: the per-feature trigonometric expansion's seeds (cos x, sin x of
// every pattern and feature), stored once per data set for the float32
// fitness kernel, which would otherwise evaluate them in every chromosome
// tile (Sec. 4.1: trigonometric terms computed once, not every iteration).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "rows.h"

namespace game {

namespace {

// sin x and cos x in float64 of a float32 angle.  Up to kFastAngle the nearest
// multiple n of pi/2 is taken off in two parts (the first fused product is
// exact, n times what the second part leaves out is below 1e-28), and both
// Taylor series run to their terms below half a unit of 2^-53 for |r| <= pi/4:
// sin to r^17/17!, cos to r^18/18!.  Larger angles, infinities and NaN go to
// the library's sincos.
constexpr float kFastAngle = 65536.f;

// a * b + c with a uniform c in scalar registers.  (Written as fma() it
// becomes an accumulating instruction after a copy of c to vector registers.)
__device__ __forceinline__ double fma_sc(double a, double b, double c) {
  double d;
  __asm__("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

__device__ __forceinline__ void sincos_of(float xf, double& sn, double& cs) {
  const double x = (double)xf;
  if (!(fabsf(xf) <= kFastAngle)) {
    sincos(x, &sn, &cs);
    return;
  }
  const double n = rint(x * 0.63661977236758134308);           // 2 / pi
  double r = fma(-n, 1.57079632679489655800, x);               // pi / 2, nearest double
  r = fma(-n, 6.12323399573676603587e-17, r);                  // and its remainder
  const double z = r * r;
  constexpr double f3 = 6.0, f5 = 120.0, f7 = 5040.0, f9 = 362880.0, f11 = 39916800.0,
                   f13 = 6227020800.0, f15 = 1307674368000.0, f17 = 355687428096000.0;
  constexpr double f4 = 24.0, f6 = 720.0, f8 = 40320.0, f10 = 3628800.0, f12 = 479001600.0,
                   f14 = 87178291200.0, f16 = 20922789888000.0, f18 = 6402373705728000.0;
  double ps = fma_sc(z, 1.0 / f17, -1.0 / f15);
  ps = fma_sc(ps, z, 1.0 / f13);
  ps = fma_sc(ps, z, -1.0 / f11);
  ps = fma_sc(ps, z, 1.0 / f9);
  ps = fma_sc(ps, z, -1.0 / f7);
  ps = fma_sc(ps, z, 1.0 / f5);
  ps = fma_sc(ps, z, -1.0 / f3);
  const double sr = fma(r * z, ps, r);
  double pc = fma_sc(z, -1.0 / f18, 1.0 / f16);
  pc = fma_sc(pc, z, -1.0 / f14);
  pc = fma_sc(pc, z, 1.0 / f12);
  pc = fma_sc(pc, z, -1.0 / f10);
  pc = fma_sc(pc, z, 1.0 / f8);
  pc = fma_sc(pc, z, -1.0 / f6);
  pc = fma_sc(pc, z, 1.0 / f4);
  const double cr = fma(z * z, pc, fma(-0.5, z, 1.0));
  const int q = (int)n;                                        // quadrant q mod 4
  const double s0 = (q & 1) ? cr : sr, c0 = (q & 1) ? sr : cr;
  sn = (q & 2) ? -s0 : s0;
  cs = ((q + 1) & 2) ? -c0 : c0;
}

template <int D, bool STAGE, bool LDS_OUT>
__global__ __launch_bounds__(kRows) void trig_sums_kernel(const float* X, int64_t NP, int N,
                                                          float* Z) {
  extern __shared__ float rows[];
  const int FC = STAGE ? min(N, kChunk) : N;
  const int S = row_stride(FC);
  constexpr int SZ = row_stride(2 * D);
  const int64_t row0 = (int64_t)blockIdx.x * kRows;
  const int n_rows = (int)min((int64_t)kRows, NP - row0);
  const float* mine = STAGE ? rows + threadIdx.x * S
                            : X + (row0 + min((int)threadIdx.x, n_rows - 1)) * N;
  double c[D], s[D];
#pragma unroll
  for (int j = 0; j < D; ++j) c[j] = s[j] = 0.0;
  for (int f0 = 0; f0 < N; f0 += FC) {
    const int nf = min(FC, N - f0);
    if constexpr (STAGE) {
      if (f0) __syncthreads();            // the features staged before have been used
      stage_rows(rows, S, X, row0, n_rows, N, f0, nf);
      __syncthreads();
    }
    if ((int)threadIdx.x < n_rows) {
      float x = mine[0];
      for (int i = 0; i < nf; ++i) {
        const float next = mine[min(i + 1, nf - 1)];
        double sn, cs;
        sincos_of(x, sn, cs);
        x = next;
        const double m2 = 2.0 * cs;
        double cp = 1.0, cc = cs, sp = 0.0, sc = sn;     // j-1 and j terms
#pragma unroll
        for (int j = 0; j < D; ++j) {
          c[j] += cc;
          s[j] += sc;
          const double cn = fma(m2, cc, -cp), sn2 = fma(m2, sc, -sp);
          cp = cc;
          cc = cn;
          sp = sc;
          sc = sn2;
        }
      }
    }
  }
  if constexpr (LDS_OUT) __syncthreads();
  else if ((int)threadIdx.x >= n_rows) return;
  float* z = LDS_OUT ? rows + threadIdx.x * SZ : Z + (row0 + threadIdx.x) * (2 * D);
#pragma unroll
  for (int j = 0; j < D; ++j) {
    z[j] = (float)c[j];
    z[D + j] = (float)s[j];
  }
  if constexpr (!LDS_OUT) return;
  __syncthreads();
  for (int e = threadIdx.x; e < n_rows * 2 * D; e += kRows)
    Z[row0 * (2 * D) + e] = rows[e / (2 * D) * SZ + e % (2 * D)];
}

// Rows of up to one cache line, those of few workgroups and inputs of up to 14 MB,
// whose lines stay cached between a thread's reads of them, are read by their
// threads directly.  Degree 3 direct and staged: 84,086 x 17 6.5 us and 9.1, 84,086
// x 40 15.5 and 16.8, 150,000 x 32 21.6 and 17.6; 1,792,000 x 11: staging costs 10
// us of 60; 200,000 x 64 takes 47 staged, 73 with strided reads.
constexpr int64_t kDirectReads = 3500000;  // floats
template <int D, bool LDS_OUT>
hipError_t launch_out(const float* X, int64_t NP, int N, float* Z, hipStream_t s) {
  const dim3 grid((unsigned)((NP + kRows - 1) / kRows));
  const int out = LDS_OUT ? row_stride(2 * D) : 0;
  if (N <= 16 || NP * N <= kDirectReads || !stages_rows(grid.x)) {
    hipLaunchKernelGGL((trig_sums_kernel<D, false, LDS_OUT>), grid, dim3(kRows),
                       (size_t)kRows * out * sizeof(float), s, X, NP, N, Z);
  } else {
    const int most = std::max(out, row_stride(std::min(N, kChunk)));
    hipLaunchKernelGGL((trig_sums_kernel<D, true, LDS_OUT>), grid, dim3(kRows),
                       (size_t)kRows * most * sizeof(float), s, X, NP, N, Z);
  }
  return hipGetLastError();
}

// Sums of up to 32 bytes a pattern are whole sectors as their threads store them, and
// with fewer workgroups than CUs nothing covers a turn through LDS: 8,000 x 1, degree
// 12 3.0 us, 3.7 through it, but 84,086 x 1 5.6 and 4.8, 60,000 x 1, degree 8 3.7 and
// 3.4; degree 3, 84,086 x 2 3.2 and 3.5, 800,000 x 2 7.8 and 8.9.
template <int D>
hipError_t launch_d(const float* X, int64_t NP, int N, float* Z, hipStream_t s) {
  if constexpr (D > 4)
    if (NP > 192 * kRows) return launch_out<D, true>(X, NP, N, Z, s);
  return launch_out<D, false>(X, NP, N, Z, s);
}

template <int... Ds>
hipError_t dispatch(int d, const float* X, int64_t NP, int N, float* Z, hipStream_t s,
                    std::integer_sequence<int, Ds...>) {
  hipError_t e = hipErrorInvalidValue;
  ((d == Ds + 1 ? (e = launch_d<Ds + 1>(X, NP, N, Z, s), 0) : 0), ...);
  return e;
}

__global__ __launch_bounds__(256) void trig_cs_kernel(const float* X, int64_t n, float* cs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float sn, c;
  sincosf(X[i], &sn, &c);
  cs[2 * i] = c;
  cs[2 * i + 1] = sn;
}

}  // namespace

hipError_t launch_trig_cs(const float* X, int64_t NP, int N, float* cs, hipStream_t s) {
  const int64_t n = NP * N;
  hipLaunchKernelGGL(trig_cs_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, n, cs);
  return hipGetLastError();
}

hipError_t launch_trig_sums(const float* X, int64_t NP, int N, int d, float* Z, hipStream_t s) {
  return dispatch(d, X, NP, N, Z, s, std::make_integer_sequence<int, kMaxDegree>{});
}

}  // namespace game
