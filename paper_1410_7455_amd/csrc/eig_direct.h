// Eigenpairs of the R x R matrix Z_t by a direct method, all in fp64: Householder reduction to a tridiagonal matrix T,
// eigenvalues of T by multisection, eigenvectors by a twisted factorisation, back through the reflections.  (One
// Newton-Schulz step in the kernel that finishes the update makes the vectors orthogonal to working precision.)
//
// The errors of the reduction are a few eps sqrt(z_ii z_jj) where the diagonal descends, and of the eigenvalues a few eps each: the
// smallest keep their digits.  So rows and columns are sorted where the diagonal spans more than kDirectOrderSpan.  (Factors of the
// last layers' inputs of the speech-shaped network, eigenvalues over 4e10 and 3e12, about descending: 2e-13 and 1e-11 off;
// the same matrices in a random order 2e-5 and 6e-4.)
// Its chain has R columns of one barrier and a dozen serial runs of R steps; cyclic Jacobi, which it replaces, goes through
// R - 1 dependent rounds per sweep and 5 to 10 sweeps.  Factors of 512 x 5000 and 512 x 3001 matrices, fresh data: rank 80 273 us (six
// sweeps 243, the vectors 30), now 121 (reduction 75, eigenpairs 30, finish 15); rank 20 50, now 35.
// Where the eigenvalues span more than kDirectCondLimit, where a vector's residual is large or where the vectors are too far
// from orthogonal (eigenvalues that agree to working precision), the finishing kernel runs Jacobi instead.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "state.h"
#include "wave_f64.h"

namespace ngsgd {

constexpr double kDirectEps = 2.220446049250313e-16;
constexpr double kDirectCondLimit = 1.0e16;     // most that eigenvalues may span
constexpr double kDirectOrderSpan = 1.0e6;      // of the diagonal: below it the order does not matter to the digits that fp32 factors have
constexpr double kDirectResidual = 1.0e-13;     // |T x - lambda x| / |T| of a unit vector, at most
constexpr double kDirectRelResidual = 1.0e-8;   // and over lambda
constexpr double kDirectTiny = 1.0e-19;         // of the norm: eigenvalues below it are not told apart
constexpr double kDirectOrthoLimit = 1.0e-4;    // |U U^T - I| before the Newton-Schulz step, which squares it
constexpr int kDirectPasses = 16;               // multisection passes at most, a factor of 17 each

// Tile of the 16 x 16 thread grid that holds Z (rank up to 16 K), and row strides in LDS.  A stride of 4 (mod 32) doubles spreads
// the fp64 matrix unit's operand reads (16 rows x 4 columns) over the banks.
template <int K>
struct DirectShape {
  static constexpr int T = 16 * K;
  static constexpr int STRIDE = T <= 36 ? 36 : (T <= 68 ? 68 : 100);
};

// The symmetric matrix in registers of NT threads: thread (ti, tj), tj < 16, holds the elements (ti + NT/16 a, tj + 16 b).
template <int K, int NT>
struct DirectTile {
  static constexpr int ROWS = NT / 16;                  // rows of the thread grid
  static constexpr int A = (16 * K + ROWS - 1) / ROWS;   // elements of a thread: A rows, K columns
  using Regs = double[A][K];
  __device__ __forceinline__ static int ti() { return 4 * (threadIdx.x >> 6) + group16_index(); }
  __device__ __forceinline__ static int tj() { return group16_member(); }
};

// Element of column c (c / 16 is F or F + 1) of a row vector that every 16 lanes hold alike.
template <int F, int K>
__device__ __forceinline__ double direct_column(const double (&v)[K], const int c) {
  constexpr int G = F + 1 < K ? F + 1 : F;
  return read_lane_f64(c >> 4 == F ? v[F] : v[G], group16_lane(c & 15));
}

// Householder reduction by the first NT threads.  Both triangles are kept, so that a row's 16 lanes have the whole of it for a
// product with the matrix.  Column j takes one barrier.  Every 16 lanes hold the row vectors x = (row j) and
// a = (row j + 1), v and w for themselves: A x for the raw x and |x|^2 need no exchange, and with
// v = x - beta e_1, A v = A x - beta a does not wait for the reflection either.  A v is published; behind
// the barrier every thread updates its elements, A <- A - v w^T - w v^T with w = theta A v - (theta^2 / 2)(v.A v) v, and from a
// and from row j + 2 (published a column earlier) forms the next x and a as the update leaves them.
// Rows and columns that are done are left out (the loop over columns is cut into stages of 16).
// Reflection j = I - theta v v^T goes to row j of V (zero up to column j), theta to tau[j]; off-diagonal j to off[j].  These are in
// LDS: a barrier waits for a wavefront's stores, and stores to memory take longer than the rest of a column.
// Bound: a column's instructions, 300 per wavefront and SIMD, a third of them the row vectors that every wavefront forms for itself (with
// 512 threads, two wavefronts share a SIMD and form them twice: 5 % slower).
template <int K, int NT>
struct DirectLds {
  double row[3][16 * K];                 // rows 0, 1, 2; then published rows, two used alternately
  double y[2][16 * K];                   // A v, alternately
  double own[NT / 64][2][16 * K];        // x and a of every wavefront, to be read by rows
};
template <int K, int NT>
__device__ __forceinline__ void direct_reduce(typename DirectTile<K, NT>::Regs& S, const int R, DirectLds<K, NT>& lds, double* V, double* tau_out,
                                              double* off) {
  using Tile = DirectTile<K, NT>;
  constexpr int ROWS = Tile::ROWS, A = Tile::A, T = 16 * K;
  const int tid = threadIdx.x, ti = Tile::ti(), tj = Tile::tj();
  const bool first_group = group16_index() == 0;
  double(&own)[2][T] = lds.own[tid >> 6];
  if (R <= 2) return;
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (ti == u) {
#pragma unroll
      for (int b = 0; b < K; ++b) lds.row[u][tj + 16 * b] = S[0][b];
    }
  __syncthreads();
  double xc[K], ac[K];
#pragma unroll
  for (int b = 0; b < K; ++b) {
    xc[b] = tj + 16 * b > 0 ? lds.row[0][tj + 16 * b] : 0.0;
    ac[b] = tj + 16 * b > 0 ? lds.row[1][tj + 16 * b] : 0.0;
  }
  auto stage = [&](auto first) {
    constexpr int F = decltype(first)::value, FR = 16 * F / ROWS;   // what lies below holds only finished columns and rows
    for (int j = 16 * F; j < min(16 * F + 16, R - 2); ++j) {
      // x and a by rows: written and read by the wavefront itself
      if (first_group) {
#pragma unroll
        for (int b = F; b < K; ++b) {
          own[0][tj + 16 * b] = xc[b];
          own[1][tj + 16 * b] = ac[b];
        }
      }
      wave_lds_exchange();
      double xr[A], ar[A], acc[A], sigma = 0.0;
#pragma unroll
      for (int x = FR; x < A; ++x) {   // (a thread's rows beyond T reach nothing)
        xr[x] = own[0][min(ti + ROWS * x, T - 1)];
        ar[x] = own[1][min(ti + ROWS * x, T - 1)];
        acc[x] = 0.0;
      }
#pragma unroll
      for (int b = F; b < K; ++b) {
        const double tail = b > F + 1 || tj + 16 * b > j + 1 ? xc[b] : 0.0;
        sigma = fma(tail, tail, sigma);
      }
      sigma = group16_sum_f64(sigma);
      const double x0 = direct_column<F, K>(xc, j + 1), x1 = direct_column<F, K>(xc, j + 2);
#pragma unroll
      for (int b = F; b < K; ++b)
#pragma unroll
        for (int x = FR; x < A; ++x) acc[x] = fma(S[x][b], xc[b], acc[x]);
#pragma unroll
      for (int x = FR; x < A; ++x) acc[x] = group16_sum_f64(acc[x]);
      // beta = -sign(x0) |x|, v_1 = x0 - beta, theta = 2 / |v|^2 = 1 / (|x| (|x| + |x0|)); hardware estimates and a third-order step
      const double nn = fma(x0, x0, sigma);
      const bool reflects = sigma > 0.0 && nn > 1.0e-290;   // (else the column is done: v = 0)
      double r = __builtin_amdgcn_rsq(nn);
      const double er = fma(-nn * r, r, 1.0);
      r = fma(r * er, fma(0.375, er, 0.5), r);
      const double norm = nn * r, size = fabs(x0) + norm, q = norm * size;
      double th = __builtin_amdgcn_rcp(q);
      const double et = fma(-q, th, 1.0);
      th = fma(th, fma(et, et, et), th);
      const double beta = reflects ? (x0 > 0.0 ? -norm : norm) : x0, v0 = reflects ? (x0 > 0.0 ? size : -size) : 0.0;
      const double theta = reflects ? th : 0.0;
      double vr[A], yr[A], vc[K];
#pragma unroll
      for (int x = FR; x < A; ++x) {
        const int i = ti + ROWS * x;
        yr[x] = fma(-beta, ar[x], acc[x]);
        if (ROWS * x <= 16 * F + 15) yr[x] = i > j ? yr[x] : 0.0;
        vr[x] = ROWS * x <= 16 * F + 16 && i == j + 1 ? v0 : xr[x];
        if (tj == 0 && (A * ROWS == T || i < T)) lds.y[j & 1][i] = yr[x];
      }
#pragma unroll
      for (int b = F; b < K; ++b) vc[b] = b <= F + 1 && tj + 16 * b == j + 1 ? v0 : xc[b];
      __syncthreads();
      const double* const y = lds.y[j & 1];
      const double* const pub = lds.row[j == 0 ? 2 : (j & 1) ^ 1];   // row j + 2 behind column j - 1
      double yc[K], nc[K], dot[2] = {0.0, 0.0};
#pragma unroll
      for (int b = F; b < K; ++b) yc[b] = y[tj + 16 * b];
      const double y0 = y[j + 1], y1 = y[j + 2];
#pragma unroll
      for (int b = F; b < K; ++b) nc[b] = pub[tj + 16 * b];
#pragma unroll
      for (int b = F; b < K; ++b) dot[b & 1] = fma(yc[b], vc[b], dot[b & 1]);
      const double half = 0.5 * theta * theta * group16_sum_f64(dot[0] + dot[1]);
      double wr[A], wc[K];
#pragma unroll
      for (int b = F; b < K; ++b) wc[b] = fma(theta, yc[b], -half * vc[b]);
      const double v1 = reflects ? x1 : 0.0, w0 = fma(theta, y0, -half * v0), w1 = fma(theta, y1, -half * v1);
#pragma unroll
      for (int b = F; b < K; ++b) {
        xc[b] = fma(-v0, wc[b], fma(-w0, vc[b], ac[b]));
        ac[b] = fma(-v1, wc[b], fma(-w1, vc[b], nc[b]));
        if (b <= F + 1) {
          const bool live = tj + 16 * b > j + 1;
          xc[b] = live ? xc[b] : 0.0;
          ac[b] = live ? ac[b] : 0.0;
        }
      }
#pragma unroll
      for (int x = FR; x < A; ++x) wr[x] = fma(theta, yr[x], -half * vr[x]);
#pragma unroll
      for (int x = FR; x < A; ++x)
#pragma unroll
        for (int b = F; b < K; ++b) S[x][b] = fma(-vr[x], wc[b], fma(-wr[x], vc[b], S[x][b]));
#pragma unroll
      for (int x = (16 * F + 3) / ROWS; x <= min((16 * F + 18) / ROWS, A - 1); ++x) {
        if (ti + ROWS * x == j + 3) {
#pragma unroll
          for (int b = F; b < K; ++b) lds.row[j & 1][tj + 16 * b] = S[x][b];
        }
      }
      if (ti == 0) {
#pragma unroll
        for (int b = 0; b < K; ++b) V[j * T + tj + 16 * b] = b < F ? 0.0 : vc[b];
      }
      if (tid == 0) {
        tau_out[j] = theta;
        off[j] = beta;
      }
    }
  };
  stage(std::integral_constant<int, 0>());
  stage(std::integral_constant<int, 1>());
  if constexpr (K > 2) stage(std::integral_constant<int, 2>());
  if constexpr (K > 3) {
    stage(std::integral_constant<int, 3>());
    stage(std::integral_constant<int, 4>());
  }
  if constexpr (K > 5) stage(std::integral_constant<int, 5>());
}
// The barriers of direct_reduce, for the wavefronts that take no part in it.
__device__ __forceinline__ void direct_reduce_idle(const int R) {
  for (int j = 0; j < R - 1 && R > 2; ++j) __syncthreads();
}
// What the reduction leaves in the registers: the diagonal and the last off-diagonal.
template <int K, int NT>
__device__ __forceinline__ void direct_store_tridiagonal(const typename DirectTile<K, NT>::Regs& S, const int R, double* __restrict__ diag,
                                                         double* __restrict__ off) {
  const int ti = DirectTile<K, NT>::ti(), tj = DirectTile<K, NT>::tj();
#pragma unroll
  for (int x = 0; x < DirectTile<K, NT>::A; ++x)
#pragma unroll
    for (int b = 0; b < K; ++b) {
      const int i = ti + DirectTile<K, NT>::ROWS * x, c = tj + 16 * b;
      if (i == c && i < R) diag[i] = S[x][b];
      if (i == R - 2 && c == R - 1) off[i] = S[x][b];
    }
}

// T in LDS, scaled to unit norm.
template <int K>
struct DirectTridiagonal {
  static constexpr int T = 16 * K;
  double diag[T], off[T];       // as they were; off[i] couples i and i + 1, zero from R - 1 on
  double d[T], e[T], e2[T];     // scaled
  // (d[i], e2[i - 1]) from the top and (d[R - 1 - i], e2[R - 1 - i]) from the bottom; beyond R a diagonal that lies above every
  // point and changes no sign
  double2 step[2][T + 24];   // (whole blocks of eight steps, two at a time and one ahead)
};
// Scales T (diag and off are in LDS, a barrier behind them) and returns an interval that holds the scaled eigenvalues and the
// norm.  256 threads; ends with a barrier.
template <int K>
__device__ __forceinline__ void direct_scale(DirectTridiagonal<K>& t, const int R, double& lo, double& hi, double& norm) {
  const int tid = threadIdx.x, l16 = tid & 15;
  double up = -1.0e300, down = -1.0e300;
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int i = l16 + 16 * b;
    if (i >= R) continue;
    const double radius = (i > 0 ? fabs(t.off[i - 1]) : 0.0) + (i < R - 1 ? fabs(t.off[i]) : 0.0);
    up = fmax(up, t.diag[i] + radius);
    down = fmax(down, radius - t.diag[i]);
  }
  up = row16_max_f64(up);
  down = row16_max_f64(down);
  norm = fmax(fabs(up), fabs(down));
  const double inv = norm > 0.0 ? 1.0 / norm : 0.0, margin = 2.0 * kDirectEps * (double)R;
  lo = -down * inv - margin;
  hi = up * inv + margin;
  if (tid < t.T + 24) {
    const int i = tid;
    const double before = i > 0 && i < R ? t.off[i - 1] * inv : 0.0, f2 = fmax(before * before, 1.0e-60);
    if (i < R) {
      const double e = i < R - 1 ? t.off[i] * inv : 0.0;
      t.d[i] = t.diag[i] * inv;
      t.e[i] = e;
      t.e2[i] = fmax(e * e, 1.0e-60);   // never zero: the recurrences do not stop
    }
    t.step[0][i] = i < R ? make_double2(t.diag[i] * inv, f2) : make_double2(4.0, 0.0);
    const double behind = i > 0 && i < R ? t.off[R - 1 - i] * inv : 0.0;
    t.step[1][i] = i < R ? make_double2(t.diag[R - 1 - i] * inv, fmax(behind * behind, 1.0e-60)) : make_double2(4.0, 0.0);
  }
  __syncthreads();
}

// The reflections are applied four at a time; for each block of four rows of V the inner products between them, row
// (4 m + a) with row (4 m + b), a < b, in the order 01 02 03 12 13 23.  By 16 lanes each; the caller's barrier follows.
template <int K, int NT>
__device__ __forceinline__ void direct_block_products(const double* V, const int ldv, const int R, double (*s_g)[6]) {
  const int row = threadIdx.x >> 4, l16 = threadIdx.x & 15, blocks = (R - 2 + 3) / 4;
  constexpr int PA[6] = {0, 0, 0, 1, 1, 2}, PB[6] = {1, 2, 3, 2, 3, 3};
  for (int m = row; m < blocks; m += NT / 16) {   // (idle lanes of a wavefront are whole rows of 16)
    double v[4][K], g[6];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < K; ++b) v[a][b] = V[(4 * m + a) * ldv + l16 + 16 * b];
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      g[p] = 0.0;
#pragma unroll
      for (int b = 0; b < K; ++b) g[p] = fma(v[PA[p]][b], v[PB[p]][b], g[p]);
      g[p] = row16_sum_f64(g[p]);
    }
    if (l16 == 0) {
#pragma unroll
      for (int p = 0; p < 6; ++p) s_g[m][p] = g[p];
    }
  }
}

// Eigenpair k (descending) by LANES lanes.  Eigenvalue: LANES points of the interval at a time, a Sturm
// count each, by the three-term recurrence of the leading minors of T - x (rescaled every eight steps), the signs gathered
// in a bit mask.  Eigenvector, by every 16 lanes alike: the leading minors from the top (first lane) and from the bottom (second lane);
// their quotients are the pivots of the two factorisations; the twist where they meet best; the products of the pivots' quotients
// outwards from it: one step of inverse iteration from the best unit vector.  Then the reflections, last to first.
// `work` is 2 (T + 8) + 2 (K + 1) * 2 doubles of LDS for these 16 lanes; V (LDS, rows up to a multiple of four, those beyond R - 3 zero
// as their tau) has the reflections, s_g their products.
// `work` of four neighbouring rows of lanes lie kDirectWork apart.  Leaves the eigenvalue of the scaled T in lambda and the vector's
// residual (of the lanes' own pair), and in x elements member + 16 b of the unit vector, in the lanes of group16_sum: with LANES 16
// group q of a wavefront has the vector of its row of lanes q.
// Bound: serial chains of R steps, 10 (64 lanes) or 14 (16) of them for the eigenvalue.
template <int K>
constexpr int kDirectWork = 2 * (16 * K + 8) + 4 * (K + 1);
template <int K, int LANES>
__device__ __forceinline__ void direct_pair(const DirectTridiagonal<K>& t, const int R, const int k, const double lo0, const double hi0,
                                            const double* V, const int ldv, const double* tau, const double (*s_g)[6], double* const work,
                                            double (&x)[K], double& lambda, double& residual) {
  static_assert(LANES == 16 || LANES == 64, "a row of lanes or a wavefront");
  constexpr int T = 16 * K, P = T + 8;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  double lo = lo0, hi = hi0;
  const int blocks = (R + 6) / 8;   // of eight steps behind the first
  const int point = LANES == 16 ? l16 : lane;
  for (int pass = 0; pass < kDirectPasses; ++pass) {
    const double width = hi - lo;
    if (!(width > kDirectEps * fmax(hi, kDirectTiny))) break;
    // the first pass finds the eigenvalue's size: 64 binary orders below the largest
    constexpr int ORDERS = 64 / LANES;
    const double step = width * (1.0 / (LANES + 1));
    const double at = pass == 0 ? __builtin_amdgcn_ldexp(hi, -ORDERS * (point + 1)) : fma(step, (double)(point + 1), lo);
    double p = t.step[0][0].x - at, p1 = 1.0;
    uint32_t signs = (uint32_t)(__builtin_bit_cast(uint64_t, p) >> 63);
    int below = (int)signs;
    double2 de[2][8];   // two blocks of steps, one requested while the other is taken
    auto fetch = [&](const int set, const int blk) {
#pragma unroll
      for (int u = 0; u < 8; ++u) de[set][u] = t.step[0][1 + 8 * blk + u];
    };
    auto steps = [&](const int set) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double q = fma(de[set][u].x - at, p, -(de[set][u].y * p1));
        signs = __builtin_amdgcn_alignbit(signs, (uint32_t)(__builtin_bit_cast(uint64_t, q) >> 32), 31);   // shifted in
        p1 = p;
        p = q;
      }
      below += __popc((signs ^ (signs >> 1)) & 0xffu);
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p1)));
      p = __builtin_amdgcn_ldexp(p, ex);
      p1 = __builtin_amdgcn_ldexp(p1, ex);
    };
    fetch(0, 0);
    for (int blk = 0; blk < blocks; blk += 2) {   // (steps beyond R change no sign)
      fetch(1, blk + 1);
      steps(0);
      fetch(0, blk + 2);
      steps(1);
    }
    const uint64_t votes = __ballot(below <= R - 1 - k);   // points at or below the eigenvalue
    const int m = LANES == 16 ? __popc((uint32_t)(votes >> (lane & 48)) & 0xffffu) : __popcll(votes);
    const double base = lo;
    if (pass == 0) {
      const double top = hi;
      if (m > 0) lo = __builtin_amdgcn_ldexp(top, -ORDERS * (LANES - m + 1));
      if (m < LANES) hi = __builtin_amdgcn_ldexp(top, -ORDERS * (LANES - m));
    } else {
      if (m > 0) lo = fma(step, (double)m, base);
      if (m < LANES) hi = fma(step, (double)(m + 1), base);
    }
  }
  lambda = 0.5 * (lo + hi);

  // minors from both ends: element s of a list is the minor behind step s, `edge` what the next block of steps starts from (rescaled)
  if (l16 < 2) {
    const double2* const list = t.step[l16];
    double* const out = work + l16 * P;
    double* const edge = work + 2 * P + l16 * (2 * K + 2);
    double p = list[0].x - lambda, p1 = 1.0;
    out[0] = p;
    for (int blk = 0; blk < blocks; ++blk) {
      double2 de[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) de[u] = list[1 + 8 * blk + u];
      edge[blk] = p;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double q = fma(de[u].x - lambda, p, -(de[u].y * p1));
        out[1 + 8 * blk + u] = q;
        p1 = p;
        p = q;
      }
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p1)));
      p = __builtin_amdgcn_ldexp(p, ex);
      p1 = __builtin_amdgcn_ldexp(p1, ex);
    }
  }
  wave_lds_exchange();
  // reciprocal pivot at row i of the factorisation from the top (side 0) or the bottom (side 1): the minor before over the minor
  auto reciprocal_pivot = [&](const int side, const int i) {
    const int s = side == 0 ? i : R - 1 - i;
    const double den = work[side * P + s];
    const double num = s == 0 ? 1.0 : (((s - 1) & 7) == 0 ? work[2 * P + side * (2 * K + 2) + ((s - 1) >> 3)] : work[side * P + s - 1]);
    const double small = 1.0e-150 * fabs(num);
    return fabs(den) > small ? num * reciprocal_f64(den) : (den < 0.0 ? -1.0e150 : 1.0e150);
  };
  // This lane's rows from here on: K in sequence.  The factors that lead from row i + 1 up to i and from i - 1 down to i, and
  // the twist: the row whose pivot, reached from both sides, is smallest (a key of its size with the row in the low bits)
  uint32_t key = 0xffffffffu;
  double up[K], down[K];   // reciprocal pivots first
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int i = min(l16 * K + b, R - 1);
    up[b] = reciprocal_pivot(0, i);
    down[b] = reciprocal_pivot(1, i);
  }
  const double up_before = dpp_or_one_f64<0x111>(up[K - 1]), down_behind = dpp_or_one_f64<0x101>(down[0]);   // of the neighbouring lanes' rows
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int i = l16 * K + b, ic = min(i, R - 1);
    double gamma = t.d[ic] - lambda;
    if (i > 0) gamma = fma(-t.e2[max(ic - 1, 0)], b > 0 ? up[max(b - 1, 0)] : up_before, gamma);
    if (i < R - 1) gamma = fma(-t.e2[ic], b < K - 1 ? down[min(b + 1, K - 1)] : down_behind, gamma);
    if (i < R) key = min(key, (__builtin_bit_cast(uint32_t, (float)fabs(gamma)) & ~127u) | (uint32_t)i);
  }
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int i = min(l16 * K + b, R - 1);
    up[b] *= -t.e[i];
    down[b] = i > 0 ? -t.e[i - 1] * down[b] : 0.0;
  }
  key = row16_min_u32(key);
  const int twist = (int)(key & 127u);
  const double pivot = (double)__builtin_bit_cast(float, key & ~127u);
  // z_i: the product of `down` over the rows twist + 1 .. i or of `up` over i .. twist - 1; running products within a lane, then over lanes
  double z[K];
  {
    double below = 1.0, above = 1.0;
#pragma unroll
    for (int b = 0; b < K; ++b) {
      const int i = l16 * K + b;
      down[b] = i > twist && i < R ? down[b] : 1.0;
      up[b] = i < twist ? up[b] : 1.0;
      below *= down[b];
      above *= up[b];
    }
    double before = row16_scan_product<true>(below), behind = row16_scan_product<false>(above);   // of the lanes below, above this one
#pragma unroll
    for (int b = 0; b < K; ++b) {
      before *= down[b];
      z[b] = before;
    }
#pragma unroll
    for (int b = K - 1; b >= 0; --b) {
      behind *= up[b];
      z[b] = l16 * K + b < twist ? behind : z[b];
    }
  }
  double ss = 0.0;
#pragma unroll
  for (int b = 0; b < K; ++b) {
    z[b] = l16 * K + b < R ? z[b] : 0.0;
    ss = fma(z[b], z[b], ss);
  }
  ss = row16_sum_f64(ss);   // at least 1
  double rn = __builtin_amdgcn_rsq(ss);
  rn = fma(0.5 * rn, fma(-ss * rn, rn, 1.0), rn);
  rn = fma(0.5 * rn, fma(-ss * rn, rn, 1.0), rn);
  residual = pivot * rn;
#pragma unroll
  for (int b = 0; b < K; ++b) work[l16 * K + b] = z[b] * rn;   // (behind the last use of the minors)
  wave_lds_exchange();
  // the lanes of group16_sum from here on: with LANES 16 each of the four groups takes the vector of one row of lanes
  const int member = group16_member();
  const double* const mine = LANES == 16 ? work + (group16_index() - (lane >> 4)) * kDirectWork<K> : work;
#pragma unroll
  for (int b = 0; b < K; ++b) x[b] = mine[member + 16 * b];
  // four reflections at a time, 4 m + 3 first: their inner products with x as it is, corrected by the ones before
  auto reflect = [&](auto first) {
    constexpr int F = decltype(first)::value;
    for (int m = min(4 * F + 3, (R - 3) >> 2); m >= 4 * F; --m) {
      double v[4][K], dot[4] = {0.0, 0.0, 0.0, 0.0}, f[4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = F; b < K; ++b) v[a][b] = V[(4 * m + a) * ldv + member + 16 * b];
#pragma unroll
      for (int b = F; b < K; ++b)
#pragma unroll
        for (int a = 0; a < 4; ++a) dot[a] = fma(v[a][b], x[b], dot[a]);
#pragma unroll
      for (int a = 0; a < 4; ++a) dot[a] = group16_sum_f64(dot[a]);
      const double* const g = s_g[m];
      f[3] = tau[4 * m + 3] * dot[3];
      f[2] = tau[4 * m + 2] * fma(-f[3], g[5], dot[2]);
      f[1] = tau[4 * m + 1] * fma(-f[2], g[3], fma(-f[3], g[4], dot[1]));
      f[0] = tau[4 * m] * fma(-f[1], g[0], fma(-f[2], g[1], fma(-f[3], g[2], dot[0])));
#pragma unroll
      for (int a = 3; a >= 0; --a)
#pragma unroll
        for (int b = F; b < K; ++b) x[b] = fma(-f[a], v[a][b], x[b]);
    }
  };
  if (R < 3) return;
  if constexpr (K > 5) reflect(std::integral_constant<int, 5>());
  if constexpr (K > 3) {
    reflect(std::integral_constant<int, 4>());
    reflect(std::integral_constant<int, 3>());
  }
  if constexpr (K > 2) reflect(std::integral_constant<int, 2>());
  reflect(std::integral_constant<int, 1>());
  reflect(std::integral_constant<int, 0>());
}

}  // namespace ngsgd
