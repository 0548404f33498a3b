// Simple natural-gradient method (App. A): Fisher factors from the other rows of the same minibatch.
//
// For an N x D matrix X the efficient form (App. A.3) needs one symmetric positive-definite inverse of size
// n = min(N, D):  G = beta I + X^T X / (N-1)  (column space, N > D)  or  beta I + X X^T / (N-1)  (row space),
// Q = X G^{-1} resp. G^{-1} X, then a_i = x_i . q_i, b_i = 1 + a_i / (N-1-a_i), xhat_i = b_i q_i, and the
// rescaling gamma of App. A.2.
//
// The Gram matrix and Q are products for the matrix units (gemm.h).  The inverse is a blocked elimination in fp64 without
// pivoting (G is positive definite, its condition number is at most about 1 + D/alpha), in the symmetric form of it (the sweep
// operator), so that only the blocks on and above the diagonal are kept: one launch per 32-wide pivot block k replaces
//     (k,k) <- -P, P = A_kk^{-1},   (k,j) <- P A_kj,   (i,k) <- A_ik P,   (i,j) <- A_ij - A_ik P A_kj,
// reading the old matrix from one buffer and writing the new one to the other, so a launch has no ordering
// among its workgroups.  After the last pivot block the matrix is -G^{-1}.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm.h"
#include "kernels.h"
#include "state.h"
#include "wave_f64.h"

namespace ngsgd {

constexpr int kSimpleBlock = 32;      // pivot block of the inversion
constexpr int kSimpleGramTile = kSymGramTile;   // the Gram matrix is computed in tiles of this size, upper triangle only
constexpr int kSimpleMaxGroup = 16;   // matrices per grouped launch (the argument block stays within 4 KB)

struct SimpleArgs {
  float* M;         // N x D, ld: X on entry, Xhat (or gamma Xhat) on exit
  float* Q;         // N x D, ldq: scratch for Q
  int ld, ldq;
  int N, D;
  int n, np, nblk;  // size of the Gram matrix, padded to a multiple of 32, number of pivot blocks
  double alpha, epsilon;
  double* buf[2];   // np x np each; the Gram matrix is accumulated in buf[1]
  float* ginv;      // np x np, G^{-1} rounded to fp32 for the Q product
  double* pinv[2];  // 32 x 32 each: inverse of the pivot block of the current / the next elimination step
  double* prow;     // N: ||xhat_i||^2
  double* scal;     // [0] tr(X^T X), [1] beta
  double* gamma;    // gamma (App. A.2)
  float* gamma_out;     // optional copies for the caller
  float* rownorm2_out;  // optional: gamma^2 ||xhat_i||^2
};
struct SimpleGroup {
  int count;
  SimpleArgs a[kSimpleMaxGroup];
};

// Elimination of all pivots of a 32 x 32 positive-definite block A by a workgroup of 256 threads, four pivots at a time:
// A <- -A^{-1}.  Wavefront w holds the 16 x 16 quadrant (w / 2, w % 2) as a matrix-unit result: acc[r] of lane l is row
// 4 r + l / 16, column l % 16 of it.  A step takes the pivot rows U (by symmetry the pivot columns as well) with -I written over
// the pivot block, E = Q^{-1} U for the pivot block Q, and A - U^T E with the pivot rows and columns of A cleared: one product
// of depth four replaces everything.  Q^{-1} is applied by 2 x 2 blocks (both positive definite: one reciprocal of a
// determinant each), every lane for its own column.  The owners publish the next rows as soon as they have them: one barrier
// a step.  Bound: the latency of 8 such steps (and one wavefront per SIMD issues an instruction only every 7 or 8 cycles,
// hence few of them): 3.1 us, two pivots at a time on the vector units took 5.
struct PivotRows {
  double row[4][48];    // U, -I in the pivot block; the spacing keeps the rows of a read on different banks
  double q[4][4];       // Q
};
__device__ __forceinline__ void eliminate_block_32(doublex4& acc, PivotRows (&pub)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int hi = (wave >> 1) * 16, hj = (wave & 1) * 16;
  auto publish = [&](PivotRows& to, const int half, const int r) {
    if (hi != half * 16) return;
    const bool diag = hj == hi && (l16 >> 2) == r;
    if (diag) to.q[g4][l16 & 3] = acc[r];
    to.row[g4][hj + l16] = diag ? (g4 == (l16 & 3) ? -1.0 : 0.0) : acc[r];
  };
  publish(pub[0], 0, 0);
  __syncthreads();
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const PivotRows& in = pub[r & 1];
      const double q00 = in.q[0][0], q01 = in.q[0][1], q02 = in.q[0][2], q03 = in.q[0][3], q11 = in.q[1][1], q12 = in.q[1][2],
                   q13 = in.q[1][3], q22 = in.q[2][2], q23 = in.q[2][3], q33 = in.q[3][3];
      const double u0 = in.row[0][hj + l16], u1 = in.row[1][hj + l16], u2 = in.row[2][hj + l16], u3 = in.row[3][hj + l16];
      const double x = in.row[g4][hi + l16];
      // inverse of the leading 2 x 2 block, T = it times the block to its right, the Schur complement and its inverse
      const double ia = reciprocal_f64(fma(q00, q11, -(q01 * q01)));
      const double a0 = q11 * ia, a1 = -q01 * ia, a2 = q00 * ia;
      const double t00 = fma(a0, q02, a1 * q12), t01 = fma(a0, q03, a1 * q13);
      const double t10 = fma(a1, q02, a2 * q12), t11 = fma(a1, q03, a2 * q13);
      const double s00 = fma(-q12, t10, fma(-q02, t00, q22)), s01 = fma(-q12, t11, fma(-q02, t01, q23));
      const double s11 = fma(-q13, t11, fma(-q03, t01, q33));
      const double is = reciprocal_f64(fma(s00, s11, -(s01 * s01)));
      const double w0 = fma(a0, u0, a1 * u1), w1 = fma(a1, u0, a2 * u1);
      const double v2 = fma(-q12, w1, fma(-q02, w0, u2)), v3 = fma(-q13, w1, fma(-q03, w0, u3));
      const double e2 = is * fma(s11, v2, -(s01 * v3)), e3 = is * fma(s00, v3, -(s01 * v2));
      const double e0 = fma(-t01, e3, fma(-t00, e2, w0)), e1 = fma(-t11, e3, fma(-t10, e2, w1));
      const double e = g4 == 0 ? e0 : (g4 == 1 ? e1 : (g4 == 2 ? e2 : e3));
      if (hi == half * 16) acc[r] = 0.0;
      if (hj == half * 16 && (l16 >> 2) == r) acc = doublex4{0.0, 0.0, 0.0, 0.0};
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-x, e, acc, 0, 0, 0);
      if (r < 3)
        publish(pub[(r & 1) ^ 1], half, r + 1);
      else if (half == 0)
        publish(pub[0], 1, 0);
      __syncthreads();
    }
  }
}

// G = beta I + S / (N-1), blocks on and above the diagonal, S given by its tiles there, with
// beta = alpha max(tr S, epsilon) / (N D) (App. A.2); rows and columns beyond n carry the identity so that the padded matrix
// stays positive definite.  A workgroup forms 64 x 64 elements: each needs the trace, whose n loads from as many cache lines
// cost more than the rest with one workgroup per 32 x 32 (9.9 us for n = 512, 25 for ten of those).
// The workgroup of tile (0, 0) also eliminates the first pivot block.  Grid (ceil(np/64), ceil(np/64), count), 256 threads.
__global__ __launch_bounds__(256) void simple_prepare_kernel(const SimpleGroup g) {
  const SimpleArgs& a = g.a[blockIdx.z];
  const int np = a.np, n = a.n, bi = blockIdx.y * 64, bj = blockIdx.x * 64;
  if (bi > bj || bj >= np) return;
  static_assert(kSimpleGramTile == 64, "the tiles of S");
  __shared__ double scratch[16];
  __shared__ PivotRows pub[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* __restrict__ S = a.buf[1];
  double v[16];   // element (wave + 4 q, lane) of the tile
  const int j = bj + lane;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int i = bi + wave + 4 * q;
    v[q] = i < n && j < n ? S[(size_t)i * np + j] : 0.0;
  }
  double t = 0.0;
  for (int i = tid; i < n; i += 256) t += S[(size_t)i * np + i];
  const double tr = block_sum(t, scratch);
  const double beta = a.alpha * fmax(tr, a.epsilon) / ((double)a.N * (double)a.D);
  if (bj == 0 && tid == 0) {
    a.scal[0] = tr;
    a.scal[1] = beta;
  }
  const double inv_nm1 = 1.0 / (double)(a.N - 1);
  auto element = [&](const int i, const int j, const double s) {
    return i < n && j < n ? s * inv_nm1 + (i == j ? beta : 0.0) : (i == j ? 1.0 : 0.0);
  };
  double* __restrict__ G = a.buf[0];
  if (bj == 0) {   // S again in the elimination's layout: the first loads have brought it near
    doublex4 acc;
    const int i0 = (wave >> 1) * 16 + (lane >> 4), j0 = (wave & 1) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 4 * r;
      acc[r] = element(i, j0, i < n && j0 < n ? S[(size_t)i * np + j0] : 0.0);
    }
    eliminate_block_32(acc, pub);
#pragma unroll
    for (int r = 0; r < 4; ++r) a.pinv[0][(i0 + 4 * r) * kSimpleBlock + j0] = -acc[r];
  }
  if (j < np) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = bi + wave + 4 * q;
      if (i < np) G[(size_t)i * np + j] = element(i, j, v[q]);
    }
  }
}

// One pivot block k of the inversion.  256 threads; grid (s + 2, ceil(s/2), count) for s = ceil(nblk/2) rows of 64 x 64 tiles,
// of which those on and above the diagonal are kept: workgroup (x + 1, y) has tile x of row y, counted from the diagonal, and
// beyond its end of row s - 1 - y, so that no workgroup stays without one.  Wavefront w replaces block (w/2, w%2) of the tile,
// using the inverse P_k of the pivot block that the previous launch left in pinv[k % 2].  With X_m = A_mk, -I for m = k, and
// the old blocks of row and column k taken as zero, all are alike: A_ij - X_i P X_j^T.  The four X of the tile go to LDS, one per
// wavefront, and the two wavefronts of a row share X_i P.
// Bound: for one matrix the latency of loads, two products and stores, about that of the chain below; for many the blocks' traffic.
// 512 x 512: one matrix 6.9 us a launch, ten 9.9 (all blocks instead of half of them, X_i P in each wavefront: 8.1 and 15.7;
// a workgroup per 32 x 32 block: 6.7 and 10.5).
// The one workgroup of the first grid column looks ahead: it forms the next pivot block (k+1, k+1) as this step leaves it
// (a 16 x 16 quadrant per wavefront) and eliminates it into pinv[(k+1) % 2], so that is done once per matrix and step, beside
// the block updates and not before them.  Its chain bounds the launch for one matrix, so it is started first.
// v_mfma_f64_16x16x4_f64: lane l supplies A[l%16][l/16] and B[l/16][l%16]; register r of lane l holds
// row 4r + l/16, column l%16 of the 16 x 16 result.
__global__ __launch_bounds__(256) void simple_sweep_kernel(const SimpleGroup g, const int k) {
  const SimpleArgs& a = g.a[blockIdx.z];
  const int nblk = a.nblk, tiles = (nblk + 1) >> 1;
  const bool ahead = blockIdx.x == 0;
  int ty = blockIdx.y, tx = ty + (int)blockIdx.x - 1;
  if (!ahead && tx >= tiles) {
    const int over = tx - tiles;
    ty = tiles - 1 - ty;
    tx = ty + over;
    if (ty <= (int)blockIdx.y) return;   // uniform per workgroup, as all of these
  }
  if (k >= nblk || 2 * (int)blockIdx.y >= tiles) return;
  if (ahead && (blockIdx.y != 0 || k + 1 >= nblk)) return;
  if (!ahead && tx >= tiles) return;
  constexpr int B = kSimpleBlock, LD = B + 2;   // rows 4 banks apart: an operand's read takes each bank once
  __shared__ double sP[B][LD];         // P_k (symmetric)
  __shared__ double sX[4][B][LD];
  __shared__ PivotRows pub[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int np = a.np;
  const double* __restrict__ src = a.buf[k & 1];
  double* __restrict__ dst = a.buf[(k & 1) ^ 1];
  const size_t k0 = (size_t)k * B;
  const int l16 = lane & 15, g4 = lane >> 4;
  double pv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) pv[q] = a.pinv[k & 1][tid + 256 * q];
  if (ahead) {
    const size_t d0 = k0 + B;
    const int hi = (wave >> 1) * 16, hj = (wave & 1) * 16;
    double xv[4];
    doublex4 acc, t[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
    for (int q = 0; q < 4; ++q) xv[q] = src[(k0 + (tid >> 5) + 8 * q) * np + d0 + (tid & 31)];
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = src[(d0 + hi + 4 * r + g4) * np + d0 + hj + l16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sP[(tid >> 5) + 8 * q][tid & 31] = pv[q];
      sX[0][tid & 31][(tid >> 5) + 8 * q] = xv[q];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < B / 4; ++ks)
      t[ks & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[0][hi + l16][ks * 4 + g4], sP[hj + l16][ks * 4 + g4], t[ks & 1], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) sX[1][hi + 4 * r + g4][hj + l16] = -(t[0][r] + t[1][r]);
    __syncthreads();
    t[1] = doublex4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < B / 4; ks += 2) {
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[1][hi + l16][ks * 4 + g4], sX[0][hj + l16][ks * 4 + g4], acc, 0, 0, 0);
      t[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[1][hi + l16][ks * 4 + 4 + g4], sX[0][hj + l16][ks * 4 + 4 + g4], t[1], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] += t[1][r];
    eliminate_block_32(acc, pub);
#pragma unroll
    for (int r = 0; r < 4; ++r) a.pinv[(k + 1) & 1][(hi + 4 * r + g4) * B + hj + l16] = -acc[r];
    return;
  }
  const int bi = 2 * ty + (wave >> 1), bj = 2 * tx + (wave & 1);
  const bool active = bi <= bj && bj < nblk;
  const size_t i0 = (size_t)bi * B, j0 = (size_t)bj * B;

  // everything this wavefront needs is requested up front: P_k, its X (stored transposed below the pivot), A_ij
  const int bx = wave < 2 ? 2 * ty + wave : 2 * tx + (wave & 1);
  const size_t x0 = bx < k ? (size_t)bx * B * np + k0 : k0 * np + (size_t)bx * B;
  const bool stored = bx != k && bx < nblk;
  double xv[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = (lane >> 5) + 2 * q, c = lane & 31;
    xv[q] = stored ? src[x0 + (size_t)r * np + c] : (bx == k && r == c ? -1.0 : 0.0);
  }
  doublex4 acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int nj = 0; nj < 2; ++nj)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc[mi][nj][r] = active && bi != k && bj != k ? src[(i0 + mi * 16 + 4 * r + g4) * np + j0 + nj * 16 + l16] : 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) sP[(tid >> 5) + 8 * q][tid & 31] = pv[q];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = (lane >> 5) + 2 * q, c = lane & 31;
    if (bx < k)
      sX[wave][r][c] = xv[q];
    else
      sX[wave][c][r] = xv[q];
  }
  __syncthreads();

  // half of -X_i P: columns 16 (w % 2) on
  const int row = wave >> 1, tc = (wave & 1) * 16;
  doublex4 t[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
  for (int ks = 0; ks < B / 4; ++ks) {
    const double pf = -sP[tc + l16][ks * 4 + g4];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
      t[mi] = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[row][mi * 16 + l16][ks * 4 + g4], pf, t[mi], 0, 0, 0);
  }
  __syncthreads();
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int r = 0; r < 4; ++r) sX[row][mi * 16 + 4 * r + g4][tc + l16] = t[mi][r];
  __syncthreads();
  if (!active) return;
#pragma unroll
  for (int ks = 0; ks < B / 4; ++ks) {
    double af[2], bf[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      af[m] = sX[row][m * 16 + l16][ks * 4 + g4];
      bf[m] = sX[2 + (wave & 1)][m * 16 + l16][ks * 4 + g4];
    }
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nj = 0; nj < 2; ++nj)
        acc[mi][nj] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[mi], bf[nj], acc[mi][nj], 0, 0, 0);
  }
  if (k < nblk - 1) {
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nj = 0; nj < 2; ++nj)
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(i0 + mi * 16 + 4 * r + g4) * np + j0 + nj * 16 + l16] = acc[mi][nj][r];
  } else {   // G^{-1}, both halves
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nj = 0; nj < 2; ++nj)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const size_t i = i0 + mi * 16 + 4 * r + g4, j = j0 + nj * 16 + l16;
          const float v = -(float)acc[mi][nj][r];
          a.ginv[i * np + j] = v;
          if (bi != bj) a.ginv[j * np + i] = v;
        }
  }
}

// a_i = x_i . q_i, b_i = 1 + a_i / (N - 1 - a_i), xhat_i = b_i q_i (App. A.3), ||xhat_i||^2.  With LATE b_i goes to the elimination's
// first buffer (done with by then) and xhat_i is left to the kernel that scales; a row's first 5120 columns are then requested at once
// (512 x 5000: 9.4 -> 5.5 us).  The matrices of a network fill the chip with rows, and the registers of that would cost them more wavefronts than
// it gives: eight matrices of 512 rows and 60 to 901 columns 14.6 instead of 11.7 us, twelve of 700 rows and 200 to 1000 columns 21.5 instead of
// 17.1 (the speech-shaped network's ten 22 either way).  Grid (N_max, count).
template <bool LATE>
__global__ __launch_bounds__(256) void simple_rows_kernel(const SimpleGroup g) {
  const SimpleArgs& a = g.a[blockIdx.y];
  const int i = blockIdx.x;
  if (i >= a.N) return;
  constexpr int AHEAD = LATE ? 5 : 0;
  __shared__ double scratch[16];
  const int tid = threadIdx.x, D = a.D, D4 = D >> 2;
  float* __restrict__ x = a.M + (size_t)i * a.ld;           // rows start on 16-byte boundaries
  const float* __restrict__ q = a.Q + (size_t)i * a.ldq;
  float4* __restrict__ x4 = reinterpret_cast<float4*>(x);
  const float4* __restrict__ q4 = reinterpret_cast<const float4*>(q);
  float4 xr[LATE ? AHEAD : 1], qr[LATE ? AHEAD : 1];
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    const int c = min(tid + 256 * u, max(D4 - 1, 0));
    xr[u] = D4 > 0 ? x4[c] : q4[c];   // (a last row shorter than a piece may end the caller's memory)
    qr[u] = q4[c];
  }
  double dot = 0.0, qq = 0.0;
  auto piece = [&](const float4& xv, const float4& qv) {
    dot += (double)xv.x * qv.x + (double)xv.y * qv.y + (double)xv.z * qv.z + (double)xv.w * qv.w;
    qq += (double)qv.x * qv.x + (double)qv.y * qv.y + (double)qv.z * qv.z + (double)qv.w * qv.w;
  };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (tid + 256 * u < D4) piece(xr[u], qr[u]);
  for (int c = tid + 256 * AHEAD; c < D4; c += 256) piece(x4[c], q4[c]);
  for (int c = 4 * D4 + tid; c < D; c += 256) {
    const double xv = x[c], qv = q[c];
    dot += xv * qv;
    qq += qv * qv;
  }
  dot = block_sum(dot, scratch);
  qq = block_sum(qq, scratch);
  const double b = 1.0 + dot / ((double)(a.N - 1) - dot);
  if (!LATE) {
    for (int c = tid; c < D4; c += 256) {
      const float4 qv = q4[c];
      x4[c] = make_float4((float)(b * qv.x), (float)(b * qv.y), (float)(b * qv.z), (float)(b * qv.w));
    }
    for (int c = 4 * D4 + tid; c < D; c += 256) x[c] = (float)(b * (double)q[c]);
  }
  if (tid == 0) {
    a.prow[i] = b * b * qq;
    if (LATE) a.buf[0][i] = b;
  }
}

// gamma as below by every workgroup, and gamma Xhat from Q and what simple_rows_kernel<true> left: X is written once (a launch each for
// Xhat, gamma and the scaling, 512 x 5000: 9.4 + 4.0 + 6.8 us; now 5.5 + 9.4).  Grid (ceil(N_max / 2), count), 256 threads, two rows.
constexpr int kSimpleScaleRows = 2;
__global__ __launch_bounds__(256) void simple_scale_kernel(const SimpleGroup g) {
  const SimpleArgs& a = g.a[blockIdx.y];
  constexpr int WIDTH = 256 / kSimpleScaleRows, AHEAD = 10;
  __shared__ double scratch[16];
  const int tid = threadIdx.x, D = a.D, D4 = D >> 2, row0 = blockIdx.x * kSimpleScaleRows, i = row0 + tid / WIDTH, c0 = tid % WIDTH;
  if (row0 >= a.N) return;
  const int ic = min(i, a.N - 1);
  const float* __restrict__ q = a.Q + (size_t)ic * a.ldq;
  const float4* __restrict__ q4 = reinterpret_cast<const float4*>(q);
  float* __restrict__ x = a.M + (size_t)ic * a.ld;
  float4* __restrict__ x4 = reinterpret_cast<float4*>(x);
  float4 qr[AHEAD];
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) qr[u] = q4[min(c0 + WIDTH * u, max(D4 - 1, 0))];
  const double b = a.buf[0][ic], p = a.prow[ic];
  double den = 0.0;
  for (int r = tid; r < a.N; r += 256) den += a.prow[r];
  den = block_sum(den, scratch);
  const double gamma = den > 0.0 ? sqrt(a.scal[0] / den) : 1.0;
  if (blockIdx.x == 0 && tid == 0) {
    *a.gamma = gamma;
    if (a.gamma_out != nullptr) *a.gamma_out = (float)gamma;
  }
  if (i >= a.N) return;
  if (c0 == 0 && a.rownorm2_out != nullptr) a.rownorm2_out[i] = (float)(gamma * gamma * p);
  const float s = (float)gamma;
  auto scaled = [&](const float4& v) {
    return make_float4(s * (float)(b * v.x), s * (float)(b * v.y), s * (float)(b * v.z), s * (float)(b * v.w));
  };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (c0 + WIDTH * u < D4) x4[c0 + WIDTH * u] = scaled(qr[u]);
  for (int c = c0 + WIDTH * AHEAD; c < D4; c += WIDTH) x4[c] = scaled(q4[c]);
  if (c0 < D - 4 * D4) x[4 * D4 + c0] = s * (float)(b * (double)q[4 * D4 + c0]);
}

// gamma = sqrt(tr(X^T X) / tr(Xhat^T Xhat)), 1 if the denominator is 0 (App. A.2).  Grid (count), 256 threads.
__global__ __launch_bounds__(256) void simple_gamma_kernel(const SimpleGroup g) {
  const SimpleArgs& a = g.a[blockIdx.x];
  __shared__ double scratch[16];
  const int tid = threadIdx.x;
  double den = 0.0;
  for (int i = tid; i < a.N; i += 256) den += a.prow[i];
  den = block_sum(den, scratch);
  const double gamma = den > 0.0 ? sqrt(a.scal[0] / den) : 1.0;
  if (tid == 0) {
    *a.gamma = gamma;
    if (a.gamma_out != nullptr) *a.gamma_out = (float)gamma;
  }
  if (a.rownorm2_out != nullptr)
    for (int i = tid; i < a.N; i += 256) a.rownorm2_out[i] = (float)(gamma * gamma * a.prow[i]);
}

}  // namespace ngsgd
