// Initialisation of the online natural-gradient state from the first minibatch (App. B.3.2):
// top-R eigenpairs of S_0 = X_0^T X_0 / N, rho_0, D_0, then W_0 = E_0^{1/2} R_0.
//
// The eigenproblem is solved on the smaller of the D x D covariance and the N x N Gram matrix (same
// non-zero spectrum; an eigenvector u of the Gram matrix gives X_0^T u / sqrt(N lambda)), in fp64 throughout:
//   1. Householder reduction to a tridiagonal matrix, Q^T A Q = T: up to 1024 rows one launch of many workgroups that keep the
//      matrix in registers and exchange vectors (above, a launch per column, each a pass over the trailing matrix);
//      the last 160 columns by one workgroup with the matrix in registers;
//   2. the R largest eigenvalues of T by multisection with Sturm counts, a wavefront each;
//   3. their eigenvectors by inverse iteration from random vectors, a thread each, then orthonormalised together
//      (twice, through the inverse Cholesky factor of their Gram matrix): vectors of equal eigenvalues start out
//      independent and any orthonormal basis of their space serves;
//   4. back with the reflections, a vector per wavefront.
// The error is a few eps |A| whatever the spectrum.  Bound: the chain of n columns.  Ten instances of the
// speech-shaped network, five of them with n = 512: 2.0 ms, of it 352 columns 0.73 (a launch each, 14 us for reading and writing 2 MB per
// instance, falling to 6 us: 2.6), the last 160 columns 0.38 ms, eigenvalues 0.14, inverse iteration 0.27,
// orthonormalisation 0.2, back transformation 0.15, rows of W 0.11.  A reduction needs no iteration; block Jacobi took
// 11 to 18 sweeps of 32 launches and did not settle on softmax derivatives within them (12.8 ms).
// This runs once per process (and after each parameter-averaging round), never inside the steady-state step.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "gemm.h"
#include "kernels.h"
#include "wave_f64.h"
#include "state.h"

namespace ngsgd {

constexpr double kNullEigRatio = 1.0e-12;          // eigenvalues of S_0 at or below this ratio carry no direction
constexpr double kCompletionMinResidual = 0.1;     // Gram-Schmidt completion threshold
constexpr int kInitPad = 64;                       // the matrix is padded with zeros to a multiple of this
constexpr double kInitEps = 2.220446049250313e-16;

struct InitArgs {
  PrecondScalars* st;
  const float* M;      // N x D first minibatch
  int ld;
  int N, D, R;
  int n;               // min(N, D): size of the eigenproblem
  int np;              // n rounded up to a multiple of kInitPad
  int rq;              // R rounded up to a multiple of 16
  int use_cov;         // 1: n = D, matrix X^T X; 0: n = N, matrix X X^T
  double* A;           // np x np matrix, reduced in place; then scratch of the inverse iteration (4 np rq), at last the
                       // eigenvectors, rq x np
  double* V;           // reflection j in row j (np x np), zero up to column j
  double* X;           // np x rq: eigenvectors of T
  double* T;           // 11 np: vectors of the tridiagonal form
  int* idx;            // R: row of the eigenvector matrix for each kept eigenpair, -1 if the direction is null
  float* W;            // R x ldw
  int ldw;
  int place;           // rows kept on the chip: launch x kTriDies + die, -1: not
  double* vwork;       // kMaxRank + D doubles

  __device__ double* G() const { return X + (size_t)np * rq; }   // rq x rq: Gram matrix of X, then the inverse of its Cholesky factor
  __device__ double* lam() const { return G() + (size_t)rq * rq; }   // R eigenvalues, descending
  __device__ double* diag() const { return T; }                  // T / N
  __device__ double* off() const { return T + np; }
  __device__ double* tau() const { return T + 2 * np; }          // the reflections' factors
  __device__ double* y(const int parity) const { return T + (3 + parity) * (size_t)np; }   // A v of the last two columns
  // Rows kept on the chip: what column j leaves for the next, A v and the next row, four columns in turn (before sdiag and bounds
  // are there); the count of workgroups that are running and their dies, and behind a closed gate the units taken and done
  __device__ double* ring(const int j) const { return T + (3 + 2 * (j & 3)) * (size_t)np; }
  __device__ int* gate() const { return st->gate; }
  __device__ double* bounds() const { return T + 5 * (size_t)np; }   // interval that holds T's eigenvalues, largest magnitude in it
  __device__ double* sdiag() const { return T + 6 * (size_t)np; }    // T scaled to unit norm: diagonal, squared off-diagonal
  __device__ double* soff2() const { return T + 7 * (size_t)np; }
  __device__ double* vec() const { return T + 8 * (size_t)np; }  // 3 np: used instead of LDS where that is too small
};
struct InitGroup {
  int count;
  double alpha, epsilon;
  InitArgs a[kMaxInstances];
};

// The initialisation is some hundreds of small launches: the instance list is stored in device memory once and the
// kernels take a pointer to it (a launch that carries the list by value costs the host three times as much).
__global__ void init_store_group_kernel(const InitGroup g, InitGroup* __restrict__ dst) {
  const uint32_t* src = reinterpret_cast<const uint32_t*>(&g);
  uint32_t* out = reinterpret_cast<uint32_t*>(dst);
  for (int i = threadIdx.x; i < (int)(sizeof(InitGroup) / sizeof(uint32_t)); i += blockDim.x) out[i] = src[i];
}

constexpr uint64_t kRingEmpty = 0x7ff8dead00c0ffeeULL;   // a NaN that no product leaves (of fp32 operands the low 29 bits are zero)

// The Gram product fills the 64 x 64 tiles on and above the diagonal; this copies them below it.  The first workgroup empties the
// ring and the gate.  Grid (np/32, np/32, instance), 256 threads.
__global__ __launch_bounds__(256) void init_mirror_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.z];
  const int np = a.np, i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    uint64_t* const ring = reinterpret_cast<uint64_t*>(a.ring(0));
    for (int i = threadIdx.x; i < 8 * np; i += 256) ring[i] = kRingEmpty;
    if (threadIdx.x < kGateWords) a.gate()[threadIdx.x] = 0;
  }
  if (i0 >= np || j0 >= np || i0 / kSymGramTile <= j0 / kSymGramTile) return;
  __shared__ double t[32][33];
  const int c = threadIdx.x & 31, r = threadIdx.x >> 5;
#pragma unroll
  for (int q = 0; q < 32; q += 8) t[r + q][c] = a.A[(size_t)(j0 + r + q) * np + i0 + c];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 32; q += 8) a.A[(size_t)(i0 + r + q) * np + j0 + c] = t[c][r + q];
}

// Column j of the reduction.  Every workgroup forms the vectors for itself: w from the last column's product y = A v
// (w = tau y - (tau^2 / 2)(y.v) v), row j of the matrix as that column's update A - v w^T - w v^T leaves it, and from it
// the next reflection.  Then it updates its rows of the trailing matrix and multiplies them with the new vector in the
// same pass.  Row j itself is only read.  Grid (16-row groups, instance), 256 threads, four rows per wavefront; the
// first 512 columns of its rows are requested before anything else.
// phases: 3 both; where three vectors do not fit into LDS (n > kTriLdsCols) 1, the vectors, to a.vec() by one workgroup
// per instance, then 2.
constexpr int kTriTail = 160;                 // columns left to the kernel that keeps the matrix in registers
constexpr int kTriRows = 4;                   // rows per wavefront
constexpr int kTriChunks = 8;                 // 64-column chunks held in registers
constexpr int kTriCols = 2;                   // columns per thread requested together in the vector phase
constexpr int kTriLdsCols = 2048;
__host__ __device__ inline int tri_step_units(const int n, const int j) { return (n - j - 1 + 4 * kTriRows - 1) / (4 * kTriRows); }
__device__ __forceinline__ void tri_step(const InitArgs& a, const int j, const int phases, const int unit, double* const dyn_tri) {
  const int n = a.n, np = a.np, wg_row = j + 1 + unit * 4 * kTriRows;
  __shared__ double red[2][4];
  double* const vo = phases == 3 ? dyn_tri : a.vec();   // the last column's v and w, and the new v
  double* const wo = vo + np;
  double* const vn = wo + np;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c0 = (j + 1) & ~63, chunks = (np - c0) / 64;
  const int row0 = wg_row + wave * kTriRows;
  double buf[kTriRows][kTriChunks];
  double* rowp[kTriRows];
#pragma unroll
  for (int q = 0; q < kTriRows; ++q) rowp[q] = a.A + (size_t)min(row0 + q, n - 1) * np + c0 + lane;
  auto load = [&](const int k0) {
#pragma unroll
    for (int q = 0; q < kTriRows; ++q)
#pragma unroll
      for (int k = 0; k < kTriChunks; ++k)
        if (k0 + k < chunks) buf[q][k] = rowp[q][(size_t)(k0 + k) * 64];
  };
  if (phases & 2) load(0);
  if (phases & 1) {
    const double* const v = a.V + (size_t)(j > 0 ? j - 1 : 0) * np;
    const double* const y = a.y((j & 1) ^ 1);
    const double* const rowj = a.A + (size_t)j * np;
    const int b0 = j & ~63;
    double tau = 0.0, vj = 0.0, yj = 0.0;
    if (j > 0) {
      tau = a.tau()[j - 1];
      vj = v[j];
      yj = y[j];
    }
    // this thread's columns: the first kTriCols of them are requested together
    double pv[kTriCols], py[kTriCols], px[kTriCols];
#pragma unroll
    for (int t = 0; t < kTriCols; ++t) {
      const int c = b0 + tid + 256 * t;
      const bool in = c >= j && c < n;
      pv[t] = in && j > 0 ? v[c] : 0.0;
      py[t] = in && j > 0 ? y[c] : 0.0;
      px[t] = in ? rowj[c] : 0.0;
    }
    double half = 0.0;
    if (j > 0) {
      double s = 0.0;
#pragma unroll
      for (int t = 0; t < kTriCols; ++t) s += py[t] * pv[t];
      for (int c = b0 + tid + 256 * kTriCols; c < n; c += 256) s += y[c] * v[c];
      half = 0.5 * tau * tau * block256_sum_f64(s, red[0]);
    }
    const double wj = tau * yj - half * vj;
    double sigma = 0.0;
    auto column = [&](const int c, const double vc, const double yc, const double xc) {
      const double wc = tau * yc - half * vc;
      const double x = xc - vj * wc - wj * vc;
      vo[c] = vc;
      wo[c] = wc;
      vn[c] = x;
      if (c > j + 1) sigma += x * x;
    };
#pragma unroll
    for (int t = 0; t < kTriCols; ++t)
      if (b0 + tid + 256 * t < np) column(b0 + tid + 256 * t, pv[t], py[t], px[t]);
    for (int c = b0 + tid + 256 * kTriCols; c < np; c += 256) {
      const bool in = c < n;
      column(c, in && j > 0 ? v[c] : 0.0, in && j > 0 ? y[c] : 0.0, in ? rowj[c] : 0.0);
    }
    sigma = block256_sum_f64(sigma, red[1]);   // also makes vn visible to all
    const Reflection h = reflection(vn[j + 1], sigma);
    const double dj = vn[j];
    __syncthreads();
    for (int c = b0 + tid; c < np; c += 256) vn[c] = c > j + 1 ? vn[c] * h.scale : (c == j + 1 ? 1.0 : 0.0);
    if (unit == 0 && tid == 0) {
      a.diag()[j] = dj;
      a.off()[j] = h.beta;
      a.tau()[j] = h.tau;
    }
    __syncthreads();
    if (unit == 0)
      for (int c = tid; c < np; c += 256) a.V[(size_t)j * np + c] = c > j ? vn[c] : 0.0;
  }
  if (!(phases & 2)) return;
  double acc[kTriRows], vr[kTriRows], wr[kTriRows];
#pragma unroll
  for (int q = 0; q < kTriRows; ++q) {
    acc[q] = 0.0;
    vr[q] = vo[min(row0 + q, n - 1)];
    wr[q] = wo[min(row0 + q, n - 1)];
  }
  for (int k0 = 0; k0 < chunks; k0 += kTriChunks) {
    if (k0 > 0) load(k0);
#pragma unroll
    for (int k = 0; k < kTriChunks; ++k) {
      if (k0 + k >= chunks) break;
      const int c = c0 + (k0 + k) * 64 + lane;
      const double vc = vo[c], wc = wo[c], xc = vn[c];
#pragma unroll
      for (int q = 0; q < kTriRows; ++q) {
        const double t = buf[q][k] - vr[q] * wc - wr[q] * vc;
        acc[q] += t * xc;
        if (row0 + q < n) rowp[q][(size_t)(k0 + k) * 64] = t;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kTriRows; ++q) {
    acc[q] = wave_sum_uniform(acc[q]);
    if (lane == 0 && row0 + q < n) a.y(j & 1)[row0 + q] = acc[q];
  }
}
__global__ __launch_bounds__(256) void init_tri_step_kernel(const InitGroup* __restrict__ gp, const int j, const int phases) {
  const InitArgs& a = gp->a[blockIdx.y];
  if (j >= a.n - kTriTail) return;   // uniform over the workgroup, as below
  if ((int)blockIdx.x >= (phases == 1 ? 1 : tri_step_units(a.n, j))) return;
  extern __shared__ double dyn_tri[];
  tri_step(a, j, phases, blockIdx.x, dyn_tri);
}

// The same columns in one launch: every workgroup keeps its rows in registers (CH 64-column chunks, ROWS rows per wavefront) and the
// workgroups of an instance exchange A v and the next row, element i of both from the workgroup of row i, through memory.
// The data are their own signal: a slot is empty (kRingEmpty) until its element is there, and the readers look at the slots themselves.
// Behind the one barrier of a column every wavefront forms w, the row and its reflection for itself; the product with the row
// does not wait for the reflection (A v = scale A x + column j + 1).
// A slot is emptied by its writer two columns later (all of the instance have then read it: the elements of the column between were
// sent behind that) and written again two columns after that; the wait for the counter of memory operations between makes the
// emptying visible before the writer's next elements, which a reader of the new ones has seen.
// Where all of an instance run on one die (matrices of up to 512 rows are dealt to the dies, the largest first to the one with the
// fewest workgroups, workgroup b to die b mod 8; the workgroups tell each
// other where they are before they start) ordinary stores do, which a reader behind the same L2 cache sees after 0.25 us; otherwise
// stores at device scope, 0.6 to 0.8 us.
// Progress: a workgroup first waits until all of its instance are running, for at most `limit` ticks.  If they are not, one closes the gate,
// all leave, and the kernel behind reduces the matrix from memory, as if a wait inside takes longer than kTriLost.  The matrix in memory
// stays as it was until then; the last 160 rows and columns go to the same places of V.
// Launches of several streams fill the chip together: an instance whose last workgroups are not placed yet waits for another one's
// reduction to end.
// Bound: the exchange and the chain of two sums over a wavefront.  One instance of 512 rows 2.07 us a column, the ten of a speech-shaped network 2.09 (with stores at
// device scope 3.9 us in the first version, 3.35 one alone; dealt in turn, two dies with two large ones, 2.5); 1024 rows 3.1 us.
constexpr int kTriResident = 1024;                    // largest padded size
constexpr int kTriDies = 8, kTriDieUnits = 2 * 32;    // workgroups of a die: two per compute unit
constexpr int kTriResidentUnits = kTriDies * kTriDieUnits;
constexpr long long kTriLost = 100000000;             // ticks (10 ns)
constexpr bool tri_on_one_die(const int np) { return np <= 512; }
constexpr int tri_resident_rows(const int np) { return np <= 512 ? 16 : 8; }   // rows of a workgroup
__host__ __device__ inline int tri_resident_units(const int n, const int rows) { return n > kTriTail ? (n + rows - 1) / rows : 0; }

// 0: not all are; 2: all on one die; 1 otherwise.
__device__ __forceinline__ int init_all_running(int* const gate, const int units, const long long limit) {
  if (limit == 0) {   // no time to wait
    __hip_atomic_fetch_or(gate, kGateClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 0;
  }
  const int die = __builtin_amdgcn_s_getreg(20 | (3 << 11));   // HW_REG_XCC_ID
  const int others = __hip_atomic_fetch_or(gate + 1, 1 << die, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" : : "v"(others) : "memory");   // it has been performed
  int seen = __hip_atomic_fetch_add(gate, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
  const long long t0 = wall_clock64();
  while (seen < units) {
    if (wall_clock64() - t0 >= limit) {   // closes the gate unless the last one came meanwhile
      if (__hip_atomic_compare_exchange_strong(gate, &seen, seen | kGateClosed, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        return 0;
      continue;
    }
    __builtin_amdgcn_s_sleep(16);
    seen = __hip_atomic_load(gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (seen >= kGateClosed) return 0;
  const int dies = __hip_atomic_load(gate + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (dies & (dies - 1)) == 0 ? 2 : 1;
}
__device__ __forceinline__ void ring_store(uint64_t* const p, const uint64_t v, const bool near) {
  if (near)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int CH, int ROWS>
__global__ __launch_bounds__(256, 2) void init_tri_resident_kernel(const InitGroup* __restrict__ gp, const int launch,
                                                                   const long long limit) {
  constexpr int C = 64 * CH, T = CH / 4;
  constexpr bool kDeal = tri_on_one_die(C);
  // the instance: those of this launch one after the other, or those of this launch and die
  const int bin = launch * kTriDies + (kDeal ? (int)blockIdx.x % kTriDies : 0), count = gp->count;
  int at = 0, unit = kDeal ? blockIdx.x / kTriDies : blockIdx.x, units = 0;
  for (; at < count; ++at) {
    if (gp->a[at].place != bin) continue;
    units = tri_resident_units(gp->a[at].n, 4 * ROWS);
    if (unit < units) break;
    unit -= units;
  }
  if (at >= count) return;
  const InitArgs& a = gp->a[at];
  const int n = a.n, np = a.np, end = n - kTriTail;
  __shared__ double sy[2][C], sx[2][C], sv[2][C];   // A v, the row and the reflection of the last column, alternately
  __shared__ int s_run, s_lost;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wg_row = unit * 4 * ROWS, row0 = wg_row + wave * ROWS;
  const bool last_wg = unit == units - 1;
  double S[ROWS][CH], v[CH];
#pragma unroll
  for (int k = 0; k < CH; ++k) {
    v[k] = 0.0;
#pragma unroll
    for (int q = 0; q < ROWS; ++q) S[q][k] = a.A[(size_t)min(row0 + q, n - 1) * np + min(64 * k, np - 64) + lane];
  }
#pragma unroll
  for (int k = 0; k < CH; ++k)
#pragma unroll
    for (int q = 0; q < ROWS; ++q) S[q][k] = 64 * k < np ? S[q][k] : 0.0;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int c = tid + 256 * t;
    sy[0][c] = sv[0][c] = 0.0;
    sx[0][c] = c < n ? a.A[c] : 0.0;
  }
  if (tid == 0) {
    s_lost = 0;
    s_run = init_all_running(a.gate(), units, limit);
  }
  __syncthreads();
  if (s_run == 0) return;
  const bool near = s_run == 2;
  // this lane's slots: rows row0 .. of A v, then of the next row
  const int mine = row0 + (lane & (ROWS - 1));
  const size_t place = (lane < ROWS ? 0 : (size_t)np) + mine;
  const bool sends = lane < 2 * ROWS && mine < n;
  double tau = 0.0;
  int stop = min(end, min(wg_row + 4 * ROWS, n) - 1);   // the columns left of the workgroup's last row
  // Columns of chunks F to G - 1: the chunks before are done.  (A branch per chunk waits for LDS in each: 2.9 us a column.)
  auto stage = [&](auto first_chunk) {
    constexpr int F = decltype(first_chunk)::value, G = F + CH / 4;
    for (int j = 64 * F; j < min(64 * G, stop); ++j) {
      const int par = j & 1;
      if (j > 0) {
        const uint64_t* const slot = reinterpret_cast<const uint64_t*>(a.ring(j - 1));
        uint64_t gy[T], gx[T];
        long long t0 = 0;
        for (int turn = 0;; ++turn) {
          bool empty = false;
#pragma unroll
          for (int t = 0; t < T; ++t) {
            const int c = max(min(tid + 256 * t, n - 1), j);
            gy[t] = __hip_atomic_load(slot + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            gx[t] = __hip_atomic_load(slot + np + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
#pragma unroll
          for (int t = 0; t < T; ++t) empty |= gy[t] == kRingEmpty || gx[t] == kRingEmpty;
          if (!empty) break;
          if ((turn & 63) == 63) {
            if (turn == 63) t0 = wall_clock64();
            if (wall_clock64() - t0 > kTriLost) {
              s_lost = 1;
              break;
            }
          }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const int c = tid + 256 * t;
          const bool in = c >= j && c < n;
          sy[par][c] = in ? __builtin_bit_cast(double, gy[t]) : 0.0;
          sx[par][c] = in ? __builtin_bit_cast(double, gx[t]) : 0.0;
        }
        __syncthreads();
      }
      const int lost = s_lost;
      asm volatile("s_waitcnt vmcnt(0)" : : : "memory");   // what was emptied a column ago is seen as empty
      if (j >= 2 && sends) ring_store(reinterpret_cast<uint64_t*>(a.ring(j - 2)) + place, kRingEmpty, near);
      double w[CH], x[CH], vr[ROWS], wr[ROWS], dot[2] = {0.0, 0.0};
#pragma unroll
      for (int k = F; k < CH; ++k) w[k] = sy[par][64 * k + lane];
#pragma unroll
      for (int k = F; k < CH; ++k) x[k] = sx[par][64 * k + lane];
#pragma unroll
      for (int q = 0; q < ROWS; ++q) {
        vr[q] = sv[par][min(row0 + q, n - 1)];
        wr[q] = sy[par][min(row0 + q, n - 1)];
      }
      const double vj = sv[par][j], yj = sy[par][j], xj = sx[par][j];
      const double vj1 = sv[par][j + 1], yj1 = sy[par][j + 1], xj1 = sx[par][j + 1];
#pragma unroll
      for (int k = F; k < CH; ++k) dot[k & 1] = fma(w[k], v[k], dot[k & 1]);
      const double half = 0.5 * tau * tau * wave_sum_f64(dot[0] + dot[1]);
      const double wj = fma(tau, yj, -half * vj), wj1 = fma(tau, yj1, -half * vj1);
      double sigma[2] = {0.0, 0.0};
#pragma unroll
      for (int k = F; k < CH; ++k) {
        w[k] = fma(tau, w[k], -half * v[k]);
        x[k] = fma(-wj, v[k], fma(-vj, w[k], x[k]));
        if (k <= G) x[k] = 64 * k + lane > j + 1 ? x[k] : 0.0;
        sigma[k & 1] = fma(x[k], x[k], sigma[k & 1]);
      }
      const double total = wave_sum_f64(sigma[0] + sigma[1]);
#pragma unroll
      for (int q = 0; q < ROWS; ++q) wr[q] = fma(tau, wr[q], -half * vr[q]);
      const double dj = fma(-wj, vj, fma(-vj, wj, xj));
      double acc[ROWS], next[ROWS];
#pragma unroll
      for (int q = 0; q < ROWS; ++q) acc[q] = next[q] = 0.0;
#pragma unroll
      for (int k = F; k < CH; ++k)
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
          S[q][k] = fma(-wr[q], v[k], fma(-vr[q], w[k], S[q][k]));
          acc[q] = fma(S[q][k], x[k], acc[q]);
        }
#pragma unroll
      for (int q = 0; q < ROWS; ++q) acc[q] = wave_sum_f64(acc[q]);
#pragma unroll
      for (int k = F; k <= min(G, CH - 1); ++k) {
        if (k != (j + 1) >> 6) continue;   // (uniform)
#pragma unroll
        for (int q = 0; q < ROWS; ++q) next[q] = read_lane_f64(S[q][k], (j + 1) & 63);
      }
      const Reflection h = reflection(fma(-wj, vj1, fma(-vj, wj1, xj1)), total);
      double send = 0.0;
#pragma unroll
      for (int q = 0; q < ROWS; ++q) {
        const double p = fma(h.scale, acc[q], next[q]);
        send = lane == q ? p : (lane == ROWS + q ? next[q] : send);
      }
      if (sends && mine > j) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, send);
        ring_store(reinterpret_cast<uint64_t*>(a.ring(j)) + place, bits == kRingEmpty ? 0x7ff8000000000000ULL : bits, near);
      }
      tau = h.tau;
#pragma unroll
      for (int k = F; k < CH; ++k) {
        v[k] = x[k] * h.scale;
        if (k <= G) v[k] = 64 * k + lane == j + 1 ? 1.0 : v[k];
        if (wave == 0) sv[par ^ 1][64 * k + lane] = v[k];
      }
      if (last_wg) {
#pragma unroll
        for (int k = 0; k < CH; ++k)
          if ((k & 3) == wave && 64 * k < np) a.V[(size_t)j * np + 64 * k + lane] = k >= F ? v[k] : 0.0;
        if (tid == 0) {
          a.diag()[j] = dj;
          a.off()[j] = h.beta;
          a.tau()[j] = h.tau;
        }
      }
      if (lost != 0) {   // (uniform) some elements never came
        if (tid == 0) __hip_atomic_fetch_or(a.gate(), kGateClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stop = 0;
      }
    }
  };
  stage(std::integral_constant<int, 0>());
  stage(std::integral_constant<int, CH / 4>());
  stage(std::integral_constant<int, CH / 2>());
  if constexpr (64 * CH - kTriTail > 48 * CH) stage(std::integral_constant<int, 3 * CH / 4>());
#pragma unroll
  for (int k = 0; k < CH; ++k)
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
      const int i = row0 + q, c = 64 * k + lane;
      if (i >= end && i < n && c >= end && c < n) a.V[(size_t)i * np + c] = S[q][k];
    }
}

// The same columns from memory, for the instances whose gate was closed: whatever workgroups are running take the units of
// init_tri_step_kernel's launches one after the other, column by column.  A unit begins when all of the columns before its own are
// done; the workgroups that hold those are running, so every wait ends, however few there are and whenever the others come.
// Order across the dies as at the boundaries of launches: a workgroup's stores are written back before its unit counts as done, what
// its die holds of the others' is dropped before it begins the next.
// Bound: that exchange, as for the launches: 512 rows 3.27 ms a call, 1024 rows 10.97 (a launch per column 3.37 and 10.2, rows kept
// on the chip 1.86 and 5.2).  By one workgroup a network's first factors of 1024 rows took 0.65 s.  With all gates open 4.5 us.
// All 13 of them and the smaller ones from memory: 44.8 ms a step that restarts, instead of 21.4 (launches 23.9).  With 32 workgroups for a matrix 36 ms,
// but one matrix of 1024 rows then 13.9; few go this way at a time.
// Grid (units, instance), 256 threads, 3 np doubles of LDS.
constexpr int kTriSharedUnits = 64;   // workgroups of an instance
__global__ __launch_bounds__(256) void init_tri_shared_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.y];
  const int n = a.n, end = n - kTriTail, tid = threadIdx.x;
  if (end <= 0 || *a.gate() < kGateClosed) return;
  extern __shared__ double dyn_tri[];
  __shared__ int s_unit;
  int j = 0, before = 0;   // units of the columns before j
  for (;;) {
    if (tid == 0) s_unit = __hip_atomic_fetch_add(a.gate() + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int unit = s_unit;
    for (; j < end && unit - before >= tri_step_units(n, j); ++j) before += tri_step_units(n, j);
    if (j >= end) return;   // (uniform)
    if (tid == 0) {
      while (__hip_atomic_load(a.gate() + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < before) __builtin_amdgcn_s_sleep(4);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    tri_step(a, j, 3, unit - before, dyn_tri);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");   // every wavefront's stores are in the die's L2 cache
    __syncthreads();
    if (tid == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_fetch_add(a.gate() + 3, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The last (at most 160) columns, the matrix in registers: 16 x 16 threads, thread (ti, tj) holds rows ti + 16 a and columns
// tj + 16 b as a 10 x 10 tile.  Two barriers per column: row j is
// published, every wavefront forms the reflection for itself; the products are published, every wavefront forms w for
// itself.  Row blocks that are done are skipped (a branch per element costs more than the finished columns).  Bound: fp64 multiply-adds, then the chain of two sums over
// the workgroup per column.  (1024 threads spend their time on the parts that every wavefront repeats: 2.7 us a column
// with 4 x 4 tiles of 128 columns, 3.9 us with 6 x 6 of 192; a 12 x 12 tile no longer fits into 256 registers: 2.8 us.)  Also divides T by N and scales it for the kernels that
// follow.  One workgroup of 256 threads per instance.
constexpr int kTriTile = kTriTail / 16;
__global__ __launch_bounds__(256) void init_tri_tail_kernel(const InitGroup* __restrict__ gp, const int resident) {
  const InitArgs& a = gp->a[blockIdx.x];
  constexpr int T = kTriTail, K = kTriTile;
  constexpr int TP = (T + 63) / 64 * 64;   // the vectors are padded with zeros for a wavefront's lanes
  static_assert(T % 16 == 0 && T <= 256, "tile and lane counts");
  __shared__ double srow[TP], sy[TP], scratch[16];
  __shared__ double sv[4][TP], sw[4][TP];   // every wavefront's own copy of v and w
  const int n = a.n, np = a.np, j0 = max(0, n - T), m = n - j0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ti = tid >> 4, tj = tid & 15;
  const double inv_n = 1.0 / (double)a.N;
  double* const v = sv[wave];
  double* const w = sw[wave];
  const bool kept = resident != 0 && j0 > 0 && *a.gate() < kGateClosed;   // (uniform) the columns before have left their rest in V
  const double* const from = kept ? a.V : a.A;
  double S[K][K];
#pragma unroll
  for (int x = 0; x < K; ++x)
#pragma unroll
    for (int b = 0; b < K; ++b) {
      const int i = ti + 16 * x, c = tj + 16 * b;
      S[x][b] = i < m && c < m ? from[(size_t)(j0 + i) * np + j0 + c] : 0.0;
    }
  // the last column that the other kernel took (none: a reflection with tau = 0)
  double tau = j0 > 0 ? a.tau()[j0 - 1] : 0.0;
  for (int c = lane; c < TP; c += 64) v[c] = j0 > 0 && c < T ? a.V[(size_t)(j0 - 1) * np + j0 + c] : 0.0;   // j0 > 0: all T columns exist
  if (tid < TP) srow[tid] = 0.0;
  if (tid < TP) sy[tid] = j0 > 0 && tid < T ? (kept ? a.ring(j0 - 1) : a.y((j0 - 1) & 1))[j0 + tid] : 0.0;
  for (int i = tid; i < j0; i += 256) {
    a.diag()[i] *= inv_n;
    a.off()[i] *= inv_n;
  }
  __syncthreads();
  for (int j = 0;; ++j) {
    // A <- A - v w^T - w v^T with the reflection of column j - 1, whose product A v is in sy
    {
      double yl[TP / 64], vl[TP / 64], dot = 0.0;
#pragma unroll
      for (int t = 0; t < TP / 64; ++t) {
        yl[t] = sy[lane + 64 * t];
        vl[t] = v[lane + 64 * t];
        dot = fma(yl[t], vl[t], dot);
      }
      const double half = 0.5 * tau * tau * wave_sum_uniform(dot);
#pragma unroll
      for (int t = 0; t < TP / 64; ++t) w[lane + 64 * t] = fma(tau, yl[t], -half * vl[t]);
    }
    wave_lds_exchange();   // w
    {
      double vc[K], wc[K];
#pragma unroll
      for (int b = 0; b < K; ++b) {
        vc[b] = v[tj + 16 * b];
        wc[b] = w[tj + 16 * b];
      }
#pragma unroll
      for (int x = 0; x < K; ++x) {
        if (16 * x + 15 < j) continue;   // uniform
        const double vr = v[ti + 16 * x], wr = w[ti + 16 * x];
#pragma unroll
        for (int b = 0; b < K; ++b) S[x][b] = fma(-vr, wc[b], fma(-wr, vc[b], S[x][b]));
        if (x == j >> 4 && ti == (j & 15)) {
#pragma unroll
          for (int b = 0; b < K; ++b) srow[tj + 16 * b] = S[x][b];
        }
      }
    }
    __syncthreads();
    if (tid == 0) a.diag()[j0 + j] = srow[j] * inv_n;
    if (j == m - 1) break;
    double xl[TP / 64], sigma = 0.0;
#pragma unroll
    for (int t = 0; t < TP / 64; ++t) {
      xl[t] = lane + 64 * t > j + 1 ? srow[lane + 64 * t] : 0.0;
      sigma = fma(xl[t], xl[t], sigma);
    }
    const Reflection h = reflection(srow[j + 1], wave_sum_uniform(sigma));
    tau = h.tau;
    if (tid == 0) {
      a.off()[j0 + j] = h.beta * inv_n;
      a.tau()[j0 + j] = h.tau;
    }
    double* const Vj = a.V + (size_t)(j0 + j) * np;
#pragma unroll
    for (int t = 0; t < TP / 64; ++t) {
      const int c = lane + 64 * t;
      xl[t] = c == j + 1 ? 1.0 : xl[t] * h.scale;
      v[c] = xl[t];
      if (wave == 0 && j0 + c < n) Vj[j0 + c] = xl[t];
    }
    for (int c = tid; c < np; c += 256)
      if (c < j0 || c >= n) Vj[c] = 0.0;
    wave_lds_exchange();   // v
    double vc[K], acc[K];
#pragma unroll
    for (int b = 0; b < K; ++b) vc[b] = v[tj + 16 * b];
#pragma unroll
    for (int x = 0; x < K; ++x) {
      acc[x] = 0.0;
      if (16 * x + 15 <= j) continue;
#pragma unroll
      for (int b = 0; b < K; ++b) acc[x] = fma(S[x][b], vc[b], acc[x]);
      acc[x] = row16_sum_f64(acc[x]);
    }
    if (tj == 0) {
#pragma unroll
      for (int x = 0; x < K; ++x) sy[ti + 16 * x] = ti + 16 * x > j ? acc[x] : 0.0;
    }
    __syncthreads();
  }
  if (tid == 0) a.off()[n - 1] = 0.0;
  __threadfence_block();
  __syncthreads();
  // interval that holds the eigenvalues (Gershgorin), and T scaled to unit norm; a squared off-diagonal of zero becomes
  // negligibly small instead, so that the Sturm sequences never stop at a zero
  double lo = 1.0e300, hi = -1.0e300;
  for (int i = tid; i < n; i += 256) {
    const double radius = (i > 0 ? fabs(a.off()[i - 1]) : 0.0) + fabs(a.off()[i]), d = a.diag()[i];
    lo = fmin(lo, d - radius);
    hi = fmax(hi, d + radius);
  }
  hi = block_max(hi, scratch);
  lo = -block_max(-lo, scratch);
  const double norm = fmax(fabs(lo), fabs(hi)), inv = norm > 0.0 ? 1.0 / norm : 0.0;
  for (int i = tid; i < n; i += 256) {
    const double e = a.off()[i] * inv;
    a.sdiag()[i] = a.diag()[i] * inv;
    a.soff2()[i] = fmax(e * e, 1.0e-60);
  }
  if (tid == 0) {
    a.bounds()[0] = lo;
    a.bounds()[1] = hi;
    a.bounds()[2] = norm;
  }
}

// Eigenvalue k (descending) of T: a wavefront counts the eigenvalues below 64 points of the interval at once, six bits
// a pass.  The count is the number of sign changes of the leading minors of T - x, by their three-term recurrence (one
// multiply-add on the critical path; with quotients instead, a reciprocal per step, 306 us for n = 512), rescaled every
// eight steps: a step changes their size by at most a factor of four upwards and far less than 2^-128 downwards.
// Grid (R, instance), 64 threads.
constexpr int kSectionPasses = 12;
__global__ __launch_bounds__(64) void init_eigenvalue_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.y];
  const int k = blockIdx.x, lane = threadIdx.x, n = a.n;
  if (k >= a.R) return;
  const double norm = a.bounds()[2], inv = norm > 0.0 ? 1.0 / norm : 0.0;
  const double margin = 2.0 * kInitEps * (double)n;
  double lo = a.bounds()[0] * inv - margin, hi = a.bounds()[1] * inv + margin;
  const double* __restrict__ d = a.sdiag();
  const double* __restrict__ e2 = a.soff2();
  for (int pass = 0; pass < kSectionPasses; ++pass) {
    const double width = hi - lo;
    if (!(width > 0.5 * kInitEps)) break;
    const double step = width / 65.0, x = lo + step * (double)(lane + 1);
    double p = d[0] - x, p1 = 1.0;
    uint32_t below = (uint32_t)(__builtin_bit_cast(uint64_t, p) >> 63);
    auto advance = [&](const int i) {
      const double q = fma(d[i] - x, p, -(e2[i - 1] * p1));
      below += (uint32_t)((__builtin_bit_cast(uint64_t, q) ^ __builtin_bit_cast(uint64_t, p)) >> 63);
      p1 = p;
      p = q;
    };
    int i = 1;
    for (; i + 8 <= n; i += 8) {
#pragma unroll
      for (int t = 0; t < 8; ++t) advance(i + t);
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p1)));
      p = __builtin_amdgcn_ldexp(p, ex);
      p1 = __builtin_amdgcn_ldexp(p1, ex);
    }
    for (; i < n; ++i) advance(i);
    const int m = __popcll(__ballot((int)below <= n - 1 - k));   // points at or below the eigenvalue
    const double base = lo;
    if (m > 0) lo = base + step * (double)m;
    if (m < 64) hi = base + step * (double)(m + 1);
  }
  if (lane == 0) a.lam()[k] = 0.5 * (lo + hi) * norm;
}

// Eigenvectors of T by inverse iteration: T - sigma = P L U with row exchanges once, then three solves from a random
// vector.  sigma lies 64 eps |T| above the eigenvalue: within a cluster of equal eigenvalues, which rounding spreads over
// a few eps |T|, every direction is then amplified alike and the vectors stay as independent as they started.  (With
// sigma on the eigenvalue itself those nearest to it win: of 80 vectors from the spectrum of one-hot rows the smallest
// eigenvalue of the Gram matrix came down to 1e-12 and at times to nothing; with the shift it is 1e-6 to 1e-3.)
// A thread per vector; everything is laid out with the vector index running fastest.
// Bound: the serial chains of n steps.  What they read does not depend on them, so every solve goes in blocks of eight
// steps whose operands are requested a block ahead (n = 512, ten instances: 900 us with plain loops in device memory,
// where every load waits behind the stores, 546 us in blocks, 270 us in blocks and LDS).
// Where a few vectors' factors fit into LDS (40 bytes per element) a workgroup takes `count` vectors there, otherwise 64 in
// device memory.  Grid (ceil(rq / count), instance), 64 threads.
constexpr int kInverseSolves = 3;
constexpr int kInverseLds = 150 * 1024, kInverseLdsMin = 4, kInverseLdsMax = 16;   // bytes; vectors of a workgroup
constexpr double kInverseShift = 64.0 * kInitEps;
constexpr int kInverseBlock = 8;
constexpr int kInversePad = 3 * kInverseBlock;   // blocks are requested whole, and one ahead
__host__ __device__ constexpr size_t inverse_lds_bytes(const int np) { return (5 * (size_t)(np + 2 * kInversePad) + 1) * sizeof(double); }
// Uniform in [-1, 1): an integer hash whose finisher (shifts and multipliers) is "lowbias32" of C. Wellons, "Prospecting for
// hash functions", 2018.
__device__ __forceinline__ double inverse_start(const int i, const int k) {
  uint32_t h = (uint32_t)i * 0x9E3779B9u ^ (uint32_t)(k + 1) * 0x85EBCA6Bu;
  h = (h ^ (h >> 16)) * 0x7FEB352Du;
  h = (h ^ (h >> 15)) * 0x846CA68Bu;
  h ^= h >> 16;
  return (double)(int32_t)h * (1.0 / 2147483648.0);
}
template <bool LDS>
__global__ __launch_bounds__(64) void init_eigenvector_kernel(const InitGroup* __restrict__ gp, const int count) {
  const InitArgs& a = gp->a[blockIdx.y];
  constexpr int B = kInverseBlock;
  extern __shared__ double dyn_inv[];
  const int k = blockIdx.x * count + threadIdx.x, n = a.n;
  if ((int)threadIdx.x >= count || k >= a.rq) return;
  const double norm = a.bounds()[2];
  const double lambda = k < a.R ? a.lam()[k] : 0.0;
  if (!(k < a.R && lambda > kNullEigRatio * a.lam()[0] && norm > 0.0)) {
    for (int i = 0; i < n; ++i) a.X[(size_t)i * a.rq + k] = 0.0;
    return;
  }
  // In LDS a vector's factors are contiguous, kInversePad elements around each of the five rows, and the vectors an odd
  // number of doubles apart; in device memory the vector index runs fastest.
  const int rq = LDS ? 1 : a.rq;   // stride of an element
  const size_t plane = LDS ? (size_t)(a.np + 2 * kInversePad) : (size_t)a.np * rq;
  double* const __restrict__ r0 = LDS ? dyn_inv + threadIdx.x * (5 * plane + 1) + kInversePad : a.A + k;   // 1 / diagonal of U, its two superdiagonals,
  double* const __restrict__ u1 = r0 + plane;                               // multipliers of L (lowest bit: rows exchanged)
  double* const __restrict__ u2 = r0 + 2 * plane;
  double* const __restrict__ ml = r0 + 3 * plane;
  double* const __restrict__ X = LDS ? r0 + 4 * plane : a.X + k;
  const double* __restrict__ d = a.diag();
  const double* __restrict__ e = a.off();
  const double tiny = kInitEps * norm, sigma = lambda + kInverseShift * norm;
  {
    double p = d[0] - sigma, b = e[0];
#pragma unroll 4
    for (int i = 0; i < n - 1; ++i) {
      const double s = e[i], dn = d[i + 1] - sigma, en = e[i + 1];
      const bool swap = fabs(p) < fabs(s);
      double piv = swap ? s : p;
      if (fabs(piv) < tiny) piv = piv < 0.0 ? -tiny : tiny;
      const double inv = reciprocal_f64(piv);
      const double l = (swap ? p : s) * inv;
      const double x1 = swap ? dn : b, x2 = swap ? en : 0.0;
      const size_t at = (size_t)i * rq;
      r0[at] = inv;
      u1[at] = x1;
      u2[at] = x2;
      ml[at] = __builtin_bit_cast(double, (__builtin_bit_cast(uint64_t, l) & ~1ull) | (swap ? 1ull : 0ull));
      p = swap ? fma(-l, dn, b) : fma(-l, b, dn);
      b = swap ? -l * en : en;
    }
    if (fabs(p) < tiny) p = p < 0.0 ? -tiny : tiny;
    r0[(size_t)(n - 1) * rq] = reciprocal_f64(p);
    u1[(size_t)(n - 1) * rq] = u2[(size_t)(n - 1) * rq] = 0.0;
  }
  double scale = 1.0;
  for (int it = 0; it < kInverseSolves; ++it) {
    if (it > 0) {   // L y = P x, in place: step i takes x_{i+1} and leaves y_i
      double bl[2][B], bx[2][B];
      auto fetch = [&](const int i0, const int set) {   // steps beyond n - 2 are read from it and not taken
#pragma unroll
        for (int t = 0; t < B; ++t) {
          const size_t at = (size_t)(LDS ? i0 + t : min(i0 + t, n - 2)) * rq;
          bl[set][t] = ml[at];
          bx[set][t] = X[at + rq];
        }
      };
      double cur = X[0] * scale;
      auto steps = [&](const int i0, const int set) {
#pragma unroll
        for (int t = 0; t < B; ++t) {
          if (i0 + t >= n - 1) break;
          const double l = bl[set][t], nxt = bx[set][t] * scale;
          const bool swap = (__builtin_bit_cast(uint64_t, l) & 1ull) != 0;
          X[(size_t)(i0 + t) * rq] = swap ? nxt : cur;
          cur = swap ? fma(-l, nxt, cur) : fma(-l, cur, nxt);
        }
      };
      fetch(0, 0);
      for (int i0 = 0; i0 < n - 1; i0 += 2 * B) {   // a block writes elements below those that the next one reads
        fetch(i0 + B, 1);
        steps(i0, 0);
        fetch(i0 + 2 * B, 0);
        steps(i0 + B, 1);
      }
      X[(size_t)(n - 1) * rq] = cur;
    }
    double x1 = 0.0, x2 = 0.0, ss = 0.0;
    double b0[2][B], b1[2][B], b2[2][B], by[2][B];
    auto fetch = [&](const int i0, const int set) {   // rows i0, i0 - 1, ...; those below 0 are read from row 0 and not taken
#pragma unroll
      for (int t = 0; t < B; ++t) {
        const int i = LDS ? i0 - t : max(i0 - t, 0);
        const ptrdiff_t at = (ptrdiff_t)i * rq;
        b0[set][t] = r0[at];
        b1[set][t] = u1[at];
        b2[set][t] = u2[at];
        by[set][t] = it > 0 ? X[at] : inverse_start(i, k);
      }
    };
    auto steps = [&](const int i0, const int set) {   // U x = y
#pragma unroll
      for (int t = 0; t < B; ++t) {
        if (i0 - t < 0) break;
        const double x = fma(-b1[set][t], x1, fma(-b2[set][t], x2, by[set][t])) * b0[set][t];
        X[(size_t)(i0 - t) * rq] = x;
        ss = fma(x, x, ss);
        x2 = x1;
        x1 = x;
      }
    };
    fetch(n - 1, 0);
    for (int i0 = n - 1; i0 >= 0; i0 -= 2 * B) {
      fetch(i0 - B, 1);
      steps(i0, 0);
      fetch(i0 - 2 * B, 0);
      steps(i0 - B, 1);
    }
    scale = 1.0 / sqrt(ss);
  }
#pragma unroll 8
  for (int i = 0; i < n; ++i) a.X[(size_t)i * a.rq + k] = X[(size_t)i * rq] * scale;
}

// G = X^T X, a 16 x 16 tile per workgroup of four wavefronts.  Grid (rq/16, rq/16, instance).
// v_mfma_f64_16x16x4_f64: lane l supplies A[l%16][l/16] and B[l/16][l%16]; register r holds row 4r + l/16, column l%16.
// `second`: X is what the first orthonormalisation left.
__device__ __forceinline__ double* init_ortho_input(const InitArgs& a, const int second) {
  return second ? a.A + (size_t)a.np * a.rq : a.X;   // behind the place of the final vectors
}
__global__ __launch_bounds__(256) void init_ortho_gram_kernel(const InitGroup* __restrict__ gp, const int second) {
  const InitArgs& a = gp->a[blockIdx.z];
  const int rq = a.rq, a0 = blockIdx.y * 16, b0 = blockIdx.x * 16;
  if (a0 >= rq || b0 >= rq) return;
  typedef double doublex4 __attribute__((ext_vector_type(4)));
  __shared__ double part[4][256];
  const double* __restrict__ X = init_ortho_input(a, second);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  doublex4 acc = {0, 0, 0, 0};
  for (int i0 = wave * 4; i0 < a.n; i0 += 16) {
    const int i = i0 + g4;
    const double x = i < a.n ? X[(size_t)i * rq + a0 + l16] : 0.0, y = i < a.n ? X[(size_t)i * rq + b0 + l16] : 0.0;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) part[wave][(4 * r + g4) * 16 + l16] = acc[r];
  __syncthreads();
  const int t = threadIdx.x;
  a.G()[(size_t)(a0 + (t >> 4)) * rq + b0 + (t & 15)] = (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]);
}

// G = L L^T replaced by L^-1: elimination without pivoting of [G | I], the right half growing in the columns that become
// zero, one barrier per pivot.  A null vector (zero row) is left out.  One workgroup of 1024 threads per instance.
__global__ __launch_bounds__(1024) void init_ortho_factor_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.x];
  __shared__ double S[kMaxRank][kMaxRank + 8];
  __shared__ double s_piv[kMaxRank];
  const int rq = a.rq, tid = threadIdx.x, r = tid >> 3, q8 = tid & 7;   // eight threads per row (all in one wavefront)
  for (int e = tid; e < rq * rq; e += 1024) S[e / rq][e % rq] = a.G()[e];
  __syncthreads();
  for (int k = 0; k < rq; ++k) {
    const double piv = S[k][k];
    const double inv = piv > 1.0e-30 ? reciprocal_f64(piv) : 0.0;
    if (tid == 0) s_piv[k] = inv;
    if (r > k && r < rq) {
      const double f = S[r][k] * inv;
#pragma unroll 4
      for (int c = q8; c < rq; c += 8) {
        const double s = S[r][c] - f * S[k][c];
        S[r][c] = c == k ? -f : s;
      }
    }
    __syncthreads();
  }
  for (int e = tid; e < rq * rq; e += 1024) {
    const int i = e / rq, c = e % rq;
    a.G()[e] = sqrt(s_piv[i]) * (c < i ? S[i][c] : (c == i ? 1.0 : 0.0));
  }
}

// X L^-T: first to the input of the second pass, then transposed to its place (rq x np, zero beyond n).
// Grid (np/64, instance), 256 threads: a wavefront owns 16 rows of X.
__global__ __launch_bounds__(256) void init_ortho_apply_kernel(const InitGroup* __restrict__ gp, const int second) {
  const InitArgs& a = gp->a[blockIdx.y];
  const int rq = a.rq, n = a.n, np = a.np;
  if ((int)blockIdx.x * 64 >= np) return;
  typedef double doublex4 __attribute__((ext_vector_type(4)));
  const double* __restrict__ X = init_ortho_input(a, second);
  double* __restrict__ out = second ? a.A : init_ortho_input(a, 1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int i0 = blockIdx.x * 64 + wave * 16;
  for (int b0 = 0; b0 < rq; b0 += 16) {
    doublex4 acc = {0, 0, 0, 0};
#pragma unroll 4
    for (int k0 = 0; k0 < b0 + 16; k0 += 4) {   // L^-1 is lower triangular
      const double x = i0 + l16 < n ? X[(size_t)(i0 + l16) * rq + k0 + g4] : 0.0;
      const double l = a.G()[(size_t)(b0 + l16) * rq + k0 + g4];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, l, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 4 * r + g4, k = b0 + l16;
      out[second ? (size_t)k * np + i : (size_t)i * rq + k] = acc[r];
    }
  }
}

// Inner products between the reflections of four neighbouring columns, 4 m + p with 4 m + q, p < q, in the order 01 02 03 12 13 23, for
// the back transformation; to X, which is free by then.  A wavefront per four.  Grid (ceil(n / 16), instance), 256 threads.
__global__ __launch_bounds__(256) void init_back_products_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.y];
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, n = a.n, np = a.np;
  if (4 * m > n - 2) return;
  const double* V[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) V[p] = a.V + (size_t)min(4 * m + p, n - 2) * np;
  double g[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int c = (4 * m & ~63) + lane; c < np; c += 64) {
    const double v0 = V[0][c], v1 = V[1][c], v2 = V[2][c], v3 = V[3][c];
    g[0] = fma(v0, v1, g[0]);
    g[1] = fma(v0, v2, g[1]);
    g[2] = fma(v0, v3, g[2]);
    g[3] = fma(v1, v2, g[3]);
    g[4] = fma(v1, v3, g[4]);
    g[5] = fma(v2, v3, g[5]);
  }
#pragma unroll
  for (int p = 0; p < 6; ++p) g[p] = wave_sum_f64(g[p]);
#pragma unroll
  for (int p = 0; p < 6; ++p)
    if (lane == p) a.X[6 * m + p] = g[p];
}

// Eigenvectors of T -> of A: the reflections, last to first, on a vector per wavefront, which it holds in registers
// (NC 64-element chunks).  B reflections at a time: their inner products with the vector as it is, corrected by the ones before through
// the products between them, so that a chain of two sums serves B; those of the next two blocks are on their way.  Only the
// loads leave out chunks where a reflection is zero: a branch around work waits for loads in each chunk.
// n = 512: 148 us and 5 for the products, one reflection at a time 278 (n = 1024, two at a time: 533 and 807; three blocks in flight 173,
// all chunks without a branch 150 and 642).  Grid (ceil(R/4), instance), 256 threads.
template <int NC, int B>
__device__ __forceinline__ void init_back_registers(const InitArgs& a, double* __restrict__ xk, const int lane) {
  static_assert(B == 2 || B == 4, "pairs within the products of four");
  const int n = a.n, np = a.np;
  const double* __restrict__ V = a.V + lane;
  const double* __restrict__ tau = a.tau();
  const double* __restrict__ products = a.X;
  double x[NC], v[2][B][NC], f[2][B], g[2][6];
#pragma unroll
  for (int c = 0; c < NC; ++c) x[c] = 64 * c < np ? xk[64 * c + lane] : 0.0;
  auto fetch = [&](const int m, const int set) {   // reflections B m .. B m + B - 1; beyond the last one tau is zero
    if (m < 0) return;
#pragma unroll
    for (int p = 0; p < B; ++p) {
      const int j = min(B * m + p, n - 2);
      f[set][p] = B * m + p <= n - 2 ? tau[j] : 0.0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        v[set][p][c] = 0.0;
        if (64 * c < np && 64 * c + 63 > j) v[set][p][c] = V[(size_t)j * np + 64 * c];
      }
    }
#pragma unroll
    for (int p = 0; p < (B == 4 ? 6 : 1); ++p) g[set][p] = products[B == 4 ? 6 * m + p : 6 * (m >> 1) + 5 * (m & 1)];
  };
  auto step = [&](const int m, const int set) {
    if (m < 0) return;
    double dot[B];
#pragma unroll
    for (int p = 0; p < B; ++p) dot[p] = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int p = 0; p < B; ++p) dot[p] = fma(v[set][p][c], x[c], dot[p]);
#pragma unroll
    for (int p = 0; p < B; ++p) dot[p] = wave_sum_f64(dot[p]);
    double* const t = f[set];
    if constexpr (B == 4) {
      const double* const q = g[set];
      t[3] *= dot[3];
      t[2] *= fma(-t[3], q[5], dot[2]);
      t[1] *= fma(-t[2], q[3], fma(-t[3], q[4], dot[1]));
      t[0] *= fma(-t[1], q[0], fma(-t[2], q[1], fma(-t[3], q[2], dot[0])));
    } else {
      t[1] *= dot[1];
      t[0] *= fma(-t[1], g[set][0], dot[0]);
    }
#pragma unroll
    for (int p = B - 1; p >= 0; --p)
#pragma unroll
      for (int c = 0; c < NC; ++c) x[c] = fma(-t[p], v[set][p][c], x[c]);
  };
  int m = (n - 2) / B;   // n = 1: nothing
  if (n < 2) return;
  fetch(m, 0);
  fetch(m - 1, 1);
  for (; m >= 0; m -= 2) {
    step(m, 0);
    fetch(m - 2, 0);
    step(m - 1, 1);
    fetch(m - 3, 1);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (64 * c < np) xk[64 * c + lane] = x[c];
}
__global__ __launch_bounds__(256) void init_back_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.y];
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, n = a.n, np = a.np;
  if (k >= a.R) return;
  double* const x = a.A + (size_t)k * np;
  if (np <= 128) {
    init_back_registers<2, 4>(a, x, lane);
  } else if (np <= 256) {
    init_back_registers<4, 4>(a, x, lane);
  } else if (np <= 512) {
    init_back_registers<8, 4>(a, x, lane);
  } else if (np <= 1024) {
    init_back_registers<16, 2>(a, x, lane);
  } else {
    for (int j = n - 2; j >= 0; --j) {   // a lane reads and writes only its own elements of x
      const double* const v = a.V + (size_t)j * np;
      double dot = 0.0;
      for (int c = (j & ~63) + lane; c < np; c += 64) dot = fma(v[c], x[c], dot);
      dot = a.tau()[j] * wave_sum_uniform(dot);
      for (int c = (j & ~63) + lane; c < np; c += 64) x[c] = fma(-dot, v[c], x[c]);
    }
  }
}

// rho_0, D_0, E_0 from the top-R eigenvalues (App. B.3.2 with eq. beta2, etii).  One workgroup per instance.
__global__ __launch_bounds__(256) void init_select_kernel(const InitGroup* __restrict__ gp) {
  __shared__ double scratch[16];
  const InitArgs& a = gp->a[blockIdx.x];
  const int n = a.n, R = a.R, D = a.D, k = threadIdx.x;
  static_assert(kMaxRank <= 256, "a thread per eigenvalue");
  PrecondScalars* st = a.st;
  double tr = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) tr += a.diag()[i];
  tr = block_sum(tr, scratch);
  const double lmax = a.lam()[0];
  const double l = k < R ? a.lam()[k] : 0.0;
  const bool keep = lmax > 0.0 && l > kNullEigRatio * lmax;
  const double sum_l = block_sum(keep ? l : 0.0, scratch);
  const double rho0 = fmax((tr - sum_l) / (double)(D - R), gp->epsilon);
  const double d = fmax(gp->epsilon, (keep ? l : 0.0) - rho0);
  const double sum_d = block_sum(k < R ? d : 0.0, scratch);
  const double beta = rho0 * (1.0 + gp->alpha) + gp->alpha / (double)D * sum_d;
  if (k < R) {
    a.idx[k] = keep ? k : -1;
    a.vwork[k] = keep ? l : 0.0;   // for the Gram route's 1 / sqrt(N lambda)
    st->d[k] = d;
    st->e[k] = 1.0 / (beta / d + 1.0);
  }
  if (k == 0) {
    st->rho = rho0;
    st->beta = beta;
    st->trace_S0 = tr;
    st->flags = 0;
    st->sweeps = 0;   // nothing iterates here
  }
}

// W_0 rows of the kept eigenpairs: sqrt(e_i) v_i with v_i an eigenvector (covariance route) or X_0^T u_i / sqrt(N lambda_i)
// (Gram route, on the fp64 matrix unit); zero for null directions.  A workgroup forms all rows for 64 columns, 16 per
// wavefront, so that X_0 is read once; the vectors go through LDS in blocks of 32 elements.
// Grid (64-column blocks, instance), 256 threads.
constexpr int kInitRowsK = 32;
template <int TR>   // 16-row tiles
__device__ __forceinline__ void init_rows_block(const InitArgs& a, double* sU) {
  typedef double doublex4 __attribute__((ext_vector_type(4)));
  constexpr int LD = kInitRowsK + 2;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int col = blockIdx.x * 64 + (tid >> 6) * 16 + l16;
  const int np = a.np, R = a.R;
  doublex4 acc[TR];   // register r: row 4 r + lane / 16 of a tile, column lane % 16
#pragma unroll
  for (int t = 0; t < TR; ++t) acc[t] = doublex4{0, 0, 0, 0};
  if (a.use_cov) {
#pragma unroll
    for (int t = 0; t < TR; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * t + 4 * r + g4;
        if (i < R && col < a.D) acc[t][r] = a.A[(size_t)i * np + col];
      }
  } else {
    const float* __restrict__ m = a.M + min(col, a.D - 1);   // columns beyond D reach no row that is stored
    float x[kInitRowsK / 4];
    auto fetch = [&](const int r0) {
#pragma unroll
      for (int ks = 0; ks < kInitRowsK / 4; ++ks) x[ks] = m[(size_t)min(r0 + 4 * ks + g4, a.N - 1) * a.ld];
    };
    fetch(0);
    for (int r0 = 0; r0 < a.N; r0 += kInitRowsK) {
      __syncthreads();
      for (int e = tid; e < 16 * TR * kInitRowsK; e += 256) {
        const int r = e % kInitRowsK, i = e / kInitRowsK;
        sU[i * LD + r] = i < R && r0 + r < a.N ? a.A[(size_t)i * np + r0 + r] : 0.0;
      }
      __syncthreads();
      float cur[kInitRowsK / 4];
#pragma unroll
      for (int ks = 0; ks < kInitRowsK / 4; ++ks) cur[ks] = x[ks];
      if (r0 + kInitRowsK < a.N) fetch(r0 + kInitRowsK);
#pragma unroll
      for (int ks = 0; ks < kInitRowsK / 4; ++ks)
#pragma unroll
        for (int t = 0; t < TR; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(sU[(16 * t + l16) * LD + 4 * ks + g4], (double)cur[ks], acc[t], 0, 0, 0);
    }
  }
  if (col >= a.ldw) return;
#pragma unroll
  for (int t = 0; t < TR; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * t + 4 * r + g4;
      if (i >= R) continue;
      double v = 0.0;
      if (a.idx[i] >= 0 && col < a.D) {
        double scale = sqrt(a.st->e[i]);
        if (!a.use_cov) scale /= sqrt((double)a.N * a.vwork[i]);
        v = acc[t][r] * scale;
      }
      a.W[(size_t)i * a.ldw + col] = (float)v;
    }
}
__global__ __launch_bounds__(256) void init_rows_kernel(const InitGroup* __restrict__ gp) {
  const InitArgs& a = gp->a[blockIdx.y];
  if ((int)blockIdx.x * 64 >= a.ldw) return;
  __shared__ double sU[kMaxRank * (kInitRowsK + 2)];
  if (a.R <= 32) {
    init_rows_block<2>(a, sU);
  } else {
    init_rows_block<kMaxRank / 16>(a, sU);
  }
}

// Rows of R_0 for null directions: Gram-Schmidt completion from the standard basis e_0, e_1, ... (each
// candidate orthogonalised twice against all rows fixed so far, accepted when its residual exceeds 0.1).
// One workgroup per instance; returns at once when every direction was kept.  A pass takes all its inner
// products against the same vector (every wavefront a share of the fixed rows) and then subtracts them together.
__global__ __launch_bounds__(1024) void init_complete_kernel(const InitGroup* __restrict__ gp) {
  __shared__ double scratch[16];
  __shared__ int s_fixed[kMaxRank];
  __shared__ double s_dot[kMaxRank], s_inv[kMaxRank];
  __shared__ int s_nfixed, s_missing;
  const InitArgs& a = gp->a[blockIdx.x];
  const int R = a.R, D = a.D, ldw = a.ldw;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  if (tid == 0) {
    int nf = 0, miss = 0;
    for (int k = 0; k < R; ++k) {
      if (a.idx[k] >= 0) s_fixed[nf++] = k; else ++miss;
    }
    s_nfixed = nf;
    s_missing = miss;
  }
  __syncthreads();
  if (s_missing == 0) return;
  double* v = a.vwork + kMaxRank;   // first kMaxRank entries hold the eigenvalues
  float* W = a.W;
  const PrecondScalars* st = a.st;
  for (int k = tid; k < R; k += nt) s_inv[k] = 1.0 / sqrt(st->e[k]);   // rows of W are sqrt(e) times rows of R_0
  __syncthreads();
  int cand = 0;
  for (int i = 0; i < R; ++i) {
    if (a.idx[i] >= 0) continue;    // uniform
    bool accepted = false;
    while (!accepted && cand < D) {
      for (int c = tid; c < D; c += nt) v[c] = c == cand ? 1.0 : 0.0;
      ++cand;
      __syncthreads();
      const int nf = s_nfixed;
      for (int pass = 0; pass < 2; ++pass) {
        for (int f = wave; f < nf; f += nw) {
          const int j = s_fixed[f];
          const float* wj = W + (size_t)j * ldw;
          double dot = 0.0;
          for (int c = lane; c < D; c += 64) dot += (double)wj[c] * v[c];
          dot = wave_sum(dot);
          if (lane == 0) s_dot[f] = dot * s_inv[j];
        }
        __syncthreads();
        for (int c = tid; c < D; c += nt) {
          double x = v[c];
          for (int f = 0; f < nf; ++f) {
            const int j = s_fixed[f];
            x -= s_dot[f] * (double)W[(size_t)j * ldw + c] * s_inv[j];
          }
          v[c] = x;
        }
        __syncthreads();
      }
      double nrm = 0.0;
      for (int c = tid; c < D; c += nt) nrm += v[c] * v[c];
      nrm = sqrt(block_sum(nrm, scratch));
      if (nrm > kCompletionMinResidual) {
        const double s = sqrt(st->e[i]) / nrm;
        for (int c = tid; c < ldw; c += nt) W[(size_t)i * ldw + c] = c < D ? (float)(s * v[c]) : 0.f;
        __syncthreads();
        if (tid == 0) s_fixed[s_nfixed++] = i;
        __syncthreads();
        accepted = true;
      }
    }
  }
}

}  // namespace ngsgd
