// The R x R part of the online natural-gradient update, entirely on the device (App. B.3, B.3.1).
//
// Z_t is formed from K_t and L_t (eq. zt:compute) and its eigenpairs come from the direct method of eig_direct.h, in one
// kernel up to rank 32 and in three above (reduction, a workgroup per instance; eigenpairs, four per workgroup; the rest).
// The finishing kernel floors the eigenvalues and produces rho_{t+1}, D_{t+1}, E_{t+1} and A_t (eq. wt1).  Where the direct
// method's checks fail it runs cyclic Jacobi first: only Z is rotated, its upper triangle in LDS in "position space"
// (Brent-Luk: the members of pair k stand at positions 2k and 2k+1, and a fixed permutation between rounds brings the
// next partners together), in two copies used alternately, so a round costs one barrier; the eigenvectors' rows go through
// the rotations in registers.
// orth_fix_kernel: the orthogonality check of App. B.3.1 and, when it fails, the Cholesky fix folded into A_t.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "eig_direct.h"
#include "gemm.h"
#include "kernels.h"
#include "state.h"
#include "wave_f64.h"

namespace ngsgd {

constexpr int kSmallThreads = 1024;          // orthogonality fix kernel
constexpr int kEigThreads = 1024;            // finishing kernel of the R x R update above rank 32
constexpr int kEigReduceThreads = 256;
// Up to here one kernel does it all: its 32 rows of lanes take all eigenpairs at once.  Update of a 512 x 3001 matrix: rank 20
// 94 us with one kernel, 100 with three; rank 32 106 and 113.  (Above, the pairs of one workgroup would come in turns.)
constexpr int kEigSmallRank = 32;
constexpr int kEigSmallThreads = 512;
constexpr int kMaxSweeps = 20;
constexpr int kMaxHalf = kMaxRank / 2;
constexpr double kJacobiTol = 1.0e-13;       // a pair is left alone once |z_pq| <= tol * sqrt(z_pp z_qq)
constexpr double kJacobiAbsTol = 1.0e-13;    // ... or once |z_pq| <= this * max_i z_ii (rounding noise level)
constexpr double kJacobiLargeTol = 1.0e-6;   // a sweep without a rotated entry above this (same measure) ...
constexpr double kJacobiLargeAbs = 1.0e3;    // ... and above this many absolute thresholds is the last
constexpr double kOrthoCondLimit = 1.0e6;    // App. B.3.1
constexpr double kOrthoTolerance = 1.0e-3;   // App. B.3.1

constexpr size_t direct_scratch_doubles(const int R) { return (size_t)R * (2 * kMaxRank + 7) + 2; }
struct SmallArgs {
  PrecondScalars* st;
  double* K;         // R x R, J J^T; cleared on exit (the orthogonality check accumulates W W^T into it)
  const double* L;   // R x R, H^T H
  float* At;         // out: A_t (eq. wt1), R x ldat
  int ldat;
  int R, D, N;
  float* bt;                  // out: R factors of W_t's rows in B_t
  const double* sumsq_part;   // partial sums of tr(X X^T) left by the H product
  int n_sumsq;
  // What the kernels of the direct method hand on: R rows of `ldv` doubles of reflections and of eigenvectors, seven vectors, rho_t; and
  // how many workgroups have left K alone.
  double* direct;
  __device__ double* V() const { return direct; }
  __device__ double* U(const int ldv) const { return direct + (size_t)R * ldv; }
  __device__ double* vec(const int ldv, const int which) const { return direct + (size_t)R * (2 * ldv + which); }
  __device__ double* tau(const int ldv) const { return vec(ldv, 0); }
  __device__ double* diag(const int ldv) const { return vec(ldv, 1); }
  __device__ double* off(const int ldv) const { return vec(ldv, 2); }
  __device__ double* lambda(const int ldv) const { return vec(ldv, 3); }
  __device__ double* residual(const int ldv) const { return vec(ldv, 4); }
  __device__ double* order(const int ldv) const { return vec(ldv, 5); }
  __device__ double* d_rho(const int ldv) const { return vec(ldv, 6); }   // diag(D_t), then rho_t
  __device__ int* k_tickets(const int ldv) const { return reinterpret_cast<int*>(d_rho(ldv) + R + 1); }
};
struct SmallGroup {
  int count;
  double alpha, epsilon, num_samples_history;
  SmallArgs a[kMaxInstances];
};

// Coupled Newton (Goldschmidt) iteration from the hardware estimate: on return g = sqrt(x), h = 1 / (2 sqrt(x)).
// Two dependent operations per step instead of the three of the plain Newton step for 1/sqrt.
__device__ __forceinline__ void sqrt_pair(double x, double& g, double& h) {
  const double y = __builtin_amdgcn_rsq(x);
  g = x * y;
  h = 0.5 * y;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
  }
}

// Rotation that diagonalises [[app, apq], [apq, aqq]] as J^T A J with J = [[c, s], [-s, c]] (the inner rotation,
// c >= 1/sqrt 2).  Returns false (and the identity) when the off-diagonal entry is already negligible: relative
// to the diagonal pair (that relative test is what gives small eigenvalues of a graded positive definite matrix
// their relative accuracy) or in absolute terms (abs_tol2 is the squared absolute threshold).  `large` reports
// whether the entry was above kJacobiLargeTol relative to the pair and well above the absolute noise threshold:
// Jacobi converges quadratically, so a sweep whose rotations were all smaller than that leaves entries of the order
// of their square and needs no further sweep.  With
// h = (aqq - app) / 2 and r = sqrt(h^2 + apq^2):  c^2 = (1 + |h| / r) / 2,  s = sign(h) apq / (2 r c).  Written
// this way the rotation costs two reciprocal square roots in sequence and no division: it sits on the critical
// path of every round.
__device__ __forceinline__ bool jacobi_rotation(double app, double aqq, double apq, double abs_tol2, double& c,
                                                double& s, bool& large) {
  c = 1.0;
  s = 0.0;
  large = false;
  const double apq2 = apq * apq, scale2 = fabs(app * aqq);
  if (!(apq2 > kJacobiTol * kJacobiTol * scale2) || !(apq2 > abs_tol2) || !(apq2 > 1.0e-290)) return false;
  large = apq2 > kJacobiLargeTol * kJacobiLargeTol * scale2 && apq2 > kJacobiLargeAbs * kJacobiLargeAbs * abs_tol2;
  const double h = 0.5 * (aqq - app);
  double r, half_rinv, half_cinv;
  sqrt_pair(fma(h, h, apq2), r, half_rinv);
  const double sa = (h >= 0.0 ? apq : -apq) * half_rinv;   // sign(h) apq / (2 r)
  sqrt_pair(fma(fabs(h), half_rinv, 0.5), c, half_cinv);
  s = sa * (half_cinv + half_cinv);
  return true;
}

// The Jacobi iteration works in "position space" (Brent-Luk): position 2k is the first and 2k+1 the second
// member of pair k, rotations always act on (2k, 2k+1), and after every round the matrix is permuted so that the
// next round's partners sit together again.  The permutation is the same every round,
//   first_k -> first_{k-1} (k >= 1),  first_0 -> second_1,  second_k -> second_{k+1} (1 <= k < half-1),
//   second_{half-1} -> first_{half-1},  second_0 stays,
// which is the circle method of a round-robin tournament with `second_0` as the fixed player: over m-1 rounds
// every two players meet once.  Because it is fixed, every thread reads and writes the same LDS addresses in
// every round and needs no index arithmetic in the loop.
__device__ __forceinline__ int next_position(int pos, int half) {
  if (half == 1) return pos;
  const int k = pos >> 1;
  if ((pos & 1) == 0) return k >= 1 ? 2 * (k - 1) : 3;          // first members
  if (k == 0) return 1;                                          // the fixed player
  return k == half - 1 ? 2 * (half - 1) : 2 * (k + 1) + 1;       // second members
}
// Player standing at `pos` after `rounds` rounds; players m-1-k start as second members, m-1 is the fixed one.
__device__ __forceinline__ int player_at(int pos, int rounds, int m) {
  const int k = pos >> 1;
  if (m == 2) return pos;
  const int r = rounds % (m - 1);
  if ((pos & 1) == 0) return (r + k) % (m - 1);
  return k == 0 ? m - 1 : (r - k + (m - 1)) % (m - 1);
}

// Factors of Z_t and the scalars around it (eq. eta:ns, beta2, etii).
struct UpdateFactors {
  double eta, rho, sum_d;
  double ck, cl, cd;   // of K, of L (with D_ii + rho + D_jj + rho), of the diagonal
};
// Every wavefront forms the sums for itself (two elements per lane: no barrier); s_ise and s_dr (beyond the rank 1 and 0) are
// written by the first one and visible to all on return.
static_assert(kMaxRank <= 128, "two elements per lane");
__device__ __forceinline__ UpdateFactors update_factors(const SmallArgs& a, const SmallGroup& g, const double* d_t, const double rho, double* s_ise,
                                                        double* s_dr, const int padded) {
  const int lane = threadIdx.x & 63, R = a.R;
  UpdateFactors f;
  f.rho = rho;
  double d[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) d[u] = lane + 64 * u < R ? d_t[lane + 64 * u] : 0.0;
  f.eta = 1.0 - exp(-(double)a.N / g.num_samples_history);
  f.sum_d = wave_sum_uniform(d[0] + d[1]);
  const double beta = f.rho * (1.0 + g.alpha) + g.alpha / (double)a.D * f.sum_d;
  if (threadIdx.x < 64) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = lane + 64 * u;
      if (i >= padded) continue;
      s_ise[i] = i < R ? 1.0 / sqrt(1.0 / (beta / d[u] + 1.0)) : 1.0;   // E_ii^{-1/2}
      s_dr[i] = i < R ? d[u] + f.rho : 0.0;
    }
  }
  f.ck = (f.eta / a.N) * (f.eta / a.N);
  f.cl = f.eta * (1.0 - f.eta) / a.N;
  f.cd = (1.0 - f.eta) * (1.0 - f.eta);
  __syncthreads();
  return f;
}
// Entry (i, j) of Z_t (eq. zt:compute), from the elements of K_t and L_t.
__device__ __forceinline__ double z_entry(const UpdateFactors& f, const int i, const int j, const double k, const double l, const double* s_ise,
                                          const double* s_dr) {
  const double z = (f.ck * k + f.cl * l * (s_dr[i] + s_dr[j])) * s_ise[i] * s_ise[j];
  return i == j ? fma(f.cd * s_dr[i], s_dr[i], z) : z;
}

// Whole shifts by one lane through the DPP path of the vector ALU (no LDS traffic), of a wavefront or of each of its rows of 16
// lanes: lane i receives the value of lane i-1 (up) or i+1 (down); the lane without a source receives zero.
template <int CTRL>
__device__ __forceinline__ double shift_lane(const double x) {
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true);
  hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Rows of U_t that go through Jacobi's rotations with the matrix.  U <- U J only mixes two columns, so rows are independent: a
// wavefront has one, with K = 2 (ranks up to 32) one in each of its rows of 16 lanes, and keeps it in registers.  Lane k holds the
// two columns that pair k rotates; between rounds the columns move to the neighbouring lanes exactly as the players of the
// round-robin schedule do (the first lane's second player never moves).  All wavefronts but the first, whose rotations bound a
// round, take rows in turn.
// (With the rotations in a log in memory, replayed by the first workgroup alone, it took longer than the iteration: 881 us a call of
// 512 x 1000 at rank 80 with equal eigenvalues, now 629.)
template <int K, int NT>
struct JacobiRows {
  static constexpr int PER_WAVE = K == 2 ? 4 : 1, LANES = 64 / PER_WAVE, SHARE = (NT / 64 - 1) * PER_WAVE;
  static constexpr int COUNT = K == 2 ? 16 * K : 16;           // rows of a workgroup
  static constexpr int SETS = (COUNT + SHARE - 1) / SHARE;
  double top[SETS], bot[SETS];
  __device__ __forceinline__ static int lane() { return (threadIdx.x & 63) % LANES; }
  __device__ __forceinline__ static int first_of(const int set) { return ((int)(threadIdx.x >> 6) - 1) * PER_WAVE + set * SHARE; }   // uniform
  __device__ __forceinline__ static bool has(const int set) { return threadIdx.x >= 64 && first_of(set) < COUNT; }
  __device__ __forceinline__ static int row(const int set) { return first_of(set) + (threadIdx.x & 63) / LANES; }   // of the workgroup's
  __device__ __forceinline__ void start(const int first_row, const int m) {
#pragma unroll
    for (int q = 0; q < SETS; ++q) {   // players of round 0: first k, second m-1-k (lane 0: the fixed player m-1)
      const int i = first_row + row(q), k = lane();
      top[q] = k < m / 2 && k == i ? 1.0 : 0.0;
      bot[q] = k < m / 2 && m - 1 - k == i ? 1.0 : 0.0;
    }
  }
  // cs: this round's rotations.  Lanes beyond the last pair repeat it on zeros: nothing of theirs reaches another (a lane takes from
  // its lower neighbour, and the last active lane takes its own second member).
  __device__ __forceinline__ void rotate(const double2* cs_of, const int half) {
    const int k = lane();
    const double2 cs = cs_of[min(k, half - 1)];
    const bool last_lane = k == half - 1, lane0 = k == 0, lane1 = k == 1, single = half == 1;   // one pair: nothing moves
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
      if (!has(q)) continue;   // uniform
      const double t = top[q] * cs.x - bot[q] * cs.y, b = top[q] * cs.y + bot[q] * cs.x;
      // firsts move one lane down (the last lane takes its own second), seconds one lane up (lane 1 takes lane 0's first)
      const double t_down = shift_lane<PER_WAVE == 1 ? 0x130 : 0x101>(t);
      const double b_up = shift_lane<PER_WAVE == 1 ? 0x138 : 0x111>(b);
      const double t_up = shift_lane<PER_WAVE == 1 ? 0x138 : 0x111>(t);
      top[q] = last_lane ? (single ? t : b) : t_down;
      bot[q] = lane0 ? b : (lane1 ? t_up : b_up);
    }
  }
  // As columns of A_t (eq. wt1), after `rounds` rounds.
  __device__ __forceinline__ void store(const SmallArgs& a, const int first_row, const int m, const int rounds, const int* s_rank, const double* s_col,
                                        const double* s_ise) const {
    const int k = lane(), R = a.R;
    if (k >= m / 2) return;
    const int tp = player_at(2 * k, rounds, m), bp = player_at(2 * k + 1, rounds, m);
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
      const int j = first_row + row(q);
      if (!has(q) || row(q) >= COUNT || j >= R) continue;
      if (tp < R) a.At[(size_t)s_rank[tp] * a.ldat + j] = (float)(s_col[s_rank[tp]] * top[q] * s_ise[j]);
      if (bp < R) a.At[(size_t)s_rank[bp] * a.ldat + j] = (float)(s_col[s_rank[bp]] * bot[q] * s_ise[j]);
    }
  }
};

// Eigenvalues of Z_t by cyclic Jacobi (upper triangle in position space, two LDS copies used alternately), `rows` with them.
// A round: the first wavefront computes the next round's rotations from the old copy while the others rotate
// the 2x2 blocks into their next positions in the other copy | barrier.
// On return s_c[i] is the eigenvalue that player i carries; K and L have been read.  All threads of the workgroup.
template <int ITEMS, int NT, typename ROWS>
__device__ __forceinline__ void jacobi_eigenvalues(const SmallArgs& a, const UpdateFactors& f, const double* s_ise, const double* s_dr, double* dyn,
                                                   double* scratch, double2 (*s_cs)[kMaxHalf], int* s_rotated, double* s_c, ROWS& rows, int& sweeps_out,
                                                   int& rounds_out, bool& converged_out) {
  const int R = a.R, tid = threadIdx.x;
  constexpr int nt = NT;
  const int m = (R + 1) & ~1;
  const int half = m / 2;
  // Z_t from K_t and L_t (eq. zt:compute), symmetrised, laid out by position in four planes: plane 2a+b holds the
  // entry (2 bi + a, 2 bj + b) of every 2x2 block bi <= bj.  Blocks are numbered diagonal by diagonal (first the
  // blocks (k, k), then (k, k+1), ...): the permutation between rounds moves a block along its diagonal or to
  // the second next one, the block waves own runs of one diagonal, and the rotation lanes need the blocks (k, k)
  // and (k-1, k+1); with this numbering neighbouring lanes touch neighbouring addresses in all of these accesses
  // (8-byte LDS accesses without bank conflicts).  The padding player of an odd R has an all-zero row and column
  // and is never rotated.
  const int n_blocks = half * (half + 1) / 2;
  const int np = n_blocks;        // plane stride
  const int zcopy = 4 * np;       // offset of the second copy (offsets, not pointers: accesses stay LDS instructions)
  auto diag_start = [half](int d) { return d * half - d * (d - 1) / 2; };   // number of the block (0, d)
  auto slot = [&](int bi, int bj) { return diag_start(bj - bi) + bi; };    // number of the block (bi, bj), bi <= bj
  auto place = [&](int pa, int pb) {   // LDS offset of the entry at positions (pa, pb) within a copy
    const int lo = pa < pb ? pa : pb, hi = pa < pb ? pb : pa;
    const int bi = lo >> 1, bj = hi >> 1;
    return (2 * (lo & 1) + (hi & 1)) * np + slot(bi, bj);
  };
  for (int idx = tid; idx < 2 * zcopy; idx += nt) dyn[idx] = 0.0;
  __syncthreads();
  double zmax = 0.0;
  for (int idx = tid; idx < m * m; idx += nt) {
    const int pa = idx / m, pb = idx % m;
    if (pa > pb) continue;
    const int i = player_at(pa, 0, m), j = player_at(pb, 0, m);
    double z = 0.0;
    if (i < R && j < R) {
      z = z_entry(f, i, j, 0.5 * (a.K[i * R + j] + a.K[j * R + i]), 0.5 * (a.L[i * R + j] + a.L[j * R + i]), s_ise, s_dr);
      if (i == j) zmax = fmax(zmax, z);
    }
    dyn[place(pa, pb)] = z;
  }
  zmax = block_max(zmax, scratch);
  const double abs_tol = kJacobiAbsTol * zmax;
  const double abs_tol2 = abs_tol * abs_tol;

  // The off-diagonal blocks (bi < bj) this thread owns (the threads after the first wavefront, diagonal by
  // diagonal), where they are stored, and the (fixed) destinations of their four entries.  The diagonal blocks
  // are handled apart (three entries, a different formula), so this path is branch-free.
  const int n_off = half * (half - 1) / 2;
  int blk_i[ITEMS], blk_j[ITEMS], blk_t[ITEMS];
  int dst[ITEMS][4];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int item = (tid - 64) + it * (nt - 64);
    const int it_no = (item >= 0 && item < n_off) ? item : 0;
    // diagonal d holds the blocks (0, d), ..., (half-1-d, half-1), numbers (d-1) half - d (d-1) / 2 onwards
    auto first_of = [half](const int d) { return (d - 1) * half - d * (d - 1) / 2; };
    const float w = (float)half - 0.5f;
    int d = max(1, min(half - 1, 1 + (int)(w - sqrtf(fmaxf(w * w - 2.f * (float)it_no, 0.f)))));
    while (d > 1 && first_of(d) > it_no) --d;
    while (d < half - 1 && first_of(d + 1) <= it_no) ++d;
    const int rem = it_no - first_of(d);
    const int bi = rem, bj = min(rem + d, half - 1);   // (an idle thread of a single-pair problem: bj = bi = 0)
    blk_i[it] = bi;
    blk_j[it] = bj;
    blk_t[it] = (item >= 0 && item < n_off) ? slot(bi, bj) : -1;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      dst[it][e] = place(next_position(2 * bi + (e >> 1), half), next_position(2 * min(bj, half - 1) + (e & 1), half));
  }
  // The diagonal block (k, k) is rotated by lane k of the second wavefront (on top of its off-diagonal block): the
  // rotation lanes' chain bounds the round and is kept as short as possible.  Destinations of (t,t), (t,b), (b,b):
  const int diag_k = tid - 64;
  const bool diag_lane = diag_k >= 0 && diag_k < half;
  int diag_t = 0, diag_dst[3] = {0, 0, 0};
  if (diag_lane) {
    diag_t = slot(diag_k, diag_k);
    diag_dst[0] = place(next_position(2 * diag_k, half), next_position(2 * diag_k, half));
    diag_dst[1] = place(next_position(2 * diag_k, half), next_position(2 * diag_k + 1, half));
    diag_dst[2] = place(next_position(2 * diag_k + 1, half), next_position(2 * diag_k + 1, half));
  }
  const bool odd_pad = (R & 1) != 0;   // pair 0 then holds the padding player

  // Rotation lanes (the first wavefront): while the 2x2 blocks of round r are being rotated, lane k of this wave
  // prepares pair k's rotation for round r+1.  The pair that will stand at (2k, 2k+1) is made of member A (the
  // later column) and member B (the earlier row) of the present layout; the lane recomputes their two diagonal
  // entries and their common entry after this round's rotations from the old copy, so a round needs one barrier.
  const int rot_k = tid;   // the first wavefront: the oldest wave of a SIMD is served first
  const bool rot_lane = rot_k < half;
  int rz_blk = 0, rz_da = 0, rz_db = 0, rz_pa = 0, rz_pb = 0;
  bool rz_sa0 = true, rz_sb0 = true;
  if (rot_lane && half >= 2) {
    const int k = rot_k;
    const int pa = k < half - 1 ? k + 1 : half - 1, sa = k < half - 1 ? 0 : 1;   // first member of the new pair
    const int pb = k >= 2 ? k - 1 : 0, sb = k == 1 ? 0 : 1;                       // second member (pb < pa)
    rz_pa = pa;
    rz_pb = pb;
    rz_sa0 = sa == 0;
    rz_sb0 = sb == 0;
    rz_blk = slot(pb, pa);
    rz_da = slot(pa, pa);
    rz_db = slot(pb, pb);
  }
  if (tid < 64) __builtin_amdgcn_s_setprio(3);   // the rotation wave's dependent chain bounds the round
  if (tid < 2) s_rotated[tid] = 0;
  __syncthreads();
  if (rot_lane) {   // rotations of the very first round
    const int t = slot(rot_k, rot_k);
    double c = 1.0, s = 0.0;
    bool large = false;
    if (!(odd_pad && rot_k == 0)) jacobi_rotation(dyn[t], dyn[3 * np + t], dyn[np + t], abs_tol2, c, s, large);
    if (large) s_rotated[0] = 1;
    s_cs[0][rot_k] = make_double2(c, s);
  }
  __syncthreads();

  // cyclic Jacobi; a sweep in which no pair needed a large rotation ends the iteration
  int sweeps = 0, rounds = 0, cur = 0;
  bool converged = false;
  for (; sweeps < kMaxSweeps && !converged; ++sweeps) {
    for (int r = 0; r < m - 1; ++r, ++rounds, cur ^= 1) {
      const int co = cur ? zcopy : 0, no = cur ? 0 : zcopy;
      const double2* cs = s_cs[cur];
      if (rot_lane) {
        double c = 1.0, s = 0.0;
        if (half >= 2 && !(odd_pad && rot_k == 0)) {
          const double2 csi = cs[rz_pb], csj = cs[rz_pa];
          const double ci = csi.x, si = csi.y, cj = csj.x, sj = csj.y;
          const double x00 = dyn[co + rz_blk], x01 = dyn[co + np + rz_blk];
          const double x10 = dyn[co + 2 * np + rz_blk], x11 = dyn[co + 3 * np + rz_blk];
          const double da_tt = dyn[co + rz_da], da_tb = dyn[co + np + rz_da], da_bb = dyn[co + 3 * np + rz_da];
          const double db_tt = dyn[co + rz_db], db_tb = dyn[co + np + rz_db], db_bb = dyn[co + 3 * np + rz_db];
          __builtin_amdgcn_sched_barrier(0);   // all reads are in flight before the first use
          // a first member takes (c, -s) of its pair's rotation, a second member (s, c)
          const double r0 = rz_sb0 ? ci : si, r1 = rz_sb0 ? -si : ci;
          const double q0 = rz_sa0 ? cj : sj, q1 = rz_sa0 ? -sj : cj;
          const double zab = q0 * (r0 * x00 + r1 * x10) + q1 * (r0 * x01 + r1 * x11);
          const double zaa = q0 * q0 * da_tt + 2.0 * q0 * q1 * da_tb + q1 * q1 * da_bb;
          const double zbb = r0 * r0 * db_tt + 2.0 * r0 * r1 * db_tb + r1 * r1 * db_bb;
          // whether this rotation belongs to the present sweep or opens the next one
          bool large = false;
          jacobi_rotation(zaa, zbb, zab, abs_tol2, c, s, large);
          if (large) s_rotated[(sweeps + (r == m - 2 ? 1 : 0)) & 1] = 1;
        }
        s_cs[cur ^ 1][rot_k] = make_double2(c, s);
      }
      if (diag_lane) {   // this round's rotation of pair diag_k, applied to its diagonal block
        const double2 csk = cs[diag_k];
        const double ck = csk.x, sk = csk.y;
        const double att = dyn[co + diag_t], atb = dyn[co + np + diag_t], abb = dyn[co + 3 * np + diag_t];
        dyn[no + diag_dst[0]] = ck * ck * att - 2.0 * ck * sk * atb + sk * sk * abb;
        dyn[no + diag_dst[2]] = sk * sk * att + 2.0 * ck * sk * atb + ck * ck * abb;
        dyn[no + diag_dst[1]] = sk == 0.0 ? atb : 0.0;
      }
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        const int t = blk_t[it];
        if (t < 0) continue;
        const int bi = blk_i[it], bj = blk_j[it];
        const double2 csi = cs[bi], csj = cs[bj];
        const double ci = csi.x, si = csi.y, cj = csj.x, sj = csj.y;
        const double x00 = dyn[co + t], x01 = dyn[co + np + t], x10 = dyn[co + 2 * np + t], x11 = dyn[co + 3 * np + t];
        const double y00 = ci * x00 - si * x10, y01 = ci * x01 - si * x11;
        const double y10 = si * x00 + ci * x10, y11 = si * x01 + ci * x11;
        dyn[no + dst[it][0]] = y00 * cj - y01 * sj;
        dyn[no + dst[it][1]] = y00 * sj + y01 * cj;
        dyn[no + dst[it][2]] = y10 * cj - y11 * sj;
        dyn[no + dst[it][3]] = y10 * sj + y11 * cj;
      }
      rows.rotate(cs, half);
      __syncthreads();
    }
    if (s_rotated[sweeps & 1] == 0) converged = true;   // same value for every thread: read after the barrier
    __syncthreads();                                    // everyone has read the flag before it is cleared again
    if (tid == 0) s_rotated[sweeps & 1] = 0;
  }

  const int fo = cur ? zcopy : 0;
  for (int pos = tid; pos < m; pos += nt) {
    const int i = player_at(pos, rounds, m);
    if (i < R) s_c[i] = dyn[fo + place(pos, pos)];
  }
  if (tid < 64) __builtin_amdgcn_s_setprio(0);
  sweeps_out = sweeps;
  rounds_out = rounds;
  converged_out = converged;
}

// Z_t in the registers of NT threads (see eig_direct.h), all elements of K_t and L_t requested together.
template <int K, int NT>
struct ZLoad {
  static constexpr int A = DirectTile<K, NT>::A, ROWS = DirectTile<K, NT>::ROWS;
  double k[A][K], l[A][K];
  template <typename ORDER>
  __device__ __forceinline__ void request(const SmallArgs& a, ORDER order) {
    const int ti = DirectTile<K, NT>::ti(), tj = DirectTile<K, NT>::tj(), last = a.R - 1;
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int b = 0; b < K; ++b) {
        const int at = order(min(ti + ROWS * x, last)) * a.R + order(min(tj + 16 * b, last));
        k[x][b] = a.K[at];
        l[x][b] = a.L[at];
      }
  }
  template <typename ORDER>
  __device__ __forceinline__ void form(const SmallArgs& a, const UpdateFactors& f, const double* s_ise, const double* s_dr, double (&S)[A][K],
                                       ORDER order) const {
    const int ti = DirectTile<K, NT>::ti(), tj = DirectTile<K, NT>::tj();
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int b = 0; b < K; ++b) {
        const int i = ti + ROWS * x, j = tj + 16 * b;
        S[x][b] = i < a.R && j < a.R ? z_entry(f, order(i), order(j), k[x][b], l[x][b], s_ise, s_dr) : 0.0;
      }
  }
  // Behind request(): Z_t, with rows and columns sorted by the diagonal where that spans much; s_order[i] is the index that
  // stands at i.  All threads of the workgroup; s_diag is scratch.
  __device__ __forceinline__ void ordered(const SmallArgs& a, const UpdateFactors& f, const double* s_ise, const double* s_dr, double (&S)[A][K],
                                          double* s_diag, int* s_order) {
    const int tid = threadIdx.x, lane = tid & 63, R = a.R;
    auto same = [](const int i) { return i; };
    form(a, f, s_ise, s_dr, S, same);
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int b = 0; b < K; ++b) {
        const int i = DirectTile<K, NT>::ti() + ROWS * x;
        if (i == DirectTile<K, NT>::tj() + 16 * b && i < R) s_diag[i] = S[x][b];
      }
    if (tid < 16 * K) s_order[tid] = tid;
    __syncthreads();
    const double d0 = s_diag[min(lane, R - 1)], d1 = s_diag[min(lane + 64, R - 1)];
    const double up = row16_max_f64(fmax(d0, d1)), down = row16_max_f64(-fmin(d0, d1));
    const double largest = fmax(fmax(read_lane_f64(up, 0), read_lane_f64(up, 16)), fmax(read_lane_f64(up, 32), read_lane_f64(up, 48)));
    const double smallest = -fmax(fmax(read_lane_f64(down, 0), read_lane_f64(down, 16)), fmax(read_lane_f64(down, 32), read_lane_f64(down, 48)));
    if (!(largest > kDirectOrderSpan * smallest)) return;   // the same for all threads
    __syncthreads();
    if (tid < R) {
      const double z = s_diag[tid];
      int rank = 0;
      for (int j = 0; j < R; ++j) rank += s_diag[j] > z || (s_diag[j] == z && j < tid) ? 1 : 0;
      s_order[rank] = tid;   // (a NaN leaves some as they are: all stay indices)
    }
    __syncthreads();
    auto sorted = [&](const int i) { return s_order[i]; };
    request(a, sorted);
    form(a, f, s_ise, s_dr, S, sorted);
  }
};

// A call that updates one instance on one stream: what does not wait for the eigen-problem, which leaves the chip idle, runs beside it in
// the same launches.  Xhat beside the first kernel; gamma, row norms and the scaling beside the eigenpairs or, up to rank 32, beside
// W_(t+1).  The eigen-problem's workgroups come first.  512 x 5000 rank 80: Xhat 9.3, finishing 10.0 us and their gaps off the call.
constexpr int kBesideFirst = kXcds;   // workgroups in front, so that a die's units stay a contiguous share
struct Beside {
  GemmGroupOf<1> xhat;
  FinishArgs finish;
  static constexpr int kBk = 16;
  static int row_blocks(const int N) { return (N + kFinishScaleRows - 1) / kFinishScaleRows; }
  int xhat_blocks() const { return (xhat.total_tiles + kXcds - 1) / kXcds * kXcds; }
};
struct NothingBeside {};   // (what the other launches carry)
template <bool BESIDE>
using BesideArg = std::conditional_t<BESIDE, Beside, NothingBeside>;
// 256 threads; block counts from the first workgroup beside.
__device__ __forceinline__ void beside_products(const Beside& b, const int block) {
  const int per = (b.xhat.total_tiles + kXcds - 1) / kXcds, unit = block % kXcds * per + block / kXcds;
  if (unit < b.xhat.total_tiles) gemm_unit<64, 64, Beside::kBk, 2, 2, true, false, EPI_SUB_ROWNORM, false, 0, false, kPrefetch>(b.xhat, 0, unit);
}

// Factors of B_t = J_t + (N (1 - eta) / eta) (D_t + rho_t I) W_t (eq. wt1), while D_t and rho_t are there.
__device__ __forceinline__ void store_bt_factors(const SmallArgs& a, const UpdateFactors& f, const double* s_dr) {
  if ((int)threadIdx.x < a.R) a.bt[threadIdx.x] = (float)((double)a.N * (1.0 - f.eta) / f.eta * s_dr[threadIdx.x]);
}

// Above rank 32, first kernel: Z_t and its reduction.  A workgroup per instance.
template <int K, bool BESIDE>
__global__ __launch_bounds__(kEigReduceThreads) void eig_reduce_kernel(const SmallGroup g, const BesideArg<BESIDE> beside) {
  if constexpr (BESIDE) {
    if ((int)blockIdx.x >= kBesideFirst) {
      beside_products(beside, (int)blockIdx.x - kBesideFirst);
      return;
    }
    if ((int)blockIdx.x >= g.count) return;
  }
  using Shape = DirectShape<K>;
  constexpr int NT = kEigReduceThreads;
  constexpr int T = Shape::T;
  extern __shared__ double eig_reserved[];   // not used: see the launch
  __shared__ double s_ise[T], s_dr[T], s_tau[T], s_diag[T], s_off[T];
  __shared__ int s_order[T];
  __shared__ DirectLds<K, NT> lds;
  __shared__ __attribute__((aligned(16))) double s_V[T * T];
  const SmallArgs& a = g.a[blockIdx.x];
  const int R = a.R, tid = threadIdx.x;
  ZLoad<K, NT> load;
  load.request(a, [](const int i) { return i; });
  const double rho = a.st->rho;
  const UpdateFactors f = update_factors(a, g, a.st->d, rho, s_ise, s_dr, T);
  store_bt_factors(a, f, s_dr);
  // handed on: the last kernel's workgroups cannot read what one of them replaces
  for (int i = tid; i <= R; i += NT) a.d_rho(T)[i] = i < R ? a.st->d[i] : rho;
  if (tid == 0) *a.k_tickets(T) = 0;
  typename DirectTile<K, NT>::Regs S;
  load.ordered(a, f, s_ise, s_dr, S, s_diag, s_order);
  direct_reduce<K, NT>(S, R, lds, s_V, s_tau, s_off);
  direct_store_tridiagonal<K, NT>(S, R, s_diag, s_off);
  __syncthreads();
  for (int e = tid; e < (R - 2) * T / 2; e += NT) reinterpret_cast<double2*>(a.V())[e] = reinterpret_cast<const double2*>(s_V)[e];
  if (tid < R) {
    a.order(T)[tid] = (double)s_order[tid];
    a.diag(T)[tid] = s_diag[tid];
    if (tid < R - 1) a.off(T)[tid] = s_off[tid];
    if (tid < R - 2) a.tau(T)[tid] = s_tau[tid];
  }
}

// Second kernel: four eigenpairs per workgroup of 256 threads.  Grid (instance, ceil(R / 4)); beside them, of the one instance, all in the
// first extent, which holds any number of rows.
template <int K, bool BESIDE>
__global__ __launch_bounds__(256) void eig_pairs_kernel(const SmallGroup g, const BesideArg<BESIDE> beside) {
  const int instance = BESIDE ? 0 : blockIdx.x, block = BESIDE ? blockIdx.x : blockIdx.y;
  if constexpr (BESIDE) {
    const int pairs = (g.a[0].R + 3) / 4;
    if (block >= pairs) {
      finish_rows<true>(beside.finish, block - pairs);
      return;
    }
  }
  using Shape = DirectShape<K>;
  constexpr int T = Shape::T;
  __shared__ DirectTridiagonal<K> t;
  __shared__ double s_tau[T], s_work[4][kDirectWork<K>], s_g[T / 4][6];
  __shared__ __attribute__((aligned(16))) double s_V[T * T];
  const SmallArgs& a = g.a[instance];
  const int R = a.R, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (block * 4 >= R) return;
  if (tid < T) {
    t.diag[tid] = tid < R ? a.diag(T)[tid] : 0.0;
    t.off[tid] = tid < R - 1 ? a.off(T)[tid] : 0.0;
    s_tau[tid] = tid < R - 2 ? a.tau(T)[tid] : 0.0;
  }
  const double2* const v_in = reinterpret_cast<const double2*>(a.V());
#pragma unroll 4
  for (int e = tid; e < T * T / 2; e += 256)
    reinterpret_cast<double2*>(s_V)[e] = e < (R - 2) * T / 2 ? v_in[e] : make_double2(0.0, 0.0);
  __syncthreads();
  direct_block_products<K, 256>(s_V, T, R, s_g);
  double lo, hi, norm, x[K], lambda, residual;
  direct_scale<K>(t, R, lo, hi, norm);   // ends with a barrier
  const int k = block * 4 + wave;
  if (k >= R) return;   // uniform over the wavefront
  direct_pair<K, 64>(t, R, k, lo, hi, s_V, T, s_tau, s_g, s_work[wave], x, lambda, residual);
  if (group16_index() == 0) {
#pragma unroll
    for (int b = 0; b < K; ++b) a.U(T)[(size_t)k * T + group16_member() + 16 * b] = x[b];
  }
  if (lane == 0) {
    a.lambda(T)[k] = lambda * norm;
    a.residual(T)[k] = residual;
  }
}

// What only the one-kernel form keeps in LDS.
template <int K, int NT, bool FUSED>
struct FusedLds {
  DirectLds<K, 256> reduce;
  double s_tau[16 * K], s_res[16 * K], s_work[NT / 16][kDirectWork<K>], s_g[4 * K][6];
  double V[16 * K * 16 * K];
  DirectTridiagonal<K> t;
};
template <int K, int NT>
struct FusedLds<K, NT, false> {};

// The last kernel, and with FUSED the only one: checks the eigenvectors U (rows) and makes them orthogonal to working
// precision, U <- (3/2 - U U^T / 2) U on the fp64 matrix unit, or has Jacobi find them; then the floors, rho_{t+1}, D_{t+1}, E_{t+1}
// (eq. rhodash2, dt1, rhot1, beta2, etii) and A_t (eq. wt1).  Above rank 32 a workgroup per 16 rows of A_t: each checks all
// vectors, by the same arithmetic so that all decide alike, and takes its rows' share of the second product; the first one does what is left.
// Grid (instance, FUSED ? 1 : ceil(R / 16)).
template <int K, int ITEMS, int NT, bool FUSED, bool BESIDE>
__global__ __launch_bounds__(NT) void eig_finish_kernel(const SmallGroup g, const BesideArg<BESIDE> beside) {
  if constexpr (BESIDE) {
    if ((int)blockIdx.x >= kBesideFirst) {
      if (threadIdx.x < 256) beside_products(beside, (int)blockIdx.x - kBesideFirst);
      return;
    }
    if ((int)blockIdx.x >= g.count) return;
  }
  using Shape = DirectShape<K>;
  constexpr int T = Shape::T, SU = Shape::STRIDE, NW = NT / 64;
  typedef double doublex4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) double dyn[];   // U, then 3/2 - U U^T / 2; or Jacobi's two copies of Z
  __shared__ double scratch[16];
  __shared__ double s_ise[T], s_dr[T], s_col[T], s_c[kMaxRank + 1];
  __shared__ __attribute__((aligned(16))) double2 s_cs[2][kMaxHalf];
  __shared__ int s_perm[kMaxRank], s_rank[kMaxRank], s_order[T];
  __shared__ int s_rotated[2];
  __shared__ FusedLds<K, NT, FUSED> s_fused;
  static_assert(kMaxRank <= NT && T <= NT, "a thread per eigenvalue");
  const SmallArgs& a = g.a[blockIdx.x];
  const int R = a.R, D = a.D, N = a.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  if (16 * (int)blockIdx.y >= R) return;
  const bool lead = blockIdx.y == 0;
  PrecondScalars* st = a.st;
  double* const U = dyn;
  double* const M = dyn + T * SU;
  double lambda = 0.0, residual = 0.0;   // of pair tid
  double tr_part = 0.0;   // tr(X X^T), summed here: the kernel that finishes the output may still be running
  for (int i = tid; i < a.n_sumsq; i += NT) tr_part += a.sumsq_part[i];
  if constexpr (!FUSED) {
    for (int e = tid; e < T * (T / 2); e += NT) {
      const int k = e / (T / 2), c = e % (T / 2);
      const double2 v = k < R ? reinterpret_cast<const double2*>(a.U(T))[(size_t)k * (T / 2) + c] : make_double2(0.0, 0.0);
      U[k * SU + 2 * c] = v.x;
      U[k * SU + 2 * c + 1] = v.y;
    }
    if (tid < R) {
      lambda = a.lambda(T)[tid];
      residual = a.residual(T)[tid];
    }
    if (tid < T) s_order[tid] = tid < R ? (int)a.order(T)[tid] : tid;
  }
  ZLoad<K, 256> load;
  if constexpr (FUSED) load.request(a, [](const int i) { return i; });   // (the upper half of the threads as well, and drops it)
  const UpdateFactors f = update_factors(a, g, FUSED ? st->d : a.d_rho(T), FUSED ? st->rho : a.d_rho(T)[R], s_ise, s_dr, T);
  if constexpr (FUSED) {
    store_bt_factors(a, f, s_dr);
    static_assert(NT >= 256 && NT >= 16 * T, "all pairs at once");
    typename DirectTile<K, 256>::Regs S;
    load.ordered(a, f, s_ise, s_dr, S, s_fused.t.diag, s_order);
    if (tid < 256) {
      direct_reduce<K, 256>(S, R, s_fused.reduce, s_fused.V, s_fused.s_tau, s_fused.t.off);
      direct_store_tridiagonal<K, 256>(S, R, s_fused.t.diag, s_fused.t.off);
    } else {
      for (int e = max(R - 2, 0) * T + tid - 256; e < T * T; e += NT - 256) s_fused.V[e] = 0.0;
      for (int e = max(R - 2, 0) + tid - 256; e < T; e += NT - 256) s_fused.s_tau[e] = 0.0;
      direct_reduce_idle(R);
    }
    __syncthreads();
    direct_block_products<K, NT>(s_fused.V, T, R, s_fused.s_g);
    double lo, hi, norm;
    direct_scale<K>(s_fused.t, R, lo, hi, norm);
    const int k = tid >> 4;
    double x[K], l, r;
    if ((k & ~3) < R) {   // (uniform over a wavefront)
      direct_pair<K, 16>(s_fused.t, R, min(k, R - 1), lo, hi, s_fused.V, T, s_fused.s_tau, s_fused.s_g, s_fused.s_work[k], x, l, r);
      if (l16 == 0 && k < R) {
        s_c[k] = l * norm;
        s_fused.s_res[k] = r;
      }
    }
    const int kx = 4 * wave + group16_index();   // whose vector this lane has
#pragma unroll
    for (int b = 0; b < K; ++b) U[kx * SU + group16_member() + 16 * b] = kx < R ? x[b] : 0.0;
    __syncthreads();
    if (tid < R) {
      lambda = s_c[tid];
      residual = s_fused.s_res[tid];
    }
  }
  if (tid < R) s_c[tid] = lambda;
  tr_part = wave_sum_uniform(tr_part);
  if (lane == 0) scratch[wave] = tr_part;
  __syncthreads();
  double tr_M = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) tr_M += scratch[w];

  // M = 3/2 - U U^T / 2 in fp64 and the check of U U^T.  v_mfma_f64_16x16x4_f64: lane l supplies A[l%16][l/16] and B[l/16][l%16];
  // register r holds row 4r + l/16, column l%16 (v_mfma_f32_16x16x4_f32 row 4 (l/16) + r).  With FUSED both by the tiles on and above
  // the diagonal.  Otherwise the first K wavefronts form this workgroup's rows of M, and the others check all tiles on and above
  // the diagonal with fp32 products (a quarter of the time, and the limit is far above their rounding): the same products
  // and sums in every workgroup of the instance, so that all decide alike however near the limit an element lies.
  const int first_row = FUSED ? 0 : 16 * (int)blockIdx.y;
  bool bad = false;
  auto product_f64 = [&](const int i0, const int j0) {
    const double* const ui = U + (i0 + l16) * SU + g4;
    const double* const uj = U + (j0 + l16) * SU + g4;
    doublex4 part[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    for (int s0 = 0; s0 < R; s0 += 16) {
#pragma unroll
      for (int s = 0; s < 16; s += 4) part[(s >> 2) & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ui[s0 + s], uj[s0 + s], part[(s >> 2) & 1], 0, 0, 0);
    }
    return part[0] + part[1];
  };
  auto tile_of = [](int tile, int& ti, int& tj) {
    for (ti = 0; tile >= K - ti; ++ti) tile -= K - ti;
    tj = ti + tile;
  };
  if constexpr (FUSED) {
    for (int tile = wave; tile < K * (K + 1) / 2; tile += NW) {
      int ti, tj;
      tile_of(tile, ti, tj);
      if (16 * tj >= R) continue;   // uniform
      const doublex4 acc = product_f64(16 * ti, 16 * tj);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + 4 * r + g4, j = 16 * tj + l16;
        const double one = i == j ? 1.0 : 0.0;
        if (i < R && j < R) bad |= !(fabs(acc[r] - one) <= kDirectOrthoLimit);   // (NaN fails)
        M[i * SU + j] = M[j * SU + i] = fma(-0.5, acc[r], 1.5 * one);
      }
    }
  } else if (wave < K) {
    if (16 * wave < R) {
      const doublex4 acc = product_f64(first_row, 16 * wave);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 4 * r + g4, j = 16 * wave + l16;
        M[i * SU + j] = fma(-0.5, acc[r], first_row + i == j ? 1.5 : 0.0);
      }
    }
  } else {
    for (int tile = wave - K; tile < K * (K + 1) / 2; tile += NW - K) {
      int ti, tj;
      tile_of(tile, ti, tj);
      if (16 * tj >= R) continue;   // uniform
      const double* const ui = U + (16 * ti + l16) * SU + g4;
      const double* const uj = U + (16 * tj + l16) * SU + g4;
      floatx4 part[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
      for (int s0 = 0; s0 < R; s0 += 16) {
#pragma unroll
        for (int s = 0; s < 16; s += 4)
          part[(s >> 2) & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)ui[s0 + s], (float)uj[s0 + s], part[(s >> 2) & 1], 0, 0, 0);
      }
      const floatx4 acc = part[0] + part[1];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + 4 * g4 + r, j = 16 * tj + l16;
        if (i < R && j < R) bad |= !(fabsf(acc[r] - (i == j ? 1.f : 0.f)) <= (float)kDirectOrthoLimit);   // (NaN fails)
      }
    }
  }
  if (tid < R) {
    const double largest = s_c[0], smallest = s_c[R - 1];
    bad |= !(residual <= kDirectResidual && residual * largest <= kDirectRelResidual * lambda);
    bad |= !(lambda <= largest && smallest > 0.0 && largest <= kDirectCondLimit * smallest);
  }
  const bool direct = __syncthreads_or(bad ? 1 : 0) == 0;   // (M is complete behind it)

  // Jacobi: all workgroups of the instance find the same rotations, each takes its rows of U through them, and the last to have read K
  // clears it.
  int sweeps = 1, rounds = 0;
  bool converged = true, clears = lead;
  JacobiRows<K, NT> rows;
  if (!direct) {
    rows.start(first_row, (R + 1) & ~1);
    jacobi_eigenvalues<ITEMS, NT>(a, f, s_ise, s_dr, dyn, scratch, s_cs, s_rotated, s_c, rows, sweeps, rounds, converged);
    if (!FUSED && tid == 0)
      s_rotated[0] = __hip_atomic_fetch_add(a.k_tickets(T), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (R + 15) / 16 - 1 ? 1 : 0;
    __syncthreads();
    if (!FUSED) clears = s_rotated[0] != 0;
  }

  // Every wavefront handles all eigenvalues, two per lane.  Floor (after eq. zt:eig:repeat), decreasing order:
  const double floor_c = (1.0 - f.eta) * (1.0 - f.eta) * f.rho * f.rho;
  bool floored = false;
  double c[2];
  int rank[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = lane + 64 * u;
    rank[u] = i;
    c[u] = i < R ? s_c[i] : 1.0;
    if (i < R && !(c[u] >= floor_c)) {
      c[u] = floor_c;
      floored = true;
    }
  }
  if (!direct) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = lane + 64 * u;
      if (wave == 0 && i < R) s_c[i] = c[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = lane + 64 * u;
      if (i >= R) continue;
      rank[u] = 0;
      for (int j = 0; j < R; ++j) rank[u] += (s_c[j] > c[u] || (s_c[j] == c[u] && j < i)) ? 1 : 0;
      if (wave == 0) {
        s_perm[rank[u]] = i;   // s_perm[k] = index of the k-th largest eigenvalue
        s_rank[i] = rank[u];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (lane + 64 * u < R) c[u] = s_c[s_perm[lane + 64 * u]];   // eigenpair at position lane + 64 u
  }
  // eq. rhodash2, dt1, rhot1
  double root[2], dn[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) root[u] = lane + 64 * u < R ? sqrt(c[u]) : 0.0;
  const double sum_sqrt = wave_sum_uniform(root[0] + root[1]);
  const double rho_dash = ((f.eta / N) * tr_M + (1.0 - f.eta) * ((double)D * f.rho + f.sum_d) - sum_sqrt) / (double)(D - R);
  const double rho_new = fmax(g.epsilon, rho_dash);
#pragma unroll
  for (int u = 0; u < 2; ++u) dn[u] = lane + 64 * u < R ? fmax(root[u] - rho_dash, g.epsilon) : 0.0;
  const double beta_new = rho_new * (1.0 + g.alpha) + g.alpha / (double)D * wave_sum_uniform(dn[0] + dn[1]);
  const bool any_floored = __any(floored);
  if (wave == 0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = lane + 64 * u;
      if (k >= R) continue;
      const double en = 1.0 / (beta_new / dn[u] + 1.0);
      s_col[k] = (f.eta / N) * sqrt(en / c[u]);   // A_t = (eta/N) E_{t+1}^{1/2} C_t^{-1/2} U_t^T E_t^{-1/2}  (eq. wt1)
      if (lead) {
        st->d[k] = dn[u];
        st->e[k] = en;
      }
      if (k == R - 1) s_c[kMaxRank] = c[u];
      if (k == 0) s_cs[0][0].x = c[u];
    }
  }
  __syncthreads();
  if (lead && tid == 0) {
    int flags = 0;
    if (any_floored) flags |= kFlagFloored | kFlagOrthCheck;
    if (s_cs[0][0].x > kOrthoCondLimit * s_c[kMaxRank]) flags |= kFlagOrthCheck;
    if (!converged) flags |= kFlagNoConverge;
    st->flags = flags;
    st->sweeps = sweeps;
    st->rho = rho_new;
    st->beta = beta_new;
  }
  if (direct) {
    constexpr int TILES = FUSED ? K * K : K;
    for (int tile = wave; tile < TILES; tile += NW) {
      const int ti = FUSED ? tile / K : 0, tj = tile % K;
      if (16 * ti >= R || 16 * tj >= R) continue;   // uniform
      doublex4 acc = {0, 0, 0, 0};
      for (int s0 = 0; s0 < R; s0 += 16) {   // (M has no columns beyond the last tile)
#pragma unroll
        for (int s = s0; s < s0 + 16; s += 4)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(M[(16 * ti + l16) * SU + s + g4], U[(s + g4) * SU + 16 * tj + l16], acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = first_row + 16 * ti + 4 * r + g4, j = 16 * tj + l16;
        if (i < R && j < R) a.At[(size_t)i * a.ldat + s_order[j]] = (float)(s_col[i] * acc[r] * s_ise[s_order[j]]);
      }
    }
  } else {
    rows.store(a, first_row, (R + 1) & ~1, rounds, s_rank, s_col, s_ise);
  }
  if (clears)
    for (int idx = tid; idx < R * R; idx += NT) a.K[idx] = 0.0;
}

// App. B.3.1 on the new factor: O = E^{-1/2} (W W^T) E^{-1/2}; if any entry is off the identity by more than
// 1e-3, W <- E^{1/2} L^{-1} E^{-1/2} W with O = L L^T.  Runs only when the update asked for the check.
struct OrthArgs {
  PrecondScalars* st;
  double* G;         // R x R, W W^T of the new factor (accumulated only when the check was requested), its 16 x 16 tiles on and
                     // above the diagonal; cleared on exit
  float* At;         // R x R (ldat): A_t on entry; when the fix is needed, E^{1/2} L^{-1} E^{-1/2} A_t on return
  int ldat;
  int R;
  // what the update accumulated into besides G (arrival counters and H, contiguous; L): cleared here, behind their last
  // readers, so that the next call needs no clearing launch in front of it
  float* clear_ptr;
  double* L;
  int clear_floats;   // a multiple of 4
};
constexpr int kOrthClearBlocks = 8;   // workgroups per instance, the first one checks and the others clear
// Several instances of a larger rank are left to a launch of small workgroups in front of the next update: 1024 threads and
// 50 KB of LDS each wait for a compute unit behind the layer products (eight replicas of the speech-shaped network: 9.23
// instead of 9.0 ms per period).
constexpr int kOrthClearRank = 32;
struct OrthGroup {
  int count;
  OrthArgs a[kMaxInstances];
};

// The augmented matrix [O | B], R x 2R: O = E^{-1/2} (W W^T) E^{-1/2} (full, symmetric) and B = E^{-1/2} A_t.
// Gaussian elimination without pivoting (O is symmetric positive definite) turns O into D L1^T and B into
// L1^{-1} B, where O = L1 D L1^T with unit lower triangular L1; the Cholesky factor is L = L1 D^{1/2}, so
// L^{-1} B = D^{-1/2} (L1^{-1} B).  The matrix lives in registers as 4 x CT tiles: thread (ti, tj) holds the rows
// 4 ti .. 4 ti + 3 and the columns tj, tj + 32, ... (CT of them: the kernel is instantiated per rank class).  What a step
// needs from other threads (the pivot row, the pivot column and the reciprocal of the pivot) is published in LDS by
// its owners at the end of the step before, in one of two buffers used alternately; a step (two pivots, see below)
// is then one barrier, LDS reads without address arithmetic and multiply-adds (a tile needs 2.3 times fewer reads
// per element than a strip of one row); wavefronts whose rows all lie above the pivot skip the step.
constexpr int kOrthTileRows = 4;
constexpr int kOrthTileStride = 32;   // columns tj, tj + 32, ...: the threads of a row of tiles
constexpr int kOrthRowsPerWave = (64 / kOrthTileStride) * kOrthTileRows;
static_assert((kMaxRank + kOrthTileRows - 1) / kOrthTileRows * kOrthTileStride <= kSmallThreads, "one thread per tile");
inline int orth_columns_per_thread(int R) { return (2 * R + kOrthTileStride - 1) / kOrthTileStride; }

template <int CT>
__global__ __launch_bounds__(kSmallThreads) void orth_fix_kernel(const OrthGroup g) {
  extern __shared__ __attribute__((aligned(16))) double dyn[];   // W W^T of the instance, R x (R + 1)
  __shared__ double scratch[16];
  __shared__ double s_ise[kMaxRank];                       // E_ii^{-1/2}
  __shared__ double s_prow[2][2][kOrthTileStride * CT];    // the two pivot rows of a step
  __shared__ double s_pcol[2][2][kMaxRank + kOrthTileRows];   // the two pivot columns of a step
  __shared__ double s_invp[2];                             // reciprocal of the first pivot of a step
  __shared__ double s_dinv[kMaxRank];                      // D_ii^{-1/2}
  const OrthArgs& a = g.a[blockIdx.x];
  PrecondScalars* st = a.st;
  const int R = a.R;
  const int tid = threadIdx.x, nt = blockDim.x;
  if (blockIdx.y > 0) {
    const int at = ((int)blockIdx.y - 1) * nt + tid, step = (kOrthClearBlocks - 1) * nt;
    float4* const z = reinterpret_cast<float4*>(a.clear_ptr);
    for (int i = at; i < a.clear_floats / 4; i += step) z[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = at; i < R * R; i += step) a.L[i] = 0.0;
    return;
  }
  if (!(st->flags & kFlagOrthCheck)) return;   // uniform over the workgroup; G was cleared by the R x R update
  // the check: G and E through LDS (coalesced reads), O symmetrised from there
  double* const Gs = dyn;   // R x (R + 1)
  const int SG = R + 1;
  for (int idx = tid; idx < R * R; idx += nt) {
    const int r = idx / R, c = idx % R;
    if (r / 16 > c / 16) continue;
    const double v = a.G[idx];
    Gs[r * SG + c] = v;
    if (r / 16 < c / 16) Gs[c * SG + r] = v;
  }
  for (int k = tid; k < R; k += nt) s_ise[k] = rsqrt(st->e[k]);
  __syncthreads();
  double dev = 0.0;
  for (int idx = tid; idx < R * R; idx += nt) {
    const int r = idx / R, c = idx % R;
    a.G[idx] = 0.0;   // its content is in LDS
    if (c < r) continue;
    const double o = 0.5 * (Gs[r * SG + c] + Gs[c * SG + r]) * s_ise[r] * s_ise[c];
    dev = fmax(dev, fabs(o - (r == c ? 1.0 : 0.0)));
  }
  dev = block_max(dev, scratch);
  if (!(dev > kOrthoTolerance)) {
    __syncthreads();
    if (tid == 0) st->flags &= ~kFlagOrthCheck;
    return;
  }
  // The fix W <- E^{1/2} L^{-1} E^{-1/2} W is applied to the factor it came from: W = A_t B_t, so the triangular
  // mixing matrix goes into A_t and the product with B_t (still in its buffer) is simply launched again, gated on
  // the flag set below.
  const int ti = tid / kOrthTileStride, tj = tid % kOrthTileStride;
  const int row0 = ti * kOrthTileRows;
  const int wave_row0 = (tid >> 6) * kOrthRowsPerWave;   // first row held by this wavefront
  double v[kOrthTileRows][CT];
#pragma unroll
  for (int r = 0; r < kOrthTileRows; ++r) {
    const int i = row0 + r;
    const double ise_i = s_ise[min(i, R - 1)];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int j = tj + kOrthTileStride * c;
      v[r][c] = 0.0;
      if (i < R && j < R) v[r][c] = 0.5 * (Gs[i * SG + j] + Gs[j * SG + i]) * ise_i * s_ise[j];
      if (i < R && j >= R && j < 2 * R) v[r][c] = (double)a.At[i * a.ldat + (j - R)] * ise_i;
    }
  }
  // Two pivots per barrier.  What the pair (k, k + 1) reads: rows k and k + 1 as they stand after pivot k - 1 (with zeros
  // in the columns up to k, which the pair must leave alone), columns k and k + 1 likewise, and the reciprocal of
  // pivot k.  Every thread derives from them what pivot k makes of row k + 1, of column k + 1 and of pivot k + 1 (a
  // few operations on values it has read anyway) and applies both eliminations to its tile at once.  The four lines
  // of the next pair are published by their owners behind the update, in the other of two buffers: the registers of a
  // row or column are met in unrolled loops under uniform compares, so no register is picked by index.
  auto publish = [&](const int kn, const int nb) {   // rows and columns kn, kn + 1 and 1 / pivot kn into buffer nb
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ku = kn + u;
      const int kr = ku % kOrthTileRows, kti = ku / kOrthTileRows;
      const int kc = ku / kOrthTileStride, ktj = ku % kOrthTileStride;
#pragma unroll
      for (int r = 0; r < kOrthTileRows; ++r) {
        if (r == kr && ti == kti) {
#pragma unroll
          for (int c = 0; c < CT; ++c)
            s_prow[nb][u][tj + kOrthTileStride * c] = (tj + kOrthTileStride * c > kn) ? v[r][c] : 0.0;
        }
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        if (c == kc && tj == ktj) {
#pragma unroll
          for (int r = 0; r < kOrthTileRows; ++r) {
            s_pcol[nb][u][row0 + r] = v[r][c];
            if (u == 0 && row0 + r == kn) s_invp[nb] = 1.0 / fmax(v[r][c], 1.0e-300);
          }
        }
      }
    }
  };
  if (row0 < R) publish(0, 0);
  for (int k = 0; k < R - 1; k += 2) {
    const int buf = (k >> 1) & 1, nb = buf ^ 1;
    __syncthreads();
    if (wave_row0 + kOrthRowsPerWave - 1 > k && wave_row0 < R) {   // (uniform over the wavefront) some row lies below k
      const int k1 = k + 1;   // (k1 <= R - 1: a row of the matrix; as the last row it eliminates nothing)
      const double inv0 = s_invp[buf];
      const double m = s_pcol[buf][0][k1] * inv0;            // what pivot k takes off row k + 1
      const double a01 = s_prow[buf][0][k1];                 // entry (k, k + 1)
      const double inv1 = 1.0 / fmax(s_pcol[buf][1][k1] - m * a01, 1.0e-300);   // pivot k + 1 after pivot k
      double f[kOrthTileRows], gq[kOrthTileRows], p0[CT], q1[CT];
#pragma unroll
      for (int r = 0; r < kOrthTileRows; ++r) {
        const int i = row0 + r;
        const double c0 = s_pcol[buf][0][i], c1 = s_pcol[buf][1][i];
        f[r] = (i > k && i < R) ? c0 * inv0 : 0.0;
        gq[r] = (i > k1 && i < R) ? (c1 - f[r] * a01) * inv1 : 0.0;
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const int j = tj + kOrthTileStride * c;
        p0[c] = s_prow[buf][0][j];
        q1[c] = (j > k1) ? s_prow[buf][1][j] - m * p0[c] : 0.0;   // row k + 1 after pivot k, dead columns zero
      }
#pragma unroll
      for (int r = 0; r < kOrthTileRows; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) v[r][c] -= f[r] * p0[c] + gq[r] * q1[c];
      if (k + 2 < R - 1) publish(k + 2, nb);
    }
  }
  // D_ii is the diagonal entry of row i as it stood when the row became the pivot row: rows are not touched afterwards
#pragma unroll
  for (int r = 0; r < kOrthTileRows; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c)
      if (row0 + r < R && tj + kOrthTileStride * c == row0 + r) s_dinv[row0 + r] = rsqrt(fmax(v[r][c], 1.0e-300));
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kOrthTileRows; ++r) {
    const int i = row0 + r;
    if (i >= R) continue;
    const double scale = s_dinv[i] / s_ise[i];   // E_ii^{1/2} D_ii^{-1/2}
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int j = tj + kOrthTileStride * c;
      if (j >= R && j < 2 * R) a.At[i * a.ldat + (j - R)] = (float)(scale * v[r][c]);
    }
  }
  if (tid == 0) st->flags = (st->flags & ~kFlagOrthCheck) | kFlagReorth;
}

// W_{t+1} = A_t B_t with B_t = J_t + (its factors) W_t (eq. wt1), and for the instances whose update asked for the orthogonality check
// (App. B.3.1) W W^T of the new factor, added to K in fp64, and B_t over J, for the second product if the check fails.  A workgroup
// takes all rows of 64 columns, so it alone reads the columns of W_t that it replaces; a wavefront has 16 of them in registers.
// Bound: latency, above rank 80 with many columns the atomic additions of W W^T (all its tiles instead of those on and above the diagonal:
// 5000 columns rank 80 / 96 15.2 / 19.4 us instead of 13.6 / 17.1, 50000 columns 63.6 / 86.9 instead of 55.8 / 75.6).  As three launches
// (B_t, the product, the gated Gram matrix of its own) 22 / 25 and 64 / 72 us and two gaps of some 2 us.
struct NewFactorArgs {
  const PrecondScalars* st;
  const float* At;
  const float* bt;
  float* J;
  float* W;
  double* K;
  int ldat, ld, R, D;
  int begin;             // first workgroup
};
struct NewFactorGroup {
  int count, total;
  NewFactorArgs a[kMaxInstances];
};
template <int RC>
__device__ __forceinline__ void new_factor_unit(const NewFactorArgs& a, const int chunk) {
  constexpr int TJ = RC / 16, LDA = RC + 4, LDT = 68;
  __shared__ __attribute__((aligned(16))) float lds[RC * (LDA > LDT ? LDA : LDT)];   // A_t, then the workgroup's part of W_(t+1)
  __shared__ float s_f[RC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int R = a.R, D = a.D, col = chunk * 64 + wave * 16 + l16, cc = min(col, D - 1);
  // lane group g takes k = 16 b + 4 g + q in step (b, q), of both operands
  float jv[TJ][4], wv[TJ][4];
#pragma unroll
  for (int b = 0; b < TJ; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t at = (size_t)min(16 * b + 4 * g4 + q, R - 1) * a.ld + cc;
      jv[b][q] = a.J[at];
      wv[b][q] = a.W[at];
    }
  for (int e = tid; e < RC * RC / 4; e += 256) {
    const int i = e / (RC / 4), k = e % (RC / 4) * 4;
    float4 v = *reinterpret_cast<const float4*>(a.At + (size_t)min(i, R - 1) * a.ldat + k);
    const int left = i < R ? R - k : 0;
    v.x = left > 0 ? v.x : 0.f;
    v.y = left > 1 ? v.y : 0.f;
    v.z = left > 2 ? v.z : 0.f;
    v.w = left > 3 ? v.w : 0.f;
    *reinterpret_cast<float4*>(&lds[i * LDA + k]) = v;
  }
  if (tid < RC) s_f[tid] = tid < R ? a.bt[tid] : 0.f;
  const bool check = (a.st->flags & kFlagOrthCheck) != 0;   // (uniform)
  __syncthreads();
#pragma unroll
  for (int b = 0; b < TJ; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * b + 4 * g4 + q;
      const float v = fmaf(s_f[k], wv[b][q], jv[b][q]);
      jv[b][q] = k < R ? v : 0.f;
      if (check && k < R && col < D) a.J[(size_t)k * a.ld + col] = v;
    }
  floatx4 acc[TJ];
#pragma unroll
  for (int t = 0; t < TJ; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int b = 0; b < TJ; ++b) {
    float4 af[TJ];
#pragma unroll
    for (int t = 0; t < TJ; ++t) af[t] = *reinterpret_cast<const float4*>(&lds[(16 * t + l16) * LDA + 16 * b + 4 * g4]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int t = 0; t < TJ; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(pick4(af[t], q), jv[b][q], acc[t], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < TJ; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 16 * t + 4 * g4 + q;
      if (i < R && col < D) a.W[(size_t)i * a.ld + col] = acc[t][q];
    }
  if (!check) return;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TJ; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) lds[(16 * t + 4 * g4 + q) * LDT + wave * 16 + l16] = col < D ? acc[t][q] : 0.f;
  __syncthreads();
  for (int tile = wave; tile < TJ * TJ; tile += 4) {
    const int i0 = tile / TJ * 16, j0 = tile % TJ * 16;
    if (i0 > j0) continue;   // (uniform)
    doublex4 c = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 64; k += 4)
      c = __builtin_amdgcn_mfma_f64_16x16x4f64((double)lds[(i0 + l16) * LDT + k + g4], (double)lds[(j0 + l16) * LDT + k + g4], c, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 4 * r + g4, j = j0 + l16;
      if (i < R && j < R) unsafeAtomicAdd(a.K + (size_t)i * R + j, c[r]);
    }
  }
}
// Grid: 64-column blocks of all instances; 256 threads.
template <int RC>
__global__ __launch_bounds__(256) void new_factor_kernel(const NewFactorGroup g) {
  int pi = 0;
  for (int i = 1; i < g.count; ++i)
    if ((int)blockIdx.x >= g.a[i].begin) pi = i;
  new_factor_unit<RC>(g.a[pi], (int)blockIdx.x - g.a[pi].begin);
}
// Up to rank 32, one instance: beside it what finishes the call's output.
__global__ __launch_bounds__(256) void new_factor_finish_kernel(const NewFactorArgs a, const int chunks, const FinishArgs finish) {
  if ((int)blockIdx.x >= chunks)
    finish_rows<true>(finish, (int)blockIdx.x - chunks);
  else
    new_factor_unit<32>(a, blockIdx.x);
}

}  // namespace ngsgd
