// Element-wise and row-reduction kernels of the NG-SGD step (gfx950, 64-lane wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "state.h"
#include "wave_f64.h"

namespace ngsgd {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// Sum over a workgroup (any multiple of 64 threads up to 1024); `scratch` holds >= 16 doubles.
__device__ __forceinline__ double block_sum(double v, double* scratch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < nw; ++w) t += scratch[w];
  return t;
}
__device__ __forceinline__ double block_max(double v, double* scratch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  double t = scratch[0];
  for (int w = 1; w < nw; ++w) t = fmax(t, scratch[w]);
  return t;
}

// ---- fills and copies ----------------------------------------------------------------------------
__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// Clears several buffers in one launch: grid (blocks, count).
struct FillGroup {
  int count;
  uint32_t* ptr[kMaxInstances];
  size_t n[kMaxInstances];
};
__global__ void fill_zero_group_kernel(const FillGroup g) {
  uint32_t* p = g.ptr[blockIdx.y];
  const size_t n = g.n[blockIdx.y];
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// out[n][0..D) = x[n][0..D), out[n][D] = 1, out[n][D+1..ldo) = 0   (input with the bias 1 appended, Sec. 4.4)
// Also clears *clear (the step's objective accumulator), if given.
__global__ void copy_append_ones_kernel(const float* __restrict__ x, int ldx, float* __restrict__ out, int ldo,
                                        int N, int D, double* __restrict__ clear) {
  const int row = blockIdx.y;
  if (row >= N) return;   // the grid's second dimension is the row count
  if (clear != nullptr && row == 0 && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0.0;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < ldo; c += gridDim.x * blockDim.x)
    out[(size_t)row * ldo + c] = c < D ? x[(size_t)row * ldx + c] : (c == D ? 1.f : 0.f);
}

// dense rows x cols  <->  padded (ld) copies
__global__ void copy2d_kernel(const float* __restrict__ src, int lds_, float* __restrict__ dst, int ldd, int rows,
                              int cols, float scale, const double* scale_dev) {
  const int row = blockIdx.y;
  if (row >= rows) return;   // the grid's second dimension is the row count
  float s = scale;
  if (scale_dev != nullptr) s *= (float)(*scale_dev);
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < cols; c += gridDim.x * blockDim.x)
    dst[(size_t)row * ldd + c] = s * src[(size_t)row * lds_ + c];
}

// Rows are 16-byte aligned and ld is a multiple of 4 (checked by the callers): 16 bytes per lane, tail by elements.
__global__ void scale_rows_kernel(float* __restrict__ M, int ld, int N, int D, const double* __restrict__ gamma) {
  const int row = blockIdx.y;
  if (row >= N) return;   // the grid's second dimension is the row count
  const float s = (float)(*gamma);
  float* m = M + (size_t)row * ld;
  const int d4 = D & ~3;
  for (int c = 4 * (blockIdx.x * blockDim.x + threadIdx.x); c < d4; c += 4 * gridDim.x * blockDim.x) {
    float4 v = *reinterpret_cast<float4*>(m + c);
    v.x *= s; v.y *= s; v.z *= s; v.w *= s;
    *reinterpret_cast<float4*>(m + c) = v;
  }
  if (blockIdx.x == 0 && threadIdx.x < D - d4) m[d4 + threadIdx.x] *= s;
}

// ---- nonlinearities ------------------------------------------------------------------------------
// The derivative w.r.t. a layer's input arrives as n_slabs partial products (split-K slabs of the backward
// GEMM, slab_stride floats apart) that are summed here in a fixed order.
// The loads of up to eight slabs are requested together (backward kernel of a p-norm layer,
// 512 rows of 300 groups of ten, eight slabs: 6.7 us, now 5.9).
template <int AT_ONCE>
__device__ __forceinline__ float slab_sum_batched(const float* __restrict__ p, int n_slabs, size_t slab_stride) {
  float v = 0.f;
  for (int s0 = 0; s0 < n_slabs; s0 += AT_ONCE) {
    float x[AT_ONCE];
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) x[u] = p[(size_t)min(s0 + u, n_slabs - 1) * slab_stride];
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) v = s0 + u < n_slabs ? (s0 + u == 0 ? x[u] : v + x[u]) : v;
  }
  return v;
}
__device__ __forceinline__ float slab_sum(const float* __restrict__ p, int n_slabs, size_t slab_stride) {
  if (n_slabs == 1) return p[0];   // uniform
  return n_slabs <= 4 ? slab_sum_batched<4>(p, n_slabs, slab_stride) : slab_sum_batched<8>(p, n_slabs, slab_stride);
}

// O[n][j] = dY[n][j] * (1 - Y[n][j]^2)
__global__ void tanh_backward_kernel(const float* __restrict__ dY, int ldd, int n_slabs, size_t slab_stride,
                                     const float* __restrict__ Y, int ldy, float* __restrict__ O, int ldo, int N,
                                     int D) {
  const int row = blockIdx.y;
  if (row >= N) return;   // the grid's second dimension is the row count
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < D; c += gridDim.x * blockDim.x) {
    const float y = Y[(size_t)row * ldy + c];
    O[(size_t)row * ldo + c] = slab_sum(dY + (size_t)row * ldd + c, n_slabs, slab_stride) * (1.f - y * y);
  }
}

// Workgroup-wide float sum / max for NT-thread workgroups (NT / 64 wavefronts); `red` holds >= NT / 64 floats.
template <int NT>
__device__ __forceinline__ float block_sum_f(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) r += red[w];
  return r;
}
template <int NT>
__device__ __forceinline__ float block_max_f(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) r = fmaxf(r, red[w]);
  return r;
}
__device__ __forceinline__ float block256_sum(float v, float* red) { return block_sum_f<256>(v, red); }
__device__ __forceinline__ float block256_max(float v, float* red) { return block_max_f<256>(v, red); }

// p-norm (p = 2) over groups of G adjacent columns, one NT-thread workgroup per row:
//   y_j = sqrt(sum_k a_{Gj+k}^2);  with renorm: y <- y / max(rms(y), floor), sigma[n] = that divisor.
// Writes Y[n][0..groups), Y[n][groups] = 1, padding zero.
constexpr float kRenormFloor = 1.0e-20f;

template <int NT>
__global__ __launch_bounds__(NT) void pnorm_forward_kernel(const float* __restrict__ A, int lda,
                                                            float* __restrict__ Y, int ldy,
                                                            float* __restrict__ sigma, int N, int groups, int G,
                                                            int renorm) {
  __shared__ float red[NT / 64];
  const int row = blockIdx.x;
  if (row >= N) return;   // one workgroup per row (uniform over the workgroup)
  const float* a = A + (size_t)row * lda;
  float* y = Y + (size_t)row * ldy;
  float ss = 0.f;
  // a thread keeps the (few) groups it computes in registers until the row's scale is known
  constexpr int kMaxOwn = 2048 / NT;   // groups per thread: rows of up to 2048 groups stay in registers
  float own[kMaxOwn];
#pragma unroll
  for (int u = 0; u < kMaxOwn; ++u) {
    const int j = threadIdx.x + u * NT;
    float s = 0.f;
    if (j < groups) {
      const float* g = a + (size_t)j * G;
      if ((G & 1) == 0) {
        for (int k = 0; k < G; k += 2) {
          const float2 v = *reinterpret_cast<const float2*>(g + k);
          s += v.x * v.x + v.y * v.y;
        }
      } else {
        for (int k = 0; k < G; ++k) s += g[k] * g[k];
      }
    }
    own[u] = sqrtf(s);
    ss += s;
  }
  for (int j = threadIdx.x + kMaxOwn * NT; j < groups; j += NT) {   // very wide rows: through memory
    float s = 0.f;
    for (int k = 0; k < G; ++k) s += a[(size_t)j * G + k] * a[(size_t)j * G + k];
    y[j] = sqrtf(s);
    ss += s;
  }
  float inv = 1.f;
  if (renorm) {
    ss = block_sum_f<NT>(ss, red);
    const float sg = fmaxf(sqrtf(ss / (float)groups), kRenormFloor);
    inv = 1.f / sg;
    if (threadIdx.x == 0) sigma[row] = sg;
    for (int j = threadIdx.x + kMaxOwn * NT; j < groups; j += NT) y[j] *= inv;   // written by this thread above
  }
#pragma unroll
  for (int u = 0; u < kMaxOwn; ++u) {
    const int j = threadIdx.x + u * NT;
    if (j < groups) y[j] = own[u] * inv;
  }
  for (int c = groups + threadIdx.x; c < ldy; c += NT) y[c] = c == groups ? 1.f : 0.f;
}

// Backward through (renorm o p-norm), one NT-thread workgroup per row, in place over the affine outputs:
//   AO[n][Gj+k] <- dy_j * a_{Gj+k} / y_j   (0 where y_j = 0)
// with dy = dYn, y = Yn without renorm; with renorm  y = Yn*sigma, dy = (dYn - Yn * mean_j(dYn_j Yn_j)) / sigma.
// dYn arrives as n_slabs partial products (see slab_sum).  The per-group factor dy_j / y_j goes through LDS.
constexpr int kPnormMaxGroupsLds = 4096;
constexpr int kPnormPrefetchPairs = 2048;   // float2 per row held in registers across the reductions (4096 outputs)

template <int NT>
__global__ __launch_bounds__(NT) void pnorm_backward_kernel(const float* __restrict__ dYn, int ldd, int n_slabs,
                                                             size_t slab_stride,
                                                             const float* __restrict__ Yn, int ldy,
                                                             const float* __restrict__ sigma,
                                                             float* __restrict__ AO, int lda, int N, int groups,
                                                             int G, int renorm) {
  constexpr int kPnormPrefetch = kPnormPrefetchPairs / NT;
  __shared__ float red[NT / 64];
  __shared__ float s_f[kPnormMaxGroupsLds];   // first dy_j, then the factor dy_j / y_j
  const int row = blockIdx.x;
  if (row >= N) return;   // one workgroup per row (uniform over the workgroup)
  const float* dy = dYn + (size_t)row * ldd;
  const float* yn = Yn + (size_t)row * ldy;
  float* ao = AO + (size_t)row * lda;
  const int D = groups * G;
  // the affine outputs this thread will rescale are requested first: they arrive while the row's factors are made
  const bool vec2 = (G & 1) == 0 && (lda & 1) == 0;
  float2* ao2 = reinterpret_cast<float2*>(ao);
  float2 pre[kPnormPrefetch];
  if (vec2) {
#pragma unroll
    for (int u = 0; u < kPnormPrefetch; ++u) {
      const int c2 = threadIdx.x + u * NT;
      if (c2 < D / 2) pre[u] = ao2[c2];
    }
  }
  float dot = 0.f;
  for (int j = threadIdx.x; j < groups; j += NT) {
    const float d = slab_sum(dy + j, n_slabs, slab_stride);
    s_f[j] = d;
    dot += d * yn[j];
  }
  float proj = 0.f, sg = 1.f;
  if (renorm) {
    dot = block_sum_f<NT>(dot, red);
    sg = sigma[row];
    proj = sg > kRenormFloor ? dot / (float)groups : 0.f;
  }
  const float inv_sg = 1.f / sg;
  for (int j = threadIdx.x; j < groups; j += NT) {   // each thread rewrites the entries it wrote above
    const float ynj = yn[j];
    const float d = (s_f[j] - ynj * proj) * inv_sg;
    const float yj = ynj * sg;
    s_f[j] = yj > 0.f ? d / yj : 0.f;
  }
  __syncthreads();
  if (vec2) {
    const int half_g = G / 2;
#pragma unroll
    for (int u = 0; u < kPnormPrefetch; ++u) {
      const int c2 = threadIdx.x + u * NT;
      if (c2 < D / 2) {
        const float f = s_f[c2 / half_g];
        ao2[c2] = make_float2(pre[u].x * f, pre[u].y * f);
      }
    }
    for (int c2 = threadIdx.x + kPnormPrefetch * NT; c2 < D / 2; c2 += NT) {
      const float f = s_f[c2 / half_g];
      float2 v = ao2[c2];
      v.x *= f;
      v.y *= f;
      ao2[c2] = v;
    }
  } else {
    for (int c = threadIdx.x; c < D; c += NT) ao[c] *= s_f[c / G];
  }
}

// ---- log-softmax, objective and its derivative (Sec. 2) ------------------------------------------
// One NT-thread workgroup per row, in place: AO[n][c] <- [c == y_n] - softmax(a_n)_c;
// rowobj[n] = log p(y_n | x_n), also added to *total.  Rows of up to 4 * kSoftmaxRowVec classes are read once and kept in registers.
constexpr int kSoftmaxRowVec = 2048;   // float4 per row held in registers

template <int NT>
__global__ __launch_bounds__(NT) void softmax_xent_kernel(float* __restrict__ AO, int ld,
                                                           const int32_t* __restrict__ labels, int N, int C,
                                                           double* __restrict__ rowobj, double* __restrict__ total) {
  constexpr int kSoftmaxVec = kSoftmaxRowVec / NT;   // float4 per thread
  __shared__ float red[NT / 64];
  const int row = blockIdx.x;
  if (row >= N) return;   // one workgroup per row (uniform over the workgroup)
  float* a = AO + (size_t)row * ld;
  const int y = labels[row];
  const bool valid = y >= 0 && y < C;        // an out-of-range label yields NaN, never an out-of-bounds access
  if (C <= 4 * kSoftmaxRowVec) {
    float4 v[kSoftmaxVec];
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < kSoftmaxVec; ++u) {
      const int c = (threadIdx.x + u * NT) * 4;
      float4 t = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      if (c + 3 < C) {
        t = *reinterpret_cast<const float4*>(a + c);
      } else if (c < C) {
        t.x = a[c];
        if (c + 1 < C) t.y = a[c + 1];
        if (c + 2 < C) t.z = a[c + 2];
      }
      v[u] = t;
      m = fmaxf(fmaxf(m, fmaxf(t.x, t.y)), fmaxf(t.z, t.w));
    }
    m = block_max_f<NT>(m, red);
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < kSoftmaxVec; ++u) {
      v[u].x = expf(v[u].x - m);
      v[u].y = expf(v[u].y - m);
      v[u].z = expf(v[u].z - m);
      v[u].w = expf(v[u].w - m);
      s += (v[u].x + v[u].y) + (v[u].z + v[u].w);
    }
    s = block_sum_f<NT>(s, red);
    if (threadIdx.x == 0) {
      const double lp = valid ? (double)a[y] - ((double)m + log((double)s)) : (double)NAN;
      rowobj[row] = lp;
      unsafeAtomicAdd(total, lp);   // the objective, cleared at the start of the step (fp64: order does not matter)
    }
    __syncthreads();   // a[y] is read before any thread overwrites the row
    const float inv = 1.f / s;
#pragma unroll
    for (int u = 0; u < kSoftmaxVec; ++u) {
      const int c = (threadIdx.x + u * NT) * 4;
      float4 o;
      o.x = (c == y ? 1.f : 0.f) - v[u].x * inv;
      o.y = (c + 1 == y ? 1.f : 0.f) - v[u].y * inv;
      o.z = (c + 2 == y ? 1.f : 0.f) - v[u].z * inv;
      o.w = (c + 3 == y ? 1.f : 0.f) - v[u].w * inv;
      if (c + 3 < C) {
        *reinterpret_cast<float4*>(a + c) = o;
      } else if (c < C) {
        a[c] = o.x;
        if (c + 1 < C) a[c + 1] = o.y;
        if (c + 2 < C) a[c + 2] = o.z;
      }
    }
    return;
  }
  // wider rows: three passes over memory
  float m = -INFINITY;
  for (int c = threadIdx.x; c < C; c += NT) m = fmaxf(m, a[c]);
  m = block_max_f<NT>(m, red);
  float s = 0.f;
  for (int c = threadIdx.x; c < C; c += NT) s += expf(a[c] - m);
  s = block_sum_f<NT>(s, red);
  const float lse = m + logf(s);
  if (threadIdx.x == 0) {
    const double lp = valid ? (double)a[y] - ((double)m + log((double)s)) : (double)NAN;
    rowobj[row] = lp;
    unsafeAtomicAdd(total, lp);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < C; c += NT) a[c] = (c == y ? 1.f : 0.f) - expf(a[c] - lse);
}

// ---- preconditioner helpers -----------------------------------------------------------------------
// After Xhat = X - H W: gamma_t = sqrt(tr(X X^T) / tr(Xhat Xhat^T)) (eq. gammat; 1 if the denominator is 0), the
// squared norms of the output's rows and, with SCALE, gamma Xhat in place of Xhat.
struct FinishArgs {
  PrecondScalars* st;
  const double* sumsq_part;  // partial sums of squares of X
  const double* hat_part;    // and of Xhat, one per tile of the kernel that formed it
  int n_sumsq, n_hat;
  const float* rownorm_part; // [n_col_tiles][N] partial row norms of Xhat
  int n_col_tiles;
  int N;
  double* prow;              // out: p_i (eq. pi), N doubles
  float* gamma_out;          // optional
  float* rownorm2_out;       // optional, gamma^2 p_i
  float* X;                  // N x D, Xhat in place
  int ldx, D;
  // patches the fused apply kernel left undone (its bounded wait ran out): Xhat = X - H W is completed here
  const int* deferred;       // rb * n_col_tiles + chunk for each such patch of 64 rows x chunk_cols columns
  const float* W;            // R x D
  float* H;                  // N x ldh, final
  int ldw, ldh, R, chunk_cols;
  // what the fused apply kernel accumulated into, H and the arrival counters: cleared here, so that the
  // next call without a factor update needs no clearing launch in front of it
  int* arrive;               // [n_arrive], then kFinishSlots numbers that are zero on entry, but for the last one, and on exit:
  int n_arrive;              // 0: not behind the fused apply kernel
  __device__ int* ticket() const { return arrive + n_arrive; }         // workgroups that are done with their deferred patches
  __device__ int* ready() const { return arrive + n_arrive + 1; }      // not 0: gamma is known
  __device__ int* claim() const { return arrive + n_arrive + 2; }      // rows handed out for scaling, by workgroup shares
  __device__ int* left() const { return arrive + n_arrive + 3; }       // workgroups that use none of these any more
  __device__ int* deferred_count() const { return arrive + n_arrive + 4; }
};
constexpr int kFinishSlots = 5;
struct FinishGroup {
  int count;
  FinishArgs a[kMaxInstances];
};

// The sums of both arguments over the 256 threads, to all of them; `red` holds 8 doubles.
__device__ __forceinline__ void block256_sum_pair(double& x, double& y, double* red) {
  x = wave_sum_uniform(x);
  y = wave_sum_uniform(y);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = x;
    red[4 + (threadIdx.x >> 6)] = y;
  }
  __syncthreads();
  x = (red[0] + red[1]) + (red[2] + red[3]);
  y = (red[4] + red[5]) + (red[6] + red[7]);
}

// The way where patches were deferred, of all workgroups of an instance.  They take the patches in turn (plain dot products over
// the rank, 16 threads per row); the one with the last ticket finds all done, forms the sums and gamma and hands out the rows to be
// scaled and the rows of H to be cleared, to itself and to those of the last tickets, which wait for it for a bounded time (nothing
// depends on them).  512 x 5000 rank 80, all patches deferred: 0.41 ms a call (by one workgroup
// 84; the patches by one of 1024 threads and the scaling by a launch of its own 27).
constexpr int kFinishRows = 64, kFinishScaleRows = 2;   // rows of a workgroup, without and with the scaling
constexpr int kFinishHelpers = 512;            // two per compute unit
constexpr long long kFinishWait = 100000;      // 1 ms at the clock's 100 MHz
template <bool SCALE>
__device__ __forceinline__ void finish_deferred(const FinishArgs& a, const int block, const int n_deferred, const int groups, double* red) {
  constexpr int ROWS = SCALE ? kFinishScaleRows : kFinishRows, WIDTH = 256 / ROWS;
  __shared__ int s_at;
  const int tid = threadIdx.x, sub = tid & 15;
  for (int e = block; e < n_deferred; e += groups) {
    const int id = a.deferred[e];
    const int rb = id / a.n_col_tiles, chunk = id % a.n_col_tiles;
    const int c_end = min(a.D, (chunk + 1) * a.chunk_cols);
    for (int r = rb * 64 + (tid >> 4); r < rb * 64 + 64; r += 16) {
      float sq = 0.f;
      if (r < a.N) {
        const float* h = a.H + (size_t)r * a.ldh;
        float* x = a.X + (size_t)r * a.ldx;
        for (int c = chunk * a.chunk_cols + sub; c < c_end; c += 16) {
          float s = 0.f;
          for (int j = 0; j < a.R; ++j) s = fmaf(h[j], a.W[(size_t)j * a.ldw + c], s);
          const float v = x[c] - s;
          x[c] = v;
          sq = fmaf(v, v, sq);
        }
      }
      sq += __shfl_xor(sq, 1);
      sq += __shfl_xor(sq, 2);
      sq += __shfl_xor(sq, 4);
      sq += __shfl_xor(sq, 8);
      if (r < a.N && sub == 0) const_cast<float*>(a.rownorm_part)[(size_t)chunk * a.N + r] = sq;
    }
  }
  __threadfence();   // on all dies before the ticket
  __syncthreads();   // and every wavefront has the deferred count
  if (tid == 0) s_at = __hip_atomic_fetch_add(a.ticket(), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int before = s_at;
  bool ready = before == groups - 1;
  if (ready) {
    __threadfence();   // (what this die holds of the others' patches)
    double t = 0.0, ph = 0.0;
    for (int i = tid; i < a.n_sumsq; i += 256) t += a.sumsq_part[i];
    for (int r = tid; r < a.N; r += 256) {
      double p = 0.0;
      for (int c = 0; c < a.n_col_tiles; ++c) p += (double)a.rownorm_part[(size_t)c * a.N + r];
      a.prow[r] = p;
      ph += p;
    }
    block256_sum_pair(t, ph, red);
    const double gamma = ph > 0.0 ? sqrt(t / ph) : 1.0;
    for (int r = tid; r < a.N && a.rownorm2_out != nullptr; r += 256) a.rownorm2_out[r] = (float)(gamma * gamma * a.prow[r]);   // (its own rows)
    if (tid == 0) {
      a.st->gamma = gamma;
      a.st->tr_M = t;
      a.st->tr_Mhat = ph;
      if (a.gamma_out != nullptr) *a.gamma_out = (float)gamma;
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) __hip_atomic_store(a.ready(), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (before >= groups - 1 - kFinishHelpers) {   // (uniform)
    __syncthreads();
    if (tid == 0) {
      const long long t0 = wall_clock64();
      int seen = 0;
      while ((seen = __hip_atomic_load(a.ready(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0 && wall_clock64() - t0 < kFinishWait)
        __builtin_amdgcn_s_sleep(16);
      s_at = seen;
    }
    __syncthreads();
    ready = s_at != 0;
    __threadfence();
  }
  while (ready) {
    __syncthreads();
    if (tid == 0) s_at = __hip_atomic_fetch_add(a.claim(), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_at >= groups) break;
    const int row0 = s_at * ROWS, row = row0 + tid / WIDTH;
    if (SCALE && row < a.N) {
      const float s = (float)__hip_atomic_load(&a.st->gamma, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      float* const x = a.X + (size_t)row * a.ldx;
      for (int c = tid % WIDTH; c < a.D >> 2; c += WIDTH) {
        float4 v = reinterpret_cast<const float4*>(x)[c];
        v.x *= s; v.y *= s; v.z *= s; v.w *= s;
        reinterpret_cast<float4*>(x)[c] = v;
      }
      for (int c = (a.D & ~3) + tid % WIDTH; c < a.D; c += WIDTH) x[c] *= s;
    }
    float4* const h = reinterpret_cast<float4*>(a.H + (size_t)row0 * a.ldh);
    for (int i = tid; i < min(ROWS, a.N - row0) * a.ldh / 4; i += 256) h[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  if (tid == 0) s_at = __hip_atomic_fetch_add(a.left(), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (s_at == groups - 1)
    for (int i = tid; i < a.n_arrive + kFinishSlots; i += 256) __hip_atomic_store(a.arrive + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Grid (ceil(N / ROWS), instance), 256 threads: every workgroup sums the tiles' partial sums for itself (a few hundred numbers) and
// takes ROWS rows.  Bound: the latency of loads from memory that no cache of
// the workgroup's die holds yet.  With one workgroup per instance, which summed the row norms for the traces and cleared H, and a
// launch of its own for the scaling: 512 x 5000 10.1 + 7.9 us, 512 x 3001 7.8 + 4.9.
template <bool SCALE>
__device__ void finish_rows(const FinishArgs& a, int block);
template <bool SCALE>
__global__ __launch_bounds__(256) void finish_apply_kernel(const FinishGroup g) {
  finish_rows<SCALE>(g.a[blockIdx.y], blockIdx.x);
}
template <bool SCALE>
__device__ __forceinline__ void finish_rows(const FinishArgs& a, const int block) {
  constexpr int ROWS = SCALE ? kFinishScaleRows : kFinishRows;
  __shared__ double red[8], s_row[4][ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, N = a.N, D = a.D;
  const int row0 = block * ROWS, groups = (N + ROWS - 1) / ROWS;
  if (row0 >= N) return;
  const int n_deferred = a.n_arrive > 0 ? *a.deferred_count() : 0;
  // Everything is requested before the first wait: the row pieces that this wavefront scales (256 / ROWS threads take a row) ...
  constexpr int AHEAD = 10, WIDTH = 256 / ROWS;
  float4 x[AHEAD];
  float4* const xrow = reinterpret_cast<float4*>(a.X + (size_t)min(row0 + tid / WIDTH, N - 1) * a.ldx);
  const int d4 = D >> 2, c0 = tid % WIDTH;   // whole pieces
  if (SCALE) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) x[u] = xrow[min(c0 + WIDTH * u, max(d4 - 1, 0))];   // (a row has at least a piece, see ld)
  }
  // ... the partial sums ...
  double t = 0.0, ph = 0.0;
  for (int i = tid; i < a.n_sumsq; i += 256) t += a.sumsq_part[i];
  for (int i = tid; i < a.n_hat; i += 256) ph += a.hat_part[i];
  // ... and the rows' partial norms: 256 / ROWS threads share a row and add every so many'th column tile
  const int r = row0 + tid % ROWS;
  constexpr int STEP = 256 / ROWS;
  float part[2] = {0.f, 0.f};
  if (r < N) {
    for (int c = tid / ROWS; c < a.n_col_tiles; c += 8 * STEP) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = a.rownorm_part[(size_t)min(c + STEP * u, a.n_col_tiles - 1) * N + r];
#pragma unroll
      for (int u = 0; u < 8; ++u) part[u & 1] += c + STEP * u < a.n_col_tiles ? v[u] : 0.f;
    }
  }
  if (n_deferred > 0) {   // (the same for all wavefronts of the instance: it is cleared when all workgroups have left)
    finish_deferred<SCALE>(a, block, n_deferred, groups, red);
    return;
  }
  double p = (double)part[0] + (double)part[1];
#pragma unroll
  for (int off = ROWS; off < 64; off <<= 1) p += __shfl_xor(p, off);
  if (lane < ROWS) s_row[wave][lane] = p;
  block256_sum_pair(t, ph, red);
  const double gamma = ph > 0.0 ? sqrt(t / ph) : 1.0;
  if (tid < ROWS && r < N) {
    p = (s_row[0][tid] + s_row[1][tid]) + (s_row[2][tid] + s_row[3][tid]);
    a.prow[r] = p;
    if (a.rownorm2_out != nullptr) a.rownorm2_out[r] = (float)(gamma * gamma * p);
  }
  if (block == 0 && tid == 0) {
    a.st->gamma = gamma;
    a.st->tr_M = t;
    a.st->tr_Mhat = ph;
    if (a.gamma_out != nullptr) *a.gamma_out = (float)gamma;
  }
  if (SCALE && row0 + tid / WIDTH < N) {
    const float s = (float)gamma;
    auto scaled = [&](float4 v) {
      v.x *= s; v.y *= s; v.z *= s; v.w *= s;
      return v;
    };
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (c0 + WIDTH * u < d4) xrow[c0 + WIDTH * u] = scaled(x[u]);
    for (int c = c0 + WIDTH * AHEAD; c < d4; c += WIDTH) xrow[c] = scaled(xrow[c]);
    if (c0 < D - 4 * d4) reinterpret_cast<float*>(xrow)[4 * d4 + c0] *= s;
  }
  if (a.n_arrive > 0) {   // (no workgroup reads H or the counters: nothing was deferred)
    const int rows = min(ROWS, N - row0);
    float4* const h = reinterpret_cast<float4*>(a.H + (size_t)row0 * a.ldh);
    for (int i = tid; i < rows * a.ldh / 4; i += 256) h[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (block == 0)
      for (int i = tid; i < a.n_arrive; i += 256) a.arrive[i] = 0;
  }
}

// Rank 0: no factor, the output is the input; only the row norms are produced.  One workgroup per row block.
__global__ __launch_bounds__(256) void rownorm_kernel(const float* __restrict__ M, int ld, int N, int D,
                                                      double* __restrict__ prow, float* __restrict__ rownorm2_out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= N) return;
  float s = 0.f;
  for (int c = lane; c < D; c += 64) {
    const float v = M[(size_t)row * ld + c];
    s += v * v;
  }
  s = wave_sum(s);
  if (lane == 0) {
    prow[row] = (double)s;
    if (rownorm2_out != nullptr) rownorm2_out[row] = s;
  }
}

// W = E^{1/2} R from a state given in definitional form (eq. beta2, etii, wt:def).  One workgroup per row.
__global__ __launch_bounds__(256) void set_state_kernel(const double* __restrict__ Rm, const double* __restrict__ d,
                                                        double rho, double alpha, int R, int D,
                                                        float* __restrict__ W, int ld, PrecondScalars* st) {
  const int i = blockIdx.x;
  double sum_d = 0.0;
  for (int k = 0; k < R; ++k) sum_d += d[k];
  const double beta = rho * (1.0 + alpha) + alpha / (double)D * sum_d;
  const double e = 1.0 / (beta / d[i] + 1.0);
  const double s = sqrt(e);
  for (int c = threadIdx.x; c < ld; c += blockDim.x) W[(size_t)i * ld + c] = c < D ? (float)(s * Rm[(size_t)i * D + c]) : 0.f;
  if (threadIdx.x == 0) {
    st->d[i] = d[i];
    st->e[i] = e;
    if (i == 0) {
      st->rho = rho;
      st->beta = beta;
      st->flags = 0;
    }
  }
}

// ---- parameter averaging (Sec. 3.1) -------------------------------------------------------------
struct AverageArgs {
  int n;
  size_t count;
  float* params[kMaxReplicas];
};
__global__ void average_kernel(const AverageArgs a) {
  const float inv = 1.f / (float)a.n;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < a.count; i += (size_t)gridDim.x * blockDim.x) {
    float s = 0.f;
    for (int r = 0; r < a.n; ++r) s += a.params[r][i];
    s *= inv;
    for (int r = 0; r < a.n; ++r) a.params[r][i] = s;
  }
}

}  // namespace ngsgd
