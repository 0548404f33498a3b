// fp32 matrix products on the bf16 matrix unit of gfx950, without giving up fp32 precision.
//
// Every fp32 operand, times 2^23, is written as the sum of three bf16 numbers, x = h + m + l, each the round-to-nearest
// bf16 of what the ones before left over.  bf16 has the exponent range of fp32 and 8 significant bits, so the three
// together hold all 24 bits of x exactly; with the factor that is so down to the smallest subnormal number, whose last bit
// becomes the smallest normal bf16 number (without it l is subnormal from 2^-109 on, and operands of 2^-118 give results
// with errors of 1e-5 to 1e-4).  A product of two bf16 numbers is exact in fp32, and of the nine partial products
//     a b = hh + (hm + mh) + (hl + mm + lh) + (ml + lm) + ll
// the last three are below 2^-24 |a b| together, half a unit in the last place of an fp32 product: the kernel adds
// the other six.  The matrix unit does them 16 times faster than fp32 products (2.5 PFLOP/s against 157 TFLOP/s), so
// six of them cost 3/8 of one fp32 product.
// At the other end the factor leaves room for operands up to 2^104 and sums up to 2^81; infinities do not split, and
// partial products of different signs may overflow where their sum is an infinity.  All of that ends as an infinity or a
// NaN in the sum: a wavefront that finds one forms that 16 x 16 tile again on the fp32 matrix unit (redo_tile), and that
// result stands: a product is infinite, NaN or large exactly where the fp32 product is.
// Accumulation is fp32 as before.  An instruction adds 32 products instead of 4 (v_mfma_f32_16x16x4_f32), and the matrix
// unit does not round its accumulator additions to nearest, so the shorter chains make long sums more accurate, not less.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm.h"

namespace ngsgd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uint32x2 __attribute__((ext_vector_type(2)));

// What a layer product has besides its operands.
constexpr int kActNone = 0, kActTanh = 1, kActTanhBackward = 2;
struct LayerProblem : GemmProblem {
  // kActTanh: C = tanh(alpha A B), column N of C is one (the bias input) and those up to pad_to are zero.
  // kActTanhBackward: C = alpha A B (1 - Y^2).  Both without split-K and with beta = 0.
  int pad_to, ldy;   // the kernel's ACT
  const float* Y;
  // Maximum parameter change (App. C.3): alpha is multiplied by min(1, mc_bound / (alpha sum_i sqrt(mc_prow[0][i] mc_prow[1][i]))) over
  // mc_rows rows, with the device scalars in alpha, and that factor is stored in *mc_out (mc_out == nullptr: not).
  int mc_rows;
  const double* mc_prow[2];
  double* mc_out;
  double mc_bound;
};
using LayerGroup = GemmGroupOf<kMaxGroup, LayerProblem>;
static_assert(sizeof(LayerGroup) <= 4096, "kernel arguments");
inline void plan_extra(const GemmDesc& d, LayerProblem& p) {
  p.pad_to = d.pad_to; p.ldy = d.ldy;
  p.Y = d.Y;
  p.mc_rows = d.mc_rows;
  p.mc_prow[0] = d.mc_prow[0]; p.mc_prow[1] = d.mc_prow[1];
  p.mc_out = d.mc_out;
  p.mc_bound = d.mc_bound;
}

constexpr int kSplitPlanes = 3;
constexpr float kSplitScale = 0x1p23f, kSplitUnscale = 0x1p-46f;   // of an operand; of a product of two

// (x0, x1) -> three words, each holding the two elements' h, m and l.
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t (&out)[kSplitPlanes]) {
  x0 *= kSplitScale;
  x1 *= kSplitScale;
#pragma unroll
  for (int p = 0; p < kSplitPlanes; ++p) {
    const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x0, x1}), bf16x2));
    out[p] = w;
    if (p + 1 < kSplitPlanes) {
      x0 -= __builtin_bit_cast(float, w << 16);
      x1 -= __builtin_bit_cast(float, w & 0xffff0000u);
    }
  }
}

// LDS image of an operand's K-block: three planes of ROWS x BK bf16, 16-byte chunks of eight k values.  The chunks of a
// 128-byte line are permuted so that eight lanes (what one cycle serves) touch every bank once, whether they read one
// chunk of eight consecutive rows, write all chunks of one line or write one chunk of every other row.
template <int ROWS, int BK>
struct SplitTile {
  static_assert(BK == 32 || BK == 64, "one or two rows per 128-byte line");
  static constexpr int PLANE = ROWS * BK * 2;   // bytes
  static constexpr int BYTES = kSplitPlanes * PLANE;
  __device__ __forceinline__ static int chunk_at(int row, int c) {   // byte offset of chunk c of a row in its plane
    if (BK == 64) return row * 128 + ((c ^ (row & 7)) << 4);
    const int slot = ((((row & 1) ^ ((row >> 2) & 1)) << 2) | (c ^ ((row >> 1) & 3)));
    return (row >> 1) * 128 + (slot << 4);
  }
};

// Staging of a K-contiguous operand (element (row, k) at base[row * ld + k]): a piece is four k values of one row.
// Rows beyond the operand are read from a clamped address and left as they are (they only reach rows or columns of C
// that are not stored); the K tail is zeroed in a tile's last K-block.
template <int ROWS, int BK, int NT>
struct SplitStageKC {
  using Tile = SplitTile<ROWS, BK>;
  static constexpr int KQ = BK / 4;
  static constexpr int TOTAL = ROWS * KQ;
  static constexpr int ITER = (TOTAL + NT - 1) / NT;
  using Regs = floatx4[ITER];
  const float* ptr[ITER];
  int kq[ITER];
  int lds_off[ITER];   // -1: surplus lane

  __device__ __forceinline__ void init(const float* __restrict__ base, int ld, int row0, int rows_total, int k_begin, int tid) {
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
      const int f = min(tid + i * NT, TOTAL - 1);
      const int r = f / KQ, q = f % KQ;
      kq[i] = 4 * q;
      ptr[i] = base + (size_t)min(row0 + r, rows_total - 1) * ld + k_begin + kq[i];
      lds_off[i] = (TOTAL % NT == 0 || tid + i * NT < TOTAL) ? Tile::chunk_at(r, q >> 1) + (q & 1) * 8 : -1;
    }
  }
  template <bool LAST>   // the block may reach past k_end
  __device__ __forceinline__ void load(Regs& reg, int k0, int k_end) {
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
      const float* p = ptr[i];
      if (LAST) p -= max(0, k0 + kq[i] - ((k_end - 1) & ~3));   // stay inside the row: the piece is masked anyway
      reg[i] = *reinterpret_cast<const floatx4*>(p);
      ptr[i] += BK;
    }
  }
  __device__ __forceinline__ void mask_tail(Regs& reg, int k0, int k_end) const {
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
      const int left = k_end - (k0 + kq[i]);
      reg[i].x = left > 0 ? reg[i].x : 0.f;
      reg[i].y = left > 1 ? reg[i].y : 0.f;
      reg[i].z = left > 2 ? reg[i].z : 0.f;
      reg[i].w = left > 3 ? reg[i].w : 0.f;
    }
  }
  __device__ __forceinline__ void store(const Regs& reg, char* lds) const {
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
      uint32_t a[kSplitPlanes], b[kSplitPlanes];
      split_pair(reg[i].x, reg[i].y, a);
      split_pair(reg[i].z, reg[i].w, b);
      if (TOTAL % NT == 0 || lds_off[i] >= 0) {
#pragma unroll
        for (int p = 0; p < kSplitPlanes; ++p)
          *reinterpret_cast<uint32x2*>(lds + p * Tile::PLANE + lds_off[i]) = uint32x2{a[p], b[p]};
      }
    }
  }
};

// Staging of a row-contiguous operand (element (row, k) at base[k * ld + row]): a piece is four k values of four
// adjacent rows, four 16-byte loads turned into four rows' half chunks.  (Two rows per piece, so that every staging
// thread of a small tile has one, was slower: twice the loads and address arithmetic for the same bytes.)
template <int ROWS, int BK, int NT>
struct SplitStageRC {
  using Tile = SplitTile<ROWS, BK>;
  static constexpr int KQ = BK / 4;
  static constexpr int RG = ROWS / 4;
  static constexpr int TOTAL = KQ * RG;
  static constexpr int ITER = (TOTAL + NT - 1) / NT;
  static_assert(KQ % 8 == 0 && RG % 8 == 0, "a wavefront covers eight k quadruples by eight row groups");
  using Regs = floatx4[ITER][4];
  const float* ptr[ITER];
  int kq[ITER];
  int lds_off[ITER][4];
  bool ok[ITER];
  int ld_;

  __device__ __forceinline__ void init(const float* __restrict__ base, int ld, int row0, int rows_total, int k_begin, int tid) {
    ld_ = ld;
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
      const int f = min(tid + i * NT, TOTAL - 1);
      // 128-byte segments of the k rows are read whole, and sixteen lanes write to different LDS banks
      const int q = (f & 7) + 8 * ((f >> 6) % (KQ / 8)), rg = ((f >> 3) & 7) + 8 * ((f >> 6) / (KQ / 8));
      kq[i] = 4 * q;
      ptr[i] = base + (size_t)(k_begin + kq[i]) * ld + min(row0 + 4 * rg, (rows_total - 1) & ~3);
      ok[i] = TOTAL % NT == 0 || tid + i * NT < TOTAL;
#pragma unroll
      for (int j = 0; j < 4; ++j) lds_off[i][j] = Tile::chunk_at(4 * rg + j, q >> 1) + (q & 1) * 8;
    }
  }
  template <bool LAST>   // the block may reach past k_end
  __device__ __forceinline__ void load(Regs& reg, int k0, int k_end) {
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* p = ptr[i] + (size_t)e * ld_;
        if (LAST) p -= (size_t)max(0, k0 + kq[i] + e - (k_end - 1)) * ld_;   // stay inside the operand: masked anyway
        reg[i][e] = *reinterpret_cast<const floatx4*>(p);
      }
      ptr[i] += (size_t)BK * ld_;
    }
  }
  __device__ __forceinline__ void mask_tail(Regs& reg, int k0, int k_end) const {
#pragma unroll
    for (int i = 0; i < ITER; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = k0 + kq[i] + e < k_end;
#pragma unroll
        for (int j = 0; j < 4; ++j) reg[i][e][j] = in ? reg[i][e][j] : 0.f;
      }
  }
  __device__ __forceinline__ void store(const Regs& reg, char* lds) const {
#pragma unroll
    for (int i = 0; i < ITER; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t a[kSplitPlanes], b[kSplitPlanes];
        split_pair(reg[i][0][j], reg[i][1][j], a);
        split_pair(reg[i][2][j], reg[i][3][j], b);
        if (TOTAL % NT == 0 || ok[i]) {
#pragma unroll
          for (int p = 0; p < kSplitPlanes; ++p)
            *reinterpret_cast<uint32x2*>(lds + p * Tile::PLANE + lds_off[i][j]) = uint32x2{a[p], b[p]};
        }
      }
  }
};

template <bool KC, int ROWS, int BK, int NT>
struct SplitStageSelect {
  using type = SplitStageKC<ROWS, BK, NT>;
};
template <int ROWS, int BK, int NT>
struct SplitStageSelect<false, ROWS, BK, NT> {
  using type = SplitStageRC<ROWS, BK, NT>;
};

constexpr int kSplitFold = 4;   // K-blocks per MFMA chain

// Four elements (row, k), ..., (row, k + 3) of an operand; TAIL: those from k_end on are zero.
template <bool KC, bool TAIL>
__device__ __forceinline__ floatx4 load_k4(const float* __restrict__ base, const int ld, const int row, const int k, const int k_end) {
  if (KC && !TAIL) return *reinterpret_cast<const floatx4*>(base + (size_t)row * ld + k);
  floatx4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int at = TAIL ? min(k + e, k_end - 1) : k + e;
    const float x = KC ? base[(size_t)row * ld + at] : base[(size_t)at * ld + row];
    v[e] = !TAIL || k + e < k_end ? x : 0.f;
  }
  return v;
}

// The 16 x 16 tile of A B at row m0 and column n0 on the fp32 matrix unit, from memory, laid out as in the kernel below
// (a lane owns four adjacent columns of one row), for tiles that the split cannot form.  Bound: the latency of the loads, the
// operands of up to 64 k values at a time.
template <bool A_KC, bool B_KC>
__device__ __forceinline__ floatx4 redo_tile(const GemmProblem& P, const int m0, const int n0, const int k_begin, const int k_end, const int lane) {
  constexpr int BATCH = A_KC && B_KC ? 4 : (A_KC || B_KC ? 2 : 1);   // (more for row-contiguous operands takes registers from the kernel)
  const int m = min(m0 + (lane & 15), P.M - 1), n = min(n0 + (lane & 15), P.N - 1), k4 = 4 * (lane >> 4);
  floatx4 total = {0.f, 0.f, 0.f, 0.f}, acc = total;
  auto add = [&](const floatx4 a, const floatx4 b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(b[e], a[e], acc, 0, 0, 0);
  };
  int k = k_begin;
  for (; k + 16 * BATCH <= k_end; k += 16 * BATCH) {
    floatx4 a[BATCH], b[BATCH];
#pragma unroll
    for (int t = 0; t < BATCH; ++t) {
      a[t] = load_k4<A_KC, false>(P.A, P.lda, m, k + 16 * t + k4, k_end);
      b[t] = load_k4<B_KC, false>(P.B, P.ldb, n, k + 16 * t + k4, k_end);
    }
#pragma unroll
    for (int t = 0; t < BATCH; ++t) add(a[t], b[t]);
    total += acc;   // chains of at most 64 products
    acc = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  for (; k < k_end; k += 16) add(load_k4<A_KC, true>(P.A, P.lda, m, k + k4, k_end), load_k4<B_KC, true>(P.B, P.ldb, n, k + k4, k_end));
  return total + acc;
}

// C = alpha A B [+ beta C] (slab `split` of it at C + split * c_split_stride), see gemm_kernel for the operands.
// WGM x WGN wavefronts cover the BM x BN tile, WGK of them share the k values of a K-block (their sums are added
// through LDS at the end).  Another PW wavefronts only stage: they load the next K-block, split it and write it to the
// other LDS buffer.  Splitting costs as much vector-ALU time as the products cost matrix-unit time; with both in the
// same wavefronts, in step with each other through the barrier, the two added up (1024 x 2048 x 2049: 55 us with
// eight wavefronts that do both, 50 us with eight that multiply and eight that stage; 512 x 3000 x 301: 11.1 and 10.4 us;
// the factor 2^23 and the look for infinities have since added 6 %).  What bounds it: matrix unit 39 - 52 % busy, LDS 20 - 35 %
// without conflicts, vector ALU issuing in 39 - 58 % of its slots for products of 1024 rows; the rest is the two roles' wait
// for each other at the barrier of every K-block.
template <int BM, int BN, int BK, int WGM, int WGN, int WGK, int PW, bool A_KC, bool B_KC, int ACT>
__global__ __launch_bounds__((WGM * WGN * WGK + PW) * 64) void split_gemm_kernel(const LayerGroup g) {
  constexpr int CW = WGM * WGN * WGK;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int KS = BK / 32 / WGK;   // 32-deep steps of a wavefront per K-block
  static_assert(WM % 16 == 0 && WN % 16 == 0 && KS >= 1 && KS * WGK * 32 == BK, "tile shape");
  using StageA = typename SplitStageSelect<A_KC, BM, BK, PW * 64>::type;
  using StageB = typename SplitStageSelect<B_KC, BN, BK, PW * 64>::type;
  using TileA = SplitTile<BM, BK>;
  using TileB = SplitTile<BN, BK>;
  constexpr int BUF = TileA::BYTES + TileB::BYTES;
  static_assert(WGK <= 2 && (WGK == 1 || TM * TN % 2 == 0), "each K share finishes half of the tiles");
  constexpr int RED = (WGK - 1) * WGM * WGN * 64 * TM * TN * 16;
  __shared__ __attribute__((aligned(16))) char lds[2 * BUF > RED ? 2 * BUF : RED];
  __shared__ double mc_part[CW];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // die-aware numbering of the units, see gemm_kernel
  const int per_xcd = (g.total_tiles + kXcds - 1) / kXcds;
  const int unit = ((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds;
  if (unit >= g.total_tiles) return;   // the grid is rounded up to a multiple of the die count
  int pi = 0;
  for (int i = 1; i < g.count; ++i)
    if (unit >= g.p[i].tile_begin) pi = i;
  const LayerProblem& P = g.p[pi];
  int local = unit - P.tile_begin;
  const int split = local / P.per_split;
  local -= split * P.per_split;
  int tm, tn;
  if (P.tiles_m <= P.tiles_n) {
    tm = local % P.tiles_m;
    tn = local / P.tiles_m;
  } else {
    tn = local % P.tiles_n;
    tm = local / P.tiles_n;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  const int k_begin = split * P.k_per_split;
  const int k_end = min(P.K, k_begin + P.k_per_split);
  const int M = P.M, N = P.N;
  const int nk = (k_end - k_begin + BK - 1) / BK;

  // K-block i is multiplied out of buffer i & 1 while block i + 1 is written to the other one: both roles pass the
  // same nk + 1 barriers (one more where K shares are added).
  if (wave >= CW) {
    const int stid = tid - CW * 64;
    StageA sa;
    StageB sb;
    typename StageA::Regs ra;
    typename StageB::Regs rb;
    sa.init(P.A, P.lda, m0, M, k_begin, stid);
    sb.init(P.B, P.ldb, n0, N, k_begin, stid);
    auto fetch = [&](const int blk) {
      const int k0 = k_begin + blk * BK;
      if (blk < nk - 1) {
        sa.template load<false>(ra, k0, k_end);
        sb.template load<false>(rb, k0, k_end);
      } else {
        sa.template load<true>(ra, k0, k_end);
        sb.template load<true>(rb, k0, k_end);
      }
    };
    auto store = [&](const int blk) {
      sa.store(ra, lds + (blk & 1) * BUF);
      sb.store(rb, lds + (blk & 1) * BUF + TileA::BYTES);
    };
    auto commit = [&](const int blk) {
      if (blk == nk - 1) {
        sa.mask_tail(ra, k_begin + blk * BK, k_end);
        sb.mask_tail(rb, k_begin + blk * BK, k_end);
      }
      store(blk);
    };
    if (nk > 0) {
      fetch(0);
      commit(0);
    }
    if (nk > 1) fetch(1);
    __syncthreads();
    int i = 0;
    for (; i + 3 < nk; ++i) {   // neither block is the last: straight-line code, a piece is reloaded as soon as it is split
      store(i + 1);
      sa.template load<false>(ra, 0, k_end);
      sb.template load<false>(rb, 0, k_end);
      __syncthreads();
    }
    for (; i < nk; ++i) {
      if (i + 1 < nk) commit(i + 1);
      if (i + 2 < nk) fetch(i + 2);
      __syncthreads();
    }
    if (WGK > 1) __syncthreads();
    return;
  }

  const int wk = wave / (WGM * WGN), wmn = wave % (WGM * WGN), wm = wmn / WGN, wn = wmn % WGN;
  const int r16 = lane & 15, g4 = lane >> 4;
  // The product is formed transposed (B's rows as the rows of the MFMA tile): a lane then owns four adjacent columns
  // of one row of C, register q of lane (r16, g4) being C[.. + r16][.. + 4 g4 + q].
  // Two-level sums: an MFMA chain runs over kSplitFold K-blocks and is then added to the total with an ordinary fp32
  // add.  The error grows little with K (update products over 301 / 2049 / 8000 rows: 1.1e-7, 1.3e-7, 1.6e-7 of the result's
  // norm; unbroken chains of fp32 MFMAs: 3.2e-7, 7.8e-7, 1.6e-6).
  floatx4 acc[TM][TN], total[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = total[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        total[i][j] += acc[i][j];
        acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
  };
  // while the first K-block is on its way: alpha, and the maximum-change sum (update products), a share of the rows each
  double alpha_f64 = (double)P.alpha;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (P.alpha_dev[i] != nullptr) alpha_f64 *= *P.alpha_dev[i];
  if (!A_KC && P.mc_out != nullptr) {
    double sum = 0.0;
    for (int r = tid; r < P.mc_rows; r += CW * 64) sum += sqrt(P.mc_prow[0][r] * P.mc_prow[1][r]);
    sum = wave_sum_uniform(sum);
    if (lane == 0) mc_part[wave] = sum;
  }
  __syncthreads();
  for (int i = 0; i < nk; ++i) {
    const char* a_lds = lds + (i & 1) * BUF;
    const char* b_lds = a_lds + TileA::BYTES;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int c = (wk * KS + ks) * 4 + g4;
      bf16x8 af[kSplitPlanes][TM], bf[kSplitPlanes][TN];
#pragma unroll
      for (int p = 0; p < kSplitPlanes; ++p) {
#pragma unroll
        for (int t = 0; t < TM; ++t)
          af[p][t] = *reinterpret_cast<const bf16x8*>(a_lds + p * TileA::PLANE + TileA::chunk_at(wm * WM + t * 16 + r16, c));
#pragma unroll
        for (int t = 0; t < TN; ++t)
          bf[p][t] = *reinterpret_cast<const bf16x8*>(b_lds + p * TileB::PLANE + TileB::chunk_at(wn * WN + t * 16 + r16, c));
      }
      // one product over all tiles at a time: consecutive MFMAs are independent
      constexpr int PA[6] = {0, 1, 0, 1, 2, 0}, PB[6] = {0, 0, 1, 1, 0, 2};
#pragma unroll
      for (int x = 0; x < 6; ++x)
#pragma unroll
        for (int ti = 0; ti < TM; ++ti)
#pragma unroll
          for (int tj = 0; tj < TN; ++tj)
            acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[PB[x]][tj], af[PA[x]][ti], acc[ti][tj], 0, 0, 0);
    }
    if (i % kSplitFold == kSplitFold - 1) fold();
    __syncthreads();
  }
  fold();

  // With two K shares each of them finishes half of the tiles: the other half's sums are handed over through LDS.
  auto owned = [&](const int i, const int j) { return WGK == 1 || (TM % 2 == 0 ? i / ((TM + 1) / 2) : j / ((TN + 1) / 2)) == wk; };
  if (WGK > 1) {
    floatx4* red = reinterpret_cast<floatx4*>(lds);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if (!owned(i, j)) red[(wmn * (TM * TN) + i * TN + j) * 64 + lane] = total[i][j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if (owned(i, j)) total[i][j] += red[(wmn * (TM * TN) + i * TN + j) * 64 + lane];
  }

  if (!A_KC && P.mc_out != nullptr) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < CW; ++w) sum += mc_part[w];
    const double change = alpha_f64 * sum;
    const double inverse = change < 1.0e300 ? reciprocal_f64(change) : 0.0;   // (its steps make a NaN of an infinity)
    const double scale = change > 0.0 ? fmin(1.0, P.mc_bound * inverse) : 1.0;
    if (unit == P.tile_begin && tid == 0) *P.mc_out = scale;
    alpha_f64 *= scale;
  }
  const float alpha = (float)alpha_f64;
  const float beta = P.beta;
  float* const C = static_cast<float*>(P.C) + (size_t)split * P.c_split_stride;
  auto store = [&](const int i, const int j, const floatx4 sum) {
    const int row = m0 + wm * WM + i * 16 + r16, col = n0 + wn * WN + j * 16 + 4 * g4;
    if (row >= M || col >= N) return;
    float* c = C + (size_t)row * P.ldc + col;
    floatx4 v = alpha * sum;
    if (ACT == kActTanh) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = tanhf(v[q]);
    } else if (ACT == kActTanhBackward) {
      const float* y = P.Y + (size_t)row * P.ldy + col;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float t = y[min(q, N - 1 - col)];
        v[q] *= 1.f - t * t;
      }
    }
    if (col + 4 <= N && (reinterpret_cast<uintptr_t>(c) & 15) == 0) {
      if (beta != 0.f) v += beta * *reinterpret_cast<const floatx4*>(c);
      *reinterpret_cast<floatx4*>(c) = v;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (col + q < N) c[q] = beta != 0.f ? v[q] + beta * c[q] : v[q];
    }
  };
  if (ACT == kActTanh && n0 + BN >= N && n0 < N) {   // behind the last columns: the bias input and the padding
    const int width = P.pad_to - N;
    for (int e = tid; e < BM * width; e += CW * 64) {
      const int row = m0 + e / width, c = e % width;
      if (row < M) C[(size_t)row * P.ldc + N + c] = c == 0 ? 1.f : 0.f;
    }
  }
  bool lost = false;   // an element of C is an infinity or a NaN (rows and columns beyond C hold whatever lies there)
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    float nan_if = 0.f;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (!owned(i, j)) continue;   // uniform, as below
#pragma unroll
      for (int q = 0; q < 4; ++q) nan_if = fmaf(n0 + wn * WN + j * 16 + 4 * g4 + q < N ? total[i][j][q] : 0.f, 0.f, nan_if);
    }
    lost |= m0 + wm * WM + i * 16 + r16 < M && nan_if != 0.f;
  }
  if (!__any(lost)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if (owned(i, j)) store(i, j, kSplitUnscale * total[i][j]);
    return;
  }
  uint32_t redo = 0;   // tiles with such an element
  static_assert(TM * TN <= 32, "a bit per tile");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (!owned(i, j)) continue;
      float nan_if = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) nan_if = fmaf(total[i][j][q], 0.f, nan_if);
      if (__any(nan_if != 0.f)) {
        redo |= 1u << (i * TN + j);
      } else {
        store(i, j, kSplitUnscale * total[i][j]);
      }
    }
  while (redo != 0) {   // uniform
    const int t = __builtin_ctz(redo), i = t / TN, j = t % TN;
    redo &= redo - 1;
    store(i, j, redo_tile<A_KC, B_KC>(P, m0 + wm * WM + i * 16, n0 + wn * WN + j * 16, k_begin, k_end, lane));
  }
}

// Of a GemmDesc the kernel uses the operands, alpha, alpha_dev, beta, the splits and what LayerProblem adds; `gate`, `sym`, `aux` and `sumsq` are
// for gemm_kernel.
// All problems of a launch have the same `act`; tanh goes with the forward layout, its derivative with the backward one.
template <int BM, int BN, int BK, int WGM, int WGN, int WGK, int PW, bool A_KC, bool B_KC>
inline hipError_t launch_split_gemm(const GemmDesc* descs, int count, hipStream_t stream) {
  constexpr int ACT = A_KC ? (B_KC ? kActTanh : kActTanhBackward) : kActNone;
  const int act = count > 0 ? descs[0].act : kActNone;
  for (int i = 0; i < count; ++i) {
    if (descs[i].gate != nullptr || descs[i].sym || descs[i].aux != nullptr || descs[i].sumsq != nullptr) return hipErrorInvalidValue;
    if (descs[i].act != act || (act != kActNone && (act != ACT || descs[i].splits > 1 || descs[i].beta != 0.f))) return hipErrorInvalidValue;
    if (A_KC && descs[i].mc_out != nullptr) return hipErrorInvalidValue;
  }
  constexpr int THREADS = (WGM * WGN * WGK + PW) * 64;
  if constexpr (ACT != kActNone) {
    if (act == ACT) return launch_unit_kernel<BM, BN, BK>(split_gemm_kernel<BM, BN, BK, WGM, WGN, WGK, PW, A_KC, B_KC, ACT>, THREADS, descs, count, stream);
  }
  return launch_unit_kernel<BM, BN, BK>(split_gemm_kernel<BM, BN, BK, WGM, WGN, WGK, PW, A_KC, B_KC, kActNone>, THREADS, descs, count, stream);
}

}  // namespace ngsgd
