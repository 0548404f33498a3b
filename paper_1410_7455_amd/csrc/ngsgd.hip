// C ABI of the NG-SGD minibatch-step library: host-side orchestration of the HIP kernels.
// Declarations and argument contracts are in include/ngsgd.h.
#include "ngsgd.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "fused_apply.h"
#include "gemm.h"
#include "init.h"
#include "kernels.h"
#include "simple_ng.h"
#include "small_update.h"
#include "split_gemm.h"
#include "state.h"

using namespace ngsgd;

namespace {

thread_local int g_last_hip_error = 0;

#define HIP_TRY(expr)                         \
  do {                                        \
    hipError_t e__ = (expr);                  \
    if (e__ != hipSuccess) {                  \
      g_last_hip_error = (int)e__;            \
      return NGSGD_EHIP;                      \
    }                                         \
  } while (0)
#define NG_TRY(expr)                \
  do {                              \
    int rc__ = (expr);              \
    if (rc__ != NGSGD_OK) return rc__; \
  } while (0)
#define LAUNCH_CHECK() HIP_TRY(hipGetLastError())

inline int pad32(int x) { return (x + 31) / 32 * 32; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Carves typed arrays out of a caller-provided device workspace; with base == nullptr it only sizes.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <typename T>
  T* take(size_t n) {
    off = align_up(off, 256);
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += n * sizeof(T);
    return p;
  }
};

// ---- optional per-category kernel timing with HIP events on the launch stream ----------------------
struct Profiler {
  bool on = false;
  std::vector<hipEvent_t> pool;
  struct Rec {
    int cat;
    size_t e0;
  };
  std::vector<Rec> recs;
  size_t used = 0;
  size_t dropped = 0;   // launch groups that found the event pool full since the last read
};
Profiler g_prof;
constexpr size_t kProfMaxEvents = 1 << 16;

struct ProfScope {
  hipStream_t s;
  bool active = false;
  size_t e0 = 0;
  ProfScope(int cat, hipStream_t stream) : s(stream) {
    if (!g_prof.on) return;
    if (g_prof.used + 2 > kProfMaxEvents) {
      g_prof.dropped += 1;
      return;
    }
    while (g_prof.pool.size() < g_prof.used + 2) {
      hipEvent_t e;
      if (hipEventCreate(&e) != hipSuccess) return;
      g_prof.pool.push_back(e);
    }
    e0 = g_prof.used;
    g_prof.used += 2;
    g_prof.recs.push_back({cat, e0});
    active = hipEventRecord(g_prof.pool[e0], s) == hipSuccess;
  }
  ~ProfScope() {
    if (active) (void)hipEventRecord(g_prof.pool[e0 + 1], s);
  }
};

// A group whose work another group's kernel does: no events, time or count, but its place among the groups that are kept between
// reads, so that a program that reads every so many steps meets the limit where it did.
void prof_place() {
  if (!g_prof.on) return;
  if (g_prof.used + 2 > kProfMaxEvents)
    g_prof.dropped += 1;
  else
    g_prof.used += 2;
}

constexpr int kSumsqMax = 1024;   // partial sums of squares per preconditioner call of up to 65536 rows
constexpr int kWideRow = 2048;    // rows at least this wide get 512-thread workgroups in the row-wise kernels
constexpr int kTargetBlocks = 512;

inline int rank_class(int rank) { return rank <= 32 ? 32 : (rank <= 80 ? 80 : 96); }

}  // namespace

// The factor updates of a network's instances run on side streams so that they overlap the rest of the step and
// the next step's forward / backward pass; the new factor is first needed by the next preconditioning.  The
// instances are split over kSideStreams streams by the moment their matrix exists (the last layer's derivatives
// and all layer inputs after the forward pass, the other derivatives as the backward pass produces them), so that
// each group's products H, J and its R x R work start as early as possible.
constexpr int kSideStreams = 3;          // most
// Without the caller's choice one stream, or two (the last layer's derivatives and the layer inputs; the other
// derivatives after the backward pass).  The second one takes the early group out of the chain that the next step waits
// for, and costs a dozen launches and some events per update, and longer gaps on every queue.  It pays where the chain is long
// (ranks above 80, see the tiles of the update) and the early group is most of it: many layers and a last one much wider than the
// others.  Time per step with two over that with one, 180 networks on fresh minibatches:
//   rank above 80, five layers or more, ten times as many classes as the widest hidden layer has outputs or more: 0.979
//   on average (29 networks, 0.92 - 1.03), five to ten times as many 0.996 (12), fewer 1.016 (22), fewer layers 1.005 (17);
//   rank 64 to 80: 1.030 (82, 0.97 - 1.08), 1.017 with that many layers and classes (24); rank 24 to 60: 1.065 (23);
//   the speech-shaped network (rank 80) 1.03: 0.369 - 0.373 ms with one, 0.380 with two.
// A third stream, which starts the upper hidden layers' derivatives in the middle of the backward pass, measured 1 - 2 %
// slower than two on the speech-shaped network.
constexpr int kTwoStreamsAboveRank = 80, kTwoStreamsFromLayers = 5, kTwoStreamsClasses = 10;
inline int default_side_streams(const ngsgd_config& cfg) {
  const int widest = *std::max_element(cfg.dims + 1, cfg.dims + std::max(cfg.n_layers, 2));
  return std::max(cfg.rank_in, cfg.rank_out) > kTwoStreamsAboveRank && cfg.n_layers >= kTwoStreamsFromLayers &&
                 cfg.dims[cfg.n_layers] / kTwoStreamsClasses >= widest
             ? 2
             : 1;
}
struct SideSync {
  hipStream_t stream = nullptr;
  hipEvent_t inputs_ready = nullptr;   // recorded on the caller's stream: the group's matrices exist
  hipEvent_t hj_done = nullptr;        // recorded on the side stream: H, J and the partial sums of tr(X X^T) are final
  hipEvent_t outputs_done = nullptr;   // recorded on the caller's stream: the last reader of W_t (Xhat) has been enqueued
  hipEvent_t done = nullptr;           // recorded on the side stream: W_{t+1}, D_{t+1}, rho_{t+1} are final
  bool pending = false;                // `done` has been recorded and the stepping stream has not waited for it yet
  hipStream_t owner = nullptr;         // the stream the network's latest step was issued on
};

// ---------------------------------------------------------------------------------------------------
struct ngsgd_precond {
  int dim = 0, rank = 0, max_batch = 0;
  double alpha = 4.0, num_samples_history = 2000.0, epsilon = 1e-10;
  int update_period = 4, always_update_first = 10;
  int64_t t = 0;
  int ldw = 0;   // leading dimension of W and J
  int ldh = 0;   // leading dimension of H and A_t (= rank class)
  PrecondScalars* st = nullptr;
  float* zero_region = nullptr;   // [arrival counters, deferred count | H | K | L], cleared before each call
  bool kl_clean = false;          // K and L are known to be clear
  int clean_rows = 0;             // the counters and this many rows of H are known to be clear (left so by the
                                  // finishing kernel of a call that went through the fused apply kernel)
  size_t zero_floats_all = 0;
  size_t arrive_slots = 0;        // arrival counters of the fused apply kernel, one per block of 64 rows, and (last five
  int* arrive = nullptr;          // slots) the finishing kernel's, of which the last is the number of deferred patches; padded to 256 bytes
  int* deferred = nullptr;        // list of deferred patches
  float* H = nullptr;
  float* J = nullptr;
  double* K = nullptr;
  double* L = nullptr;
  float* W = nullptr;
  float* At = nullptr;
  float* rownorm_part = nullptr;
  double* hat_part = nullptr;     // sums of squares of Xhat per tile
  int max_col_tiles = 0;
  double* sumsq_part = nullptr;
  double* prow = nullptr;
  // initialisation scratch
  int n_init_max = 0;
  double* Ai = nullptr;
  double* Vi = nullptr;
  double* Xi = nullptr;
  double* ti = nullptr;
  InitGroup* init_group = nullptr;   // device copy of the instance list of an initialisation this instance leads
  int* idx = nullptr;
  double* vwork = nullptr;
  double* direct = nullptr;       // scratch of a factor update's eigen-problem
  float* bt = nullptr;            // factors of W_t's rows in B_t, from the eigen-problem to the new factor
  bool owned_by_net = false;
  SideSync* sync = nullptr;   // set for instances of a network
  int last_N = 0;             // rows of the latest call
  int fused_columns = kFusedChunk;   // columns of a patch in the last fused launch
  int n_sumsq = 0;            // partial sums of tr(X X^T) its H product left in sumsq_part
};

namespace {

void precond_layout(ngsgd_precond& p, Carver& c) {
  const int R = p.rank, D = p.dim, NB = p.max_batch;
  p.ldw = pad32(D);
  p.ldh = R > 0 ? rank_class(R) : 0;
  p.st = c.take<PrecondScalars>(1);
  p.prow = c.take<double>(NB);
  if (R == 0) return;
  const size_t h_floats = (size_t)NB * p.ldh, kl_floats = (size_t)4 * R * R;   // ldh is a multiple of 16
  p.arrive_slots = align_up((size_t)(NB + kFusedRows - 1) / kFusedRows + kFinishSlots, 64);
  p.zero_floats_all = p.arrive_slots + h_floats + kl_floats;
  p.zero_region = c.take<float>(p.zero_floats_all);
  if (p.zero_region) {
    p.arrive = reinterpret_cast<int*>(p.zero_region);
    p.H = p.zero_region + p.arrive_slots;
    p.K = reinterpret_cast<double*>(p.H + h_floats);
    p.L = p.K + (size_t)R * R;
  }
  p.J = c.take<float>((size_t)R * p.ldw);
  p.W = c.take<float>((size_t)R * p.ldw);
  p.At = c.take<float>((size_t)R * p.ldh);
  p.max_col_tiles = (D + 63) / 64;
  p.rownorm_part = c.take<float>((size_t)p.max_col_tiles * NB);
  p.hat_part = c.take<double>((size_t)p.max_col_tiles * ((NB + 63) / 64));   // (the fused kernel's patches are larger than 64 x 64)
  p.sumsq_part = c.take<double>(std::max(kSumsqMax, (NB + 63) / 64));   // (the H product leaves one per 64 rows at least)
  p.deferred = c.take<int>(kSumsqMax);
  p.n_init_max = NB < D ? NB : D;
  const size_t np_init = align_up(p.n_init_max, kInitPad), rq = align_up(R, 16);
  p.Ai = c.take<double>(std::max(np_init * np_init, 4 * np_init * rq));
  p.Vi = c.take<double>(np_init * np_init);
  p.Xi = c.take<double>(np_init * rq + rq * rq + rq);
  p.ti = c.take<double>(11 * np_init);
  p.init_group = c.take<InitGroup>(1);
  p.idx = c.take<int>(kMaxRank);
  p.vwork = c.take<double>((size_t)kMaxRank + D);
  p.direct = c.take<double>(direct_scratch_doubles(R));
  p.bt = c.take<float>(R);
}

int precond_check_config(int dim, int rank, int max_batch, float alpha, float S, float eps, int period, int first) {
  if (dim < 1 || rank < 0 || rank > NGSGD_MAX_RANK || rank >= dim || max_batch < 1) return NGSGD_EINVAL;
  if (!(alpha >= 0.f) || !(S > 0.f) || !(eps > 0.f) || period < 1 || first < 0) return NGSGD_EINVAL;
  return NGSGD_OK;
}

void precond_configure(ngsgd_precond& p, int dim, int rank, int max_batch, float alpha, float S, float eps,
                       int period, int first) {
  p.dim = dim;
  p.rank = rank;
  p.max_batch = max_batch;
  p.alpha = alpha;
  p.num_samples_history = S;
  p.epsilon = eps;
  p.update_period = period;
  p.always_update_first = first;
  p.t = 0;
}

bool g_attr_done = false;
constexpr int kEigLdsReserve = 126 * 1024;   // dynamic LDS of a large eigen-update workgroup (of 160 KB per compute unit)
constexpr int kEigReserveFromRank = 48;

// Of the first kernel's LDS the reflections take a part already.
template <int K>
constexpr int kEigReduceReserve = kEigLdsReserve - DirectShape<K>::T * DirectShape<K>::T * (int)sizeof(double);
template <int K, int ITEMS>
hipError_t eig_attributes() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(eig_reduce_kernel<K, false>), hipFuncAttributeMaxDynamicSharedMemorySize, kEigReduceReserve<K>);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(eig_finish_kernel<K, ITEMS, kEigThreads, false, false>),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             kEigLdsReserve);
}
// The three kernels of an R x R update above rank 32.  A large eigen-problem is a long sequential chain bound by latency, on which
// the next step waits: its single workgroups ask for most of the compute unit's LDS, so that no workgroup of the layer
// products (which live on LDS bandwidth) is placed next to them.  That costs the products one compute unit in 256 per instance.
// With work beside them there are no layer products to keep away.
template <int K, int ITEMS>
hipError_t launch_eig(const SmallGroup& g, const int n, const int r_max, const Beside* beside, hipStream_t s) {
  if (beside != nullptr) {
    hipLaunchKernelGGL((eig_reduce_kernel<K, true>), dim3(kBesideFirst + beside->xhat_blocks()), dim3(kEigReduceThreads), 0, s, g, *beside);
    hipLaunchKernelGGL((eig_pairs_kernel<K, true>), dim3((r_max + 3) / 4 + Beside::row_blocks(beside->finish.N)), dim3(256), 0, s, g, *beside);
  } else {
    const size_t reserve = r_max >= kEigReserveFromRank ? kEigReduceReserve<K> : 0;
    hipLaunchKernelGGL((eig_reduce_kernel<K, false>), dim3(n), dim3(kEigReduceThreads), reserve, s, g, NothingBeside());
    hipLaunchKernelGGL((eig_pairs_kernel<K, false>), dim3(n, (r_max + 3) / 4), dim3(256), 0, s, g, NothingBeside());
  }
  const int half = (r_max + 1) / 2;
  const size_t jacobi = (size_t)2 * 4 * (half * (half + 1) / 2) * sizeof(double);   // two copies of four planes of 2 x 2 blocks
  const size_t direct = (size_t)(DirectShape<K>::T + 16) * DirectShape<K>::STRIDE * sizeof(double);
  hipLaunchKernelGGL((eig_finish_kernel<K, ITEMS, kEigThreads, false, false>), dim3(n, (r_max + 15) / 16), dim3(kEigThreads), std::max(jacobi, direct), s, g,
                     NothingBeside());
  return hipGetLastError();
}
static_assert((kMaxRank / 2) * (kMaxRank / 2 - 1) / 2 <= 2 * (kEigThreads - 64), "2 x 2 blocks of Jacobi's off-diagonal per thread: two");

int ensure_kernel_attributes() {
  if (g_attr_done) return NGSGD_OK;
  HIP_TRY((eig_attributes<3, 1>()));
  HIP_TRY((eig_attributes<5, 1>()));
  HIP_TRY((eig_attributes<6, 2>()));
  {
    const int orth_dyn = kMaxRank * (kMaxRank + 1) * (int)sizeof(double);
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(orth_fix_kernel<2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, orth_dyn));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(orth_fix_kernel<3>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, orth_dyn));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(orth_fix_kernel<5>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, orth_dyn));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(orth_fix_kernel<6>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, orth_dyn));
  }
  HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(init_tri_step_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 3 * kTriLdsCols * (int)sizeof(double)));
  HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(init_eigenvector_kernel<true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kInverseLds));
  g_attr_done = true;
  return NGSGD_OK;
}

inline int choose_splits(int tiles, int ksteps) {
  int s = kTargetBlocks / (tiles > 0 ? tiles : 1);
  if (s < 1) s = 1;
  if (s > ksteps) s = ksteps;
  return s < 1 ? 1 : s;
}

// ---- GEMM dispatch ---------------------------------------------------------------------------------
constexpr int BK = 16;

enum LayerGemm { GEMM_FWD, GEMM_BWD, GEMM_UPD };
constexpr int kMaxBwdSplits = 8;    // split-K slabs of the backward GEMM, summed by the nonlinearity's backward kernel
constexpr int kComputeUnits = 256;

// Tile shapes of the layer GEMMs.  The products of a minibatch step are small next to the chip (a few hundred 64 x 64
// tiles for 256 compute units), so what decides the time is how evenly the tiles fill it: every shape is priced as
// launch + rounds x (fill + K-blocks x time per K-block), and the cheapest is taken.
enum LayerTile { TILE_32x64, TILE_64x64, TILE_64x96, TILE_64x128, TILE_128x128, TILE_64x64_SHALLOW, TILE_COUNT };
constexpr int kTileBM[TILE_COUNT] = {32, 64, 64, 64, 128, 64};
constexpr int kTileBN[TILE_COUNT] = {64, 64, 96, 128, 128, 64};
constexpr int kTileBK[TILE_COUNT] = {64, 64, 64, 64, 32, 32};
// Microseconds: what a round spends besides its K-blocks (first loads, stores), and what 64 k values add per tile of a
// compute unit.  The latter by operand layout (forward: both K-contiguous; backward: A; update: neither), measured on
// 512 x 3000 x 301, 1024 x 2048 x 2049, 600 x 1000 x 1000 (forward), 512 x 300 x 3000 in 8 slabs, 1024 x 2048 x 2048
// (backward) and the grouped update products of both networks.  Three workgroups of the shallow 64 x 64 tile share a
// compute unit: their time per block is per tile all the same, but they are filled together.
constexpr double kTileLaunch = 1.5;
constexpr double kTileFill[TILE_COUNT] = {1.7, 2.1, 2.5, 2.8, 3.5, 2.1};
constexpr int kTileResident[TILE_COUNT] = {1, 1, 1, 1, 1, 3};
constexpr double kTileBlock[3][TILE_COUNT] = {{0.58, 0.90, 1.05, 1.40, 2.15, 0.90},
                                              {0.75, 1.10, 1.30, 1.55, 2.40, 1.06},
                                              {1.00, 1.55, 1.90, 2.10, 2.90, 1.20}};
LayerTile pick_layer_tile(LayerGemm layout, const GemmDesc* d, int n, double* cost_out = nullptr) {
  LayerTile best = TILE_64x64_SHALLOW;
  double best_cost = 0.0;
  for (int t = 0; t < TILE_COUNT; ++t) {
    if (t == TILE_64x64 && layout != GEMM_FWD) continue;   // the shallow one is cheaper for any size, and the only one built
    long long tiles = 0;
    double depth = 0.0;   // k values per tile, averaged over the tiles
    for (int i = 0; i < n; ++i) {
      const int splits = std::max(1, d[i].splits);
      const long long here = (long long)((d[i].M + kTileBM[t] - 1) / kTileBM[t]) *
                             ((d[i].N + kTileBN[t] - 1) / kTileBN[t]) * splits;
      tiles += here;
      depth += (double)here * ((d[i].K + splits - 1) / splits);
    }
    if (tiles == 0) continue;
    const double blocks = std::ceil(depth / (double)tiles / 64.0);
    const double rounds = (double)((tiles + kComputeUnits - 1) / kComputeUnits);
    const double fills = std::ceil(rounds / kTileResident[t]);
    const double cost = kTileLaunch + fills * kTileFill[t] + rounds * blocks * kTileBlock[layout][t];
    if (best_cost == 0.0 || cost < best_cost) {
      best_cost = cost;
      best = (LayerTile)t;
    }
  }
  if (cost_out != nullptr) *cost_out = best_cost;
  return best;
}

template <bool A_KC, bool B_KC>
hipError_t launch_layer_tile(LayerTile t, const GemmDesc* d, int n, hipStream_t s) {
  switch (t) {
    case TILE_32x64: return launch_split_gemm<32, 64, 64, 2, 2, 2, 8, A_KC, B_KC>(d, n, s);
    case TILE_64x96: return launch_split_gemm<64, 96, 64, 2, 2, 2, 8, A_KC, B_KC>(d, n, s);
    case TILE_64x128: return launch_split_gemm<64, 128, 64, 2, 2, 2, 8, A_KC, B_KC>(d, n, s);
    case TILE_128x128: return launch_split_gemm<128, 128, 32, 2, 2, 1, 4, A_KC, B_KC>(d, n, s);
    case TILE_64x64:
      if constexpr (A_KC && B_KC) return launch_split_gemm<64, 64, 64, 2, 2, 2, 8, A_KC, B_KC>(d, n, s);
      break;
    default: break;
  }
  return launch_split_gemm<64, 64, 32, 2, 2, 1, 4, A_KC, B_KC>(d, n, s);
}

// Whether the backward product of a tanh layer is formed without split-K, so that its epilogue can apply the
// derivative: where the longer sums cost less than the launch that would sum the slabs.
constexpr double kTanhBackwardLaunch = 3.0;   // microseconds: 2.6 for 64 x 128, 7.7 for 1024 x 2048 (never split)
bool backward_in_one(GemmDesc d) {
  if (d.splits <= 1) return true;
  double split = 0.0, whole = 0.0;
  (void)pick_layer_tile(GEMM_BWD, &d, 1, &split);
  d.splits = 1;
  (void)pick_layer_tile(GEMM_BWD, &d, 1, &whole);
  return whole <= split + kTanhBackwardLaunch;
}

// `slabs` (optional): how many split-K slabs of the first problem are written.
int launch_layer_gemms(LayerGemm layout, const GemmDesc* d, int n, hipStream_t s, int* slabs = nullptr) {
  const LayerTile t = pick_layer_tile(layout, d, n);
  if (slabs != nullptr) *slabs = kTileBK[t] == 64 ? planned_splits<64, 64, 64>(d[0]) : planned_splits<64, 64, 32>(d[0]);
  switch (layout) {
    case GEMM_FWD: HIP_TRY((launch_layer_tile<true, true>(t, d, n, s))); break;
    case GEMM_BWD: HIP_TRY((launch_layer_tile<true, false>(t, d, n, s))); break;
    case GEMM_UPD: HIP_TRY((launch_layer_tile<false, false>(t, d, n, s))); break;
  }
  return NGSGD_OK;
}

// H = X W^T (split over D, float atomics) with the sum of squares of X as a by-product; two-level accumulation
// (MFMA chains of 64 products) keeps the rounding error of a long split at the level of a short one
constexpr int HBK = 32;          // K-block of the H product
constexpr int kHAccChunk = 2;
template <int RC>
hipError_t launch_h(const GemmDesc* d, int n, hipStream_t s) {
  return launch_gemm_group<64, RC, HBK, 4, 1, true, true, EPI_ATOMIC_F32, true, kHAccChunk>(d, n, s);
}
// J = H^T X, accumulated in fp64 and rounded once to fp32; narrow column tiles instead of a split over the rows
template <int RC>
hipError_t launch_j(const GemmDesc* d, int n, hipStream_t s) {
  if (RC == 32) return launch_gemm_group<32, 32, 32, 2, 2, false, false, EPI_STORE, false, 0, true>(d, n, s);
  return launch_gemm_group<RC, 32, 32, RC / 16, 2, false, false, EPI_STORE, false, 0, true>(d, n, s);
}
// W_{t+1} = A_t B_t
template <int RC>
hipError_t launch_wnew(const GemmDesc* d, int n, hipStream_t s) {
  return launch_gemm_group<RC, 64, BK, RC / 16, 2, true, false, EPI_STORE, false>(d, n, s);
}

template <typename F32, typename F80, typename F96>
hipError_t by_rank_class(int rc, F32 f32, F80 f80, F96 f96) {
  return rc == 32 ? f32() : (rc == 80 ? f80() : f96());
}

// R x R Gram products of the factor update (K = J J^T, L = H^T H, W W^T), fp64 accumulation across the splits of the
// long dimension.  Ranks up to 32: one 32 x 32 tile per instance; above: 64 x 64 tiles (a single 80 x 80 tile with one
// row of MFMA tiles per wavefront was measured slower at rank 80: 399 instead of 387 us for the 512 x 5000 call,
// fewer and longer workgroups)
hipError_t launch_small_gram(int rc, const GemmDesc* d, int n, hipStream_t s) {
  if (rc == 32) return launch_gram_group<32, 32, BK, 2, 1>(d, n, s);
  return launch_gram_group<64, 64, BK, 2, 2>(d, n, s);
}
constexpr int kGramMinSplitSteps = 4;   // K-blocks per split of a 32 x 32 tile at least: below that the atomic epilogue dominates
inline int gram_splits(int rc, int rank, int instances, int k) {
  const int ksteps = (k + BK - 1) / BK;
  if (rc == 32) return std::min(choose_splits(instances, ksteps), std::max(1, ksteps / kGramMinSplitSteps));
  const int tiles = ((rank + 63) / 64) * ((rank + 63) / 64);
  return choose_splits(tiles * instances, ksteps);
}

struct PrecondCall {
  ngsgd_precond* p;
  float* M;
  int ld;
  int N;
  float* gamma_out;
  float* rownorm2_out;
};

// How long a workgroup of the fused apply kernel waits for the other column chunks of its row block before it
// leaves its patch to the finishing kernel (microseconds; the kernels' clock runs at 100 MHz).
std::atomic<long long> g_fused_wait_us{2000};
// One of the initialisation's reduction waits so many times as long for the others of its matrix to be running: what other streams
// have in front of them are reductions like its own, of up to 0.74 and 2.7 ms.  Three and four replicas on streams, 13 matrices of
// 1024 rows each: with 2 ms up to 7 of them went through memory (52 -> 68 ms, 65 -> 73), from 4 ms on none.
constexpr int tri_wait_factor(const int np_max) { return tri_on_one_die(np_max) ? 2 : 6; }

// Deals the instances to launches of as many workgroups as can be resident together, and to the dies where an instance fits one: the
// largest first, each to the die with the fewest workgroups.
void plan_resident(InitGroup& g, const int np_max, std::vector<int>& launch_units) {
  const bool deal = tri_on_one_die(np_max);
  const int bins = deal ? kTriDies : 1, room = deal ? kTriDieUnits : kTriResidentUnits;
  int order[kMaxInstances], load[kTriDies] = {};
  for (int i = 0; i < g.count; ++i) order[i] = i;
  std::stable_sort(order, order + g.count, [&](const int x, const int y) { return g.a[x].n > g.a[y].n; });
  for (int o = 0; o < g.count; ++o) {
    InitArgs& a = g.a[order[o]];
    const int u = tri_resident_units(a.n, tri_resident_rows(np_max));
    a.place = -1;
    if (u == 0) continue;
    int* bin = std::min_element(load, load + bins);
    if (launch_units.empty() || *bin + u > room) {
      launch_units.push_back(0);
      std::fill(load, load + bins, 0);
      bin = load;
    }
    a.place = ((int)launch_units.size() - 1) * kTriDies + (int)(bin - load);
    *bin += u;
    launch_units.back() = bins * *std::max_element(load, load + bins);
  }
}

int run_init(const std::vector<PrecondCall>& calls, hipStream_t s) {
  ProfScope prof(NGSGD_PROF_INIT, s);
  size_t done = 0;
  while (done < calls.size()) {
    InitGroup g;
    const int n = (int)std::min<size_t>(kMaxInstances, calls.size() - done);
    g.count = n;
    int n_max = 0, ldw_max = 0, r_max = 0;
    for (int i = 0; i < n; ++i) {
      const PrecondCall& c = calls[done + i];
      ngsgd_precond& p = *c.p;
      InitArgs& a = g.a[i];
      a.st = p.st;
      a.M = c.M;
      a.ld = c.ld;
      a.N = c.N;
      a.D = p.dim;
      a.R = p.rank;
      a.use_cov = p.dim <= c.N ? 1 : 0;
      a.n = a.use_cov ? p.dim : c.N;
      a.np = (int)align_up(a.n, kInitPad);
      a.rq = (int)align_up(a.R, 16);
      a.A = p.Ai;
      a.V = p.Vi;
      a.X = p.Xi;
      a.T = p.ti;
      a.idx = p.idx;
      a.W = p.W;
      a.ldw = p.ldw;
      a.vwork = p.vwork;
      n_max = std::max(n_max, a.n);
      ldw_max = std::max(ldw_max, p.ldw);
      r_max = std::max(r_max, p.rank);
      g.alpha = p.alpha;       // one configuration per group (instances of one net share it)
      g.epsilon = p.epsilon;
    }
    const int np_max = (int)align_up(n_max, kInitPad), rq_max = (int)align_up(r_max, 16);
    const bool resident = np_max <= kTriResident;
    std::vector<int> launch_units;   // workgroups of each launch of the reduction that keeps the rows on the chip
    if (resident) plan_resident(g, np_max, launch_units);
    InitGroup* gd = calls[done].p->init_group;
    static_assert(sizeof(InitGroup) % sizeof(uint32_t) == 0 && sizeof(InitGroup) <= 4096, "copied word by word");
    hipLaunchKernelGGL(init_store_group_kernel, dim3(1), dim3(256), 0, s, g, gd);
    LAUNCH_CHECK();
    {
      FillGroup fg;
      fg.count = n;
      std::vector<GemmDesc> rows, cols;
      for (int i = 0; i < n; ++i) {
        const InitArgs& a = g.a[i];
        fg.ptr[i] = reinterpret_cast<uint32_t*>(a.A);
        fg.n[i] = (size_t)a.np * a.np * 2;
        GemmDesc d;
        d.A = a.M; d.lda = a.ld;
        d.C = a.A; d.ldc = a.np;
        d.M = a.n;
        d.K = a.use_cov ? a.N : a.D;
        (a.use_cov ? cols : rows).push_back(d);
      }
      hipLaunchKernelGGL(fill_zero_group_kernel, dim3((unsigned)std::min<size_t>(((size_t)np_max * np_max * 2 + 2047) / 2048, 256), n),
                         dim3(256), 0, s, fg);
      LAUNCH_CHECK();
      if (!rows.empty()) HIP_TRY(launch_sym_gram<true>(rows.data(), (int)rows.size(), s));
      if (!cols.empty()) HIP_TRY(launch_sym_gram<false>(cols.data(), (int)cols.size(), s));
      hipLaunchKernelGGL(init_mirror_kernel, dim3(np_max / 32, np_max / 32, n), dim3(256), 0, s, gd);
      LAUNCH_CHECK();
    }
    const long long limit = g_fused_wait_us.load() * 100 * tri_wait_factor(np_max);
    for (size_t l = 0; l < launch_units.size(); ++l) {
      if (tri_on_one_die(np_max))
        hipLaunchKernelGGL((init_tri_resident_kernel<8, 4>), dim3(launch_units[l]), dim3(256), 0, s, gd, (int)l, limit);
      else
        hipLaunchKernelGGL((init_tri_resident_kernel<16, 2>), dim3(launch_units[l]), dim3(256), 0, s, gd, (int)l, limit);
      LAUNCH_CHECK();
    }
    if (!launch_units.empty()) {   // what of it could not run at once
      hipLaunchKernelGGL(init_tri_shared_kernel, dim3(std::min(kTriSharedUnits, tri_step_units(n_max, 0)), n), dim3(256), 3 * np_max * sizeof(double), s, gd);
      LAUNCH_CHECK();
    }
    for (int j = 0; !resident && j < n_max - kTriTail; ++j) {
      const int groups = tri_step_units(n_max, j);
      if (np_max <= kTriLdsCols) {
        hipLaunchKernelGGL(init_tri_step_kernel, dim3(groups, n), dim3(256), 3 * np_max * sizeof(double), s, gd, j, 3);
      } else {
        hipLaunchKernelGGL(init_tri_step_kernel, dim3(1, n), dim3(256), 0, s, gd, j, 1);
        hipLaunchKernelGGL(init_tri_step_kernel, dim3(groups, n), dim3(256), 0, s, gd, j, 2);
      }
    }
    hipLaunchKernelGGL(init_tri_tail_kernel, dim3(n), dim3(256), 0, s, gd, resident ? 1 : 0);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(init_eigenvalue_kernel, dim3(r_max, n), dim3(64), 0, s, gd);
    LAUNCH_CHECK();
    const int lds_vectors = std::min(kInverseLdsMax, (int)(kInverseLds / inverse_lds_bytes(np_max)));
    if (lds_vectors >= kInverseLdsMin) {
      hipLaunchKernelGGL(init_eigenvector_kernel<true>, dim3((rq_max + lds_vectors - 1) / lds_vectors, n), dim3(64),
                         inverse_lds_bytes(np_max) * lds_vectors, s, gd, lds_vectors);
    } else {
      hipLaunchKernelGGL(init_eigenvector_kernel<false>, dim3((rq_max + 63) / 64, n), dim3(64), 0, s, gd, 64);
    }
    LAUNCH_CHECK();
    for (int second = 0; second < 2; ++second) {
      hipLaunchKernelGGL(init_ortho_gram_kernel, dim3(rq_max / 16, rq_max / 16, n), dim3(256), 0, s, gd, second);
      hipLaunchKernelGGL(init_ortho_factor_kernel, dim3(n), dim3(1024), 0, s, gd);
      hipLaunchKernelGGL(init_ortho_apply_kernel, dim3(np_max / 64, n), dim3(256), 0, s, gd, second);
    }
    LAUNCH_CHECK();
    hipLaunchKernelGGL(init_back_products_kernel, dim3((n_max + 15) / 16, n), dim3(256), 0, s, gd);
    hipLaunchKernelGGL(init_back_kernel, dim3((r_max + 3) / 4, n), dim3(256), 0, s, gd);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(init_select_kernel, dim3(n), dim3(256), 0, s, gd);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(init_rows_kernel, dim3((ldw_max + 63) / 64, n), dim3(256), 0, s, gd);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(init_complete_kernel, dim3(n), dim3(1024), 0, s, gd);
    LAUNCH_CHECK();
    done += n;
  }
  return NGSGD_OK;
}

// Makes stream s wait for a factor update still running on the side stream.  Any stream may ask (an inspection
// call, an averaging call); the update only stops being pending once the stream that steps the network has
// waited for it, because that is the stream the next step's readers of the new factor are ordered on.
int join_side(SideSync* sync, hipStream_t s) {
  if (sync != nullptr && sync->pending) {
    HIP_TRY(hipStreamWaitEvent(s, sync->done, 0));
    if (s == sync->owner) sync->pending = false;
  }
  return NGSGD_OK;
}

// Split-K factor of the H = X W^T product of an N x D input (bounded by the room for its sum-of-squares partials).
// `group` is the number of instances that share the launch: the split only has to fill the chip once for all of
// them, and a split shorter than kMinSplitSteps K-blocks would spend its time in the atomic epilogue.
constexpr int kMinSplitSteps = 6;
int h_splits(int N, int D, int group) {
  const int tiles_m = (N + 63) / 64, ksteps = (D + HBK - 1) / HBK;
  int splits = choose_splits(tiles_m * (group > 0 ? group : 1), ksteps);
  splits = std::min(splits, std::max(1, ksteps / kMinSplitSteps));
  while (splits > 1 && splits * tiles_m > kSumsqMax) --splits;
  return splits;
}

// The online natural-gradient call (App. B.5) for a list of independent instances, in two phases.
//
// precond_apply: everything that touches the N x D matrices (initialisation on the first call, H, J when the
// factor is going to be updated, Xhat, gamma).  With scale_output the matrices are left as gamma * Xhat; without
// it they are left as Xhat and gamma stays in the instance's state for the caller to fold into a later product.
// The instances whose factor is due for an update are appended to `to_update`.
//
// factor_begin / factor_finish: the R x R work and the new factor for those instances (App. B.3); they read only
// what the first phase left in the instances' buffers, so a network runs them on side streams (ngsgd_step).
int precond_validate(const std::vector<PrecondCall>& calls) {
  for (auto& c : calls) {
    const ngsgd_precond& p = *c.p;
    if (c.N < 1 || c.N > p.max_batch || c.ld < p.dim || (c.ld & 3) || !aligned16(c.M)) return NGSGD_EINVAL;
    if (p.rank > 0 && p.t == 0 && c.N <= p.rank) return NGSGD_EINVAL;
  }
  return NGSGD_OK;
}

inline bool factor_due(const ngsgd_precond& p) { return p.t < p.always_update_first || p.t % p.update_period == 0; }

// Clears the accumulation buffers of the listed instances (H always; K, L when the factor is updated) as far as they
// are not still clear from the kernel that ended their last use (the finishing kernel of the fused path, the
// orthogonality check of an update); no kernel is launched when that holds for all of them.
// A call that is being captured runs later and any number of times: it always clears, and clears nothing for the others.
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) != hipSuccess) {
    (void)hipGetLastError();   // (the NULL stream beside a capture: a launch there reports that itself)
    return false;
  }
  return status == hipStreamCaptureStatusActive;
}
int clear_accumulators(const std::vector<PrecondCall>& list, hipStream_t s, const bool captured) {
  for (size_t done = 0; done < list.size();) {
    FillGroup fg;
    const int n = (int)std::min<size_t>(kMaxInstances, list.size() - done);
    fg.count = n;
    size_t n_max = 0;
    for (int i = 0; i < n; ++i) {
      const PrecondCall& c = list[done + i];
      ngsgd_precond& p = *c.p;
      fg.ptr[i] = reinterpret_cast<uint32_t*>(p.zero_region);
      fg.n[i] = factor_due(p) ? p.zero_floats_all : p.arrive_slots + (size_t)c.N * p.ldh;
      if (!captured && p.clean_rows >= c.N && (!factor_due(p) || p.kl_clean)) fg.n[i] = 0;
      p.clean_rows = 0;   // until the kernel that clears them again has been enqueued
      if (factor_due(p)) p.kl_clean = false;
      n_max = std::max(n_max, fg.n[i]);
    }
    done += n;
    if (n_max == 0) continue;
    ProfScope prof(NGSGD_PROF_PRECOND_MISC, s);
    const unsigned blocks = (unsigned)std::min<size_t>((n_max + 2047) / 2048, 64);
    hipLaunchKernelGGL(fill_zero_group_kernel, dim3(blocks > 0 ? blocks : 1, n), dim3(256), 0, s, fg);
    LAUNCH_CHECK();
  }
  return NGSGD_OK;
}

// H = X W^T   (eq. ht) and the partial sums of tr(X X^T) for the listed instances in one launch: the tile is as
// wide as the widest rank class present (a narrower instance wastes matrix-unit work that is small next to the
// cost of a launch of its own).
int launch_h_products(std::vector<PrecondCall>& list, hipStream_t s) {
  if (list.empty()) return NGSGD_OK;
  int rc = 0;
  int class_count[3] = {0, 0, 0};   // the split of an instance is chosen for the instances of its own rank class:
  for (auto& c : list) {            // they carry comparable work, the narrower classes add little to the launch
    rc = std::max(rc, c.p->ldh);
    class_count[c.p->ldh == 32 ? 0 : (c.p->ldh == 80 ? 1 : 2)] += 1;
  }
  std::vector<GemmDesc> d;
  for (auto& c : list) {
    ngsgd_precond& p = *c.p;
    GemmDesc g;
    g.A = c.M; g.lda = c.ld;
    g.B = p.W; g.ldb = p.ldw;
    g.C = p.H; g.ldc = p.ldh;
    g.M = c.N; g.N = p.rank; g.K = p.dim;
    g.sumsq = p.sumsq_part;
    g.splits = h_splits(c.N, p.dim, class_count[p.ldh == 32 ? 0 : (p.ldh == 80 ? 1 : 2)]);
    p.last_N = c.N;
    {
      GemmDesc hd = g;
      p.n_sumsq = planned_sumsq_partials<64, 32, HBK>(hd);   // independent of the tile width
    }
    d.push_back(g);
  }
  ProfScope prof(NGSGD_PROF_PRECOND_H, s);
  HIP_TRY(by_rank_class(rc, [&] { return launch_h<32>(d.data(), (int)d.size(), s); },
                        [&] { return launch_h<80>(d.data(), (int)d.size(), s); },
                        [&] { return launch_h<96>(d.data(), (int)d.size(), s); }));
  return NGSGD_OK;
}

// J = H^T X for the listed instances (must read X before it is overwritten by Xhat).
int launch_j_products(std::vector<PrecondCall>& list, hipStream_t s) {
  for (int rc : {32, 80, 96}) {
    std::vector<GemmDesc> d;
    for (auto& c : list) {
      ngsgd_precond& p = *c.p;
      if (p.ldh != rc) continue;
      GemmDesc g;
      g.A = p.H; g.lda = p.ldh;
      g.B = c.M; g.ldb = c.ld;
      g.C = p.J; g.ldc = p.ldw;
      g.M = p.rank; g.N = p.dim; g.K = c.N;
      d.push_back(g);
    }
    if (d.empty()) continue;
    ProfScope prof(NGSGD_PROF_PRECOND_J, s);
    HIP_TRY(by_rank_class(rc, [&] { return launch_j<32>(d.data(), (int)d.size(), s); },
                          [&] { return launch_j<80>(d.data(), (int)d.size(), s); },
                          [&] { return launch_j<96>(d.data(), (int)d.size(), s); }));
  }
  return NGSGD_OK;
}


inline int fused_chunks(int D, int columns = kFusedChunk) { return (D + columns - 1) / columns; }
inline int fused_row_blocks(int N) { return (N + kFusedRows - 1) / kFusedRows; }

// Whether the fused kernel's bookkeeping has room for this call (partial sums of tr(X X^T) per patch).
inline bool fused_fits(const ngsgd_precond& p, int N) {
  return fused_chunks(p.dim) * fused_row_blocks(N) <= kSumsqMax && (size_t)fused_row_blocks(N) + kFinishSlots <= p.arrive_slots;
}

// Columns of a patch in the launch of calls list[done .. done + n).  Every patch adds its part of H to memory by
// float atomics, and workgroups that run at the same time wait for the slowest of these: wide patches need half as many, but
// are fewer and have two wavefronts per SIMD instead of three.  They are taken from four narrow patches per compute unit on, if
// that takes work off the busiest die (a chunk of columns has one die, and few chunks leave dies idle).  160 / 320 columns, rank
// 80: p-norm network with 512 rows (952 narrow patches) 64 / 78 us, 576 (1071) 82 / 83, 640 (1190) 90 / 89, 700 (1309) 108 / 92, 1024
// (1904) 167 / 125; tanh network of 2048 with 1024 rows (3344) 268 / 178; one matrix of 512 x 5000 (256) 24 / 33, 2048 x 5000
// (1024) 88 / 59, 8192 x 1280 (1024, four wide chunks for eight dies) 69 / 93.
constexpr int kFusedWideUnits = 1023;
int busiest_die(const std::vector<PrecondCall>& list, size_t done, int n, int columns) {
  int load[kXcds] = {}, chunk = 0;
  for (int i = 0; i < n; ++i) {
    const PrecondCall& c = list[done + i];
    for (int k = fused_chunks(c.p->dim, columns); k > 0; --k) load[chunk++ % kXcds] += fused_row_blocks(c.N);
  }
  return *std::max_element(load, load + kXcds);
}
int fused_columns(const std::vector<PrecondCall>& list, size_t done, int n, int rc) {
  int units = 0;
  for (int i = 0; i < n; ++i) units += fused_row_blocks(list[done + i].N) * fused_chunks(list[done + i].p->dim);
  if (rc <= 32 || units <= kFusedWideUnits) return kFusedChunk;
  return 4 * busiest_die(list, done, n, kFusedWide) <= 3 * busiest_die(list, done, n, kFusedChunk) ? kFusedWide : kFusedChunk;
}

template <int RC>
void launch_fused(const FusedGroup& g, int columns, hipStream_t s) {
  if constexpr (RC > 32)
    if (columns == kFusedWide) {
      hipLaunchKernelGGL((fused_apply_kernel<RC, kFusedWide, 64>), dim3(g.total_units), dim3(kFusedThreads), 0, s, g);
      return;
    }
  hipLaunchKernelGGL((fused_apply_kernel<RC, kFusedChunk, kFusedChunk>), dim3(g.total_units), dim3(kFusedThreads), 0, s, g);
}

// Xhat = X - (X W^T) W, row-norm partials and the partial sums of tr(X X^T) in one pass over each matrix
// (eq. ht, hatxt:compute:2, pi), for instances whose factor is not updated by this call.
int launch_fused_apply(std::vector<PrecondCall>& list, hipStream_t s) {
  for (size_t done = 0; done < list.size();) {
    FusedGroup g;
    const int n = (int)std::min<size_t>(kMaxInstances, list.size() - done);
    g.count = n;
    g.spin_limit = g_fused_wait_us.load() * 100;
    int units = 0, chunks = 0, rc = 0;
    for (int i = 0; i < n; ++i) rc = std::max(rc, list[done + i].p->ldh);
    const int columns = fused_columns(list, done, n, rc);
    for (int i = 0; i < n; ++i) {
      const PrecondCall& c = list[done + i];
      ngsgd_precond& p = *c.p;
      FusedArgs& a = g.a[i];
      a.X = c.M; a.ldx = c.ld;
      a.Xout = c.M; a.ldo = c.ld;
      a.W = p.W; a.ldw = p.ldw;
      a.H = p.H; a.ldh = p.ldh;
      a.arrive = p.arrive;
      a.deferred_count = p.arrive + (p.arrive_slots - 1);
      a.deferred = p.deferred;
      a.rownorm_part = p.rownorm_part;
      a.sumsq_part = p.sumsq_part;
      a.hat_part = p.hat_part;
      a.N = c.N; a.D = p.dim; a.R = p.rank;
      a.n_rb = fused_row_blocks(c.N);
      a.n_chunks = fused_chunks(p.dim, columns);
      a.n_chunks_pad = (a.n_chunks + kXcds - 1) / kXcds * kXcds;
      a.first_die = chunks % kXcds;
      chunks += a.n_chunks;
      a.unit_begin = units;
      units += a.n_rb * a.n_chunks_pad;
      p.last_N = c.N;
      p.n_sumsq = a.n_chunks * a.n_rb;
      p.fused_columns = columns;
    }
    g.total_units = units;
    ProfScope prof(NGSGD_PROF_PRECOND_FUSED, s);
    if (rc == 32) {
      launch_fused<32>(g, columns, s);
    } else if (rc == 80) {
      launch_fused<80>(g, columns, s);
    } else {
      launch_fused<96>(g, columns, s);
    }
    LAUNCH_CHECK();
    done += n;
  }
  return NGSGD_OK;
}

// Xhat = X - H W   (eq. hatxt:compute:2), row-norm partials (eq. pi)
GemmDesc xhat_product(const PrecondCall& c) {
  ngsgd_precond& p = *c.p;
  GemmDesc g;
  g.A = p.H; g.lda = p.ldh;
  g.B = p.W; g.ldb = p.ldw;
  g.C = c.M; g.ldc = c.ld;
  g.M = c.N; g.N = p.dim; g.K = p.rank;
  g.aux = p.rownorm_part;
  g.sumsq = p.hat_part;
  return g;
}
// gamma_t, tr(X X^T), tr(Xhat Xhat^T), row norms; gamma Xhat
FinishArgs finish_args(const PrecondCall& c, const bool fused) {
  ngsgd_precond& p = *c.p;
  FinishArgs a;
  a.st = p.st;
  a.sumsq_part = p.sumsq_part;
  a.hat_part = p.hat_part;
  a.n_sumsq = p.n_sumsq;
  a.n_hat = fused ? fused_chunks(p.dim, p.fused_columns) * fused_row_blocks(c.N) : ((p.dim + 63) / 64) * ((c.N + 63) / 64);
  a.rownorm_part = p.rownorm_part;
  a.n_col_tiles = fused ? fused_chunks(p.dim, p.fused_columns) : (p.dim + 63) / 64;
  a.N = c.N;
  a.prow = p.prow;
  a.gamma_out = c.gamma_out;
  a.rownorm2_out = c.rownorm2_out;
  a.X = c.M; a.ldx = c.ld; a.D = p.dim;
  a.deferred = p.deferred;
  a.W = p.W; a.ldw = p.ldw;
  a.H = p.H; a.ldh = p.ldh;
  a.R = p.rank;
  a.chunk_cols = p.fused_columns;
  a.arrive = p.arrive;
  a.n_arrive = fused ? (int)p.arrive_slots - kFinishSlots : 0;
  return a;
}

// With hj_ready the caller has already produced H and J of every instance (all due for an update, none at t = 0)
// and ordered s behind them; only Xhat and gamma remain.
// do_products / do_finish select the two halves of the work on the matrices (the products; the reduction of the
// partial sums to gamma and the row norms), so that a caller can issue the products of different instances at
// different times and reduce once.
int precond_apply(std::vector<PrecondCall>& calls, bool scale_output, hipStream_t s,
                  std::vector<PrecondCall>& to_update_out, bool hj_ready = false, bool do_products = true,
                  bool do_finish = true, Beside* beside = nullptr) {
  std::vector<PrecondCall> full, to_init, to_update;
  const bool captured = capturing(s);
  for (auto& c : calls) {
    ngsgd_precond& p = *c.p;
    if (p.rank == 0) {
      hipLaunchKernelGGL(rownorm_kernel, dim3((c.N + 3) / 4), dim3(256), 0, s, c.M, c.ld, c.N, p.dim, p.prow,
                         c.rownorm2_out);
      LAUNCH_CHECK();
      if (c.gamma_out != nullptr) {
        const uint32_t one_bits = 0x3f800000u;
        hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(c.gamma_out),
                           (size_t)1, one_bits);
        LAUNCH_CHECK();
      }
      continue;
    }
    full.push_back(c);
    if (p.t == 0) to_init.push_back(c);
    if (factor_due(p)) to_update.push_back(c);
  }
  // No factor is updated by this call: one fused pass per matrix instead of the H and Xhat products.
  bool fused = !hj_ready && to_update.empty() && !full.empty();
  for (auto& c : full) fused = fused && fused_fits(*c.p, c.N);
  if (!do_products) {
    // the caller has issued the products already
  } else if (fused) {
    NG_TRY(clear_accumulators(full, s, captured));
    NG_TRY(launch_fused_apply(full, s));
  } else if (!hj_ready) {
    if (!to_init.empty()) NG_TRY(run_init(to_init, s));
    NG_TRY(clear_accumulators(full, s, captured));
    NG_TRY(launch_h_products(full, s));
    NG_TRY(launch_j_products(to_update, s));
  }
  if (beside != nullptr && !to_update.empty()) {   // the rest of this call's output goes with the eigen-problem
    const GemmDesc d = xhat_product(to_update[0]);
    plan_tiles<64, 64, Beside::kBk>(d, beside->xhat.p[0]);
    beside->xhat.p[0].tile_begin = 0;
    beside->xhat.count = 1;
    beside->xhat.total_tiles = beside->xhat.p[0].per_split * beside->xhat.p[0].splits;
    beside->finish = finish_args(to_update[0], false);
    prof_place();   // (the groups of Xhat and of the finishing kernel)
    prof_place();
    to_update_out.push_back(to_update[0]);
    return NGSGD_OK;
  }
  if (!fused && do_products && !full.empty()) {
    std::vector<GemmDesc> d;
    for (auto& c : full) d.push_back(xhat_product(c));
    ProfScope prof(NGSGD_PROF_PRECOND_XHAT, s);
    HIP_TRY((launch_gemm_group<64, 64, BK, 2, 2, true, false, EPI_SUB_ROWNORM, false>(d.data(), (int)d.size(), s)));
  }
  for (size_t done = 0; do_finish && done < full.size();) {
    ProfScope prof(NGSGD_PROF_PRECOND_MISC, s);
    FinishGroup g;
    const int n = (int)std::min<size_t>(kMaxInstances, full.size() - done);
    g.count = n;
    int n_max = 0;
    for (int i = 0; i < n; ++i) {
      const PrecondCall& c = full[done + i];
      g.a[i] = finish_args(c, fused);
      n_max = std::max(n_max, c.N);
    }
    if (scale_output) {
      hipLaunchKernelGGL(finish_apply_kernel<true>, dim3((n_max + kFinishScaleRows - 1) / kFinishScaleRows, n), dim3(256), 0, s, g);
    } else {
      hipLaunchKernelGGL(finish_apply_kernel<false>, dim3((n_max + kFinishRows - 1) / kFinishRows, n), dim3(256), 0, s, g);
    }
    LAUNCH_CHECK();
    if (fused && !captured)
      for (int i = 0; i < n; ++i) full[done + i].p->clean_rows = full[done + i].N;
    done += n;
  }
  if (do_products) to_update_out.insert(to_update_out.end(), to_update.begin(), to_update.end());
  return NGSGD_OK;
}

// Instances of one small-kernel launch share alpha / epsilon / S (instances of one net do): length of the run
// of compatible instances that starts at `done`.
int small_chunk(const std::vector<PrecondCall>& list, size_t done) {
  const ngsgd_precond& p0 = *list[done].p;
  int n = 0;
  while (n < kMaxInstances && done + n < list.size()) {
    const ngsgd_precond& p = *list[done + n].p;
    if (p.alpha != p0.alpha || p.epsilon != p0.epsilon || p.num_samples_history != p0.num_samples_history) break;
    ++n;
  }
  return n;
}

// First half of the factor update (App. B.3): K, L, then Z_t, its eigen-decomposition, rho_{t+1}, D_{t+1}
// and A_t.  Reads H, J and the partial sums of tr(X X^T); leaves W_t alone.
int factor_begin(std::vector<PrecondCall>& to_update, hipStream_t s, Beside* beside = nullptr) {
  if (to_update.empty()) return NGSGD_OK;
  {
    // K = J J^T, L = H^T H, fp64 accumulation across the splits
    std::vector<GemmDesc> d;   // one launch for both
    int rc = 0;
    for (auto& c : to_update) rc = std::max(rc, c.p->ldh);
    for (auto& c : to_update) {
      ngsgd_precond& p = *c.p;
      GemmDesc g;
      g.A = p.J; g.lda = p.ldw;
      g.B = p.J; g.ldb = p.ldw;
      g.C = p.K; g.ldc = p.rank;
      g.M = p.rank; g.N = p.rank; g.K = p.dim;
      g.splits = gram_splits(rc, p.rank, (int)to_update.size(), p.dim);
      g.kc = 1;
      d.push_back(g);
      GemmDesc h;
      h.A = p.H; h.lda = p.ldh;
      h.B = p.H; h.ldb = p.ldh;
      h.C = p.L; h.ldc = p.rank;
      h.M = p.rank; h.N = p.rank; h.K = p.last_N;
      h.splits = gram_splits(rc, p.rank, (int)to_update.size(), p.last_N);
      d.push_back(h);
    }
    ProfScope prof(NGSGD_PROF_PRECOND_KL, s);
    HIP_TRY(launch_small_gram(rc, d.data(), (int)d.size(), s));
  }
  // Z_t, eigen-decomposition, rho_{t+1}, D_{t+1}, A_t
  for (size_t done = 0; done < to_update.size();) {
    SmallGroup g;
    const ngsgd_precond& p0 = *to_update[done].p;
    g.alpha = p0.alpha;
    g.epsilon = p0.epsilon;
    g.num_samples_history = p0.num_samples_history;
    const int n = small_chunk(to_update, done);
    int r_max = 0;
    for (int i = 0; i < n; ++i) {
      const ngsgd_precond& p = *to_update[done + i].p;
      SmallArgs& a = g.a[i];
      a.st = p.st; a.K = p.K; a.L = p.L; a.At = p.At; a.ldat = p.ldh;
      a.R = p.rank; a.D = p.dim; a.N = p.last_N;
      a.direct = p.direct;
      a.bt = p.bt;
      a.sumsq_part = p.sumsq_part;
      a.n_sumsq = p.n_sumsq;
      r_max = std::max(r_max, p.rank);
    }
    g.count = n;
    ProfScope prof(NGSGD_PROF_PRECOND_SMALL, s);
    prof_place();   // (the eigenvectors' group and B_t's)
    prof_place();
    if (r_max <= kEigSmallRank) {
      using Shape = DirectShape<kEigSmallRank / 16>;
      const size_t dyn = 2 * Shape::T * Shape::STRIDE * sizeof(double);
      if (beside != nullptr)
        hipLaunchKernelGGL((eig_finish_kernel<kEigSmallRank / 16, 1, kEigSmallThreads, true, true>), dim3(kBesideFirst + beside->xhat_blocks()),
                           dim3(kEigSmallThreads), dyn, s, g, *beside);
      else
        hipLaunchKernelGGL((eig_finish_kernel<kEigSmallRank / 16, 1, kEigSmallThreads, true, false>), dim3(n), dim3(kEigSmallThreads), dyn, s, g, NothingBeside());
      LAUNCH_CHECK();
    } else if (r_max <= 48) {
      HIP_TRY((launch_eig<3, 1>(g, n, r_max, beside, s)));
    } else if (r_max <= 80) {
      HIP_TRY((launch_eig<5, 1>(g, n, r_max, beside, s)));
    } else {
      HIP_TRY((launch_eig<6, 2>(g, n, r_max, beside, s)));
    }
    done += n;
  }
  return NGSGD_OK;
}

// Second half: W_{t+1} = A_t B_t (eq. wt1) and the orthogonality check of App. B.3.1.  Overwrites W_t, so the
// caller orders it behind the last reader of W_t.
int factor_finish(std::vector<PrecondCall>& to_update, hipStream_t s, const Beside* beside = nullptr) {
  for (size_t done = 0; done < to_update.size();) {
    OrthGroup og;
    const int n = small_chunk(to_update, done);
    int r_max = 0;
    for (int i = 0; i < n; ++i) {
      const ngsgd_precond& p = *to_update[done + i].p;
      OrthArgs& o = og.a[i];
      o.st = p.st; o.G = p.K; o.At = p.At; o.ldat = p.ldh; o.R = p.rank;
      o.clear_ptr = p.zero_region; o.L = p.L;
      o.clear_floats = (int)(p.arrive_slots + (size_t)p.last_N * p.ldh);
      r_max = std::max(r_max, p.rank);
    }
    og.count = n;
    const bool clears = n == 1 || r_max <= kOrthClearRank, counts = clears && !capturing(s);
    // W_{t+1} = A_t B_t; App. B.3.1: W W^T of the new factor, accumulated into K (cleared by the R x R kernel) only for the
    // instances whose update asked for the check
    for (int rc : {32, 80, 96}) {
      NewFactorGroup f;
      f.count = f.total = 0;
      for (int i = 0; i < n; ++i) {
        const ngsgd_precond& p = *to_update[done + i].p;
        if (p.ldh != rc) continue;
        f.a[f.count++] = NewFactorArgs{p.st, p.At, p.bt, p.J, p.W, p.K, p.ldh, p.ldw, p.rank, p.dim, f.total};
        f.total += (p.dim + 63) / 64;
      }
      if (f.count == 0) continue;
      ProfScope prof(NGSGD_PROF_PRECOND_WNEW, s);
      const dim3 grid(f.total), block(256);
      if (rc == 32 && beside != nullptr)
        hipLaunchKernelGGL(new_factor_finish_kernel, dim3(f.total + Beside::row_blocks(beside->finish.N)), block, 0, s, f.a[0], f.total, beside->finish);
      else if (rc == 32)
        hipLaunchKernelGGL(new_factor_kernel<32>, grid, block, 0, s, f);
      else if (rc == 80)
        hipLaunchKernelGGL(new_factor_kernel<80>, grid, block, 0, s, f);
      else
        hipLaunchKernelGGL(new_factor_kernel<96>, grid, block, 0, s, f);
      LAUNCH_CHECK();
    }
    auto launch_product_again = [&]() -> int {
      for (int rc : {32, 80, 96}) {
        std::vector<GemmDesc> d;
        for (int i = 0; i < n; ++i) {
          ngsgd_precond& p = *to_update[done + i].p;
          if (p.ldh != rc) continue;
          GemmDesc w;
          w.A = p.At; w.lda = p.ldh;
          w.B = p.J; w.ldb = p.ldw;
          w.C = p.W; w.ldc = p.ldw;
          w.M = p.rank; w.N = p.dim; w.K = p.rank;
          w.gate = &p.st->flags;
          w.gate_mask = kFlagReorth;
          d.push_back(w);
        }
        if (d.empty()) continue;
        ProfScope prof(NGSGD_PROF_PRECOND_MISC, s);
        HIP_TRY(by_rank_class(rc, [&] { return launch_wnew<32>(d.data(), (int)d.size(), s); },
                              [&] { return launch_wnew<80>(d.data(), (int)d.size(), s); },
                              [&] { return launch_wnew<96>(d.data(), (int)d.size(), s); }));
      }
      return NGSGD_OK;
    };
    prof_place();   // (the group of W W^T)
    {   // the check itself and, if needed, the Cholesky fix
      ProfScope prof(NGSGD_PROF_PRECOND_MISC, s);
      const size_t dyn = (size_t)r_max * (r_max + 1) * sizeof(double);   // W W^T of an instance
      const int ct = orth_columns_per_thread(r_max);   // 2 R / 32 rounded up: 1 .. 6
      if (ct <= 2) {
        hipLaunchKernelGGL(orth_fix_kernel<2>, dim3(n, clears ? kOrthClearBlocks : 1), dim3(kSmallThreads), dyn, s, og);
      } else if (ct <= 3) {
        hipLaunchKernelGGL(orth_fix_kernel<3>, dim3(n, clears ? kOrthClearBlocks : 1), dim3(kSmallThreads), dyn, s, og);
      } else if (ct <= 5) {
        hipLaunchKernelGGL(orth_fix_kernel<5>, dim3(n, clears ? kOrthClearBlocks : 1), dim3(kSmallThreads), dyn, s, og);
      } else {
        hipLaunchKernelGGL(orth_fix_kernel<6>, dim3(n, clears ? kOrthClearBlocks : 1), dim3(kSmallThreads), dyn, s, og);
      }
      LAUNCH_CHECK();
    }
    // where the check failed the kernel has folded the fix into A_t: W_{t+1} = A_t B_t once more for those
    NG_TRY(launch_product_again());
    for (int i = 0; i < n; ++i) {
      ngsgd_precond& p = *to_update[done + i].p;
      if (!counts) continue;
      p.clean_rows = p.last_N;
      p.kl_clean = true;
    }
    done += n;
  }
  return NGSGD_OK;
}

// Largest Xhat, in tiles of 64 x 64, that goes beside the eigen-problem.  The LDS of the eigen-problem's kernels leaves a compute unit three
// workgroups for it above rank 48 and two above 80, and the eigen-problem is soon the shorter part.  Time of an updating call without / with:
//   above 48: 2048 x 6000 (3008 tiles) 1.15 - 1.18, 4096 x 5000 (5056) 1.04 - 1.11, 2048 x 12000 (6016) 1.00 - 1.07, 15000 x 2000 (7520) 0.94 - 1.01,
//             30000 x 1000 (7504) 0.88 - 0.97, 8192 x 5000 (10112) 0.91 - 0.97, 65000 x 5000 (80264) 0.66 - 0.70;
//   up to 32: 12000 x 5000 (14852) 1.01 - 1.04, 16384 x 5000 (20224) 1.00 - 1.02, 65000 x 5000 0.97; 33 to 48: 1.01 - 1.02 there.
int beside_tiles(const int rank) { return rank <= kEigSmallRank ? 16384 : (rank <= 48 ? INT32_MAX : 6144); }

// Both phases for one list of instances on one stream.
int precondition_many(std::vector<PrecondCall>& calls, bool scale_output, hipStream_t s) {
  NG_TRY(ensure_kernel_attributes());
  NG_TRY(precond_validate(calls));
  std::vector<PrecondCall> to_update;
  Beside beside = {};
  Beside* alone = nullptr;
  if (calls.size() == 1 && scale_output) {
    const ngsgd_precond& p = *calls[0].p;
    const long long tiles = (long long)((calls[0].N + 63) / 64) * ((p.dim + 63) / 64);
    if (tiles <= beside_tiles(p.rank)) alone = &beside;
  }
  NG_TRY(precond_apply(calls, scale_output, s, to_update, false, true, true, alone));
  NG_TRY(factor_begin(to_update, s, alone));
  NG_TRY(factor_finish(to_update, s, alone));
  for (auto& c : calls) c.p->t += 1;
  return NGSGD_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------------
// preconditioner C ABI
// ---- simple method (App. A) --------------------------------------------------------------------------
namespace {

struct SimpleWork {   // device scratch of one matrix, carved for up to max_rows x dim
  double* scal = nullptr;
  double* prow = nullptr;
  double* buf[2] = {nullptr, nullptr};
  double* pinv[2] = {nullptr, nullptr};
  float* ginv = nullptr;
  float* Q = nullptr;
  int ldq = 0;
};

void simple_layout(SimpleWork& w, int max_rows, int dim, bool own_prow, Carver& c) {
  const size_t np = (size_t)pad32(std::min(max_rows, dim));
  w.scal = c.take<double>(4);
  w.prow = own_prow ? c.take<double>(max_rows) : nullptr;
  w.buf[0] = c.take<double>(np * np);
  w.buf[1] = c.take<double>(np * np);
  w.pinv[0] = c.take<double>(kSimpleBlock * kSimpleBlock);
  w.pinv[1] = c.take<double>(kSimpleBlock * kSimpleBlock);
  w.ginv = c.take<float>(np * np);
  w.ldq = pad32(dim);
  w.Q = c.take<float>((size_t)max_rows * w.ldq);
}

struct SimpleCall {
  float* M;
  int ld, N, D;
  double alpha, epsilon;
  SimpleWork w;
  double* prow;          // N doubles: ||xhat_i||^2
  double* gamma;         // 1 double
  float* gamma_out;      // optional
  float* rownorm2_out;   // optional
};

constexpr long long kSimpleLateColumns = 8192, kSimpleLatePerRow = 160;   // longest rows whose scaled output is written once

// Enqueues the simple method for a list of independent matrices; every stage is one grouped launch.  With
// scale_output the matrices are left as gamma * Xhat, without it as Xhat with gamma in *gamma.
int simple_many(const std::vector<SimpleCall>& calls, bool scale_output, hipStream_t s) {
  for (auto& c : calls)
    if (c.M == nullptr || c.N < 2 || c.D < 1 || c.ld < c.D || (c.ld & 3) || !aligned16(c.M) || !(c.alpha > 0.0) ||
        !(c.epsilon > 0.0))
      return NGSGD_EINVAL;
  for (size_t done = 0; done < calls.size();) {
    const int cnt = (int)std::min<size_t>(kSimpleMaxGroup, calls.size() - done);
    SimpleGroup g;
    g.count = cnt;
    int nblk_max = 0, n_max = 0;
    for (int i = 0; i < cnt; ++i) {
      const SimpleCall& c = calls[done + i];
      SimpleArgs& a = g.a[i];
      a.M = c.M; a.ld = c.ld; a.Q = c.w.Q; a.ldq = c.w.ldq;
      a.N = c.N; a.D = c.D;
      a.n = c.N > c.D ? c.D : c.N;     // column space if N > D, row space otherwise (App. A.3)
      a.np = pad32(a.n);
      a.nblk = a.np / kSimpleBlock;
      a.alpha = c.alpha; a.epsilon = c.epsilon;
      a.buf[0] = c.w.buf[0]; a.buf[1] = c.w.buf[1];
      a.pinv[0] = c.w.pinv[0]; a.pinv[1] = c.w.pinv[1];
      a.ginv = c.w.ginv;
      a.prow = c.prow; a.scal = c.w.scal; a.gamma = c.gamma;
      a.gamma_out = c.gamma_out; a.rownorm2_out = c.rownorm2_out;
      nblk_max = std::max(nblk_max, a.nblk);
      n_max = std::max(n_max, a.N);
    }
    {
      // Gram matrix in fp64 (split over the long dimension, double atomics)
      ProfScope prof(NGSGD_PROF_SIMPLE_GRAM, s);
      FillGroup fg;
      fg.count = cnt;
      size_t fill_max = 0;
      for (int i = 0; i < cnt; ++i) {
        fg.ptr[i] = reinterpret_cast<uint32_t*>(g.a[i].buf[1]);
        fg.n[i] = (size_t)g.a[i].np * g.a[i].np * 2;
        fill_max = std::max(fill_max, fg.n[i]);
      }
      const unsigned blocks = (unsigned)std::min<size_t>((fill_max + 2047) / 2048, 256);
      hipLaunchKernelGGL(fill_zero_group_kernel, dim3(blocks > 0 ? blocks : 1, cnt), dim3(256), 0, s, fg);
      LAUNCH_CHECK();
      // the Gram matrix is symmetric: only the tiles on and above the diagonal are computed, and the elimination keeps to those
      std::vector<GemmDesc> rows, cols;
      for (int i = 0; i < cnt; ++i) {
        const SimpleArgs& a = g.a[i];
        GemmDesc d;
        d.A = a.M; d.lda = a.ld;
        d.C = a.buf[1]; d.ldc = a.np;
        d.M = a.n;
        d.K = a.N > a.D ? a.N : a.D;
        (a.N > a.D ? cols : rows).push_back(d);   // X^T X: the sum runs over the rows; X X^T: over the columns
      }
      if (!rows.empty()) HIP_TRY(launch_sym_gram<true>(rows.data(), (int)rows.size(), s));
      if (!cols.empty()) HIP_TRY(launch_sym_gram<false>(cols.data(), (int)cols.size(), s));
    }
    {
      // G = beta I + Gram / (N-1), then its inverse, one launch per pivot block
      ProfScope prof(NGSGD_PROF_SIMPLE_INVERSE, s);
      const int tiles = (nblk_max + 1) / 2;   // rows of 64 x 64 tiles
      hipLaunchKernelGGL(simple_prepare_kernel, dim3(tiles, tiles, cnt), dim3(256), 0, s, g);
      LAUNCH_CHECK();
      for (int k = 0; k < nblk_max; ++k) {
        // look-ahead column first
        hipLaunchKernelGGL(simple_sweep_kernel, dim3(tiles + 2, (tiles + 1) / 2, cnt), dim3(256), 0, s, g, k);
        LAUNCH_CHECK();
      }
    }
    {
      // Q = G^{-1} X (row space) or X G^{-1} (column space), per-row factors, gamma
      ProfScope prof(NGSGD_PROF_SIMPLE_APPLY, s);
      std::vector<GemmDesc> rows, cols;
      for (int i = 0; i < cnt; ++i) {
        const SimpleArgs& a = g.a[i];
        GemmDesc d;
        d.C = a.Q; d.ldc = a.ldq;
        d.M = a.N; d.N = a.D; d.K = a.n;
        if (a.N > a.D) {
          d.A = a.M; d.lda = a.ld;         // X, N x D
          d.B = a.ginv; d.ldb = a.np;      // G^{-1} is symmetric: row d of it is column d
          cols.push_back(d);
        } else {
          d.A = a.ginv; d.lda = a.np;      // G^{-1}, N x N
          d.B = a.M; d.ldb = a.ld;         // X stored K x N
          rows.push_back(d);
        }
      }
      if (!rows.empty()) NG_TRY(launch_layer_gemms(GEMM_BWD, rows.data(), (int)rows.size(), s));
      if (!cols.empty()) NG_TRY(launch_layer_gemms(GEMM_FWD, cols.data(), (int)cols.size(), s));
      // The scaled output in one go where the elimination's buffer holds a number per row (of a tall, very narrow matrix it does not) and
      // the rows are not few and long, which leaves most of the chip to the one launch that scales with a workgroup per two rows.
      // Written twice / once: 16 x 8000 49.2 / 47.8 us a call, 12000 50.7 / 51.7, 80000 100 / 130; 64 x 8000 62.1 / 60.3, 20000 76.3 / 78.6;
      // 128 x 20000 109.7 / 108.9, 40000 141 / 146; 256 x 40000 246.1 / 244.3, 80000 417 / 420; 512 x 80000 1155 / 1149.
      bool late = scale_output;
      for (int i = 0; i < cnt; ++i)
        late = late && (size_t)g.a[i].N <= (size_t)g.a[i].np * g.a[i].np && g.a[i].D <= std::max(kSimpleLateColumns, kSimpleLatePerRow * (long long)g.a[i].N);
      if (late) {
        hipLaunchKernelGGL(simple_rows_kernel<true>, dim3(n_max, cnt), dim3(256), 0, s, g);
        LAUNCH_CHECK();
        hipLaunchKernelGGL(simple_scale_kernel, dim3((n_max + kSimpleScaleRows - 1) / kSimpleScaleRows, cnt), dim3(256), 0, s, g);
        LAUNCH_CHECK();
        done += cnt;
        continue;
      }
      hipLaunchKernelGGL(simple_rows_kernel<false>, dim3(n_max, cnt), dim3(256), 0, s, g);
      LAUNCH_CHECK();
      hipLaunchKernelGGL(simple_gamma_kernel, dim3(cnt), dim3(256), 0, s, g);
      LAUNCH_CHECK();
      if (scale_output)
        for (int i = 0; i < cnt; ++i) {
          const SimpleArgs& a = g.a[i];
          hipLaunchKernelGGL(scale_rows_kernel, dim3((a.D + 1023) / 1024, a.N), dim3(256), 0, s, a.M, a.ld, a.N, a.D,
                             a.gamma);
          LAUNCH_CHECK();
        }
    }
    done += cnt;
  }
  return NGSGD_OK;
}

}  // namespace

extern "C" int ngsgd_simple_workspace_bytes(int32_t max_rows, int32_t dim, size_t* out_bytes) {
  if (out_bytes == nullptr || max_rows < 2 || dim < 1) return NGSGD_EINVAL;
  SimpleWork w;
  Carver c(nullptr);
  simple_layout(w, max_rows, dim, true, c);
  (void)c.take<double>(1);   // gamma
  *out_bytes = align_up(c.off, 256);
  return NGSGD_OK;
}

extern "C" int ngsgd_precondition_simple(float* dev_M, int32_t N, int32_t D, int32_t ld, float alpha, float epsilon,
                                         void* dev_workspace, size_t workspace_bytes, float* dev_gamma,
                                         float* dev_rownorm2, void* hip_stream) {
  if (dev_M == nullptr || dev_workspace == nullptr || (reinterpret_cast<uintptr_t>(dev_workspace) & 255u))
    return NGSGD_EINVAL;
  size_t need = 0;
  NG_TRY(ngsgd_simple_workspace_bytes(N, D, &need));
  if (workspace_bytes < need) return NGSGD_ENOMEM;
  SimpleCall c;
  Carver carve(dev_workspace);
  simple_layout(c.w, N, D, true, carve);
  c.gamma = carve.take<double>(1);
  c.M = dev_M; c.ld = ld; c.N = N; c.D = D;
  c.alpha = alpha; c.epsilon = epsilon;
  c.prow = c.w.prow;
  c.gamma_out = dev_gamma;
  c.rownorm2_out = dev_rownorm2;
  std::vector<SimpleCall> calls(1, c);
  return simple_many(calls, true, static_cast<hipStream_t>(hip_stream));
}

// ---- the simple method without a workspace argument ------------------------------------------------------
// Scratch of ngsgd_precondition_simple_static: a fixed array in the library's device image instead of memory the
// caller brings, for callers that cannot allocate.  Every GPU holds its own copy at its own address; in host
// code the array's name is only a handle for hipGetSymbolAddress, the address it returns is what kernels get.
static __device__ __align__(256) unsigned char scratch[NGSGD_SIMPLE_STATIC_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(void** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return NGSGD_EUNSUPPORTED;
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (ptr == nullptr || (reinterpret_cast<uintptr_t>(ptr) & 255u)) return NGSGD_EHIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return NGSGD_OK;
}
}  // namespace

extern "C" int ngsgd_precondition_simple_static(float* dev_M, int32_t N, int32_t D, int32_t ld, float alpha,
                                                float epsilon, float* dev_gamma, float* dev_rownorm2,
                                                void* hip_stream) {
  if (dev_M == nullptr) return NGSGD_EINVAL;
  size_t need = 0;
  NG_TRY(ngsgd_simple_workspace_bytes(N, D, &need));
  if (need > (size_t)NGSGD_SIMPLE_STATIC_BYTES) return NGSGD_ENOMEM;   // the matrix is too large for the fixed scratch
  void* ptr = nullptr;
  NG_TRY(static_scratch(&ptr));
  // the scratch keeps the previous call's contents: the kernels clear what they accumulate into (the Gram
  // matrix) and write every other buffer before reading it, exactly as with a caller's reused workspace
  return ngsgd_precondition_simple(dev_M, N, D, ld, alpha, epsilon, ptr, (size_t)NGSGD_SIMPLE_STATIC_BYTES, dev_gamma,
                                   dev_rownorm2, hip_stream);
}

extern "C" int ngsgd_precond_workspace_bytes(int32_t dim, int32_t rank, int32_t max_batch, size_t* out_bytes) {
  if (out_bytes == nullptr) return NGSGD_EINVAL;
  NG_TRY(precond_check_config(dim, rank, max_batch, 4.f, 2000.f, 1e-10f, 4, 10));
  ngsgd_precond p;
  p.dim = dim; p.rank = rank; p.max_batch = max_batch;
  Carver c(nullptr);
  precond_layout(p, c);
  *out_bytes = align_up(c.off, 256);
  return NGSGD_OK;
}

extern "C" int ngsgd_precond_create(int32_t dim, int32_t rank, int32_t max_batch, float alpha,
                                    float num_samples_history, float epsilon, int32_t update_period,
                                    int32_t always_update_first, void* dev_workspace, size_t workspace_bytes,
                                    ngsgd_precond** out) {
  if (out == nullptr || dev_workspace == nullptr) return NGSGD_EINVAL;
  if (reinterpret_cast<uintptr_t>(dev_workspace) & 255u) return NGSGD_EINVAL;
  NG_TRY(precond_check_config(dim, rank, max_batch, alpha, num_samples_history, epsilon, update_period,
                              always_update_first));
  size_t need = 0;
  NG_TRY(ngsgd_precond_workspace_bytes(dim, rank, max_batch, &need));
  if (workspace_bytes < need) return NGSGD_ENOMEM;
  ngsgd_precond* p = new (std::nothrow) ngsgd_precond();
  if (p == nullptr) return NGSGD_ENOMEM;
  precond_configure(*p, dim, rank, max_batch, alpha, num_samples_history, epsilon, update_period,
                    always_update_first);
  Carver c(dev_workspace);
  precond_layout(*p, c);
  hipError_t e = hipMemset(dev_workspace, 0, need);
  if (e == hipSuccess) {
    PrecondScalars init;
    std::memset(&init, 0, sizeof(init));
    init.gamma = 1.0;
    e = hipMemcpy(p->st, &init, sizeof(init), hipMemcpyHostToDevice);
  }
  if (e != hipSuccess) {
    g_last_hip_error = (int)e;
    delete p;
    return NGSGD_EHIP;
  }
  *out = p;
  return NGSGD_OK;
}

extern "C" int ngsgd_precond_destroy(ngsgd_precond* p) {
  if (p == nullptr || p->owned_by_net) return NGSGD_EINVAL;
  delete p;
  return NGSGD_OK;
}

extern "C" int ngsgd_precond_reset(ngsgd_precond* p) {
  if (p == nullptr) return NGSGD_EINVAL;
  p->t = 0;
  return NGSGD_OK;
}

extern "C" int ngsgd_precondition(ngsgd_precond* p, float* dev_M, int32_t N, int32_t ld, float* dev_gamma,
                                  float* dev_rownorm2, void* hip_stream) {
  if (p == nullptr || dev_M == nullptr) return NGSGD_EINVAL;
  std::vector<PrecondCall> calls(1);
  calls[0] = PrecondCall{p, dev_M, ld, N, dev_gamma, dev_rownorm2};
  NG_TRY(join_side(p->sync, static_cast<hipStream_t>(hip_stream)));
  return precondition_many(calls, true, static_cast<hipStream_t>(hip_stream));
}

extern "C" int ngsgd_precond_get_state(const ngsgd_precond* p, float* dev_W, double* dev_d, double* dev_rho,
                                       int64_t* t_host, void* hip_stream) {
  if (p == nullptr) return NGSGD_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  NG_TRY(join_side(p->sync, s));
  if (t_host != nullptr) *t_host = p->t;
  if (p->rank == 0) {
    if (dev_rho != nullptr) HIP_TRY(hipMemsetAsync(dev_rho, 0, sizeof(double), s));
    return NGSGD_OK;
  }
  if (dev_W != nullptr)
    HIP_TRY(hipMemcpy2DAsync(dev_W, (size_t)p->dim * sizeof(float), p->W, (size_t)p->ldw * sizeof(float),
                             (size_t)p->dim * sizeof(float), p->rank, hipMemcpyDeviceToDevice, s));
  if (dev_d != nullptr)
    HIP_TRY(hipMemcpyAsync(dev_d, p->st->d, (size_t)p->rank * sizeof(double), hipMemcpyDeviceToDevice, s));
  if (dev_rho != nullptr)
    HIP_TRY(hipMemcpyAsync(dev_rho, &p->st->rho, sizeof(double), hipMemcpyDeviceToDevice, s));
  return NGSGD_OK;
}

extern "C" int ngsgd_precond_diagnostics(const ngsgd_precond* p, int32_t* flags_host, int32_t* sweeps_host,
                                         void* hip_stream) {
  if (p == nullptr) return NGSGD_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  NG_TRY(join_side(p->sync, s));
  int v[3] = {0, 0, 0};
  if (p->rank > 0) {
    HIP_TRY(hipMemcpyAsync(v, &p->st->flags, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(v + 2, p->st->gate, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
  }
  if (flags_host != nullptr) *flags_host = v[0] | (v[2] >= kGateClosed ? kFlagInitFromMemory : 0);
  if (sweeps_host != nullptr) *sweeps_host = v[1];
  return NGSGD_OK;
}

extern "C" int ngsgd_precond_set_state(ngsgd_precond* p, const double* dev_R, const double* dev_d, double rho,
                                       int64_t t, void* hip_stream) {
  if (p == nullptr || t < 1 || !(rho > 0.0)) return NGSGD_EINVAL;
  if (p->rank == 0) {
    p->t = t;
    return NGSGD_OK;
  }
  if (dev_R == nullptr || dev_d == nullptr) return NGSGD_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  NG_TRY(join_side(p->sync, s));
  hipLaunchKernelGGL(set_state_kernel, dim3(p->rank), dim3(256), 0, s, dev_R, dev_d, rho, p->alpha, p->rank, p->dim,
                     p->W, p->ldw, p->st);
  LAUNCH_CHECK();
  p->t = t;
  return NGSGD_OK;
}

// ---------------------------------------------------------------------------------------------------
// network
struct ngsgd_layer {
  int din = 0, dout = 0, in1 = 0;   // in1 = din + 1 (bias input)
  int ldw = 0, ldx = 0, lda = 0;
  int nonlin = -1;                  // nonlinearity after this layer, -1 for the last
  int groups = 0;                   // p-norm output dimension
  float* W = nullptr;               // dout x ldw
  float* Xin = nullptr;             // max_batch x ldx, [input, 1]
  float* A = nullptr;               // max_batch x lda, affine output, later O_l
  float* sigma = nullptr;           // max_batch renorm divisors
  double* mc_scale = nullptr;       // max-change scale of the latest step
  ngsgd_precond pin, pout;
  SimpleWork sin, sout;             // scratch of the simple method (only laid out when it is selected)
};

struct ngsgd_net {
  int n_layers = 0;
  int max_batch = 0;
  int pnorm_group = 10;
  int renorm = 0;
  double max_change_per_sample = 0.0;
  int method = NGSGD_METHOD_ONLINE;
  double alpha = 4.0, simple_epsilon = 1e-20;
  std::vector<ngsgd_layer> layers;
  float* params = nullptr;
  size_t n_params_padded = 0;
  float* dX = nullptr;
  int lddx = 0;
  double* rowobj = nullptr;
  double* logprob = nullptr;
  int last_N = 0;
  float last_lr = 0.f;
  SideSync side[kSideStreams];
  int n_side = kSideStreams;   // streams in use
  // ordering between the stream that steps this replica and a stream that averages it with others
  hipEvent_t step_done = nullptr;   // recorded by an averaging call on the stream of the latest step (an event per
                                    // step would cost every step a marker packet on its critical stream)
  hipStream_t step_stream = nullptr;
  bool stepped = false;
  hipEvent_t avg_done = nullptr;    // recorded behind an averaging kernel that rewrote the weights
  bool avg_pending = false;
};

namespace {

// Side stream of the output-side instance of layer l when n_side streams are in use: the last layer's derivatives
// exist after the log-softmax (group 0, with all input sides); the others appear in descending layer order during
// the backward pass, two layers per group, everything below in the last group.  With one stream there is one group.
int output_side_group(int l, int n_layers, int n_side) {
  if (n_side <= 1 || l == n_layers - 1) return 0;
  return std::min(n_side - 1, 1 + (n_layers - 2 - l) / 2);
}

int net_check_config(const ngsgd_config* cfg) {
  if (cfg == nullptr || cfg->dims == nullptr || cfg->n_layers < 1 || cfg->n_layers > NGSGD_MAX_LAYERS)
    return NGSGD_EINVAL;
  if (cfg->n_layers > 1 && cfg->nonlin == nullptr) return NGSGD_EINVAL;
  if (cfg->max_batch < 1 || cfg->pnorm_group < 1) return NGSGD_EINVAL;
  if (cfg->dims[0] < 1 || (cfg->dims[0] & 3)) return NGSGD_EINVAL;
  if (!(cfg->max_change_per_sample >= 0.f)) return NGSGD_EINVAL;
  if (cfg->method != NGSGD_METHOD_ONLINE && cfg->method != NGSGD_METHOD_SIMPLE) return NGSGD_EINVAL;
  const bool simple = cfg->method == NGSGD_METHOD_SIMPLE;
  if (cfg->side_streams < 0 || cfg->side_streams > kSideStreams) return NGSGD_EINVAL;
  if (simple && (cfg->max_batch < 2 || !(cfg->alpha > 0.f) || !(cfg->simple_epsilon > 0.f))) return NGSGD_EINVAL;
  int din = cfg->dims[0];
  for (int l = 0; l < cfg->n_layers; ++l) {
    const int dout = cfg->dims[l + 1];
    if (dout < 1) return NGSGD_EINVAL;
    // the simple method keeps no factors: the ranks are not used
    NG_TRY(precond_check_config(din + 1, simple ? 0 : cfg->rank_in, cfg->max_batch, cfg->alpha,
                                cfg->num_samples_history, cfg->epsilon, cfg->update_period, cfg->always_update_first));
    NG_TRY(precond_check_config(dout, simple ? 0 : cfg->rank_out, cfg->max_batch, cfg->alpha,
                                cfg->num_samples_history, cfg->epsilon, cfg->update_period, cfg->always_update_first));
    if (l < cfg->n_layers - 1) {
      if (cfg->nonlin[l] == NGSGD_PNORM) {
        if (dout % cfg->pnorm_group || dout / cfg->pnorm_group > kPnormMaxGroupsLds) return NGSGD_EINVAL;
        din = dout / cfg->pnorm_group;
      } else if (cfg->nonlin[l] == NGSGD_TANH) {
        din = dout;
      } else {
        return NGSGD_EINVAL;
      }
    }
  }
  return NGSGD_OK;
}

void net_layout(ngsgd_net& net, const ngsgd_config* cfg, Carver& c) {
  net.n_layers = cfg->n_layers;
  net.max_batch = cfg->max_batch;
  net.pnorm_group = cfg->pnorm_group;
  net.renorm = cfg->renorm ? 1 : 0;
  net.max_change_per_sample = cfg->max_change_per_sample;
  net.method = cfg->method;
  net.alpha = cfg->alpha;
  net.simple_epsilon = cfg->simple_epsilon;
  const bool simple = cfg->method == NGSGD_METHOD_SIMPLE;
  net.layers.assign(cfg->n_layers, ngsgd_layer());
  int din = cfg->dims[0];
  size_t n_params = 0;
  int max_ldx = 0;
  for (int l = 0; l < cfg->n_layers; ++l) {
    ngsgd_layer& L = net.layers[l];
    L.din = din;
    L.dout = cfg->dims[l + 1];
    L.in1 = din + 1;
    L.ldw = pad32(L.in1);
    L.ldx = pad32(L.in1);
    L.lda = pad32(L.dout);
    L.nonlin = l < cfg->n_layers - 1 ? cfg->nonlin[l] : -1;
    L.groups = L.nonlin == NGSGD_PNORM ? L.dout / cfg->pnorm_group : L.dout;
    n_params += (size_t)L.dout * L.ldw;
    max_ldx = std::max(max_ldx, L.ldx);
    din = L.groups;
  }
  net.n_params_padded = n_params;
  net.n_side = cfg->side_streams > 0 ? cfg->side_streams : default_side_streams(*cfg);
  net.params = c.take<float>(n_params);
  size_t off = 0;
  for (auto& L : net.layers) {
    L.W = net.params ? net.params + off : nullptr;
    off += (size_t)L.dout * L.ldw;
  }
  net.lddx = max_ldx;
  net.dX = c.take<float>((size_t)kMaxBwdSplits * net.max_batch * net.lddx);
  net.rowobj = c.take<double>(net.max_batch);
  net.logprob = c.take<double>(1);
  for (auto& L : net.layers) {
    L.Xin = c.take<float>((size_t)net.max_batch * L.ldx);
    L.A = c.take<float>((size_t)net.max_batch * L.lda);
    L.sigma = c.take<float>(net.max_batch);
    L.mc_scale = c.take<double>(1);
    precond_configure(L.pin, L.in1, simple ? 0 : cfg->rank_in, cfg->max_batch, cfg->alpha, cfg->num_samples_history,
                      cfg->epsilon, cfg->update_period, cfg->always_update_first);
    precond_configure(L.pout, L.dout, simple ? 0 : cfg->rank_out, cfg->max_batch, cfg->alpha,
                      cfg->num_samples_history, cfg->epsilon, cfg->update_period, cfg->always_update_first);
    L.pin.owned_by_net = L.pout.owned_by_net = true;
    L.pin.sync = &net.side[0];
    L.pout.sync = &net.side[output_side_group((int)(&L - net.layers.data()), cfg->n_layers, net.n_side)];
    precond_layout(L.pin, c);
    precond_layout(L.pout, c);
    if (simple) {   // gamma and the row norms go where the online method leaves them (st->gamma, prow)
      simple_layout(L.sin, cfg->max_batch, L.in1, false, c);
      simple_layout(L.sout, cfg->max_batch, L.dout, false, c);
    }
  }
}

int copy2d(const float* src, int lds_, float* dst, int ldd, int rows, int cols, float scale, const double* scale_dev,
           hipStream_t s) {
  hipLaunchKernelGGL(copy2d_kernel, dim3((cols + 1023) / 1024, rows), dim3(256), 0, s, src, lds_, dst, ldd, rows, cols,
                     scale, scale_dev);
  LAUNCH_CHECK();
  return NGSGD_OK;
}

// Orders stream s behind an averaging kernel that rewrote this replica's weights on another stream.  The wait is
// dropped once the replica's own stepping stream has taken it.
int order_after_average(ngsgd_net* net, hipStream_t s, bool stepping_stream) {
  if (net->avg_pending) {
    HIP_TRY(hipStreamWaitEvent(s, net->avg_done, 0));
    if (stepping_stream) net->avg_pending = false;
  }
  return NGSGD_OK;
}

GemmDesc update_desc(const ngsgd_layer& L, int N, float alpha, float beta, float* C, int ldc) {
  GemmDesc g;
  g.A = L.A; g.lda = L.lda;          // O_l stored N x dout: A^T
  g.B = L.Xin; g.ldb = L.ldx;        // Xbar_l stored N x in1
  g.C = C; g.ldc = ldc;
  g.M = L.dout; g.N = L.in1; g.K = N;
  g.alpha = alpha; g.beta = beta;
  g.alpha_dev[0] = &L.pout.st->gamma;
  g.alpha_dev[1] = &L.pin.st->gamma;
  g.alpha_dev[2] = L.mc_scale;
  return g;
}

}  // namespace

extern "C" int ngsgd_workspace_bytes(const ngsgd_config* cfg, size_t* out_bytes) {
  if (out_bytes == nullptr) return NGSGD_EINVAL;
  NG_TRY(net_check_config(cfg));
  ngsgd_net net;
  Carver c(nullptr);
  net_layout(net, cfg, c);
  *out_bytes = align_up(c.off, 256);
  return NGSGD_OK;
}

extern "C" int ngsgd_create(const ngsgd_config* cfg, void* dev_workspace, size_t workspace_bytes, ngsgd_net** out) {
  if (out == nullptr || dev_workspace == nullptr) return NGSGD_EINVAL;
  if (reinterpret_cast<uintptr_t>(dev_workspace) & 255u) return NGSGD_EINVAL;
  size_t need = 0;
  NG_TRY(ngsgd_workspace_bytes(cfg, &need));
  if (workspace_bytes < need) return NGSGD_ENOMEM;
  ngsgd_net* net = new (std::nothrow) ngsgd_net();
  if (net == nullptr) return NGSGD_ENOMEM;
  Carver c(dev_workspace);
  net_layout(*net, cfg, c);
  hipError_t e = hipMemset(dev_workspace, 0, need);
  PrecondScalars init;
  std::memset(&init, 0, sizeof(init));
  init.gamma = 1.0;
  const double one = 1.0;
  for (auto& L : net->layers) {
    if (e == hipSuccess) e = hipMemcpy(L.pin.st, &init, sizeof(init), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(L.pout.st, &init, sizeof(init), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(L.mc_scale, &one, sizeof(one), hipMemcpyHostToDevice);
  }
  // second stream for the factor updates: default priority, does not synchronise with the NULL stream
  if (e == hipSuccess) e = hipEventCreateWithFlags(&net->step_done, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&net->avg_done, hipEventDisableTiming);
  for (int k = 0; k < net->n_side; ++k) {
    SideSync& sd = net->side[k];
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&sd.stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&sd.inputs_ready, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&sd.hj_done, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&sd.outputs_done, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&sd.done, hipEventDisableTiming);
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    g_last_hip_error = (int)e;
    ngsgd_destroy(net);
    return NGSGD_EHIP;
  }
  *out = net;
  return NGSGD_OK;
}

extern "C" int ngsgd_destroy(ngsgd_net* net) {
  if (net == nullptr) return NGSGD_EINVAL;
  for (SideSync& sd : net->side) {
    if (sd.stream != nullptr) {
      (void)hipStreamSynchronize(sd.stream);
      (void)hipStreamDestroy(sd.stream);
    }
    for (hipEvent_t ev : {sd.inputs_ready, sd.hj_done, sd.outputs_done, sd.done})
      if (ev != nullptr) (void)hipEventDestroy(ev);
  }
  for (hipEvent_t ev : {net->step_done, net->avg_done})
    if (ev != nullptr) (void)hipEventDestroy(ev);
  delete net;
  return NGSGD_OK;
}

extern "C" int ngsgd_step(ngsgd_net* net, const float* dev_x, const int32_t* dev_labels, int32_t N, float lr,
                          double* dev_logprob_sum, void* hip_stream) {
  if (net == nullptr || dev_x == nullptr || dev_labels == nullptr) return NGSGD_EINVAL;
  if (N < 1 || N > net->max_batch || !aligned16(dev_x)) return NGSGD_EINVAL;
  if (net->method == NGSGD_METHOD_SIMPLE && N < 2) return NGSGD_EINVAL;   // nothing to hold out
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int nl = net->n_layers;
  auto& Ls = net->layers;
  for (SideSync& sd : net->side) sd.owner = s;
  NG_TRY(order_after_average(net, s, true));
  for (auto& L : Ls) {   // argument errors must leave the state untouched: check before any launch
    if (L.pin.rank > 0 && L.pin.t == 0 && N <= L.pin.rank) return NGSGD_EINVAL;
    if (L.pout.rank > 0 && L.pout.t == 0 && N <= L.pout.rank) return NGSGD_EINVAL;
  }

  // forward (Sec. 2): A_l = [X_l, 1] W_l^T, nonlinearity, log-softmax; the objective is cleared by the first
  // kernel of the step and accumulated by the log-softmax kernel
  double* const objective = dev_logprob_sum != nullptr ? dev_logprob_sum : net->logprob;
  {
    ProfScope prof(NGSGD_PROF_ELEMENTWISE, s);
    hipLaunchKernelGGL(copy_append_ones_kernel, dim3((Ls[0].ldx + 255) / 256, N), dim3(256), 0, s, dev_x, Ls[0].din,
                       Ls[0].Xin, Ls[0].ldx, N, Ls[0].din, objective);
    LAUNCH_CHECK();
  }
  for (int l = 0; l < nl; ++l) {
    ngsgd_layer& L = Ls[l];
    GemmDesc g;
    g.A = L.Xin; g.lda = L.ldx;
    g.B = L.W; g.ldb = L.ldw;
    g.C = L.A; g.ldc = L.lda;
    g.M = N; g.N = L.dout; g.K = L.in1;
    if (L.nonlin == NGSGD_TANH) {   // the next layer's input straight from the product
      ngsgd_layer& Nx = Ls[l + 1];
      g.C = Nx.Xin; g.ldc = Nx.ldx;
      g.act = kActTanh;
      g.pad_to = Nx.ldx;
    }
    {
      ProfScope prof(NGSGD_PROF_GEMM_FWD, s);
      NG_TRY(launch_layer_gemms(GEMM_FWD, &g, 1, s));
    }
    if (l == nl - 1) continue;
    if (L.nonlin == NGSGD_TANH) {
      prof_place();
    } else {
      ProfScope prof(NGSGD_PROF_ELEMENTWISE, s);
      ngsgd_layer& Nx = Ls[l + 1];
      if (L.dout >= kWideRow) {
        hipLaunchKernelGGL(pnorm_forward_kernel<512>, dim3(N), dim3(512), 0, s, L.A, L.lda, Nx.Xin, Nx.ldx,
                           L.sigma, N, L.groups, net->pnorm_group, net->renorm);
      } else {
        hipLaunchKernelGGL(pnorm_forward_kernel<256>, dim3(N), dim3(256), 0, s, L.A, L.lda, Nx.Xin, Nx.ldx,
                           L.sigma, N, L.groups, net->pnorm_group, net->renorm);
      }
      LAUNCH_CHECK();
    }
  }
  ngsgd_layer& last = Ls[nl - 1];
  {
    ProfScope prof(NGSGD_PROF_ELEMENTWISE, s);
    if (last.dout >= kWideRow) {
      hipLaunchKernelGGL(softmax_xent_kernel<512>, dim3(N), dim3(512), 0, s, last.A, last.lda, dev_labels, N,
                         last.dout, net->rowobj, objective);
    } else {
      hipLaunchKernelGGL(softmax_xent_kernel<256>, dim3(N), dim3(256), 0, s, last.A, last.lda, dev_labels, N,
                         last.dout, net->rowobj, objective);
    }
    LAUNCH_CHECK();
  }

  // On a step whose factors are all due for an update (and none needs initialising) the products H, J and the
  // R x R work of each group of instances start on the group's side stream as soon as the group's matrices
  // exist, next to the backward pass; W_t is replaced only after Xhat has read it (the second half of each group's
  // update is enqueued at the end of the step).
  bool early = net->method == NGSGD_METHOD_ONLINE;
  for (auto& L : Ls)
    for (const ngsgd_precond* p : {&L.pin, &L.pout})
      if (p->rank > 0 && (p->t == 0 || !factor_due(*p))) early = false;
  std::vector<PrecondCall> early_calls[kSideStreams];
  int ready_layer[kSideStreams];   // a group starts once the derivatives of this layer (its lowest) exist
  for (int& r : ready_layer) r = nl - 1;
  if (early) {
    NG_TRY(ensure_kernel_attributes());
    for (int l = 0; l < nl; ++l) {
      ngsgd_layer& L = Ls[l];
      const int k = output_side_group(l, nl, net->n_side);
      ready_layer[k] = std::min(ready_layer[k], l);
      if (L.pout.rank > 0) early_calls[k].push_back(PrecondCall{&L.pout, L.A, L.lda, N, nullptr, nullptr});
      if (L.pin.rank > 0) early_calls[0].push_back(PrecondCall{&L.pin, L.Xin, L.ldx, N, nullptr, nullptr});
    }
  }
  auto early_start = [&](const int k) -> int {
    if (!early || early_calls[k].empty()) return NGSGD_OK;
    SideSync& sd = net->side[k];
    HIP_TRY(hipEventRecord(sd.inputs_ready, s));
    HIP_TRY(hipStreamWaitEvent(sd.stream, sd.inputs_ready, 0));
    NG_TRY(clear_accumulators(early_calls[k], sd.stream, capturing(sd.stream)));
    NG_TRY(launch_h_products(early_calls[k], sd.stream));
    NG_TRY(launch_j_products(early_calls[k], sd.stream));
    HIP_TRY(hipEventRecord(sd.hj_done, sd.stream));
    return factor_begin(early_calls[k], sd.stream);
  };
  for (int k = 0; k < kSideStreams; ++k)
    if (ready_layer[k] == nl - 1) NG_TRY(early_start(k));   // (empty groups return at once)

  // backward on the unmodified derivatives (App. C.3, last paragraph)
  for (int l = nl - 1; l >= 1; --l) {
    ngsgd_layer& L = Ls[l];
    ngsgd_layer& P = Ls[l - 1];
    GemmDesc g;
    g.A = L.A; g.lda = L.lda;           // O_l, N x dout
    g.B = L.W; g.ldb = L.ldw;           // W_l as dout x din (bias column dropped)
    g.C = net->dX; g.ldc = net->lddx;
    g.M = N; g.N = L.din; g.K = L.dout;
    // few output tiles and a long K: split K into slabs that the nonlinearity's backward kernel sums
    const size_t slab = (size_t)net->max_batch * net->lddx;
    g.c_split_stride = (long long)slab;
    const int tiles = ((N + 63) / 64) * ((L.din + 63) / 64);
    g.splits = std::min(kMaxBwdSplits, choose_splits(tiles, (L.dout + 31) / 32));
    const bool whole = P.nonlin == NGSGD_TANH && backward_in_one(g);
    if (whole) {   // the derivative straight from the product
      g.splits = 1;
      g.C = P.A; g.ldc = P.lda;
      g.act = kActTanhBackward;
      g.Y = L.Xin; g.ldy = L.ldx;
    }
    int n_slabs = 1;
    {
      ProfScope prof(NGSGD_PROF_GEMM_BWD, s);
      NG_TRY(launch_layer_gemms(GEMM_BWD, &g, 1, s, &n_slabs));
    }
    if (whole) {
      prof_place();
    } else {
      ProfScope prof(NGSGD_PROF_ELEMENTWISE, s);
      if (P.nonlin == NGSGD_TANH) {
        hipLaunchKernelGGL(tanh_backward_kernel, dim3((P.dout + 1023) / 1024, N), dim3(256), 0, s, net->dX, net->lddx,
                           n_slabs, slab, L.Xin, L.ldx, P.A, P.lda, N, P.dout);
      } else if (P.dout >= kWideRow) {
        hipLaunchKernelGGL(pnorm_backward_kernel<512>, dim3(N), dim3(512), 0, s, net->dX, net->lddx, n_slabs, slab,
                           L.Xin, L.ldx, P.sigma, P.A, P.lda, N, P.groups, net->pnorm_group, net->renorm);
      } else {
        hipLaunchKernelGGL(pnorm_backward_kernel<256>, dim3(N), dim3(256), 0, s, net->dX, net->lddx, n_slabs, slab,
                           L.Xin, L.ldx, P.sigma, P.A, P.lda, N, P.groups, net->pnorm_group, net->renorm);
      }
      LAUNCH_CHECK();
    }
    // the derivatives of layer l - 1 exist now: start the group of which it is the lowest layer
    for (int k = 0; k < kSideStreams; ++k)
      if (ready_layer[k] == l - 1) NG_TRY(early_start(k));
  }

  // maximum parameter change (App. C.3), then W_l += lr a_l gamma_o gamma_x Ohat_l^T Xhat_l  (Sec. 4.6) for the
  // listed layers, once both of their matrices are preconditioned
  auto update_layers = [&](const std::vector<int>& layers) -> int {
    if (layers.empty()) return NGSGD_OK;
    std::vector<GemmDesc> upd;
    for (const int l : layers) {
      const ngsgd_layer& L = Ls[l];
      GemmDesc g = update_desc(L, N, lr, 1.f, L.W, L.ldw);
      if (net->max_change_per_sample > 0.0) {   // the product forms the scale and leaves it in L.mc_scale
        g.alpha_dev[2] = nullptr;
        g.mc_rows = N;
        g.mc_prow[0] = L.pout.prow;
        g.mc_prow[1] = L.pin.prow;
        g.mc_out = L.mc_scale;
        g.mc_bound = (double)N * net->max_change_per_sample;
      }
      upd.push_back(g);
    }
    ProfScope prof(NGSGD_PROF_GEMM_UPD, s);
    return launch_layer_gemms(GEMM_UPD, upd.data(), (int)upd.size(), s);
  };
  std::vector<int> all_layers;
  for (int l = 0; l < nl; ++l) all_layers.push_back(l);

  // natural gradient: both matrices of every layer (Sec. 4.6; 2I instances), grouped calls; the factor updates
  // overlap the rest of this step and the next step's forward and backward passes on the side streams
  if (net->method == NGSGD_METHOD_SIMPLE) {
    // App. A instead: the factors come from the other rows of this minibatch, no state
    std::vector<SimpleCall> calls;
    for (auto& L : Ls) {
      calls.push_back(SimpleCall{L.A, L.lda, N, L.dout, net->alpha, net->simple_epsilon, L.sout, L.pout.prow,
                                 &L.pout.st->gamma, nullptr, nullptr});
      calls.push_back(SimpleCall{L.Xin, L.ldx, N, L.in1, net->alpha, net->simple_epsilon, L.sin, L.pin.prow,
                                 &L.pin.st->gamma, nullptr, nullptr});
    }
    NG_TRY(simple_many(calls, false, s));
    NG_TRY(update_layers(all_layers));
  } else if (early) {
    std::vector<PrecondCall> calls;
    for (auto& L : Ls) {
      calls.push_back(PrecondCall{&L.pout, L.A, L.lda, N, nullptr, nullptr});
      calls.push_back(PrecondCall{&L.pin, L.Xin, L.ldx, N, nullptr, nullptr});
    }
    // Xhat and gamma behind every group's H and J; the second half of each group's factor update is enqueued
    // after the rest of this step so that the caller's stream is never short of work
    // (the group whose matrices appeared last is still busy with H and J when the backward pass ends: the Xhat
    // products of the other groups go first)
    std::vector<PrecondCall> due;
    for (int k = 0; k < kSideStreams; ++k) {
      if (early_calls[k].empty()) continue;
      HIP_TRY(hipStreamWaitEvent(s, net->side[k].hj_done, 0));
      NG_TRY(precond_apply(early_calls[k], false, s, due, true, true, false));
    }
    NG_TRY(precond_apply(calls, false, s, due, true, false, true));
    for (int k = 0; k < kSideStreams; ++k)
      if (!early_calls[k].empty()) HIP_TRY(hipEventRecord(net->side[k].outputs_done, s));
    for (auto& c : calls) c.p->t += 1;
    NG_TRY(update_layers(all_layers));
    for (int k = 0; k < kSideStreams; ++k) {
      if (early_calls[k].empty()) continue;
      SideSync& sd = net->side[k];
      HIP_TRY(hipStreamWaitEvent(sd.stream, sd.outputs_done, 0));
      NG_TRY(factor_finish(early_calls[k], sd.stream));
      HIP_TRY(hipEventRecord(sd.done, sd.stream));
      sd.pending = true;
    }
  } else {
    // No factor is due, or the first call of an instance (initialisation): everything on the caller's stream.
    // On the step after an update the group that started last may still be running: the layers that do not
    // depend on it are preconditioned and updated first, the others behind them.
    SideSync* const last_side = &net->side[net->n_side - 1];
    std::vector<PrecondCall> calls[2];
    std::vector<int> layers[2];
    const bool split = net->n_side > 1 && last_side->pending;
    for (int l = 0; l < nl; ++l) {
      ngsgd_layer& L = Ls[l];
      const int late = split && L.pout.sync == last_side ? 1 : 0;
      calls[late].push_back(PrecondCall{&L.pout, L.A, L.lda, N, nullptr, nullptr});
      calls[0].push_back(PrecondCall{&L.pin, L.Xin, L.ldx, N, nullptr, nullptr});
      layers[late].push_back(l);
    }
    for (SideSync& sd : net->side)
      if (!split || &sd != last_side) NG_TRY(join_side(&sd, s));
    NG_TRY(precondition_many(calls[0], false, s));
    NG_TRY(update_layers(layers[0]));
    if (split) {
      NG_TRY(join_side(last_side, s));
      if (!calls[1].empty()) NG_TRY(precondition_many(calls[1], false, s));
      NG_TRY(update_layers(layers[1]));
    }
  }
  net->last_N = N;
  net->last_lr = lr;
  net->step_stream = s;   // an averaging call on another stream orders itself behind this stream's work so far
  net->stepped = true;
  return NGSGD_OK;
}

extern "C" int ngsgd_join(ngsgd_net* net, void* hip_stream) {
  if (net == nullptr) return NGSGD_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  for (SideSync& sd : net->side) NG_TRY(join_side(&sd, s));
  return NGSGD_OK;
}

extern "C" int ngsgd_average(ngsgd_net* const* nets, int32_t n, int32_t reset_preconditioners, void* hip_stream) {
  if (nets == nullptr || n < 1 || n > kMaxReplicas) return NGSGD_EINVAL;
  for (int i = 0; i < n; ++i) {
    if (nets[i] == nullptr) return NGSGD_EINVAL;
    if (nets[i]->n_params_padded != nets[0]->n_params_padded || nets[i]->n_layers != nets[0]->n_layers)
      return NGSGD_EINVAL;
    for (int l = 0; l < nets[0]->n_layers; ++l)
      if (nets[i]->layers[l].dout != nets[0]->layers[l].dout || nets[i]->layers[l].din != nets[0]->layers[l].din)
        return NGSGD_EINVAL;
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  for (int i = 0; i < n; ++i) {
    // behind the replica's latest step (whatever stream it ran on), its factor updates and an earlier averaging
    if (nets[i]->stepped && nets[i]->step_stream != s) {
      HIP_TRY(hipEventRecord(nets[i]->step_done, nets[i]->step_stream));
      HIP_TRY(hipStreamWaitEvent(s, nets[i]->step_done, 0));
    }
    NG_TRY(order_after_average(nets[i], s, false));
    for (SideSync& sd : nets[i]->side) NG_TRY(join_side(&sd, s));
  }
  AverageArgs a;
  a.n = n;
  a.count = nets[0]->n_params_padded;
  for (int i = 0; i < n; ++i) a.params[i] = nets[i]->params;
  size_t blocks = (a.count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(average_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
  LAUNCH_CHECK();
  for (int i = 0; i < n; ++i) {   // the replicas' next steps (on their own streams) wait for the new weights
    HIP_TRY(hipEventRecord(nets[i]->avg_done, s));
    nets[i]->avg_pending = true;
  }
  if (reset_preconditioners)
    for (int i = 0; i < n; ++i)
      for (auto& L : nets[i]->layers) L.pin.t = L.pout.t = 0;
  return NGSGD_OK;
}

extern "C" int ngsgd_get_params(const ngsgd_net* net, int32_t layer, float* dev_out, void* hip_stream) {
  if (net == nullptr || dev_out == nullptr || layer < 0 || layer >= net->n_layers) return NGSGD_EINVAL;
  const ngsgd_layer& L = net->layers[layer];
  NG_TRY(order_after_average(const_cast<ngsgd_net*>(net), static_cast<hipStream_t>(hip_stream), false));
  return copy2d(L.W, L.ldw, dev_out, L.in1, L.dout, L.in1, 1.f, nullptr, static_cast<hipStream_t>(hip_stream));
}

extern "C" int ngsgd_set_params(ngsgd_net* net, int32_t layer, const float* dev_in, void* hip_stream) {
  if (net == nullptr || dev_in == nullptr || layer < 0 || layer >= net->n_layers) return NGSGD_EINVAL;
  ngsgd_layer& L = net->layers[layer];
  NG_TRY(order_after_average(net, static_cast<hipStream_t>(hip_stream), false));
  return copy2d(dev_in, L.in1, L.W, L.ldw, L.dout, L.in1, 1.f, nullptr, static_cast<hipStream_t>(hip_stream));
}

extern "C" int ngsgd_net_precond(ngsgd_net* net, int32_t layer, int32_t side, ngsgd_precond** out) {
  if (net == nullptr || out == nullptr || layer < 0 || layer >= net->n_layers) return NGSGD_EINVAL;
  if (side != NGSGD_SIDE_INPUT && side != NGSGD_SIDE_OUTPUT) return NGSGD_EINVAL;
  ngsgd_layer& L = net->layers[layer];
  ngsgd_precond* p = side == NGSGD_SIDE_INPUT ? &L.pin : &L.pout;
  *out = p->rank > 0 ? p : nullptr;
  return NGSGD_OK;
}

extern "C" int ngsgd_last_preconditioned(ngsgd_net* net, int32_t layer, int32_t side, float* dev_out,
                                         void* hip_stream) {
  if (net == nullptr || dev_out == nullptr || layer < 0 || layer >= net->n_layers || net->last_N < 1)
    return NGSGD_EINVAL;
  if (side != NGSGD_SIDE_INPUT && side != NGSGD_SIDE_OUTPUT) return NGSGD_EINVAL;
  ngsgd_layer& L = net->layers[layer];
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (side == NGSGD_SIDE_INPUT)
    return copy2d(L.Xin, L.ldx, dev_out, L.in1, net->last_N, L.in1, 1.f, &L.pin.st->gamma, s);
  return copy2d(L.A, L.lda, dev_out, L.dout, net->last_N, L.dout, 1.f, &L.pout.st->gamma, s);
}

extern "C" int ngsgd_last_gradient(ngsgd_net* net, int32_t layer, float* dev_out, void* hip_stream) {
  if (net == nullptr || dev_out == nullptr || layer < 0 || layer >= net->n_layers || net->last_N < 1)
    return NGSGD_EINVAL;
  ngsgd_layer& L = net->layers[layer];
  GemmDesc g = update_desc(L, net->last_N, 1.f, 0.f, dev_out, L.in1);
  return launch_layer_gemms(GEMM_UPD, &g, 1, static_cast<hipStream_t>(hip_stream));
}

extern "C" int ngsgd_last_max_change_scale(ngsgd_net* net, int32_t layer, double* dev_out, void* hip_stream) {
  if (net == nullptr || dev_out == nullptr || layer < 0 || layer >= net->n_layers) return NGSGD_EINVAL;
  HIP_TRY(hipMemcpyAsync(dev_out, net->layers[layer].mc_scale, sizeof(double), hipMemcpyDeviceToDevice,
                         static_cast<hipStream_t>(hip_stream)));
  return NGSGD_OK;
}

extern "C" const char* ngsgd_strerror(int code) {
  switch (code) {
    case NGSGD_OK: return "ok";
    case NGSGD_EINVAL: return "invalid argument";
    case NGSGD_ENOMEM: return "workspace too small";
    case NGSGD_EHIP: return "HIP runtime error";
    case NGSGD_EUNSUPPORTED: return "unsupported";
    default: return "unknown error";
  }
}

extern "C" int ngsgd_profile_enable(int32_t on) {
  g_prof.on = on != 0;
  g_prof.used = 0;
  g_prof.dropped = 0;
  g_prof.recs.clear();
  return NGSGD_OK;
}

extern "C" int ngsgd_profile_read(double* ms_out, int64_t* launches_out, int32_t n_categories) {
  if (ms_out == nullptr || launches_out == nullptr || n_categories < NGSGD_PROF_CATEGORIES) return NGSGD_EINVAL;
  for (int i = 0; i < n_categories; ++i) {
    ms_out[i] = 0.0;
    launches_out[i] = 0;
  }
  for (const auto& r : g_prof.recs) {
    HIP_TRY(hipEventSynchronize(g_prof.pool[r.e0 + 1]));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, g_prof.pool[r.e0], g_prof.pool[r.e0 + 1]));
    ms_out[r.cat] += (double)ms;
    launches_out[r.cat] += 1;
  }
  const bool complete = g_prof.dropped == 0;
  g_prof.used = 0;
  g_prof.dropped = 0;
  g_prof.recs.clear();
  return complete ? NGSGD_OK : NGSGD_ENOMEM;   // the sums miss the groups that did not fit
}

extern "C" int ngsgd_set_wait_limit_us(int64_t microseconds) {
  if (microseconds < 0) return NGSGD_EINVAL;
  g_fused_wait_us.store((long long)microseconds);
  return NGSGD_OK;
}

extern "C" int ngsgd_last_hip_error(void) { return g_last_hip_error; }
extern "C" int ngsgd_version(void) { return 100; }
