// Batched uneven GEMMs in one launch.
//
// A plan turns a list of independent problems C_i <- alpha_i A_i B_i +
// beta_i C_i into a device work list of macro-tiles (each record carries its
// problem's arguments, tile coordinates and a tile class from the tuning
// table), sorted longest first.  One launch runs a workgroup per tile in list
// order with the single-problem kernels' register-staged tiles, so a problem's
// result does not depend on what else is in the batch.  The launch is captured
// once in a HIP graph and replayed.
//
// What bounds it: memory, for a batch of small problems.  2000 problems of
// extents 16-512 (1.32 GB, 11.1 GFLOP, 17.9 on 64x64 tiles): 411 us in FP64 =
// 3.2 TB/s (on 64x64 tiles alone 419 when measured: 345 without the products,
// 325 without the C traffic, 210 with neither); FP32 236 us.  A persistent
// kernel that streamed a workgroup's tiles through one LDS ring of 4-byte
// loads (any alignment) took 650 and 401 us: four times the load instructions,
// one register allocation for every path, and a static deal of the tiles.
//
// In the paper's terms (Section 3.2): blocks are independent and are never
// synchronised with each other; they share nothing but the read-only list.
#include "grouped.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <numeric>
#include <type_traits>
#include <vector>

#include "gemm_tile.h"

namespace mg {

namespace {

// Tile classes (work divisions per problem).
constexpr int kClsBM[kNumGroupedClasses] = {64, 64, 32};
constexpr int kClsBN[kNumGroupedClasses] = {64, 32, 32};
constexpr int kScaleCls = 15;  // C <- beta*C only (alpha == 0 or k == 0)
constexpr int kScaleTile = 64;

// One macro-tile of work: the problem's arguments inline (one load per tile).
template <typename T>
struct GTileRec {
  GemmArgs<T> g;
  int tm, tn;
  int cls;
  int pad;
};

template <typename T>
__device__ __forceinline__ void scale_tile(const GemmArgs<T> &g, int m0, int n0) {
  for (int e = threadIdx.x; e < kScaleTile * kScaleTile; e += kTileThreads) {
    const int i = m0 + e / kScaleTile, j = n0 + e % kScaleTile;
    if (i < g.m && j < g.n) {
      T *p = g.C + (int64_t)i * g.ldc + j;
      *p = g.beta == T(0) ? T(0) : g.beta * *p;
    }
  }
}

// One workgroup per tile of the list, in list order (longest first): the
// dispatcher hands a finished workgroup's place to the next tile, which
// balances the CUs by the tiles' real times.  The tiles are the single-problem
// register-staged ones, which take rows of any pitch and alignment.
constexpr int kMinWaves = 3;  // wavefronts per SIMD: three 64x64 tiles per CU

// Tile record through the constant address space: the list is never written
// during the launch, so the uniform record loads become scalar loads.
template <typename T>
__device__ __forceinline__ GTileRec<T> gd_record(const GTileRec<T> *tiles, int w) {
  typedef __attribute__((address_space(4))) const GTileRec<T> CRec;
  GTileRec<T> r;
  __builtin_memcpy(&r, (const GTileRec<T> *)&((const CRec *)tiles)[w], sizeof(r));
  return r;
}

// Tile of workgroup b: the list is dealt in rounds of `round` tiles (the
// workgroups resident at once), and within a round each XCD takes a
// contiguous run (the dispatcher places workgroup b on XCD b % 8): the tiles
// of one problem, adjacent in the list, then share one L2.
__device__ __forceinline__ int gd_deal(int b, int round, int ntiles) {
  const int first = b / round * round;
  return first + xcd_remap(b - first, min(round, ntiles - first));
}

template <typename T>
__global__ __launch_bounds__(kTileThreads, kMinWaves) void grouped_kernel(
    const GTileRec<T> *__restrict__ tiles, int ntiles, int round) {
  extern __shared__ __align__(16) unsigned char lds[];
  T *smem = reinterpret_cast<T *>(lds);
  const GTileRec<T> r = gd_record(tiles, gd_deal(blockIdx.x, round, ntiles));
  // Wavefronts of ragged tiles that lie past the matrix skip the products;
  // turning the tile's parts over the wavefronts spreads them over the SIMDs.
  const int turn = (blockIdx.x >> 3) & 3;
  if (r.cls == kScaleCls) scale_tile<T>(r.g, r.tm * kScaleTile, r.tn * kScaleTile);
  else if (r.cls == 0) gemm_tile<T, 64, 64>(r.g, r.tm * 64, r.tn * 64, smem, turn);
  else if (r.cls == 1) gemm_tile<T, 64, 32>(r.g, r.tm * 64, r.tn * 32, smem, turn);
  else gemm_tile<T, 32, 32>(r.g, r.tm * 32, r.tn * 32, smem, turn);
}

template <typename T>
constexpr size_t grouped_lds_bytes() {
  return TileShape<T, 64, 64>::LDS_BYTES;  // the largest class
}

int bucket_of(int64_t x) {
  int b = 0;
  while (b < kTuneEdges - 1 && x >= (int64_t)(32 << b)) ++b;
  return b;
}

}  // namespace

int tune_bucket(int64_t m, int64_t n, int64_t k) {
  return (bucket_of(m) * kTuneEdges + bucket_of(n)) * kTuneEdges + bucket_of(k);
}

int64_t tune_bucket_rep(int b) {  // representative extent of a 1-D bucket
  if (b == 0) return 22;                       // [1, 32)
  if (b == kTuneEdges - 1) return 16 << b;     // [512, ...)
  return (int64_t)std::lround(16.0 * std::sqrt(2.0) * (1 << b));  // geometric middle
}

int grouped_class_tile(int cls, int *bm, int *bn) {
  if (cls < 0 || cls >= kNumGroupedClasses) return MG_ERR_INVALID_ARG;
  *bm = kClsBM[cls];
  *bn = kClsBN[cls];
  return MG_OK;
}

// Class when no tuning table is given: the least count of
//   tiles x (per tile + per k-step x k-steps),
// the microseconds of one CU a tile takes in a full batch, fitted to batches
// forced to each class (2000 problems of extents 16-512, 500 of 64-128, 1000
// of 16-64 and 100 of 128-512; 6 % off on average).  Per tile: the launch, the
// first loads' latency and C; per k-step: the products and the panels' loads,
// so padding counts by what it costs.  The largest tile wasting at most a
// quarter of its area, the rule before, took 467 / 280 us (FP64 / FP32) for the
// 2000 problems where this takes 411 / 241.
struct ClassCost {
  double tile, step;
};
constexpr ClassCost kCost64[kNumGroupedClasses] = {{2.6, 0.52}, {1.5, 0.29}, {1.2, 0.15}};
constexpr ClassCost kCost32[kNumGroupedClasses] = {{0.9, 0.70}, {0.95, 0.31}, {0.9, 0.162}};

namespace {

double tile_cost(int dtype, int cls, int64_t k) {
  const ClassCost &c = dtype == MG_F64 ? kCost64[cls] : kCost32[cls];
  return c.tile + c.step * (double)ceil_div(k, dtype == MG_F64 ? 16 : 32);
}

}  // namespace

int heuristic_class(int dtype, int64_t m, int64_t n, int64_t k) {
  int best = 0;
  double least = 0;
  for (int c = 0; c < kNumGroupedClasses; ++c) {
    const double cost =
        (double)(ceil_div(m, kClsBM[c]) * ceil_div(n, kClsBN[c])) * tile_cost(dtype, c, k);
    if (c == 0 || cost < least) {
      best = c;
      least = cost;
    }
  }
  return best;
}

struct Plan {
  int dtype = MG_F64;
  int device = 0;
  int64_t count = 0;
  int ntiles = 0;
  int grid = 0;
  void *d_tiles = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  mg_plan_stats stats{};
};

namespace {

template <typename T>
int build_t(int64_t count, const mg_problem *probs, const mg_tune_table *table, WorkList *out) {
  constexpr int dtype = std::is_same<T, double>::value ? MG_F64 : MG_F32;
  std::vector<GemmArgs<T>> hp((size_t)count);
  std::vector<GTileRec<T>> tiles;
  std::vector<double> cost;
  double flops = 0, bytes = 0;
  int64_t per_cls[kNumGroupedClasses + 1] = {0};
  for (int64_t i = 0; i < count; ++i) {
    const mg_problem &q = probs[i];
    GemmArgs<T> &g = hp[(size_t)i];
    g.A = static_cast<const T *>(q.A);
    g.B = static_cast<const T *>(q.B);
    g.C = static_cast<T *>(q.C);
    g.lda = q.lda;
    g.ldb = q.ldb;
    g.ldc = q.ldc;
    g.m = (int)q.m;
    g.n = (int)q.n;
    g.k = (int)q.k;
    g.alpha = (T)q.alpha;
    g.beta = (T)q.beta;
    if (q.m == 0 || q.n == 0) continue;
    if (q.k == 0 || q.alpha == 0.0) {
      const int tm = (int)ceil_div(q.m, kScaleTile), tn = (int)ceil_div(q.n, kScaleTile);
      for (int a = 0; a < tm; ++a)
        for (int b = 0; b < tn; ++b) {
          tiles.push_back(GTileRec<T>{g, a, b, kScaleCls, 0});
          cost.push_back(0.5);  // C alone
        }
      per_cls[kNumGroupedClasses] += (int64_t)tm * tn;
      bytes += (double)q.m * q.n * sizeof(T) * (q.beta != 0.0 ? 2 : 1);
      continue;
    }
    int cls = table ? table->cls[tune_bucket(q.m, q.n, q.k)] : -1;
    if (cls < 0 || cls >= kNumGroupedClasses) cls = heuristic_class(dtype, q.m, q.n, q.k);
    const int bm = kClsBM[cls], bn = kClsBN[cls];
    const int tm = (int)ceil_div(q.m, bm), tn = (int)ceil_div(q.n, bn);
    for (int a = 0; a < tm; ++a)
      for (int b = 0; b < tn; ++b) {
        tiles.push_back(GTileRec<T>{g, a, b, cls, 0});
        cost.push_back(tile_cost(dtype, cls, q.k));
      }
    per_cls[cls] += (int64_t)tm * tn;
    flops += 2.0 * q.m * q.n * q.k;
    bytes += sizeof(T) * ((double)q.m * q.k + (double)q.k * q.n +
                          (double)q.m * q.n * (q.beta != 0.0 ? 2 : 1));
  }
  if (tiles.size() > (size_t)INT32_MAX) {
    set_error("too many tiles");
    return MG_ERR_INVALID_ARG;
  }
  // Longest first: the expensive tiles start at once and the cheap ones fill
  // in at the end.
  std::vector<int> order(tiles.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
  out->dtype = dtype;
  out->tiles.resize(tiles.size() * sizeof(GTileRec<T>));
  GTileRec<T> *dst = reinterpret_cast<GTileRec<T> *>(out->tiles.data());
  for (size_t i = 0; i < order.size(); ++i) dst[i] = tiles[(size_t)order[i]];
  out->ntiles = (int)tiles.size();
  mg_plan_stats &st = out->stats;
  st = mg_plan_stats{};
  st.problems = count;
  st.tiles = out->ntiles;
  for (int c = 0; c < kNumGroupedClasses; ++c) st.tiles_per_class[c] = per_cls[c];
  st.scale_tiles = per_cls[kNumGroupedClasses];
  st.flops = flops;
  st.bytes = bytes;
  return MG_OK;
}

template <typename T>
int occupancy_t(int *cus, int *occ) {
  // Once per process (one device model), thread-safe through the static's
  // initialisation: CU count, the kernel's LDS limit, workgroups per CU.
  struct Occ {
    hipError_t err;
    const char *what;
    int cus, occ;
  };
  static const Occ o = [] {
    Occ r{hipSuccess, "", 0, 0};
    int dev = 0;
    const size_t lds = grouped_lds_bytes<T>();
    if ((r.err = hipGetDevice(&dev)) != hipSuccess) r.what = "hipGetDevice";
    else if ((r.err = hipDeviceGetAttribute(&r.cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
             hipSuccess)
      r.what = "hipDeviceGetAttribute";
    else if ((r.err = hipFuncSetAttribute(reinterpret_cast<const void *>(grouped_kernel<T>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
             hipSuccess)
      r.what = "hipFuncSetAttribute";
    else if ((r.err = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                  &r.occ, reinterpret_cast<const void *>(grouped_kernel<T>), kTileThreads,
                  lds)) != hipSuccess)
      r.what = "hipOccupancyMaxActiveBlocksPerMultiprocessor";
    r.occ = std::max(1, r.occ);
    return r;
  }();
  if (o.err != hipSuccess) {
    set_error("%s failed: %s", o.what, hipGetErrorString(o.err));
    return MG_ERR_HIP;
  }
  *cus = o.cus;
  *occ = o.occ;
  return MG_OK;
}

// A dispatch counts work-items in 32 bits: longer lists (17 M problems of one
// tile) go in whole rounds over several launches.
template <typename T>
int launch_t(const void *d_tiles, int ntiles, int grid, hipStream_t s) {
  const int most = (int)(UINT32_MAX / kTileThreads) / grid * grid;
  const GTileRec<T> *tiles = static_cast<const GTileRec<T> *>(d_tiles);
  for (int64_t first = 0; first < ntiles; first += most) {
    const int part = (int)std::min<int64_t>(most, ntiles - first);
    hipLaunchKernelGGL(grouped_kernel<T>, dim3(part), dim3(kTileThreads), grouped_lds_bytes<T>(), s,
                       tiles + first, part, grid);
    MG_HIP_TRY(hipGetLastError());
  }
  return MG_OK;
}

int launch_raw(Plan *p, hipStream_t s) {
  return launch_worklist(p->dtype, p->d_tiles, p->ntiles, p->grid, s);
}

}  // namespace

int build_worklist(int dtype, int64_t count, const mg_problem *probs, const mg_tune_table *table,
                   WorkList *out) {
  return dtype == MG_F64 ? build_t<double>(count, probs, table, out)
                         : build_t<float>(count, probs, table, out);
}

int grouped_grid(int dtype, int ntiles, int *grid, int *occupancy) {
  int cus = 0, occ = 0;
  int rc = dtype == MG_F64 ? occupancy_t<double>(&cus, &occ) : occupancy_t<float>(&cus, &occ);
  if (rc != MG_OK) return rc;
  *grid = std::max(1, std::min(ntiles, cus * occ));
  if (occupancy) *occupancy = occ;
  return MG_OK;
}

int launch_worklist(int dtype, const void *d_tiles, int ntiles, int grid, hipStream_t s) {
  if (ntiles == 0) return MG_OK;
  return dtype == MG_F64 ? launch_t<double>(d_tiles, ntiles, grid, s)
                         : launch_t<float>(d_tiles, ntiles, grid, s);
}

int plan_create(int dtype, int64_t count, const mg_problem *probs, const mg_tune_table *table,
                Plan **out) {
  WorkList wl;
  int rc = build_worklist(dtype, count, probs, table, &wl);
  if (rc != MG_OK) return rc;
  Plan *p = new Plan();
  p->dtype = dtype;
  p->count = count;
  p->ntiles = wl.ntiles;
  p->stats = wl.stats;
  int occ = 1;
  rc = grouped_grid(dtype, p->ntiles, &p->grid, &occ);
  if (rc == MG_OK) rc = (hipGetDevice(&p->device) == hipSuccess) ? MG_OK : MG_ERR_HIP;
  p->stats.workgroups = p->grid;
  p->stats.occupancy = occ;
  auto upload = [&](void **dst, const std::vector<unsigned char> &src) -> int {
    MG_HIP_TRY(hipMalloc(dst, std::max<size_t>(src.size(), 256)));
    if (!src.empty()) MG_HIP_TRY(hipMemcpy(*dst, src.data(), src.size(), hipMemcpyHostToDevice));
    return MG_OK;
  };
  if (rc == MG_OK) rc = upload(&p->d_tiles, wl.tiles);
  if (rc != MG_OK) {
    plan_destroy(p);
    return rc;
  }
  *out = p;
  return MG_OK;
}

int plan_launch(Plan *p, hipStream_t s, bool use_graph) {
  if (p->ntiles == 0) return MG_OK;
  if (!use_graph) return launch_raw(p, s);
  if (p->exec == nullptr) {
    // Capture the launch once on a private stream.
    hipStream_t cap;
    MG_HIP_TRY(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      int rc = launch_raw(p, cap);
      hipGraph_t g = nullptr;
      hipError_t e2 = hipStreamEndCapture(cap, &g);
      if (rc != MG_OK || e2 != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        (void)hipStreamDestroy(cap);
        if (rc != MG_OK) return rc;
        set_error("hipStreamEndCapture failed: %s", hipGetErrorString(e2));
        return MG_ERR_HIP;
      }
      p->graph = g;
      e = hipGraphInstantiate(&p->exec, g, nullptr, nullptr, 0);
    }
    (void)hipStreamDestroy(cap);
    if (e != hipSuccess) {
      set_error("graph capture failed: %s", hipGetErrorString(e));
      return MG_ERR_HIP;
    }
    p->stats.graph = 1;
  }
  MG_HIP_TRY(hipGraphLaunch(p->exec, s));
  return MG_OK;
}

void plan_destroy(Plan *p) {
  if (p == nullptr) return;
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  if (p->d_tiles) (void)hipFree(p->d_tiles);
  delete p;
}

const mg_plan_stats &plan_stats(const Plan *p) { return p->stats; }

// ---------------------------------------------------------------------------
// Batched launch without allocation: the work list lives in a fixed device
// array (one copy per GPU, held until the process ends) instead of memory
// the library allocates per call.

static __device__ __align__(256) unsigned char scratch[kNoAllocWorklistBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's copy of `scratch` (the array's
// name is only a host-side stand-in).  Resolved once per device, with that
// device current.
int scratch_address(void **out) {
  int dev = 0;
  MG_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("device %d beyond the %d the static work-list buffer supports", dev, kMaxDevices);
    return MG_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr) {
      set_error("hipGetSymbolAddress(scratch) failed on device %d: %s", dev,
                hipGetErrorString(e));
      return MG_ERR_HIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return MG_OK;
}

}  // namespace

int gemm_batched_noalloc(int dtype, int64_t count, const mg_problem *probs, hipStream_t s) {
  // Host work list, reused by the calling thread (the copy below reads it
  // from pageable memory, which HIP stages before the call returns).
  thread_local WorkList wl;
  int rc = build_worklist(dtype, count, probs, nullptr, &wl);
  if (rc != MG_OK) return rc;
  if (wl.ntiles == 0) return MG_OK;
  if (wl.tiles.size() > kNoAllocWorklistBytes) {
    set_error("batch needs a %zu-byte work list (%d tiles); the static buffer holds %zu bytes",
              wl.tiles.size(), wl.ntiles, kNoAllocWorklistBytes);
    return MG_ERR_INVALID_ARG;
  }
  void *ptr = nullptr;
  if ((rc = scratch_address(&ptr)) != MG_OK) return rc;
  int grid = 1;
  if ((rc = grouped_grid(dtype, wl.ntiles, &grid, nullptr)) != MG_OK) return rc;
  MG_HIP_TRY(hipMemcpyAsync(ptr, wl.tiles.data(), wl.tiles.size(), hipMemcpyHostToDevice, s));
  return launch_worklist(dtype, ptr, wl.ntiles, grid, s);
}

}  // namespace mg

namespace mg {

namespace {

constexpr int kTuneMinProblems = 48;
constexpr int kTuneMaxProblems = 4096;
constexpr int kTuneWavesOfTiles = 4;          // tiles per workgroup slot when timing
constexpr int64_t kTuneOperandElems = 1 << 24;  // per operand scratch (A, B)

// Problems per bucket: enough that even the largest tile class gives every
// workgroup slot several tiles, so a class is judged by its throughput in a
// full batch rather than by the parallelism a few problems expose.
int64_t tune_count(int64_t m, int64_t n, int grid) {
  const int64_t t0 = ceil_div(m, kClsBM[0]) * ceil_div(n, kClsBN[0]);
  const int64_t want = ceil_div((int64_t)kTuneWavesOfTiles * grid, t0);
  return std::min<int64_t>(kTuneMaxProblems, std::max<int64_t>(kTuneMinProblems, want));
}

int time_plan(Plan *p, int reps, hipStream_t s, hipEvent_t e0, hipEvent_t e1, float *ms) {
  int rc = plan_launch(p, s, false);  // warm-up
  if (rc != MG_OK) return rc;
  MG_HIP_TRY(hipEventRecord(e0, s));
  for (int r = 0; r < reps; ++r) {
    rc = plan_launch(p, s, false);
    if (rc != MG_OK) return rc;
  }
  MG_HIP_TRY(hipEventRecord(e1, s));
  MG_HIP_TRY(hipEventSynchronize(e1));
  MG_HIP_TRY(hipEventElapsedTime(ms, e0, e1));
  return MG_OK;
}

}  // namespace

int autotune(int dtype, int reps, hipStream_t s, mg_tune_table *out) {
  const size_t esz = dtype == MG_F64 ? 8 : 4;
  int grid = 0;
  int rc = grouped_grid(dtype, INT32_MAX, &grid, nullptr);
  if (rc != MG_OK) return rc;
  // C needs a private region per problem; A and B are carved round-robin
  // from fixed scratch so that consecutive problems read different memory.
  int64_t c_elems = 0;
  for (int b = 0; b < kTuneEdges; ++b)
    for (int c = 0; c < kTuneEdges; ++c) {
      const int64_t m = tune_bucket_rep(b), n = tune_bucket_rep(c);
      c_elems = std::max(c_elems, tune_count(m, n, grid) * round_up(m * n, 64));
    }
  void *dA = nullptr, *dB = nullptr, *dC = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  auto cleanup = [&]() {
    if (dA) (void)hipFree(dA);
    if (dB) (void)hipFree(dB);
    if (dC) (void)hipFree(dC);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  };
  const size_t op_bytes = (size_t)kTuneOperandElems * esz;
  if (hipMalloc(&dA, op_bytes) != hipSuccess || hipMalloc(&dB, op_bytes) != hipSuccess ||
      hipMalloc(&dC, (size_t)c_elems * esz) != hipSuccess) {
    cleanup();
    set_error("autotune: scratch allocation failed");
    return MG_ERR_NO_MEMORY;
  }
  if (hipMemset(dA, 0, op_bytes) != hipSuccess || hipMemset(dB, 0, op_bytes) != hipSuccess ||
      hipMemset(dC, 0, (size_t)c_elems * esz) != hipSuccess ||
      hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    cleanup();
    set_error("autotune: scratch setup failed");
    return MG_ERR_HIP;
  }
  out->dtype = dtype;
  std::vector<mg_problem> probs;
  mg_tune_table forced;
  for (int bm = 0; bm < kTuneEdges && rc == MG_OK; ++bm)
    for (int bn = 0; bn < kTuneEdges && rc == MG_OK; ++bn)
      for (int bk = 0; bk < kTuneEdges && rc == MG_OK; ++bk) {
        const int64_t m = tune_bucket_rep(bm), n = tune_bucket_rep(bn), k = tune_bucket_rep(bk);
        const int64_t count = tune_count(m, n, grid);
        const int64_t a_sz = round_up(m * k, 64), b_sz = round_up(k * n, 64);
        const int64_t c_sz = round_up(m * n, 64);
        probs.assign((size_t)count, mg_problem{});
        int64_t oa = 0, ob = 0;
        for (int64_t i = 0; i < count; ++i) {
          if (oa + a_sz > kTuneOperandElems) oa = 0;
          if (ob + b_sz > kTuneOperandElems) ob = 0;
          mg_problem &q = probs[(size_t)i];
          q.m = m;
          q.n = n;
          q.k = k;
          q.alpha = 1.0;
          q.beta = 1.0;
          q.A = static_cast<char *>(dA) + (size_t)oa * esz;
          q.lda = k;
          q.B = static_cast<char *>(dB) + (size_t)ob * esz;
          q.ldb = n;
          q.C = static_cast<char *>(dC) + (size_t)(i * c_sz) * esz;
          q.ldc = n;
          oa += a_sz;
          ob += b_sz;
        }
        float best = 0;
        int best_cls = heuristic_class(dtype, m, n, k);
        for (int c = 0; c < kNumGroupedClasses && rc == MG_OK; ++c) {
          forced.dtype = dtype;
          for (int b = 0; b < MG_TUNE_BUCKETS; ++b) forced.cls[b] = c;
          Plan *p = nullptr;
          rc = plan_create(dtype, count, probs.data(), &forced, &p);
          if (rc != MG_OK) break;
          float ms = 0;
          rc = time_plan(p, reps, s, e0, e1, &ms);
          plan_destroy(p);
          if (rc == MG_OK && (c == 0 || ms < best)) {
            best = ms;
            best_cls = c;
          }
        }
        out->cls[(bm * kTuneEdges + bn) * kTuneEdges + bk] = best_cls;
      }
  cleanup();
  return rc;
}

}  // namespace mg
