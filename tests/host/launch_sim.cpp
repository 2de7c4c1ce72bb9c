// Host side of libmg's launches, run without a GPU: this program defines the
// HIP runtime calls that the library makes (an executable's definitions come
// before a shared library's), so that every launch is recorded instead of
// enqueued, memory is an address that nobody reads, and the conditions a call
// has to cope with (a stream that is being captured, a pool that is exhausted,
// a stream of another device) are set from here.  Checked are the kernels a
// call picks, their grids, and their arguments.
#include <cxxabi.h>
#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "mg.h"

namespace mg {  // internal to the library, exported
bool split_refill_early(int64_t k, int64_t tiles_m, int64_t tiles_n, int64_t batch_tiles);
}

static int failures = 0;

#define EXPECT(cond)                                                              \
  do {                                                                            \
    if (!(cond)) {                                                                \
      std::fprintf(stderr, "line %d: expected %s (last error: %s)\n", __LINE__,   \
                   #cond, mg_last_error());                                       \
      ++failures;                                                                 \
    }                                                                             \
  } while (0)

// ------------------------------------------------------- the device's state
struct Launch {
  std::string kernel;
  dim3 grid, block;
  struct {  // of a product's kernel: the workspace, parts and k per part
    void *planes;
    int parts, kpart;
  } cut;
};
static struct {
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  bool pool_empty = false;
  int stream_device = 0;
} state;
static std::vector<Launch> launches;
static std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> m;  // filled by static constructors
  return m;
}
static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t s;
} config;

static std::string demangled(const char *name) {
  int st = 0;
  char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  std::string r = st == 0 ? d : name;
  std::free(d);
  return r;
}

static void *fake(uint64_t i) { return reinterpret_cast<void *>((i + 1) << 40); }

extern "C" {
void __hipRegisterFunction(void **modules, const void *host, char *dev, const char *name,
                           unsigned limit, void *a, void *b, void *c, void *d, int *e) {
  kernels()[host] = demangled(name);
  typedef void (*F)(void **, const void *, char *, const char *, unsigned, void *, void *, void *,
                    void *, int *);
  static const F real = reinterpret_cast<F>(dlsym(RTLD_NEXT, "__hipRegisterFunction"));
  real(modules, host, dev, name, limit, a, b, c, d, e);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  config = {grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *s = config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t,
                           hipStream_t) {
  Launch l = {kernels()[f], grid, block, {}};
  if (l.kernel.find("gemm_dma_kernel<") != std::string::npos ||
      l.kernel.find("gemm_native_kernel<") != std::string::npos)
    std::memcpy(&l.cut, args[3], sizeof l.cut);
  launches.push_back(l);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = state.capture;
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) {
  *d = state.stream_device;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 3;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t) {
  *p = fake(93);
  return hipSuccess;
}
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t *p, const hipMemPoolProps *) {
  *p = static_cast<hipMemPool_t>(fake(90));
  return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void **p, size_t, hipMemPool_t, hipStream_t) {
  if (state.pool_empty) return hipErrorOutOfMemory;
  *p = fake(91);
  return hipSuccess;
}
hipError_t hipFreeAsync(void *, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) {
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = static_cast<hipEvent_t>(fake(92));
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
}

// ------------------------------------------------------------------- checks
static mg_problem problem(int64_t m, int64_t n, int64_t k, int c) {
  return mg_problem{m, n, k, 1.0, 1.0, fake(1), k, fake(2), n, fake(c), n};
}

// The batched split product's lane offsets: row 15 of a slice, 15 * kp_bytes
// plus a byte of the 64-byte stage, has to fit the offset's type.
static void split_batch_offsets() {
  struct {
    int algo;
    int64_t k;
    bool wide;
  } cases[] = {{MG_SPLIT_I8, 4096, false},          {MG_SPLIT_BF16, 4096, false},
               {MG_SPLIT_BF16, 143165568, false},   {MG_SPLIT_BF16, 143165569, true},
               {MG_SPLIT_BF16, 143200000, true},    {MG_SPLIT_I8, 286331136, false},
               {MG_SPLIT_I8, 286331137, true},      {MG_SPLIT_BF16, 170000000, true}};
  for (const auto &c : cases) {
    const int64_t kp_bytes = (c.k + 63) / 64 * 64 * (c.algo == MG_SPLIT_BF16 ? 2 : 1);
    EXPECT((15 * kp_bytes + 63 > (int64_t)UINT32_MAX) == c.wide);
    launches.clear();
    const mg_problem p[2] = {problem(16, 24, 200, 3), problem(16, 64, c.k, 4)};
    EXPECT(mg_gemm_batched(MG_F64, c.algo, 2, p, nullptr) == MG_OK);
    const std::string &prod = launches.empty() ? "" : launches.back().kernel;
    EXPECT(prod.find("split_allpairs_kernel<") != std::string::npos);
    EXPECT((prod.find(", long>") != std::string::npos) == c.wide);
  }
}

// A batch's list of 64x64 tiles (C <- beta C, two rows of tiles): every tile
// runs, and no dispatch has more work-items than its 32-bit count holds.
static void batch_dispatches() {
  for (int64_t tiles : {2ll, 1000ll, (1ll << 24) - 2, 1ll << 24, (1ll << 24) + 6}) {
    const int64_t n = tiles / 2 * 64;
    const mg_problem p{65, n, 0, 0.0, 0.5, nullptr, 1, nullptr, n, fake(3), n};
    launches.clear();
    mg_plan *plan = nullptr;
    EXPECT(mg_plan_create(MG_F32, 1, &p, nullptr, &plan) == MG_OK);
    EXPECT(mg_plan_launch_direct(plan, nullptr) == MG_OK);
    int64_t run = 0;
    for (const Launch &l : launches) {
      EXPECT(l.kernel.find("grouped_kernel<") != std::string::npos);
      EXPECT((uint64_t)l.grid.x * l.block.x <= UINT32_MAX && l.grid.y == 1 && l.grid.z == 1);
      run += l.grid.x;
    }
    EXPECT(run == tiles);
    EXPECT(mg_plan_destroy(plan) == MG_OK);
  }
}

// Outputs of nearly 2^30 columns: the division picked, and the 128x128 ones
// asked for, fit a dispatch wherever 128x128 tiles on 8 wavefronts do, and the
// work-item count says so where they don't.
static void long_rows() {
  const int64_t big = 1ll << 30;
  for (int dtype : {MG_F64, MG_F32})
    for (int64_t off : {0, 8})  // 16-byte aligned operands, and not
      for (int64_t m : {1, 32, 33, 64, 65, 96, 97, 128, 129, 200})
        for (int64_t n : {(int64_t)1000, big / 8, big / 4 + 5, big / 2 - 40, big / 2, big - 128, big - 1})
          for (int cfg : {-1, 13, 17, 21, 22}) {
            char *A = static_cast<char *>(fake(1)) + off, *B = static_cast<char *>(fake(2)) + off;
            launches.clear();
            const int rc = mg_gemm_ex(dtype, cfg, 0, 0, m, n, 16, 1.0, A, 16, B, n, 0.5, fake(3), n,
                                      nullptr);
            const int64_t t128 = (m + 127) / 128 * ((n + 127) / 128);
            if (t128 * 512 <= (int64_t)UINT32_MAX) EXPECT(rc == MG_OK);
            EXPECT(rc == MG_OK || std::strstr(mg_last_error(), "too many tiles") != nullptr);
            EXPECT(launches.size() == (rc == MG_OK ? 1u : 0u));
            for (const Launch &l : launches)
              EXPECT((uint64_t)l.grid.x * l.block.x <= UINT32_MAX);
          }
}

// The 32x32 ring's instance without the unrolled loop, below the k of one pass.
static void short_ring() {
  for (int dtype : {MG_F64, MG_F32})
    for (int t = 0; t < 4; ++t)
      for (int64_t k : {1, 16, 127, 128, 255, 256, 1000}) {
        launches.clear();
        EXPECT(mg_gemm_ex(dtype, 19, t & 1, t >> 1, 64, 64, k, 1.0, fake(1), 1024, fake(2), 1024,
                          1.0, fake(3), 64, nullptr) == MG_OK);
        EXPECT(launches.size() == 1 && launches[0].kernel.find(" 32, 32, 2, 2, 4,") !=
                                           std::string::npos);
        const bool plain = launches[0].kernel.find(", true>(") != std::string::npos;
        EXPECT(plain == (k < (dtype == MG_F64 ? 128 : 256)));
      }
}

// Short k: a tile's fill and its C count, so the tile that is fastest per k is
// not the fastest (times measured, us, beside the cases).
static void short_k() {
  struct {
    int dtype;
    int64_t m, n, k;
    const char *kernel;
  } cases[] = {
      {MG_F64, 8192, 8192, 64, "gemm_dma_kernel<double, 64, 64,"},     // 128x128 332, 64x64 257
      {MG_F64, 8192, 8192, 512, "gemm_dma_kernel<double, 64, 64,"},    // 1099, 1020
      {MG_F64, 4096, 4096, 256, "gemm_dma_kernel<double, 64, 64,"},    // 165, 139
      {MG_F64, 8192, 8192, 8192, "gemm_dma_kernel<double, 128, 128,"},
      {MG_F64, 2560, 2560, 64, "gemm_dma_kernel<double, 64, 64,"},     // 64x32 31.5, 64x64 28.9
      {MG_F64, 256, 1536, 32, "gemm_dma_kernel<double, 32, 32,"},      // 64x32 4.71, 32x32 4.50
      {MG_F64, 385, 1025, 33, "gemm_native_kernel<double, 32, 32,"},   // 64x32 6.1, 32x32 5.6
      {MG_F32, 2048, 1536, 512, "gemm_dma_kernel<float, 64, 64, 4, 2,"},  // 2x2: 41.2, 4x2: 33.2
      {MG_F32, 2048, 2048, 2048, "gemm_dma_kernel<float, 128, 128,"},
  };
  for (const auto &c : cases) {
    launches.clear();
    EXPECT(mg_gemm(c.dtype, MG_NATIVE, c.m, c.n, c.k, 1.0, fake(1), c.k, fake(2), c.n, 1.0, fake(3),
                   c.n, nullptr) == MG_OK);
    EXPECT(launches.size() == 1 && launches[0].kernel.find(c.kernel) != std::string::npos);
  }
}

// The all-pairs split tile's refill (times measured, us, early / late).
static void split_refill() {
  struct {
    int64_t k, tm, tn, batch;
    bool early;
  } cases[] = {
      {1024, 16, 16, 256, true},     // 46 / 53
      {8192, 16, 16, 256, true},     // 266 / 339
      {8192, 24, 24, 576, true},     // 626 / 675
      {2048, 32, 32, 1024, true},    // 195 / 200
      {4096, 32, 32, 1024, false},   // 408 / 394
      {8192, 32, 32, 1024, false},   // 973 / 881
      {8192, 16, 64, 1024, false},   // 1066 / 930
      {4096, 12, 86, 1032, true},    // 519 / 565
      {2048, 44, 44, 1936, true},    // 345 / 365
      {4096, 44, 44, 1936, false},   // 778 / 720
      {8192, 32, 64, 2048, false},   // 2308 / 1678
      {2048, 64, 64, 4096, true},    // 731 / 778
      {4096, 64, 64, 4096, false},   // 1824 / 1517
      {4096, 16, 16, 768, true},     // three problems in a batch: 420 / 462
      {4096, 16, 16, 4096, false},   // sixteen: 2347 / 2167
      {4096, 2, 2, 2000, true},      // 500 of 4 tiles: 3211 / 3409
      {2048, 12, 12, 9216, true},    // 2797 / 2916
  };
  for (const auto &c : cases)
    EXPECT(mg::split_refill_early(c.k, c.tm, c.tn, c.batch) == c.early);
}

// Which operands the rings load: aligned rows, and pitches whose lane offsets
// fit 32 bits (255 rows along k, 31 rows of k).
static void ring_pitches() {
  for (int dtype : {MG_F64, MG_F32})
    for (int ta : {0, 1})
      for (int tb : {0, 1})
        for (int64_t a : {0, 1, 2})
          for (int64_t b : {0, 1, 2}) {
            const int64_t esz = dtype == MG_F64 ? 8 : 4;
            const int64_t pitch[3] = {(1ll << 24) / esz - 16, (1ll << 27) / esz - 16,
                                      (1ll << 27) / esz};
            launches.clear();
            EXPECT(mg_gemm_ex(dtype, -1, ta, tb, 64, 64, 64, 1.0, fake(1), pitch[a], fake(2),
                              pitch[b], 1.0, fake(3), 64, nullptr) == MG_OK);
            const bool ring = a <= (ta ? 1 : 0) && b <= (tb ? 0 : 1);
            EXPECT(launches.size() == 1 &&
                   (launches[0].kernel.find("gemm_dma_kernel<") != std::string::npos) == ring);
          }
}

// Products cut along k: the parts cover k, the grid holds every tile of every
// part, and a second kernel adds them; uncut on a stream that is captured or
// belongs to another device, and when the pool has no memory.
static void long_k() {
  struct {
    int64_t m, n, k;
  } shapes[] = {{64, 64, 16384}, {1, 3, 20001}, {65, 33, 9985}, {130, 70, 8193}, {200, 200, 12288},
                {96, 80, 16384},
                // a last part of one k: on the FP64 rings, and off the rings
                {33, 70, 19041}, {33, 70, 12097}, {33, 70, 16193}};
  int last_of_one = 0;
  for (int dtype : {MG_F64, MG_F32})
    for (int64_t odd : {0, 1})  // pitches that the rings load, and not
      for (int t = 0; t < 4; ++t)
        for (const auto &q : shapes) {
          auto run = [&] {
            launches.clear();
            return mg_gemm_ex(dtype, -1, t & 1, t >> 1, q.m, q.n, q.k, 1.5, fake(1), 20480 + odd,
                              fake(2), 20480 + odd, 0.5, fake(3), q.n, nullptr);
          };
          EXPECT(run() == MG_OK && launches.size() == 2);
          if (launches.size() != 2) continue;
          const Launch cut = launches[0];
          const int64_t parts = cut.cut.parts, kpart = cut.cut.kpart;
          EXPECT(cut.cut.planes == fake(91) && parts >= 2);
          EXPECT((parts - 1) * kpart < q.k && q.k <= parts * kpart && cut.grid.x % parts == 0);
          EXPECT(launches[1].kernel.find("add_parts_kernel<") != std::string::npos);
          last_of_one += q.k - (parts - 1) * kpart == 1;
          for (int why = 0; why < 3; ++why) {
            state.capture = why == 0 ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
            state.stream_device = why == 1;
            state.pool_empty = why == 2;
            EXPECT(run() == MG_OK && launches.size() == 1);
            EXPECT(std::strlen(mg_last_error()) == 0);
            if (launches.size() == 1)
              EXPECT(launches[0].cut.planes == nullptr && launches[0].cut.parts == 1);
          }
          state = {};
        }
  EXPECT(last_of_one >= 12);  // each of the three, in every layout
}

// FP32 A B^T: 64x64 tiles on 4 wavefronts unless three share a CU (times measured,
// us: 8 / 4 wavefronts).
static void f32_nt() {
  struct {
    int64_t m, n, k;
    const char *kernel;
  } cases[] = {{1000, 1000, 512, " 64, 64, 2, 2, 2,"},    // k = 1024: 24.3 / 20.9
               {2048, 1536, 512, " 64, 64, 4, 2, 4,"},    // k = 256: 19.8 / 23.0
               {64, 64, 16384, nullptr}};                 // cut along k: 4 wavefronts
  for (const auto &c : cases) {
    launches.clear();
    EXPECT(mg_gemm_ex(MG_F32, -1, 0, 1, c.m, c.n, c.k, 1.0, fake(1), c.k, fake(2), c.k, 1.0, fake(3),
                      c.n, nullptr) == MG_OK);
    EXPECT(launches.size() == (c.kernel ? 1u : 2u));
    EXPECT(c.kernel == nullptr || launches[0].kernel.find(c.kernel) != std::string::npos);
    EXPECT(c.kernel || launches[0].kernel.find(" 64, 64, 4, 2, 4,") == std::string::npos);
  }
}

// Workgroups of the explicit divisions whose shape depends on type or layout.
static void explicit_divisions() {
  struct {
    int dtype, cfg, ta, tb;
    int64_t odd;
    unsigned threads;
  } cases[] = {
      {MG_F64, 13, 0, 0, 0, 1024}, {MG_F64, 13, 1, 0, 0, 512}, {MG_F64, 13, 1, 1, 0, 1024},
      {MG_F32, 13, 1, 0, 0, 512},  {MG_F64, 21, 1, 0, 1, 512}, {MG_F64, 21, 1, 0, 0, 1024},
      {MG_F64, 18, 0, 1, 0, 1024}, {MG_F32, 18, 0, 1, 0, 512}, {MG_F32, 26, 1, 0, 0, 512},
  };
  for (const auto &c : cases) {
    launches.clear();
    EXPECT(mg_gemm_ex(c.dtype, c.cfg, c.ta, c.tb, 300, 300, 300, 1.0, fake(1), 304 + c.odd, fake(2),
                      304 + c.odd, 1.0, fake(3), 300, nullptr) == MG_OK);
    EXPECT(launches.size() == 1 && launches[0].block.x == c.threads);
    int threads = 0;
    EXPECT(mg_tile_cfg_info(c.dtype, c.cfg, nullptr, nullptr, nullptr, &threads) == MG_OK);
    EXPECT(c.odd || (c.cfg == 13 && c.ta && !c.tb) || threads == (int)c.threads);
  }
}

int main() {
  split_batch_offsets();
  batch_dispatches();
  long_rows();
  short_ring();
  short_k();
  split_refill();
  ring_pitches();
  long_k();
  explicit_divisions();
  f32_nt();
  std::printf("host launches: %d failures\n", failures);
  return failures != 0;
}
