// Native FP64 / FP32 GEMM: one workgroup per macro-tile of C (Section 4.2.2
// tiling), work division chosen per shape on the host.  This unit holds the
// plain-layout kernels and the host side; the transposed layouts are built
// in gemm_op_*.hip.
#include <algorithm>

#include "gemm_launch.h"
#include "split.h"

namespace mg {

namespace {

// C <- beta*C (alpha == 0 or k == 0).  beta == 0 writes zeros without reading.
template <typename T>
__global__ void scale_kernel(T *C, int64_t ldc, int m, int n, T beta) {
  const int64_t total = (int64_t)m * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / n, j = e % n;
    T *p = C + i * ldc + j;
    *p = beta == T(0) ? T(0) : beta * *p;
  }
}

struct CfgDesc {
  int bm, bn, wgm, wgn, bkm;
  int ks = 1;  // k groups of wgm x wgn wavefronts
};
// Work divisions (the order of launch_cfg): macro-tile, wavefront grid,
// k-step multiplier.  0-13 register-staged, 14-24 direct-load rings, 25 the
// naive mapping (a 16 x 16 workgroup of lanes, one output each), 26-29
// direct-load rings with two k groups of wavefronts.
constexpr CfgDesc kCfgs[] = {{128, 128, 2, 2, 1}, {128, 64, 2, 2, 1}, {64, 64, 2, 2, 1},
                             {64, 32, 2, 2, 1},   {32, 32, 2, 2, 1},  {128, 128, 4, 2, 1},
                             {128, 128, 2, 4, 1}, {64, 64, 2, 2, 2},  {128, 64, 4, 2, 1},
                             {128, 64, 2, 2, 2},  {256, 128, 4, 2, 1}, {128, 256, 2, 4, 1},
                             {256, 128, 4, 4, 1}, {128, 128, 4, 4, 1},  {64, 64, 2, 2, 1},
                             {64, 32, 2, 2, 1},   {128, 64, 2, 2, 1},  {128, 128, 2, 4, 1},
                             {256, 128, 4, 4, 1},  {32, 32, 2, 2, 1},   {64, 64, 4, 2, 1},
                             {128, 128, 2, 4, 1},  {128, 128, 2, 2, 1}, {64, 64, 2, 2, 1},
                             {64, 32, 2, 2, 1},   {16, 16, 0, 0, 0},  {64, 64, 2, 2, 1, 2},
                             {128, 64, 2, 2, 1, 2}, {64, 64, 2, 2, 1, 2},  {64, 32, 2, 1, 1, 2}};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);
constexpr int kNaiveCfg = 25;  // one output per lane, no LDS (wgm/wgn/bkm unused)

template <typename T>
int scale_c(int64_t m, int64_t n, double beta, void *C, int64_t ldc, hipStream_t s) {
  const int64_t total = m * n;
  const int blocks = (int)std::min<int64_t>((total + 255) / 256, 4096);
  hipLaunchKernelGGL(scale_kernel<T>, dim3(blocks), dim3(256), 0, s, static_cast<T *>(C), ldc,
                     (int)m, (int)n, (T)beta);
  MG_HIP_TRY(hipGetLastError());
  return MG_OK;
}

}  // namespace

bool vec_aligned(const void *p, int64_t ld, int64_t esz, int vec) {
  return (reinterpret_cast<uintptr_t>(p) % (uintptr_t)(esz * vec)) == 0 && ld % vec == 0;
}

int num_tile_cfgs() { return kNumCfgs; }

int tile_cfg_info(int dtype, int cfg, int *bm, int *bn, int *bk, int *threads) {
  if (cfg < 0 || cfg >= kNumCfgs || (dtype != MG_F64 && dtype != MG_F32)) {
    set_error("unknown tile cfg %d / dtype %d", cfg, dtype);
    return MG_ERR_INVALID_ARG;
  }
  if (bm) *bm = kCfgs[cfg].bm;
  if (bn) *bn = kCfgs[cfg].bn;
  if (cfg == kNaiveCfg) {
    if (bk) *bk = 1;
    if (threads) *threads = kCfgs[cfg].bm * kCfgs[cfg].bn;
    return MG_OK;
  }
  if (bk) *bk = kCfgs[cfg].bkm * (dtype == MG_F64 ? Mfma<double>::BK : Mfma<float>::BK);
  if (threads)
    *threads = cfg == 21 && dtype == MG_F64   ? 1024  // 16 wavefronts (launch_cfg)
               : cfg == 18 && dtype == MG_F32 ? 512
                                              : 64 * kCfgs[cfg].wgm * kCfgs[cfg].wgn * kCfgs[cfg].ks;
  return MG_OK;
}

// A lane's offset from its tile's corner spans up to 255 rows of an operand
// stored with k along its rows, but the rows of one k-step, 31 at most, of one
// stored by k rows (B, A^T): those keep the rings, 2 % faster than the
// register-staged tiles, up to pitches of 128 MiB (FP64 2048 x 2359296 x 256: 42.7
// -> 41.9 ms).
bool ring_operands(int dtype, bool ta, bool tb, const void *A, int64_t lda, const void *B,
                   int64_t ldb) {
  const int64_t esz = dtype == MG_F64 ? 8 : 4;
  const int64_t along_k = ((int64_t)1 << 24) / esz, k_rows = ((int64_t)1 << 27) / esz;
  return vec_aligned(A, lda, esz, 16 / (int)esz) && vec_aligned(B, ldb, esz, 16 / (int)esz) &&
         lda < (ta ? k_rows : along_k) && ldb < (tb ? along_k : k_rows);
}

namespace {

// Measured rate (TFLOP/s, whole chip, k = 2048, the launch itself taken off)
// of a work division when every CU has 1, 2, 3-5 and 6 or more of its tiles
// to run.  A tile takes as long whether it is full or reaches past the matrix,
// and the CU with the most tiles ends last, so a division's time is
// ceil(tiles / CUs) tiles at that rate: 128x128 tiles are the fastest per flop,
// but n = 3000 gives some CUs three of them and the others two (k = 2048: 729 us
// on 128x128 tiles, 554 on 64x64 ones, nine on every CU).
// `over`, for the same counts: what a tile costs besides its k, in k: filling
// its ring and writing C while no other workgroup of its CU covers them.  The
// FP64 128x128 ring has a CU to itself, so it wins only from k of 800 (16 tiles
// per CU) to 2200 (4 per CU) on (8192 x 8192, against 64x64 tiles: k = 64 332 against 257 us, k = 512 1099
// against 1020, k = 2048 73 against 70 TFLOP/s; 4096 x 4096: k = 256 165 against
// 139).  Fitted to 40 outputs from 32 x 32 to 8192 x 8192, k = 32 to 2048, with
// every division timed: the pick is within 1 % of the best on average.
struct TileRate {
  int cfg;
  float r[4], over[4];
};
constexpr TileRate kRing64[] = {{21, {70.f, 71.3f, 72.f, 73.f}, {64, 56, 72, 48}},
                                {23, {64.4f, 67.4f, 69.5f, 70.2f}, {48, 24, 16, 16}},
                                {15, {59.2f, 63.3f, 65.5f, 66.5f}, {16, 32, 32, 32}},
                                {19, {57.f, 59.f, 61.f, 62.f}, {0, 8, 24, 24}}};
// FP32 64x64 tiles on 8 wavefronts (20): two k-steps per stage (23) leave room
// for two workgroups per CU, so three tiles take as long as four (2048 x 1536 x
// 512: 41.2 against 33.2 us).
constexpr TileRate kRing32[] = {{22, {120.6f, 130.1f, 131.5f, 133.f}, {0, 0, 8, 0}},
                                {21, {126.f, 127.7f, 128.5f, 128.7f}, {0, 0, 8, 8}},
                                {20, {118.f, 113.f, 117.f, 120.f}, {0, 16, 0, 16}},
                                {15, {99.3f, 106.f, 107.f, 111.f}, {24, 16, 24, 24}},
                                {19, {104.f, 104.f, 105.f, 109.f}, {16, 0, 0, 16}}};
// The FP32 64x64 tiles of products cut along k, which leave a CU at most two.
constexpr TileRate kCutTile32 = {23, {106.7f, 110.7f, 115.f, 119.f}, {}};
// Operands the rings cannot load: the register-staged divisions.
constexpr TileRate kReg64[] = {{5, {61.6f, 67.9f, 67.8f, 68.f}, {24, 24, 24, 24}},
                               {8, {58.f, 64.5f, 65.f, 66.f}, {24, 24, 24, 24}},
                               {2, {52.5f, 62.4f, 64.5f, 66.8f}, {32, 32, 24, 24}},
                               {3, {46.f, 51.f, 54.f, 55.3f}, {24, 24, 16, 16}},
                               {4, {36.f, 44.f, 47.f, 49.f}, {16, 16, 16, 24}}};
constexpr TileRate kReg32[] = {{5, {116.7f, 126.9f, 128.5f, 129.f}, {16, 16, 16, 16}},
                               {8, {110.7f, 117.f, 119.f, 121.f}, {24, 16, 16, 16}},
                               {2, {81.f, 103.f, 117.f, 124.f}, {16, 8, 0, 8}},
                               {3, {74.9f, 96.1f, 106.5f, 112.f}, {24, 24, 16, 24}},
                               {4, {68.f, 84.f, 92.f, 98.f}, {24, 24, 32, 56}}};
constexpr int64_t kCus = 256;

int rate_column(int64_t per_cu) { return per_cu <= 1 ? 0 : per_cu == 2 ? 1 : per_cu <= 5 ? 2 : 3; }

// Flops per CU and k of `units` workgroups of one division, over its rate.
double division_cost(const TileRate &t, int64_t units) {
  const int64_t per_cu = ceil_div(units, kCus);
  return (double)per_cu * kCfgs[t.cfg].bm * kCfgs[t.cfg].bn / t.r[rate_column(per_cu)];
}

int64_t tiles_of(int cfg, int64_t m, int64_t n) {
  return ceil_div(m, kCfgs[cfg].bm) * ceil_div(n, kCfgs[cfg].bn);
}

// A dispatch counts work-items in 32 bits: one row of 2^29 outputs is too many
// workgroups in 32x32 tiles, not in 128x128 ones.
bool fits_dispatch(int cfg, int64_t m, int64_t n) {
  const CfgDesc &c = kCfgs[cfg];
  return tiles_of(cfg, m, n) * 64 * c.wgm * c.wgn * c.ks <= (int64_t)UINT32_MAX;
}

// 32x32 ring tiles only where an extent is below 1024: with both above, the
// wide and tall panels they re-read twice as often as 64x32 tiles are large.
// (If no division fits a dispatch, the launch of the one picked says so.)
template <size_t N>
const TileRate *best_division(const TileRate (&rates)[N], int64_t m, int64_t n, int64_t k) {
  const TileRate *best = nullptr;
  double cost = 0;
  bool fits = false;
  for (const TileRate &t : rates) {
    if (t.cfg == 19 && std::min(m, n) >= 1024) continue;
    const bool f = fits_dispatch(t.cfg, m, n);
    const int64_t tiles = tiles_of(t.cfg, m, n);
    const double c = division_cost(t, tiles) *
                     ((double)k + t.over[rate_column(ceil_div(tiles, kCus))]);
    if (best == nullptr || (f == fits ? c < cost : f)) {
      fits = f;
      best = &t;
      cost = c;
    }
  }
  return best;
}

}  // namespace

int pick_division(int dtype, bool ring, int64_t m, int64_t n, int64_t k) {
  const bool f64 = dtype != MG_F32;
  if (!ring) return (f64 ? best_division(kReg64, m, n, k) : best_division(kReg32, m, n, k))->cfg;
  const int cfg = (f64 ? best_division(kRing64, m, n, k) : best_division(kRing32, m, n, k))->cfg;
  // Between 2^20 and 2^22 outputs the 64x64 and 64x32 tiles run as two k
  // groups of wavefronts where those are about as fast: 64x64 tiles that leave a
  // CU at most one (two wavefronts per SIMD instead of one: within 3 % of the
  // one-group ring either way, 5 % in FP32), 64x32 tiles from four per CU (FP64
  // 68 against 66.5 TFLOP/s).
  const int64_t outputs = m * n;
  if (outputs >= (int64_t)1 << 20 && outputs < (int64_t)1 << 22) {
    if ((cfg == 23 || cfg == 20) && tiles_of(cfg, m, n) <= kCus) return 26;
    if (cfg == 15 && tiles_of(15, m, n) > 3 * kCus) return 29;
  }
  return cfg;
}

int pick_tile_cfg(int dtype, int64_t m, int64_t n, int64_t k) {
  return pick_division(dtype, true, m, n, k);
}

int gemm_tiles_nn(int dtype, int cfg, int64_t m, int64_t n, int64_t k, double alpha,
                  const void *A, int64_t lda, const void *B, int64_t ldb, double beta, void *C,
                  int64_t ldc, const PartPlan &pp, hipStream_t s) {
  return gemm_tiles<false, false>(dtype, cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, pp, s);
}

namespace {

// C <- alpha * (sum of the planes, in order) + beta * C: one output per lane,
// consecutive lanes along a plane.  FP32 sums are added in FP64 and rounded
// once.
template <typename T>
__global__ __launch_bounds__(256) void add_parts_kernel(const T *planes, int parts, T *C,
                                                        int64_t ldc, int m, int n, T alpha,
                                                        T beta) {
  const int64_t total = (int64_t)m * n;
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  double s = 0.0;
#pragma unroll 4
  for (int z = 0; z < parts; ++z) s += (double)planes[z * total + e];
  T *c = C + e / n * ldc + e % n;
  *c = beta != T(0) ? fma(alpha, (T)s, beta * *c) : alpha * (T)s;
}

// Whether and how to cut k.  A product whose tiles fill the chip badly and
// whose k is long (384 x 384 x 8192 FP64: 144 tiles of 32x32, each a chain of
// 512 k-steps: 69 us with 16-byte rows, 123 us without) runs `parts` times the
// workgroups on 1/parts of the k-steps each (49 us either way); that costs
// the partial sums' write and read and a second launch.  Both sides are
// counted in microseconds: the division's by its rate (kOverK: the k-steps'
// worth of time a part takes to fill and drain its ring), the planes at the
// rate a copy reaches from the L2 and the Infinity Cache, the launch as
// measured.  The host spends about 26 us on a cut call (the workspace and two
// launches), so no cut call counts for less.  The cut must win by a fifth
// (64 x 64 x 16384: 130 -> 29 us; 512 x 512 x 2048: 21 us uncut, not cut).
struct PartChoice {
  int cfg, parts, kpart;
};

PartChoice choose_parts(int dtype, bool ring, int64_t m, int64_t n, int64_t k) {
  constexpr int64_t kMinK = 1024;           // shorter k: nothing to win
  constexpr int64_t kMaxBytes = 64 << 20;   // of partial sums
  constexpr double kOverK = 64, kLaunchUs = 5, kPlaneGBps = 3500, kHostUs = 26;
  const int cfg = pick_division(dtype, ring, m, n, k);
  PartChoice best = {cfg, 1, 0};
  if (k < kMinK) return best;
  const bool f64 = dtype == MG_F64;
  const int64_t esz = f64 ? 8 : 4, bk = 128 / esz, steps = ceil_div(k, bk);
  auto find = [&](int c) -> const TileRate * {
    if (ring && !f64 && c == kCutTile32.cfg) return &kCutTile32;
    auto in = [&](const auto &tab) -> const TileRate * {
      for (const TileRate &t : tab)
        if (t.cfg == c) return &t;
      return nullptr;
    };
    return ring ? (f64 ? in(kRing64) : in(kRing32)) : (f64 ? in(kReg64) : in(kReg32));
  };
  // one flop-per-CU unit of division_cost takes 2 * kCus * 1e-6 us per k
  auto us = [&](const TileRate &t, int64_t units, double kk) {
    return division_cost(t, units) * kk * 2.0 * kCus * 1e-6;
  };
  const TileRate *t1 = find(cfg);
  if (t1 == nullptr) return best;  // a two-k-group division: the chip is full
  const double uncut = us(*t1, tiles_of(cfg, m, n), (double)k + kOverK);
  double least = 0.8 * uncut;
  if (least <= kHostUs) return best;
  const int candidates[2] = {ring ? 23 : 2, ring ? 19 : 4};
  for (int c : candidates) {
    const TileRate *t = find(c);
    const int64_t tiles = tiles_of(c, m, n);
    for (int64_t parts = 2; parts <= 64 && parts <= steps / 4; ++parts) {
      const int64_t kpart = ceil_div(steps, parts) * bk;
      if (ceil_div(k, kpart) != parts) continue;
      const double bytes = (double)parts * m * n * esz;
      if (bytes > (double)kMaxBytes) break;
      const double cost = std::max(kHostUs, us(*t, tiles * parts, (double)kpart + kOverK) +
                                                kLaunchUs + 2.0 * bytes / (kPlaneGBps * 1e3));
      if (cost < least) {
        least = cost;
        best = {c, (int)parts, (int)kpart};
      }
    }
  }
  return best;
}

template <typename T>
int add_parts(const PartPlan &pp, int64_t m, int64_t n, double alpha, double beta, void *C,
              int64_t ldc, hipStream_t s) {
  const int64_t blocks = ceil_div(m * n, 256);
  hipLaunchKernelGGL(add_parts_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s,
                     static_cast<const T *>(pp.planes), pp.parts, static_cast<T *>(C), ldc, (int)m,
                     (int)n, (T)alpha, (T)beta);
  MG_HIP_TRY(hipGetLastError());
  return MG_OK;
}

}  // namespace

namespace {

// Whether a cut call may take its workspace: not while `s` is captured, and only
// for a stream of the current device (the pool's memory is that device's, and a
// stream of another one may not reach it).
bool may_cut_on(hipStream_t s) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  int dev = 0;
  hipDevice_t stream_dev = 0;
  return hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
         hipGetDevice(&dev) == hipSuccess && hipStreamGetDevice(s, &stream_dev) == hipSuccess &&
         stream_dev == dev;
}

// The division for A B^T in place of `cfg`, with the same sums: FP32 64x64 tiles
// on 4 wavefronts (23) where one or two of them share a CU, or four and more: on
// 8 (20) each wavefront reads 16 columns of B^T for half the rows (1024 x 1024 x
// 3616 76 against 64 us).  Three per CU stay (2048 x 1536 x 256 20 against 23 us).
int division_nt(int cfg, int64_t tiles) {
  return cfg == 20 && ceil_div(tiles, kCus) != 3 ? 23 : cfg;
}

}  // namespace

int gemm_native_auto(int dtype, bool ta, bool tb, int64_t m, int64_t n, int64_t k, double alpha,
                     const void *A, int64_t lda, const void *B, int64_t ldb, double beta, void *C,
                     int64_t ldc, hipStream_t s) {
  const bool ring = ring_operands(dtype, ta, tb, A, lda, B, ldb);
  PartChoice pc = choose_parts(dtype, ring, m, n, k);
  if (alpha == 0.0) pc.parts = 1;
  if (!ta && tb) pc.cfg = division_nt(pc.cfg, tiles_of(pc.cfg, m, n));
  if (pc.parts > 1) {
    PartPlan pp;
    const int64_t bytes = (int64_t)pc.parts * m * n * (dtype == MG_F64 ? 8 : 4);
    if (may_cut_on(s) && pool_alloc(&pp.planes, bytes, s) == MG_OK) {
      pp.parts = pc.parts;
      pp.kpart = pc.kpart;
      auto run = ta ? (tb ? gemm_tiles_tt : gemm_tiles_tn) : (tb ? gemm_tiles_nt : gemm_tiles_nn);
      int rc = run(dtype, pc.cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, pp, s);
      if (rc == MG_OK)
        rc = dtype == MG_F64 ? add_parts<double>(pp, m, n, alpha, beta, C, ldc, s)
                             : add_parts<float>(pp, m, n, alpha, beta, C, ldc, s);
      const hipError_t e = hipFreeAsync(pp.planes, s);
      if (rc != MG_OK) return rc;
      MG_HIP_TRY(e);
      return MG_OK;
    }
    (void)hipGetLastError();
    clear_error();
    pc.cfg = pick_division(dtype, ring, m, n, k);
    if (!ta && tb) pc.cfg = division_nt(pc.cfg, tiles_of(pc.cfg, m, n));
  }
  return gemm_native_op(dtype, pc.cfg, ta, tb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, s);
}

int gemm_native_op(int dtype, int cfg, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                   double alpha, const void *A, int64_t lda, const void *B, int64_t ldb,
                   double beta, void *C, int64_t ldc, hipStream_t s) {
  if (dtype != MG_F64 && dtype != MG_F32) {
    set_error("unknown dtype %d", dtype);
    return MG_ERR_INVALID_ARG;
  }
  if (m == 0 || n == 0) return MG_OK;
  if (alpha == 0.0 || k == 0)
    return dtype == MG_F64 ? scale_c<double>(m, n, beta, C, ldc, s)
                           : scale_c<float>(m, n, beta, C, ldc, s);
  auto run = ta ? (tb ? gemm_tiles_tt : gemm_tiles_tn) : (tb ? gemm_tiles_nt : gemm_tiles_nn);
  return run(dtype, cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, PartPlan{}, s);
}

int gemm_native(int dtype, int cfg, int64_t m, int64_t n, int64_t k, double alpha, const void *A,
                int64_t lda, const void *B, int64_t ldb, double beta, void *C, int64_t ldc,
                hipStream_t s) {
  return gemm_native_op(dtype, cfg, false, false, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, s);
}

}  // namespace mg
