// Native FP64 / FP32 GEMM: one workgroup per macro-tile of C (Section 4.2.2
// tiling), work division chosen per shape on the host.  This unit holds the
// plain-layout kernels and the host side; the transposed layouts are built
// in gemm_op_*.hip.
#include "gemm_launch.h"

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
    *threads = cfg == 21 && dtype == MG_F64 ? 1024  // 16 wavefronts (launch_cfg)
                                            : 64 * kCfgs[cfg].wgm * kCfgs[cfg].wgn * kCfgs[cfg].ks;
  return MG_OK;
}

bool ring_operands(int dtype, const void *A, int64_t lda, const void *B, int64_t ldb) {
  const int64_t esz = dtype == MG_F64 ? 8 : 4;
  const int64_t max_ld = ((int64_t)1 << 24) / esz;
  return vec_aligned(A, lda, esz, 16 / (int)esz) && vec_aligned(B, ldb, esz, 16 / (int)esz) &&
         lda < max_ld && ldb < max_ld;
}

namespace {

// Measured rate (TFLOP/s, whole chip, k = 2048) of a work division when every
// CU has 1, 2, 3-5 and 6 or more of its tiles to run.  A tile takes as long
// whether it is full or reaches past the matrix, and the CU with the most
// tiles ends last, so a division's time is ceil(tiles / CUs) tiles at that
// rate: 128x128 tiles are the fastest per flop, but n = 3000 gives some CUs
// three of them and the others two (683 us by this count; 64x64 tiles: nine
// on every CU, 520 us; measured 1092 -> 821 us).
struct TileRate {
  int cfg;
  float r[4];
};
constexpr TileRate kRing64[] = {{21, {70.f, 71.3f, 72.f, 73.f}},
                                {23, {64.4f, 67.4f, 70.5f, 71.3f}},
                                {15, {59.2f, 63.3f, 65.5f, 66.5f}},
                                {19, {48.f, 57.f, 60.f, 62.f}}};
constexpr TileRate kRing32[] = {{22, {120.6f, 130.1f, 131.5f, 133.f}},
                                {21, {126.f, 127.7f, 128.5f, 128.7f}},
                                {23, {106.7f, 110.7f, 115.f, 119.f}},
                                {15, {99.3f, 106.f, 107.f, 111.f}},
                                {19, {85.8f, 98.5f, 102.5f, 109.f}}};
// Operands the rings cannot load: the register-staged divisions.
constexpr TileRate kReg64[] = {{5, {61.6f, 67.9f, 67.8f, 68.f}},
                               {8, {58.f, 64.5f, 65.f, 66.f}},
                               {2, {52.5f, 62.4f, 64.5f, 66.8f}},
                               {3, {42.9f, 49.6f, 54.f, 55.3f}},
                               {4, {30.7f, 42.8f, 47.f, 49.f}}};
constexpr TileRate kReg32[] = {{5, {116.7f, 126.9f, 128.5f, 129.f}},
                               {8, {110.7f, 117.f, 119.f, 121.f}},
                               {2, {81.f, 103.f, 117.f, 124.f}},
                               {3, {74.9f, 96.1f, 106.5f, 112.f}},
                               {4, {56.1f, 80.2f, 91.f, 98.f}}};
constexpr int64_t kCus = 256;

// Flops per CU of `units` workgroups of one division, over its rate.
double division_cost(const TileRate &t, int64_t units) {
  const int64_t per_cu = ceil_div(units, kCus);
  const float r = t.r[per_cu <= 1 ? 0 : per_cu == 2 ? 1 : per_cu <= 5 ? 2 : 3];
  return (double)per_cu * kCfgs[t.cfg].bm * kCfgs[t.cfg].bn / r;
}

int64_t tiles_of(int cfg, int64_t m, int64_t n) {
  return ceil_div(m, kCfgs[cfg].bm) * ceil_div(n, kCfgs[cfg].bn);
}

// 32x32 ring tiles only where an extent is below 1024: with both above, the
// wide and tall panels they re-read twice as often as 64x32 tiles are large.
template <size_t N>
const TileRate *best_division(const TileRate (&rates)[N], int64_t m, int64_t n) {
  const TileRate *best = nullptr;
  double cost = 0;
  for (const TileRate &t : rates) {
    if (t.cfg == 19 && std::min(m, n) >= 1024) continue;
    const double c = division_cost(t, tiles_of(t.cfg, m, n));
    if (best == nullptr || c < cost) {
      best = &t;
      cost = c;
    }
  }
  return best;
}

}  // namespace

int pick_division(int dtype, bool ring, int64_t m, int64_t n) {
  const bool f64 = dtype != MG_F32;
  if (!ring) return (f64 ? best_division(kReg64, m, n) : best_division(kReg32, m, n))->cfg;
  const int cfg = (f64 ? best_division(kRing64, m, n) : best_division(kRing32, m, n))->cfg;
  // Between 2^20 and 2^22 outputs the 64x64 and 64x32 tiles run as two k
  // groups of wavefronts where those are as fast: 64x64 tiles that leave a CU
  // at most one (two wavefronts per SIMD instead of one: within 3 % of the
  // one-group ring either way), 64x32 tiles from four per CU (FP64 68 against
  // 66.5 TFLOP/s).
  const int64_t outputs = m * n;
  if (outputs >= (int64_t)1 << 20 && outputs < (int64_t)1 << 22) {
    if (cfg == 23 && tiles_of(23, m, n) <= kCus) return 26;
    if (cfg == 15 && tiles_of(15, m, n) > 3 * kCus) return 29;
  }
  return cfg;
}

int pick_tile_cfg(int dtype, int64_t m, int64_t n, int64_t k) {
  (void)k;
  return pick_division(dtype, true, m, n);
}

int gemm_tiles_nn(int dtype, int cfg, int64_t m, int64_t n, int64_t k, double alpha,
                  const void *A, int64_t lda, const void *B, int64_t ldb, double beta, void *C,
                  int64_t ldc, hipStream_t s) {
  return gemm_tiles<false, false>(dtype, cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, s);
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
  return run(dtype, cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, s);
}

int gemm_native(int dtype, int cfg, int64_t m, int64_t n, int64_t k, double alpha, const void *A,
                int64_t lda, const void *B, int64_t ldb, double beta, void *C, int64_t ldc,
                hipStream_t s) {
  return gemm_native_op(dtype, cfg, false, false, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, s);
}

}  // namespace mg
