// Native FP64 / FP32 GEMM kernels and their launchers, templated on the
// operand layouts: C <- alpha*op(A)*op(B) + beta*C with op(X) = X or X^T
// (one workgroup per macro-tile of C, Section 4.2.2 tiling).  Each layout
// combination is instantiated by its own translation unit.
#pragma once

#include "gemm_dma.h"
#include "gemm_native.h"
#include "gemm_tile.h"

namespace mg {

namespace {

constexpr int kGroupM = 8;  // tile-rows walked together by the raster

// The FP64 128x128 tile on 8 wavefronts is held to 128 registers (6 spilled
// outside the k loop): two workgroups per CU cover each other's barriers
// (4 tiles per CU: 57.7 -> 59.8 TFLOP/s).
template <typename T, int BM, int BN, int WGM, int WGN, int BKM, bool TA, bool TB>
__global__ __launch_bounds__((TileShape<T, BM, BN, WGM, WGN, BKM>::THREADS),
                             (TileShape<T, BM, BN, WGM, WGN, BKM>::MINW)) void gemm_native_kernel(
    GemmArgs<T> g, int tiles_m, int tiles_n, KSplit<T> ks) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T *smem = reinterpret_cast<T *>(lds_raw);
  int tm, tn;
  const int tiles = tiles_m * tiles_n;
  const int t = take_part<T, TA, TB>(g, ks, xcd_remap(blockIdx.x, tiles * ks.parts), tiles);
  grouped_tile(t, tiles_m, tiles_n, kGroupM, tm, tn);
  gemm_tile<T, BM, BN, WGM, WGN, BKM, TA, TB>(g, tm * BM, tn * BN, smem);
}

template <typename T, int BM, int BN, int WGM, int WGN, int NS, bool TA, bool TB, int KS = 1,
          int KU = 1, bool SHORT = false>
__global__ __launch_bounds__((DmaShape<T, BM, BN, WGM, WGN, NS, KS, KU>::THREADS),
                             (DmaShape<T, BM, BN, WGM, WGN, NS, KS, KU>::MINW)) void gemm_dma_kernel(
    GemmArgs<T> g, int tiles_m, int tiles_n, KSplit<T> ks) {
  extern __shared__ __align__(16) unsigned char lds[];
  int tm, tn;
  const int tiles = tiles_m * tiles_n;
  const int t = take_part<T, TA, TB>(g, ks, xcd_remap(blockIdx.x, tiles * ks.parts), tiles);
  grouped_tile(t, tiles_m, tiles_n, kGroupM, tm, tn);
  gemm_dma_tile<T, BM, BN, WGM, WGN, NS, TA, TB, KS, KU, SHORT>(g, tm * BM, tn * BN, lds);
}

// The textbook mapping without the paper's hierarchy below the thread: one
// output per lane, no shared memory, the k loop reading A and B straight
// from global memory (the naive triple loop of Section 4.2's portability
// experiment).  Lanes of a 16 x 16 workgroup take consecutive columns, so
// B and C accesses coalesce and A values are shared by a row of lanes.
// The sum runs in increasing k with one FMA per term.
constexpr int kNaiveDim = 16;

template <typename T, bool TA, bool TB>
__global__ __launch_bounds__(kNaiveDim *kNaiveDim) void gemm_naive_kernel(GemmArgs<T> g) {
  const int j = blockIdx.x * kNaiveDim + threadIdx.x;
  const int i = blockIdx.y * kNaiveDim + threadIdx.y;
  if (i >= g.m || j >= g.n) return;
  T s = T(0);
  for (int p = 0; p < g.k; ++p) {
    const T a = TA ? g.A[(int64_t)p * g.lda + i] : g.A[(int64_t)i * g.lda + p];
    const T b = TB ? g.B[(int64_t)j * g.ldb + p] : g.B[(int64_t)p * g.ldb + j];
    s = fma(a, b, s);
  }
  T *c = g.C + (int64_t)i * g.ldc + j;
  *c = g.beta != T(0) ? fma(g.alpha, s, g.beta * *c) : g.alpha * s;
}

template <typename T, bool TA, bool TB>
int launch_naive(const GemmArgs<T> &g, hipStream_t s) {
  const int64_t bx = (g.n + kNaiveDim - 1) / kNaiveDim, by = (g.m + kNaiveDim - 1) / kNaiveDim;
  if (by > 65535 || bx * by * kNaiveDim * kNaiveDim > (int64_t)UINT32_MAX) {
    set_error("naive work division: %d x %d outputs exceed one dispatch", g.m, g.n);
    return MG_ERR_INVALID_ARG;
  }
  hipLaunchKernelGGL((gemm_naive_kernel<T, TA, TB>), dim3((unsigned)bx, (unsigned)by),
                     dim3(kNaiveDim, kNaiveDim), 0, s, g);
  MG_HIP_TRY(hipGetLastError());
  return MG_OK;
}

// Raises a kernel's dynamic LDS limit to what its ring needs; called through
// a function-local static, so once per template instance and thread-safe.
template <typename K>
hipError_t set_max_lds(K kern, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <typename T, int BM, int BN, int WGM, int WGN, int BKM, bool TA, bool TB>
int launch_one(const GemmArgs<T> &g, const KSplit<T> &ks, hipStream_t s) {
  typedef TileShape<T, BM, BN, WGM, WGN, BKM, TA, TB> S;
  const int tiles_m = (g.m + BM - 1) / BM, tiles_n = (g.n + BN - 1) / BN;
  const int64_t tiles = (int64_t)tiles_m * tiles_n * ks.parts;
  if (tiles * S::THREADS > (int64_t)UINT32_MAX) {  // 32-bit work-item count per dispatch
    set_error("too many tiles (%lld) for one dispatch", (long long)tiles);
    return MG_ERR_INVALID_ARG;
  }
  auto kern = gemm_native_kernel<T, BM, BN, WGM, WGN, BKM, TA, TB>;
  static const hipError_t attr = set_max_lds(kern, S::LDS_BYTES);  // once per instance
  MG_HIP_TRY(attr);
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(S::THREADS), S::LDS_BYTES, s, g, tiles_m,
                     tiles_n, ks);
  MG_HIP_TRY(hipGetLastError());
  return MG_OK;
}

template <typename T, int BM, int BN, int WGM, int WGN, int NS, bool TA, bool TB, int KS = 1,
          int KU = 1, bool SHORT = false>
int launch_dma(const GemmArgs<T> &g, const KSplit<T> &ks, hipStream_t s) {
  typedef DmaShape<T, BM, BN, WGM, WGN, NS, KS, KU> S;
  const int tiles_m = (g.m + BM - 1) / BM, tiles_n = (g.n + BN - 1) / BN;
  const int64_t tiles = (int64_t)tiles_m * tiles_n * ks.parts;
  if (tiles * S::THREADS > (int64_t)UINT32_MAX) {  // 32-bit work-item count per dispatch
    set_error("too many tiles (%lld) for one dispatch", (long long)tiles);
    return MG_ERR_INVALID_ARG;
  }
  auto kern = gemm_dma_kernel<T, BM, BN, WGM, WGN, NS, TA, TB, KS, KU, SHORT>;
  static const hipError_t attr = set_max_lds(kern, S::LDS_BYTES);  // once per instance
  MG_HIP_TRY(attr);
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(S::THREADS), S::LDS_BYTES, s, g, tiles_m,
                     tiles_n, ks);
  MG_HIP_TRY(hipGetLastError());
  return MG_OK;
}

// Work divisions 0-13 stage A and B through registers; 14-24 load them
// straight into an LDS ring (operands as ring_operands says: otherwise a
// register-staged division of the same macro-tile runs); 25 is the naive
// one-output-per-lane mapping; 26-29 are direct-load rings whose wavefronts
// form two k groups (twice the wavefronts per output block).  The host's table
// of shapes (kCfgs in gemm_native.hip) lists the same divisions in order.
template <typename T, bool TA, bool TB>
int launch_cfg(int cfg, bool dma_ok, const GemmArgs<T> &g, const KSplit<T> &ks, hipStream_t s) {
  // FP32 halves the matrix cores' time per k-step, so its 64x64 and 64x32
  // rings meet every second k-step (4 tiles of 64x64 per CU: 104 -> 116
  // TFLOP/s; FP64, where the deeper stage costs resident workgroups, 71 -> 66).
  // The 128x128 ring (21): FP64 on 16 wavefronts of 32x32, whose fragments
  // fit twice, 72.8 TFLOP/s at n = 4096 against 72.0 on 8 wavefronts of
  // 64x32; FP32 on 8 with two k-steps per stage, 125.6 at n = 2048 against
  // 122.8 on 16.
  constexpr bool F64 = sizeof(T) == 8;
  constexpr int KU32 = F64 ? 1 : 2;
  // 128x128 tiles on 16 wavefronts (13, the FP64 ring 21 and what 17, 21 and 22
  // fall back to) run on 8 where 16 would be more work-items than a dispatch
  // holds: the same sums.  Register-staged ones of A^T B always do: their
  // fragments do not fit 16 wavefronts' registers (n = 4096 FP64 3011 -> 1986 us,
  // FP32 1271 -> 1034; the other layouts lose by it, A B^T 1936 -> 1992).
  const bool many = ((int64_t)g.m + 127) / 128 * (((int64_t)g.n + 127) / 128) * 1024 >
                    (int64_t)UINT32_MAX;
  auto reg128 = [&] {
    if constexpr (TA && !TB) return launch_one<T, 128, 128, 4, 2, 1, TA, TB>(g, ks, s);
    else
      return many ? launch_one<T, 128, 128, 4, 2, 1, TA, TB>(g, ks, s)
                  : launch_one<T, 128, 128, 4, 4, 1, TA, TB>(g, ks, s);
  };
  switch (cfg) {
    case 0: return launch_one<T, 128, 128, 2, 2, 1, TA, TB>(g, ks, s);
    case 1: return launch_one<T, 128, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 2: return launch_one<T, 64, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 3: return launch_one<T, 64, 32, 2, 2, 1, TA, TB>(g, ks, s);
    case 4: return launch_one<T, 32, 32, 2, 2, 1, TA, TB>(g, ks, s);
    case 5: return launch_one<T, 128, 128, 4, 2, 1, TA, TB>(g, ks, s);
    case 6: return launch_one<T, 128, 128, 2, 4, 1, TA, TB>(g, ks, s);
    case 7: return launch_one<T, 64, 64, 2, 2, 2, TA, TB>(g, ks, s);
    case 8: return launch_one<T, 128, 64, 4, 2, 1, TA, TB>(g, ks, s);
    case 9: return launch_one<T, 128, 64, 2, 2, 2, TA, TB>(g, ks, s);
    case 10: return launch_one<T, 256, 128, 4, 2, 1, TA, TB>(g, ks, s);
    case 11: return launch_one<T, 128, 256, 2, 4, 1, TA, TB>(g, ks, s);
    case 12: return launch_one<T, 256, 128, 4, 4, 1, TA, TB>(g, ks, s);
    case 13: return reg128();
    case 14:
      return dma_ok ? launch_dma<T, 64, 64, 2, 2, 4, TA, TB>(g, ks, s)
                    : launch_one<T, 64, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 15:
      return dma_ok ? launch_dma<T, 64, 32, 2, 2, 4, TA, TB>(g, ks, s)
                    : launch_one<T, 64, 32, 2, 2, 1, TA, TB>(g, ks, s);
    case 16:
      return dma_ok ? launch_dma<T, 128, 64, 2, 2, 4, TA, TB>(g, ks, s)
                    : launch_one<T, 128, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 17:
      return dma_ok ? launch_dma<T, 128, 128, 2, 4, 3, TA, TB>(g, ks, s) : reg128();
    case 18:
      if (!dma_ok) return launch_one<T, 256, 128, 4, 4, 1, TA, TB>(g, ks, s);
      // FP32 on 8 wavefronts: on 16, A^T B spills (n = 4096 1236 -> 1043 us) and
      // A B^T reads B^T for fewer rows at a time (1105 -> 1026; A B 1004 -> 1016)
      if constexpr (F64) return launch_dma<T, 256, 128, 4, 4, 3, TA, TB>(g, ks, s);
      else return launch_dma<T, 256, 128, 2, 4, 3, TA, TB>(g, ks, s);
    case 19:
      if (!dma_ok) return launch_one<T, 32, 32, 2, 2, 1, TA, TB>(g, ks, s);
      return g.k < DmaShape<T, 32, 32, 2, 2, 4>::LOOP_K
                 ? launch_dma<T, 32, 32, 2, 2, 4, TA, TB, 1, 1, true>(g, ks, s)
                 : launch_dma<T, 32, 32, 2, 2, 4, TA, TB>(g, ks, s);
    case 20:
      return dma_ok ? launch_dma<T, 64, 64, 4, 2, 4, TA, TB>(g, ks, s)
                    : launch_one<T, 64, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 21:
      if (!dma_ok) return reg128();
      if constexpr (!F64) return launch_dma<T, 128, 128, 2, 4, 2, TA, TB, 1, 2>(g, ks, s);
      else
        return many ? launch_dma<T, 128, 128, 2, 4, 3, TA, TB>(g, ks, s)
                    : launch_dma<T, 128, 128, 4, 4, 3, TA, TB>(g, ks, s);
    case 22:
      return dma_ok ? launch_dma<T, 128, 128, 2, 2, 2, TA, TB>(g, ks, s) : reg128();
    case 23:
      return dma_ok ? launch_dma<T, 64, 64, 2, 2, 2, TA, TB, 1, KU32>(g, ks, s)
                    : launch_one<T, 64, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 24:
      return dma_ok ? launch_dma<T, 64, 32, 2, 2, 3, TA, TB>(g, ks, s)
                    : launch_one<T, 64, 32, 2, 2, 1, TA, TB>(g, ks, s);
    case 25: return launch_naive<T, TA, TB>(g, s);
    case 26:  // three stages of one k-step (FP32 three workgroups per CU) instead of
              // two of two (two): FP32 n = 4096 A^T B 1268 -> 1161 us, A B^T 1202 ->
              // 1132, A B 1145 -> 1139 (n = 1024 21.2 -> 21.6); FP64 1944 -> 1920
      return dma_ok ? launch_dma<T, 64, 64, 2, 2, 3, TA, TB, 2>(g, ks, s)
                    : launch_one<T, 64, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 27:  // three stages: one workgroup per CU by its registers (FP32 two), so two
              // stages hide less (FP64 n = 4096 2.53 -> 2.14 ms, FP32 1.20 -> 1.11)
      return dma_ok ? launch_dma<T, 128, 64, 2, 2, 3, TA, TB, 2>(g, ks, s)
                    : launch_one<T, 128, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 28:
      return dma_ok ? launch_dma<T, 64, 64, 2, 2, 4, TA, TB, 2>(g, ks, s)
                    : launch_one<T, 64, 64, 2, 2, 1, TA, TB>(g, ks, s);
    case 29:
      return dma_ok ? launch_dma<T, 64, 32, 2, 1, F64 ? 2 : 3, TA, TB, 2, KU32>(g, ks, s)
                    : launch_one<T, 64, 32, 2, 2, 1, TA, TB>(g, ks, s);
  }
  set_error("unknown tile cfg %d", cfg);
  return MG_ERR_INVALID_ARG;
}

template <typename T, bool TA, bool TB>
int gemm_tiles_t(int cfg, int64_t m, int64_t n, int64_t k, double alpha, const void *A,
                 int64_t lda, const void *B, int64_t ldb, double beta, void *C, int64_t ldc,
                 const PartPlan &pp, hipStream_t s) {
  GemmArgs<T> g;
  g.A = static_cast<const T *>(A);
  g.B = static_cast<const T *>(B);
  g.C = static_cast<T *>(C);
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  g.m = (int)m;
  g.n = (int)n;
  g.k = (int)k;
  g.alpha = (T)alpha;
  g.beta = (T)beta;
  const bool dma_ok = ring_operands(sizeof(T) == 8 ? MG_F64 : MG_F32, TA, TB, A, lda, B, ldb);
  const KSplit<T> ks = {static_cast<T *>(pp.planes), pp.parts, pp.kpart};
  return launch_cfg<T, TA, TB>(cfg, dma_ok, g, ks, s);
}

}  // namespace

// The tiled kernels for one layout combination (m, n, k >= 1, alpha != 0,
// arguments validated).
template <bool TA, bool TB>
int gemm_tiles(int dtype, int cfg, int64_t m, int64_t n, int64_t k, double alpha, const void *A,
               int64_t lda, const void *B, int64_t ldb, double beta, void *C, int64_t ldc,
               const PartPlan &pp, hipStream_t s) {
  if (dtype == MG_F64)
    return gemm_tiles_t<double, TA, TB>(cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, pp, s);
  return gemm_tiles_t<float, TA, TB>(cfg, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, pp, s);
}

}  // namespace mg
