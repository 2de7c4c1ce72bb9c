// One macro-tile of C <- alpha*A*B + beta*C on gfx950 matrix cores.
//
// This is the hierarchical tiling of the paper's single-source DGEMM
// (Section 4.2.2, Fig. 7): a block (workgroup) owns one tile of C, its
// threads stage tiles of A and B in shared memory (LDS), every thread
// accumulates a set of elements, and the block then moves on to the next
// A/B tiles along k.  Mapped to CDNA4:
//   grid    -> one dispatch
//   block   -> workgroup of 256 lanes = 4 wavefronts in a 2 x 2 arrangement
//   thread  -> lane; its registers hold (BM/32)*(BN/32) MFMA accumulators
//   element -> 16x16 MFMA fragments (4 values per lane) and 16-byte loads
// A and B are double buffered in LDS with one barrier per k-tile, and the
// global loads of the next PD k-tiles are in flight in registers.  With one
// k-tile in flight and element-wise loads of rows that are not 16-byte
// aligned this path was bound by memory latency and load count; 16-byte loads
// at any address and PD = 4 (32x32 tiles) or 2 (64x64) gave, FP64 and FP32,
// tightly packed odd extents: 1531 x 1033 x 2047 242 -> 169 us and 186 -> 87
// us, 4095 x 4097 x 4099 4.04 -> 2.68 ms and 2.55 -> 1.42 ms; 384 x 384 x 8192
// (A^T, aligned, 32x32 tiles, one per CU) 260 -> 175 us.  What was left was
// the latency of the fragment reads and the barrier between two k-tiles:
// with fragments read a round ahead (small wave tiles), FP64 at k = 2048 by
// tiles per CU: 32x32 1: 24 -> 31, 12: 45 -> 49; 64x64 1: 42 -> 52, 4: 56 ->
// 64, 12: 59 -> 67; 128x64 on 8 wavefronts 2: 60 -> 64; 128x128 64 -> 68
// TFLOP/s.
//
// LDS layouts (chosen for conflict-free 16-byte LDS traffic):
//   A: [BK/VEC][BM+2][VEC]  -- VEC = 16/sizeof(T) consecutive k values of one
//      row form one 16-byte chunk, written as loaded from row-major A and read
//      back with one ds_read_b128 that feeds VEC MFMAs.
//   B: [BK][BN+PB]          -- row-major like B in HBM.
// Transposed operands (op(A) = A^T with A stored k x m, op(B) = B^T with B
// stored n x k) swap layouts: a stored row of A^T is a k row of the tile, so
// it is staged like B ([BK][BM+PB], read one value per MFMA), and a stored
// row of B^T runs along k, so it is staged like A ([BK/VEC][BN+PA][VEC], read
// one 16-byte chunk per VEC MFMAs).
// Fragment k mapping: lane group g = lane/16 supplies k = VEC*(4r+g)+v to the
// v-th MFMA of round r on both operands, so A and B always agree on k, and
// every output sums its products in the same order for every layout.
#pragma once

#include "common.h"

namespace mg {

template <typename T>
struct Mfma;

template <>
struct Mfma<double> {
  typedef d4v acc_t;
  typedef d2v vec_t;  // one 16-byte chunk
  static constexpr int VEC = 2;
  static constexpr int BK = 16;
  static constexpr int PB = 8;  // B row pitch = BN + 8 doubles
  // Row (within the 16x16 block) of accumulator register r of lane group g.
  __device__ static __forceinline__ int row_of(int g, int r) { return 4 * r + g; }
  __device__ static __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

template <>
struct Mfma<float> {
  typedef f4v acc_t;
  typedef f4v vec_t;
  static constexpr int VEC = 4;
  static constexpr int BK = 32;
  static constexpr int PB = 4;
  __device__ static __forceinline__ int row_of(int g, int r) { return 4 * g + r; }
  __device__ static __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

template <typename T>
struct GemmArgs {
  const T *A;
  const T *B;
  T *C;
  int64_t lda, ldb, ldc;
  int m, n, k;
  T alpha, beta;
};

// Split of a product's k range over workgroups: part z sums k in [z*kpart,
// (z+1)*kpart) into its own m x n plane of `planes` (pitch n), and a second
// kernel adds the planes in order.  parts == 1: no split.
template <typename T>
struct KSplit {
  T *planes;
  int parts, kpart;
};

// The part of workgroup t of tiles * parts (tile t % tiles of part t / tiles):
// `g` becomes that part's product, C <- A B into its plane.
template <typename T, bool TA, bool TB>
__device__ __forceinline__ int take_part(GemmArgs<T> &g, const KSplit<T> &ks, int t, int tiles) {
  if (ks.parts == 1) return t;
  const int z = t / tiles;
  const int64_t k0 = (int64_t)z * ks.kpart;
  g.A += TA ? k0 * g.lda : k0;
  g.B += TB ? k0 : k0 * g.ldb;
  g.C = ks.planes + (int64_t)z * g.m * g.n;
  g.ldc = g.n;
  g.k = min(ks.kpart, g.k - (int)k0);
  g.alpha = T(1);
  g.beta = T(0);
  return t - z * tiles;
}

constexpr int kTileThreads = 256;

// Macro-tile BM x BN computed by WGM x WGN wavefronts (each a WM x WN wave
// tile of 16x16 MFMA blocks), k-step BK = BKM times the type's base step.
template <typename T, int BM, int BN, int WGM = 2, int WGN = 2, int BKM = 1, bool TA = false,
          bool TB = false>
struct TileShape {
  typedef Mfma<T> M;
  static constexpr int THREADS = 64 * WGM * WGN;
  static constexpr int VEC = M::VEC;
  static constexpr int BK = M::BK * BKM;
  static constexpr int ACH = BK / VEC;  // A chunks per tile row
  // A chunk-row pitch BM + PA: with ACH chunks per row written by consecutive
  // lanes, PA = 16 / ACH spreads the 16 lanes of a 16-byte LDS write over
  // all 64 banks.
  static constexpr int PA = 16 / ACH;
  static constexpr int PB = M::PB;
  static constexpr int WM = BM / WGM, WN = BN / WGN;  // wave tile
  static constexpr int FM = WM / 16, FN = WN / 16;    // MFMA blocks per wave
  static constexpr int A_CHUNKS = BM * BK / VEC;      // 16-byte chunks per A tile
  static constexpr int B_CHUNKS = BK * BN / VEC;
  static constexpr int NA = A_CHUNKS / THREADS;  // per thread
  static constexpr int NB = B_CHUNKS / THREADS;
  static constexpr int A_STAGE = TA ? BK * (BM + PB) : ACH * (BM + PA) * VEC;  // elements
  static constexpr int B_STAGE = TB ? ACH * (BN + PA) * VEC : BK * (BN + PB);
  static constexpr int STAGE = A_STAGE + B_STAGE;
  static constexpr size_t LDS_BYTES = 2 * STAGE * sizeof(T);
  // k-tiles in flight in registers: deep for the small tiles, whose k-tile is
  // far shorter than a memory round trip; one where a k-tile's products cover
  // it and the registers are needed for two workgroups per CU.
  static constexpr int PD = NA + NB <= 2 ? 4 : NA + NB <= 4 && BM * BN <= 8192 ? 2 : 1;
  // Fragments read one round ahead.  Not the FP32 64x64 tile: the second set
  // costs it a workgroup per CU (4 tiles per CU: 119 -> 112 TFLOP/s).
  static constexpr bool AHEAD =
      FM * FN <= 4 && !(sizeof(T) == 4 && FM * FN == 4 && THREADS == 256);
  // Wavefronts per SIMD the registers must leave room for (the second
  // __launch_bounds__ value): at one the compiler would keep the sums in
  // accumulation registers and copy them every k-tile.
  static constexpr int MINW = FM * FN * sizeof(T) >= 128  ? 1
                              : AHEAD && BKM == 1         ? (FM * FN < 4 || THREADS >= 512 ? 4 : 3)
                              : BM * BN == 128 * 128 && THREADS == 512 && BKM == 1 ? 4
                                                                                   : 2;
  static_assert(WM % 16 == 0 && WN % 16 == 0 && FM >= 1 && FN >= 1, "wave tile of 16x16 blocks");
  static_assert(ACH <= 16 && 16 % ACH == 0, "A chunks per row");
  static_assert(NA >= 1 && NB >= 1 && A_CHUNKS % THREADS == 0 && B_CHUNKS % THREADS == 0,
                "every thread loads whole chunks");
  static_assert(ACH % 4 == 0, "k rounds of 4 lane groups");
};

// A 16-byte chunk at any element address.  Global loads and stores of several
// dwords need dword alignment only, so a row of any pitch and base moves in
// 16-byte chunks: an element-by-element path for rows that are not 16-byte
// aligned costs VEC times the load instructions behind per-lane branches.
template <typename T>
struct Chunk {
  typedef typename Mfma<T>::vec_t V;
  typedef V __attribute__((aligned(sizeof(T)))) U;
  __device__ static __forceinline__ V load(const T *p) { return *reinterpret_cast<const U *>(p); }
  __device__ static __forceinline__ void store(T *p, V v) { *reinterpret_cast<U *>(p) = v; }
};

// Elements `s`, s+1, ... of chunk x, then zeros (s >= VEC: all zeros).
template <typename T>
__device__ __forceinline__ typename Mfma<T>::vec_t shift_chunk(typename Mfma<T>::vec_t x, int s) {
  constexpr int VEC = Mfma<T>::VEC;
  typename Mfma<T>::vec_t r = x;
#pragma unroll
  for (int b = 1; b < VEC; b *= 2) {
    typename Mfma<T>::vec_t y = r;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const T up = v + b < VEC ? r[v + b < VEC ? v + b : v] : T(0);
      y[v] = (s & b) ? up : r[v];
    }
    r = y;
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) r[v] = s >= VEC ? T(0) : r[v];
  return r;
}

// One 16-byte chunk of a row shorter than a chunk: `left` elements from p.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::vec_t load_short(const T *p, int left) {
  typename Mfma<T>::vec_t r = {};
#pragma unroll
  for (int v = 0; v < Mfma<T>::VEC; ++v)
    if (v < left) r[v] = p[v];
  return r;
}

// Swap with the neighbouring lane (lane ^ 1) through DPP quad_perm [1,0,3,2].
__device__ __forceinline__ double dpp_swap1(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  const int lo2 = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, false);
  const int hi2 = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, false);
  return __hiloint2double(hi2, lo2);
}

// Output row of accumulator register r of lane group gq in block row i.
// PA (paired block rows, FP64 direct-load tiles with a transposed A): block
// rows 2p and 2p+1 hold the even and odd rows of a 32-row span.
template <bool PA>
__device__ __forceinline__ int f64_out_row(int row0, int i, int gq, int r) {
  return PA ? row0 + 32 * (i >> 1) + 2 * Mfma<double>::row_of(gq, r) + (i & 1)
            : row0 + 16 * i + Mfma<double>::row_of(gq, r);
}

// C tile epilogue for a wave's FM x FN grid of 16x16 blocks whose top-left
// output is (row0, col0): out = alpha*acc + beta*C (C unread when beta == 0).
// In block (i, j), lane l holds column l%16 of rows row_of(l/16, r).  The C
// loads of a few block rows are all issued before the first store, so they
// are in flight together instead of each waiting behind the previous store.
// FP32 loads come from addresses clamped into the matrix, without lane
// branches (2000 problems in one launch: 265 -> 240 us); FP64 pairs are masked
// (clamped ones, read twice at the edges: 414 -> 443 us).

// Block rows whose C is in flight at once: all of a small wave tile's (the
// registers of its k loop are free by now), one of a large one's.
template <int FM, int FN>
constexpr int kEpilogueRows = FM * FN <= 4 ? FM : 1;

// Columns col, col+1 of row `row`; zeros past the matrix.
__device__ __forceinline__ d2v load_c_pair(const GemmArgs<double> &g, int row, int col) {
  d2v x = {0.0, 0.0};
  if (row >= g.m) return x;
  const double *p = g.C + (int64_t)row * g.ldc + col;
  if (col + 1 < g.n) x = Chunk<double>::load(p);
  else if (col < g.n) x[0] = p[0];
  return x;
}

__device__ __forceinline__ void store_c_pair(const GemmArgs<double> &g, int row, int col, d2v v,
                                             d2v c, bool use_c) {
  if (row >= g.m) return;
  d2v o;
#pragma unroll
  for (int e = 0; e < 2; ++e) o[e] = use_c ? fma(g.alpha, v[e], g.beta * c[e]) : g.alpha * v[e];
  double *p = g.C + (int64_t)row * g.ldc + col;
  if (col + 1 < g.n) Chunk<double>::store(p, o);
  else if (col < g.n) p[0] = o[0];
}

template <typename T>
struct Epilogue;

// FP64: neighbouring lanes (same rows, columns c and c+1) swap one value each
// so that each lane owns a 16-byte pair of adjacent columns of one row.
template <>
struct Epilogue<double> {
  template <int FM, int FN, int AM, int AN, bool PA = false>
  __device__ static __forceinline__ void store(const GemmArgs<double> &g,
                                               const d4v (&acc)[AM][AN], int row0, int col0,
                                               int lane) {
    constexpr int R = kEpilogueRows<FM, FN>;
    const int gq = lane >> 4, j = lane & 15;
    const bool odd = j & 1;
    const bool use_c = g.beta != 0.0;
#pragma unroll
    for (int i0 = 0; i0 < FM; i0 += R) {
      d2v c[R][FN][2] = {};
      if (use_c) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int jb = 0; jb < FN; ++jb)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              c[i][jb][h] = load_c_pair(g, f64_out_row<PA>(row0, i0 + i, gq, 2 * h + (odd ? 1 : 0)),
                                        col0 + 16 * jb + (j & ~1));
      }
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int jb = 0; jb < FN; ++jb)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const d4v &s = acc[i0 + i][jb];
            const int r = 2 * h;
            const double got = dpp_swap1(odd ? s[r] : s[r + 1]);
            const d2v v = {odd ? got : s[r], odd ? s[r + 1] : got};
            store_c_pair(g, f64_out_row<PA>(row0, i0 + i, gq, r + (odd ? 1 : 0)),
                         col0 + 16 * jb + (j & ~1), v, c[i][jb][h], use_c);
          }
    }
  }
};

// Epilogue of the column-paired FP64 fragment layout: block columns 2p and
// 2p+1 of a wave hold the even and odd columns of one 32-column span, so
// lane l owns columns 32p + 2(l%16) and 32p + 2(l%16) + 1 of each of its rows:
// one 16-byte C load and store per pair (at any 8-byte address), no lane
// exchange.
template <int FM, int FN, int AM, int AN, bool PA = false>
__device__ __forceinline__ void store_paired_f64(const GemmArgs<double> &g,
                                                 const d4v (&acc)[AM][AN], int row0, int col0,
                                                 int lane) {
  static_assert(FN % 2 == 0, "pairs of block columns");
  constexpr int R = kEpilogueRows<FM, FN>;
  const int gq = lane >> 4, l16 = lane & 15;
  const bool use_c = g.beta != 0.0;
#pragma unroll
  for (int i0 = 0; i0 < FM; i0 += R) {
    d2v c[R][FN / 2][4] = {};
    if (use_c) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int p = 0; p < FN / 2; ++p)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            c[i][p][r] = load_c_pair(g, f64_out_row<PA>(row0, i0 + i, gq, r),
                                     col0 + 32 * p + 2 * l16);
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int p = 0; p < FN / 2; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          store_c_pair(g, f64_out_row<PA>(row0, i0 + i, gq, r), col0 + 32 * p + 2 * l16,
                       d2v{acc[i0 + i][2 * p][r], acc[i0 + i][2 * p + 1][r]}, c[i][p][r], use_c);
  }
}

template <>
struct Epilogue<float> {
  template <int FM, int FN, int AM, int AN>
  __device__ static __forceinline__ void store(const GemmArgs<float> &g,
                                               const f4v (&acc)[AM][AN], int row0, int col0,
                                               int lane) {
    constexpr int R = kEpilogueRows<FM, FN>;
    const int gq = lane >> 4, j = lane & 15;
    const bool use_c = g.beta != 0.0f;
#pragma unroll
    for (int i0 = 0; i0 < FM; i0 += R) {
      float c[R][FN][4] = {};
      if (use_c) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int jb = 0; jb < FN; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int row = row0 + 16 * (i0 + i) + Mfma<float>::row_of(gq, r);
              c[i][jb][r] = g.C[(int64_t)min(row, g.m - 1) * g.ldc + min(col0 + 16 * jb + j, g.n - 1)];
            }
        // One wait for all loads, here: the compiler's own, in the branch of
        // each store, also waits for the stores before it (one counter): 2000
        // problems in one launch 242 -> 238 us.  FP64 tiles, whose 16-byte
        // stores are fewer, lose by it (n = 2048 249 -> 254 us).
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt 0, the others at their maxima
      }
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int jb = 0; jb < FN; ++jb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = row0 + 16 * (i0 + i) + Mfma<float>::row_of(gq, r), col = col0 + 16 * jb + j;
            const float a = acc[i0 + i][jb][r];
            if (row < g.m && col < g.n)
              g.C[(int64_t)row * g.ldc + col] =
                  use_c ? fmaf(g.alpha, a, g.beta * c[i][jb][r]) : g.alpha * a;
          }
    }
  }
};

// Workgroup barrier after this wavefront's LDS accesses (lgkmcnt 0; loads in
// flight stay in flight: vmcnt and expcnt at their maxima are not waited for).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
}

// One operand's share of a k-tile, per thread: N 16-byte chunks at any element
// alignment.  KC: the stored rows run along k (A, or stored B^T): chunk (i, j)
// is k chunk j of tile row i.  Otherwise the stored rows are k rows (B, or
// stored A^T): chunk (i, j) is columns j.. of k row i.  Rows past the matrix
// read its last row and their outputs are never stored.  A chunk that would
// run past a row's end is loaded from the row's last full chunk instead and
// shifted into place by fix(), so every load is one 16-byte instruction
// without lane branches; rows shorter than a chunk are read element by
// element.  k past the problem is zeroed by fix().
// PD k-tiles are in flight at once, k-tile kt in register set kt % PD.
template <typename T, int EXT, int BK, int THREADS, bool KC, int PD>
struct Panel {
  typedef typename Mfma<T>::vec_t V;
  static constexpr int VEC = Mfma<T>::VEC;
  static constexpr int CH = (KC ? BK : EXT) / VEC;  // chunks per stored row of the tile
  static constexpr int N = EXT * BK / VEC / THREADS;
  const T *p[N];
  V x[PD][N];

  __device__ static __forceinline__ int row_of(int tid, int u) { return (tid + THREADS * u) / CH; }
  __device__ static __forceinline__ int col_of(int tid, int u) {  // element within the row
    return (tid + THREADS * u) % CH * VEC;
  }
  // `base`: the stored matrix; c0: the tile's first row / column of `ext`.
  __device__ __forceinline__ void init(const T *base, int64_t ld, int c0, int ext, int tid) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = row_of(tid, u), j = col_of(tid, u);
      p[u] = KC ? base + (int64_t)min(c0 + i, ext - 1) * ld + j
                : base + (int64_t)i * ld + max(min(c0 + j, ext - VEC), 0);
    }
  }
  // k-tiles [0, whole_tiles) take one plain load per chunk.
  __device__ static __forceinline__ int whole_tiles(int ext, int k) {
    return KC || ext >= VEC ? k / BK : 0;
  }
  __device__ __forceinline__ void load(int64_t ld, int kt, int set) {
    const int64_t step = KC ? kt * BK : (int64_t)(kt * BK) * ld;
#pragma unroll
    for (int u = 0; u < N; ++u) x[set][u] = Chunk<T>::load(p[u] + step);
  }
  __device__ __forceinline__ void load_tail(int64_t ld, int c0, int ext, int k, int kt, int tid,
                                            int set) {
    const int kbase = kt * BK;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = row_of(tid, u), j = col_of(tid, u);
      const int64_t rows = KC ? 0 : (int64_t)(min(kbase + i, k - 1) - i) * ld;
      if ((KC ? k : ext) < VEC)
        x[set][u] = KC ? load_short<T>(p[u] + kbase, k - kbase - j)
                       : load_short<T>(p[u] + rows + c0 + j, ext - c0 - j);
      else
        x[set][u] = Chunk<T>::load(p[u] + (KC ? min(kbase + j, k - VEC) - j : rows));
    }
  }
  // Puts chunks loaded from a row's end in place and zeroes k past the
  // problem; `whole`: k-tiles that load() reads, where only columns past the
  // matrix's edge matter.
  __device__ __forceinline__ void fix(int c0, int ext, int k, int kt, int tid, int set,
                                      bool whole) {
    const int kbase = kt * BK;
    if (KC ? !whole && k >= VEC : c0 + EXT > ext && ext >= VEC) {
      const int c1 = KC ? kbase : c0, end = (KC ? k : ext) - VEC;
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int c = c1 + col_of(tid, u);
        x[set][u] = shift_chunk<T>(x[set][u], c - min(c, end));
      }
    }
    if (!KC && !whole) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const bool in = kbase + row_of(tid, u) < k;
#pragma unroll
        for (int v = 0; v < VEC; ++v) x[set][u][v] = in ? x[set][u][v] : T(0);
      }
    }
  }
  // LDS position of chunk u: [k chunk][EXT + PA][VEC] or [k row][EXT + PB].
  template <int PA, int PB>
  __device__ __forceinline__ void put(T *lds, int tid, int set) const {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = row_of(tid, u), j = col_of(tid, u);
      T *q = KC ? lds + (j / VEC * (EXT + PA) + i) * VEC : lds + i * (EXT + PB) + j;
      *reinterpret_cast<V *>(q) = x[set][u];
    }
  }
};

// Computes the BM x BN tile of C whose top-left output is (m0, n0) of
// C <- alpha*op(A)*op(B) + beta*C (op = transpose when TA / TB is set).
// `smem` holds 2 stages of TileShape::STAGE elements.  All THREADS lanes of
// the workgroup must call this together (it contains barriers).  `turn` (below
// WGM * WGN, the same for all lanes) permutes which wavefront computes which
// part of the tile.
template <typename T, int BM, int BN, int WGM = 2, int WGN = 2, int BKM = 1, bool TA = false,
          bool TB = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs<T> &g, int m0, int n0, T *smem,
                                          int turn = 0) {
  typedef TileShape<T, BM, BN, WGM, WGN, BKM, TA, TB> S;
  typedef Mfma<T> M;
  typedef typename M::vec_t V;
  typedef typename M::acc_t Acc;
  constexpr int VEC = S::VEC, BK = S::BK;
  constexpr int ACH = S::ACH;  // k chunks per tile row of A (and of stored B^T)
  constexpr int PD = S::PD;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) ^ turn;
  const int wm0 = (wave / WGN) * S::WM, wn0 = (wave % WGN) * S::WN;
  const int gq = lane >> 4, l16 = lane & 15;

  Panel<T, BM, BK, S::THREADS, !TA, PD> pa;
  Panel<T, BN, BK, S::THREADS, TB, PD> pb;
  pa.init(g.A, g.lda, m0, g.m, tid);
  pb.init(g.B, g.ldb, n0, g.n, tid);
  const int KT = (g.k + BK - 1) / BK;
  const int KW = min(pa.whole_tiles(g.m, g.k), pb.whole_tiles(g.n, g.k));
  auto load_tiles = [&](int kt, int set) {  // kt < KW
    pa.load(g.lda, kt, set);
    pb.load(g.ldb, kt, set);
  };
  auto load_any = [&](int kt, int set) {
    if (kt < KW) {
      load_tiles(kt, set);
    } else if (kt < KT) {
      pa.load_tail(g.lda, m0, g.m, g.k, kt, tid, set);
      pb.load_tail(g.ldb, n0, g.n, g.k, kt, tid, set);
    }
  };
  auto store_tiles = [&](int kt, int buf, int set, bool whole) {
    T *As = smem + buf * S::STAGE;
    pa.fix(m0, g.m, g.k, kt, tid, set, whole);
    pb.fix(n0, g.n, g.k, kt, tid, set, whole);
    pa.template put<S::PA, S::PB>(As, tid, set);
    pb.template put<S::PA, S::PB>(As + S::A_STAGE, tid, set);
  };

  Acc acc[S::FM][S::FN];
#pragma unroll
  for (int i = 0; i < S::FM; ++i)
#pragma unroll
    for (int j = 0; j < S::FN; ++j) acc[i][j] = Acc{};

  // Fragments of one round (k chunks 4r + 0..3, one per lane group): VEC
  // MFMAs per block.
  struct Frag {
    V a[S::FM];
    T b[VEC][S::FN];
  };
  auto load_frag = [&](Frag &f, int buf, int r) {
    const T *As = smem + buf * S::STAGE;
    const T *Bs = As + S::A_STAGE;
    const int kc = 4 * r + gq;  // this lane group's chunk
#pragma unroll
    for (int i = 0; i < S::FM; ++i) {
      if constexpr (!TA) {
        f.a[i] = *reinterpret_cast<const V *>(As + (kc * (BM + S::PA) + wm0 + 16 * i + l16) * VEC);
      } else {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
          f.a[i][v] = As[(kc * VEC + v) * (BM + S::PB) + wm0 + 16 * i + l16];
      }
    }
#pragma unroll
    for (int j = 0; j < S::FN; ++j) {
      if constexpr (TB) {  // transposed B: one chunk of VEC k values per block column
        const V bv =
            *reinterpret_cast<const V *>(Bs + (kc * (BN + S::PA) + wn0 + 16 * j + l16) * VEC);
#pragma unroll
        for (int v = 0; v < VEC; ++v) f.b[v][j] = bv[v];
      } else {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
          f.b[v][j] = Bs[(kc * VEC + v) * (BN + S::PB) + wn0 + 16 * j + l16];
      }
    }
  };
  auto mma_first = [&](const Frag &f) { acc[0][0] = M::mma(f.a[0][0], f.b[0][0], acc[0][0]); };
  auto mma_rest = [&](const Frag &f) {
#pragma unroll
    for (int v = 0; v < VEC; ++v)
#pragma unroll
      for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
          if (v + i + j > 0) acc[i][j] = M::mma(f.a[i][v], f.b[v][j], acc[i][j]);
  };
  constexpr int U = ACH / 4;  // rounds per k-tile

  MG_LDS_POISON_STAGE(smem, 2 * S::STAGE * (int)sizeof(T));
#pragma unroll
  for (int q = 0; q < PD; ++q) load_any(q, q);
  store_tiles(0, 0, 0, KW > 0);
  load_any(PD, 0);
  __syncthreads();
  int kt = 0;
  if constexpr (S::AHEAD) {
    // A 32x32 wavefront whose outputs all lie past the matrix only stages
    // (16x16 ones cost more in the check than they save: 528 -> 567 us for
    // 2000 problems in 32x32 tiles).
    if (S::WM * S::WN >= 1024 && (m0 + wm0 >= g.m || n0 + wn0 >= g.n)) {
      for (; kt < KT; kt += PD) {
#pragma unroll
        for (int j = 0; j < PD; ++j) {
          if (kt + j >= KT) break;
          const int buf = (kt + j + 1) & 1;
          MG_LDS_POISON_STAGE(smem + buf * S::STAGE, S::STAGE * (int)sizeof(T));
          if (kt + j + 1 < KT)
            store_tiles(kt + j + 1, buf, (j + 1) % PD, kt + j + 1 < KW);
          load_any(kt + j + 1 + PD, (j + 1) % PD);
          lds_barrier();
        }
      }
      return;
    }
    // Small wave tiles: a round's fragments are read from LDS while the
    // matrix cores work on the previous round's.  In step kt, k-tile kt+1 goes
    // to the other buffer (its last readers are behind the barrier) and the
    // loads of k-tile kt+1+PD start; before the last round the wavefronts
    // meet, with their LDS writes done and their fragments of k-tile kt in
    // registers (products may be scheduled past the barrier, so they do not
    // imply it).  The order is pinned: one product first, whose wait covers
    // only this round's fragments, then what the others hide.
    Frag f[2];
    load_frag(f[0], 0, 0);
    constexpr int UNR = PD > 1 ? PD : 2;  // buffers and register sets alternate
    static_assert(UNR % 2 == 0 && UNR * U % 2 == 0, "constant LDS and fragment addresses");
    for (; kt + UNR + PD < KW; kt += UNR) {
#pragma unroll
      for (int j = 0; j < UNR; ++j)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const Frag &cur = f[(j * U + u) & 1];
          Frag &nx = f[(j * U + u + 1) & 1];
          if (u + 1 == U) {
            lds_barrier();
            mma_first(cur);
            __builtin_amdgcn_sched_barrier(0);
            load_frag(nx, (j + 1) & 1, 0);
          } else {
            mma_first(cur);
            __builtin_amdgcn_sched_barrier(0);
            load_frag(nx, j & 1, u + 1);
            if (u == 0) {
              MG_LDS_POISON_STAGE(smem + ((j + 1) & 1) * S::STAGE, S::STAGE * (int)sizeof(T));
              store_tiles(kt + j + 1, (j + 1) & 1, (j + 1) % PD, true);
              load_tiles(kt + j + 1 + PD, (j + 1) % PD);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          mma_rest(cur);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    for (; kt < KT; kt += PD) {
#pragma unroll
      for (int j = 0; j < PD; ++j) {
        if (kt + j >= KT) break;
        const int buf = (kt + j) & 1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (u + 1 == U) {
            lds_barrier();
            if (kt + j + 1 < KT) load_frag(f[1], buf ^ 1, 0);
          } else {
            load_frag(f[1], buf, u + 1);
            if (u == 0) {
              MG_LDS_POISON_STAGE(smem + (buf ^ 1) * S::STAGE, S::STAGE * (int)sizeof(T));
              if (kt + j + 1 < KT)
                store_tiles(kt + j + 1, buf ^ 1, (j + 1) % PD, kt + j + 1 < KW);
              load_any(kt + j + 1 + PD, (j + 1) % PD);
            }
          }
          mma_first(f[0]);
          mma_rest(f[0]);
          f[0] = f[1];
        }
      }
    }
  } else {
    // Step kt puts k-tile kt+1 in the other buffer (its last readers are
    // behind the barrier) and starts the loads of k-tile kt+1+PD.  Whole
    // k-tiles run without branches around the loads, so waits count only
    // older loads.
    auto compute = [&](int t) {
      Frag f;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        load_frag(f, t & 1, u);
        mma_first(f);
        mma_rest(f);
      }
    };
    for (; kt + 2 * PD < KW; kt += PD) {
#pragma unroll
      for (int j = 0; j < PD; ++j) {
        MG_LDS_POISON_STAGE(smem + ((kt + j + 1) & 1) * S::STAGE, S::STAGE * (int)sizeof(T));
        store_tiles(kt + j + 1, (kt + j + 1) & 1, (j + 1) % PD, true);
        load_tiles(kt + j + 1 + PD, (j + 1) % PD);
        compute(kt + j);
        __syncthreads();
      }
    }
    for (; kt < KT; kt += PD) {
#pragma unroll
      for (int j = 0; j < PD; ++j) {
        if (kt + j >= KT) break;
        MG_LDS_POISON_STAGE(smem + ((kt + j + 1) & 1) * S::STAGE, S::STAGE * (int)sizeof(T));
        if (kt + j + 1 < KT)
          store_tiles(kt + j + 1, (kt + j + 1) & 1, (j + 1) % PD, kt + j + 1 < KW);
        load_any(kt + j + 1 + PD, (j + 1) % PD);
        compute(kt + j);
        __syncthreads();
      }
    }
  }

  Epilogue<T>::template store<S::FM, S::FN>(g, acc, m0 + wm0, n0 + wn0, lane);
}

}  // namespace mg
