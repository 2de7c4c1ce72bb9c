// Native GEMM tile fed by direct global->LDS loads (gfx950
// global_load_lds_dwordx4) into an NS-stage LDS ring.
//
// Same hierarchy as gemm_tile (Section 4.2.2 tiling: block = macro-tile of
// C, threads stage A/B tiles in shared memory, each lane accumulates MFMA
// fragments), but the loads of the next NS-1 stages are in flight while the
// matrix cores work on the current one, and no registers or LDS write
// instructions are spent on staging: each lane's 16 bytes land at the wave's
// LDS base + 16*lane.
//
// What bounds it: the matrix cores, once nothing else sits in a wavefront's
// instruction stream.  A k-step of a small tile is 8 to 16 MFMAs per
// wavefront; with the barrier, the waits, the refill's address arithmetic and
// branches, and the latency of the fragment reads all between two k-steps, a
// 64x64 ring reached 65 TFLOP/s (FP64) and a 32x32 tile alone on its CU 25.
// So scalar registers carry the addresses, the loop is unrolled over the ring
// (constant LDS addresses, no branches), and wavefronts with up to 2x2
// blocks read the fragments of a half step while the previous half step's
// products run.  FP64, k = 2048, by tiles per CU, before -> after (whole calls;
// the division rule's rates have the launch taken off): 64x64
// 1: 48.7 -> 64.6, 4: 65.2 -> 70.8, 16: 66.5 -> 72 TFLOP/s; 32x32 1: 25.2 ->
// 53.5, 12: 52 -> 64; 128x128 (now on 16 wavefronts) n = 2048 63.9 -> 70.3,
// 4096 69.5 -> 72.8, 8192 70.6 -> 74.1.  FP32: 32x32 1: 43 -> 84, 12: 95 ->
// 110; 64x64 1: 86 -> 107, 12: 113 -> 121; 128x128 n = 2048 120.5 -> 125.6.
// Requires 16-byte aligned operands (base aligned, pitch a multiple of the
// 16-byte element count); ragged edges are read from clamped in-bounds
// chunks and never stored, and k past the problem's k is zeroed in LDS on
// both operands before the last step's multiply (the same sums as the
// zero-filled tail of the register-staged tile).
//
// One k-step covers 128 bytes of k (16 FP64 / 32 FP32 values).  LDS stage:
//   A [BM rows][128 B], 16-byte chunk c of row r stored at chunk c ^ ((r>>1)&7)
//     so the fragment reads of 16 consecutive rows hit distinct banks;
//   B [128/size rows of k][BN*size B], row-major like B in HBM, chunks XOR-
//     swizzled per k row so the four lane groups' rows of one fragment read
//     fall on different banks.
// Transposed operands keep the stored rows intact: A^T (stored k x m) lands
// as [k rows][BM*size B] with B's swizzle and is read one value per MFMA like
// B; B^T (stored n x k) lands as [BN rows][128 B] with A's swizzle and is read
// one 16-byte chunk per VEC MFMAs like A.  Stage sizes are the same.
#pragma once

#include <type_traits>

#include "gemm_tile.h"

namespace mg {

// KS = 2 runs two groups of WGM x WGN wavefronts on the same outputs, each
// taking half of every k-step's values (16-byte k chunks 0-3 and 4-7); the
// second group's sums are added to the first's through LDS at the end.
// KU: k-steps per ring stage, so one wait and one barrier per KU k-steps.
template <typename T, int BM, int BN, int WGM, int WGN, int NS, int KS = 1, int KU = 1>
struct DmaShape {
  static constexpr int SWAVES = WGM * WGN;     // wavefronts per k group
  static constexpr int WAVES = SWAVES * KS;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int ESZ = sizeof(T);
  static constexpr int VEC = 16 / ESZ;
  static constexpr int BK = 128 / ESZ;
  static constexpr int RB = BN * ESZ;          // B row bytes in LDS
  static constexpr int CPB = RB / 16;          // 16-byte chunks per B row
  static constexpr int RA = BM * ESZ;          // row bytes of a transposed A stage
  static constexpr int CPA = RA / 16;
  static constexpr int A_BYTES = BM * 128;
  static constexpr int STEP = A_BYTES + 128 * BN;  // B block: BK rows of RB bytes
  static constexpr int STAGE = KU * STEP;
  static constexpr size_t RING_BYTES = (size_t)NS * STAGE;
  static constexpr size_t RED_BYTES = KS > 1 ? (size_t)BM * BN * ESZ : 0;  // k-group sums
  static constexpr size_t LDS_BYTES = RING_BYTES > RED_BYTES ? RING_BYTES : RED_BYTES;
  static constexpr int IA = BM / 8 / WAVES;    // 1 KB DMA instructions per wave, A
  static constexpr int IB = BN / 8 / WAVES;    // and B
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int FM = WM / 16, FN = WN / 16;
  // Fragments read one half step ahead (see the main loop).
  static constexpr bool AHEAD = FM * FN <= 4 && (ESZ == 8 || KS == 1);
  // Stages in a pass of that loop, and the k from which it can run once.
  static constexpr int UNROLL = NS * KU * (2 / KS) % 2 ? 2 * NS : NS;
  static constexpr int LOOP_K = (UNROLL + NS) * KU * BK;
  static_assert(IA >= 1 && IA * 8 * WAVES == BM, "whole A instructions per wave");
  static_assert(IB >= 1 && IB * 8 * WAVES == BN, "whole B instructions per wave");
  static_assert(FM >= 1 && FN >= 1 && WM % 16 == 0 && WN % 16 == 0, "16x16 blocks per wave");
  static_assert(CPB >= 8 && (CPB & (CPB - 1)) == 0, "B rows of 2^j >= 8 chunks");
  static_assert(NS >= 2 && LDS_BYTES <= 160 * 1024, "ring fits in LDS");
  static_assert(KS == 1 || KS == 2, "one or two k groups");
  // Wavefronts per SIMD the register allocation must leave room for (the
  // second __launch_bounds__ value): as many workgroups as the LDS ring
  // allows per CU, counted up to 4 per SIMD (128 registers each).
  static constexpr int WGS_PER_CU = (int)((160 * 1024) / LDS_BYTES);
  static constexpr int WPS = WGS_PER_CU * WAVES / 4;
  static constexpr int CAP = KS > 1 && FM * FN > 4 ? 2 : 4;  // two k groups of 64x32 outputs
  static constexpr int MINW = WPS < 1 ? 1 : WPS > CAP ? CAP : WPS;
};

__device__ __forceinline__ int dma_swz_a(int row, int c) { return c ^ ((row >> 1) & 7); }

// FP64 fragments read 8-byte values of 16 consecutive columns (128 B) from the
// rows 2(4r+g)+v of the four lane groups g: flip the 128-byte half by a bit
// that differs between any two of them.  FP32 reads 64 B from rows 4(4r+g)+v:
// rotate by 64-byte quarters with (row/4) mod 4.
template <typename T, int CPB>
__device__ __forceinline__ int dma_swz_b(int row, int c) {
  if (sizeof(T) == 8) return c ^ ((((row >> 1) ^ (row >> 2)) & 1) << 3);
  return c ^ ((((row >> 2) & 3) << 2) & (CPB - 1));
}

__device__ __forceinline__ void dma_lds16(const void *src, unsigned char *lds_dst) {
  __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds_dst, 16, 0,
                                   0);
}

template <int N>
__device__ __forceinline__ void dma_wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  // gfx9 s_waitcnt encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[15:14]
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// The same, and for every LDS access of this wavefront (lgkmcnt 0).
template <int N>
__device__ __forceinline__ void dma_wait_ring() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}
// LDS accesses only (vmcnt and expcnt at their maxima: not waited for).
__device__ __forceinline__ void dma_wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Waits until at most q stages' DMAs (DPS instructions each) are pending.
template <int DPS, int NS>
__device__ __forceinline__ void dma_wait_steps(int q) {
  if (q <= 0) dma_wait_vmcnt<0>();
  else if (q == 1 || NS <= 2) dma_wait_vmcnt<DPS>();
  else if (q == 2 || NS <= 3) dma_wait_vmcnt<2 * DPS>();
  else dma_wait_vmcnt<3 * DPS>();
}

// SHORT: the plain loop alone, for k of fewer stages than one pass of the loop
// unrolled over the ring takes.  There the unrolled loop's set-up and its
// remainder, which moves a second fragment set and has branches, cost a 32x32
// tile more than reading ahead gives: FP64 200 x 2048, k = 32 / 64: 4.27 / 5.05
// against 3.90 / 4.78 us, FP32 768 x 768 x 128 5.74 against 5.41.
template <typename T, int BM, int BN, int WGM, int WGN, int NS, bool TA = false, bool TB = false,
          int KS = 1, int KU = 1, bool SHORT = false>
__device__ __forceinline__ void gemm_dma_tile(const GemmArgs<T> &g, int m0, int n0,
                                              unsigned char *lds) {
  typedef DmaShape<T, BM, BN, WGM, WGN, NS, KS, KU> S;
  typedef Mfma<T> M;
  typedef typename M::vec_t V;
  typedef typename M::acc_t Acc;
  constexpr int ESZ = S::ESZ, VEC = S::VEC, BK = S::BK;
  constexpr int DPS = KU * (S::IA + S::IB);  // DMA instructions per stage per wave
  // FP64 with B in k rows: pair block columns 2p, 2p+1 on the even / odd
  // columns of a 32-column span, so one 16-byte LDS read feeds both.
  constexpr bool PAIR = ESZ == 8 && !TB && S::FN % 2 == 0;
  // FP64 with A in k rows (transposed A): pair block rows 2p, 2p+1 on the
  // even / odd rows of a 32-row span the same way.
  constexpr bool PAIRA = ESZ == 8 && TA && S::FM % 2 == 0;
  static_assert(!TA || (S::CPA >= 8 && (S::CPA & (S::CPA - 1)) == 0),
                "transposed A rows of 2^j >= 8 chunks");
  static_assert(ESZ == 4 || (S::CPB >= 16 && (!TA || S::CPA >= 16)), "FP64 swizzle flips bit 3");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sw = wave % S::SWAVES, kg = wave / S::SWAVES;  // output block, k group
  const int wm0 = (sw / WGN) * S::WM, wn0 = (sw % WGN) * S::WN;
  const int gq = lane >> 4, l16 = lane & 15;

  // Source of this lane's chunk in every DMA slot: a 32-bit byte offset from
  // the tile's corner of the operand (uniform, in scalar registers), so a
  // k-step advances by one scalar add per operand and costs the vector units
  // no address arithmetic (the host keeps pitches whose offsets would not fit
  // away from these divisions).
  // Rows of 128 B of k (A, or stored B^T): slot u covers rows 8q .. 8q+7
  // (q = wave*I + u), lane -> row 8q + lane/8, physical chunk lane%8 holding
  // logical chunk c.  Rows of k (B, or stored A^T): slot u covers stage bytes
  // [1024q, 1024q + 1024).  Rows past the matrix and chunks past its columns
  // are clamped to the last valid ones.
  const unsigned lda_b = (unsigned)(g.lda * ESZ), ldb_b = (unsigned)(g.ldb * ESZ);
  auto kcol_row = [&](int q) { return 8 * q + (lane >> 3); };         // [rows][128 B of k]
  auto kcol_kof = [&](int q) { return dma_swz_a(kcol_row(q), lane & 7) * VEC; };
  auto krow_row = [&](int q, int rb) { return (q * 1024 + lane * 16) / rb; };  // [k rows][rb B]
  auto slot_off = [&](auto kcols, int q, int c0, int ext, unsigned ld_b, auto cp) -> unsigned {
    constexpr bool KC = decltype(kcols)::value;
    constexpr int CP = decltype(cp)::value;
    if constexpr (KC) {
      return (unsigned)(min(c0 + kcol_row(q), ext - 1) - c0) * ld_b +
             (unsigned)kcol_kof(q) * ESZ;
    } else {
      const int row = krow_row(q, CP * 16);
      const int c = dma_swz_b<T, CP>(row, ((q * 1024 + lane * 16) % (CP * 16)) >> 4);
      return (unsigned)row * ld_b +
             (unsigned)(min(c0 + c * VEC, ((ext - 1) / VEC) * VEC) - c0) * ESZ;
    }
  };
  typedef std::integral_constant<int, S::CPA> CPA;
  typedef std::integral_constant<int, S::CPB> CPB;
  typedef std::integral_constant<bool, !TA> AKC;
  typedef std::integral_constant<bool, TB> BKC;
  const char *Abase = reinterpret_cast<const char *>(g.A) + (int64_t)m0 * (TA ? ESZ : g.lda * ESZ);
  const char *Bbase = reinterpret_cast<const char *>(g.B) + (int64_t)n0 * (TB ? g.ldb * ESZ : ESZ);
  unsigned aoff[S::IA], boff[S::IB];
#pragma unroll
  for (int u = 0; u < S::IA; ++u)
    aoff[u] = slot_off(AKC{}, wave * S::IA + u, m0, g.m, lda_b, CPA{});
#pragma unroll
  for (int u = 0; u < S::IB; ++u)
    boff[u] = slot_off(BKC{}, wave * S::IB + u, n0, g.n, ldb_b, CPB{});
  const int64_t astep = TA ? (int64_t)BK * g.lda * ESZ : 128;  // bytes per k-step
  const int64_t bstep = TB ? 128 : (int64_t)BK * g.ldb * ESZ;

  const int KT = (g.k + BK - 1) / BK;
  unsigned char *const lds_wa = lds + wave * S::IA * 1024;
  unsigned char *const lds_wb = lds + S::A_BYTES + wave * S::IB * 1024;
  // Loads of whole k-step kt into ring step `slot`.
  auto issue_whole = [&](int kt, int slot) {
    const char *ab = Abase + kt * astep, *bb = Bbase + kt * bstep;
    // opaque scalar bases: keeps the compiler from carrying one 64-bit vector
    // pointer per slot through the loop instead
    asm("" : "+s"(ab), "+s"(bb));
#pragma unroll
    for (int u = 0; u < S::IA; ++u) dma_lds16(ab + aoff[u], lds_wa + slot * S::STEP + u * 1024);
#pragma unroll
    for (int u = 0; u < S::IB; ++u) dma_lds16(bb + boff[u], lds_wb + slot * S::STEP + u * 1024);
  };
  // The same for a k-step that reaches past the problem's k: the k chunk / k
  // row is clamped to the last valid one.
  auto issue_tail = [&](int kt, int slot) {
    const int kbase = kt * BK, last_chunk = ((g.k - 1) / VEC) * VEC;
    auto back = [&](auto kcols, int q, int64_t ld, int rb) -> int64_t {
      if constexpr (decltype(kcols)::value) {
        const int ko = kcol_kof(q);
        return (int64_t)(min(kbase + ko, last_chunk) - ko) * ESZ;
      } else {
        const int kr = krow_row(q, rb);
        return (int64_t)(min(kbase + kr, g.k - 1) - kr) * ld * ESZ;
      }
    };
#pragma unroll
    for (int u = 0; u < S::IA; ++u)
      dma_lds16(Abase + aoff[u] + back(AKC{}, wave * S::IA + u, g.lda, S::RA),
                lds_wa + slot * S::STEP + u * 1024);
#pragma unroll
    for (int u = 0; u < S::IB; ++u)
      dma_lds16(Bbase + boff[u] + back(BKC{}, wave * S::IB + u, g.ldb, S::RB),
                lds_wb + slot * S::STEP + u * 1024);
  };

  Acc acc[S::FM][S::FN];
#pragma unroll
  for (int i = 0; i < S::FM; ++i)
#pragma unroll
    for (int j = 0; j < S::FN; ++j) acc[i][j] = Acc{};

  // Fragments of half a k-step (16-byte k chunks 4h + 0..3, one per lane
  // group): VEC MFMAs per block.  With two k groups, group kg owns half kg.
  struct Frag {
    V a[S::FM];
    T b[VEC][S::FN];
  };
  auto load_frag = [&](Frag &f, const unsigned char *As, int h) {
    const unsigned char *Bs = As + S::A_BYTES;
    const int kc = 4 * (KS == 2 ? kg : h) + gq;  // this lane group's 16-byte k chunk
#pragma unroll
    for (int i = 0; i < S::FM; ++i) {
      const int row = wm0 + 16 * i + l16;
      if constexpr (!TA) {
        f.a[i] = *reinterpret_cast<const V *>(As + row * 128 + dma_swz_a(row, kc) * 16);
      } else if constexpr (PAIRA) {
        if (i % 2 == 0) {  // rows wm0 + 32p + 2*l16 (block 2p) and +1 (block 2p+1)
          const int chunk = ((wm0 + 16 * i) >> 1) + l16;
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            const int kr = kc * VEC + v;
            const V aa = *reinterpret_cast<const V *>(As + kr * S::RA +
                                                      dma_swz_b<T, S::CPA>(kr, chunk) * 16);
            f.a[i][v] = aa[0];
            f.a[i + 1][v] = aa[1];
          }
        }
      } else {
        const int byte = row * ESZ;
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          const int kr = kc * VEC + v;
          f.a[i][v] = *reinterpret_cast<const T *>(
              As + kr * S::RA + dma_swz_b<T, S::CPA>(kr, byte >> 4) * 16 + (byte & 15));
        }
      }
    }
    if constexpr (TB) {  // transposed B: one chunk of VEC k values per block column
#pragma unroll
      for (int j = 0; j < S::FN; ++j) {
        const int col = wn0 + 16 * j + l16;
        const V bv = *reinterpret_cast<const V *>(Bs + col * 128 + dma_swz_a(col, kc) * 16);
#pragma unroll
        for (int v = 0; v < VEC; ++v) f.b[v][j] = bv[v];
      }
    } else {
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        const int kr = kc * VEC + v;
        if constexpr (PAIR) {
#pragma unroll
          for (int p = 0; p < S::FN / 2; ++p) {
            const int chunk = ((wn0 + 32 * p) >> 1) + l16;  // columns wn0 + 32p + 2*l16, +1
            const V bb = *reinterpret_cast<const V *>(Bs + kr * S::RB +
                                                      dma_swz_b<T, S::CPB>(kr, chunk) * 16);
            f.b[v][2 * p] = bb[0];
            f.b[v][2 * p + 1] = bb[1];
          }
        } else {
#pragma unroll
          for (int j = 0; j < S::FN; ++j) {
            const int byte = (wn0 + 16 * j + l16) * ESZ;
            f.b[v][j] = *reinterpret_cast<const T *>(
                Bs + kr * S::RB + dma_swz_b<T, S::CPB>(kr, byte >> 4) * 16 + (byte & 15));
          }
        }
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
  auto mma_frag = [&](const Frag &f) {
    mma_first(f);
    mma_rest(f);
  };

  // Last, partial k-step: zero every k >= kvalid of the landed stage (A
  // columns, B rows), so values read from clamped addresses never reach the
  // sums; the same zeros the register-staged tile loads past k.
  auto zero_krows = [&](unsigned char *X, int cp, int kvalid) {  // [k rows][cp chunks]
    for (int e = tid; e < BK * cp; e += S::THREADS)
      if (e / cp >= kvalid) *reinterpret_cast<V *>(X + e * 16) = V{};
  };
  auto zero_kcols = [&](unsigned char *X, int rows, int kvalid) {  // [rows][128 B of k]
    for (int e = tid; e < rows * 8; e += S::THREADS) {
      const int row = e >> 3, c = e & 7;
      if ((c + 1) * VEC <= kvalid) continue;
      T *p = reinterpret_cast<T *>(X + row * 128 + dma_swz_a(row, c) * 16);
#pragma unroll
      for (int v = 0; v < VEC; ++v)
        if (c * VEC + v >= kvalid) p[v] = T(0);
    }
  };
  auto zero_tail = [&](unsigned char *As, unsigned char *Bs, int kvalid) {
    if constexpr (!TA) zero_kcols(As, BM, kvalid);
    else zero_krows(As, S::CPA, kvalid);
    if constexpr (!TB) zero_krows(Bs, S::CPB, kvalid);
    else zero_kcols(Bs, BN, kvalid);
  };

  // Stages of KU k-steps.  Stages [0, SW) are whole; the one after them, if
  // any, loads k past the problem from clamped addresses (zeroed below or
  // never multiplied), so every stage has the same number of loads.
  constexpr int HPS = 2 / KS;   // half steps of this wavefront per k-step
  constexpr int U = KU * HPS;   // and per stage
  const int ST = (KT + KU - 1) / KU, SW = g.k / (KU * BK);
  auto issue_stage = [&](int st) {
    const int slot = (st % NS) * KU;
    if (st < SW) {
#pragma unroll
      for (int u = 0; u < KU; ++u) issue_whole(st * KU + u, slot + u);
    } else {
#pragma unroll
      for (int u = 0; u < KU; ++u) issue_tail(st * KU + u, slot + u);
    }
  };
  auto half = [&](Frag &f, int slot, int u) {
    load_frag(f, lds + slot * S::STAGE + u / HPS * S::STEP, u % HPS);
  };
  MG_LDS_POISON_STAGE(lds, NS * S::STAGE);
  int st = 0;
  Frag f[2];
  if constexpr (S::AHEAD && !SHORT) {
    // Small wave tiles: the fragments of a half step are read from LDS while
    // the matrix cores work on the previous half step's.  Before the last
    // half step of stage st the wavefronts meet: stage st+1 has landed (only
    // the stages issued after it may be pending), every wavefront has its
    // fragments of stage st, and its place in the ring is refilled with st+NS.
#pragma unroll
    for (int q = 0; q < NS; ++q)
      if (q < ST) issue_stage(q);
    if (SW > 0) {
      dma_wait_steps<DPS, NS>(min(ST, NS) - 1);
      __builtin_amdgcn_s_barrier();
      half(f[0], 0, 0);
    }
    // Whole stages with whole refills, unrolled over the ring: LDS addresses
    // are constants and nothing branches.
    constexpr int UNR = NS * U % 2 ? 2 * NS : NS;  // fragment registers alternate
    static_assert(UNR == S::UNROLL, "k that SHORT serves");
    for (; st + UNR + NS - 1 < SW; st += UNR) {
#pragma unroll
      for (int j = 0; j < UNR; ++j)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // The order is pinned: one product first (its wait covers only this
          // half step's fragments), then the reads and loads that the other
          // products hide.
          const Frag &cur = f[(j * U + u) & 1];
          Frag &nx = f[(j * U + u + 1) & 1];
          if (u + 1 == U) {
            dma_wait_ring<(NS - 2) * DPS>();
            __builtin_amdgcn_s_barrier();
            MG_LDS_POISON_STAGE(lds + (j % NS) * S::STAGE, S::STAGE);
          }
          mma_first(cur);
          __builtin_amdgcn_sched_barrier(0);
          if (u + 1 < U) {
            half(nx, j % NS, u + 1);
          } else {
            half(nx, (j + 1) % NS, 0);
#pragma unroll
            for (int w = 0; w < KU; ++w) issue_whole((st + j + NS) * KU + w, (j % NS) * KU + w);
          }
          __builtin_amdgcn_sched_barrier(0);
          mma_rest(cur);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    for (; st < SW; ++st) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u + 1 < U) {
          half(f[1], st % NS, u + 1);
        } else if (st + 1 < SW) {
          dma_wait_steps<DPS, NS>(min(ST - 1, st + NS - 1) - (st + 1));
          dma_wait_lds();
          __builtin_amdgcn_s_barrier();
          if (st + NS < ST) {
            MG_LDS_POISON_STAGE(lds + (st % NS) * S::STAGE, S::STAGE);
            issue_stage(st + NS);
          }
          half(f[1], (st + 1) % NS, 0);
        }
        mma_frag(f[0]);
        f[0] = f[1];
      }
    }
  } else {
    // Large wave tiles: a half step's products are long enough to hide its
    // fragment reads behind the other wavefronts', and a second fragment set
    // would cost a workgroup per CU.  Stage st's barrier also frees stage
    // st-1 (every wavefront has its fragments: the lgkmcnt wait, as products
    // may be scheduled past the barrier), refilled with st+NS-1.
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
      if (q < ST) issue_stage(q);
    for (; !SHORT && st + 2 * NS - 2 < SW; st += NS) {
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        const int rs = (j + NS - 1) % NS;  // the ring stage refilled
        dma_wait_ring<(NS - 2) * DPS>();
        __builtin_amdgcn_s_barrier();
        MG_LDS_POISON_STAGE(lds + rs * S::STAGE, S::STAGE);
#pragma unroll
        for (int w = 0; w < KU; ++w) issue_whole((st + j + NS - 1) * KU + w, rs * KU + w);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          half(f[0], j, u);
          mma_frag(f[0]);
        }
      }
    }
    for (; st < SW; ++st) {
      dma_wait_steps<DPS, NS>(min(ST - 1, st + NS - 2) - st);
      dma_wait_lds();
      __builtin_amdgcn_s_barrier();
      if (st + NS - 1 < ST) {
        MG_LDS_POISON_STAGE(lds + ((st + NS - 1) % NS) * S::STAGE, S::STAGE);
        issue_stage(st + NS - 1);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        half(f[0], st % NS, u);
        mma_frag(f[0]);
      }
    }
  }
  if (st < ST) {  // the last, partial stage: nothing else is in flight
    dma_wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    unsigned char *As = lds + (st % NS) * S::STAGE;
    for (int kt = st * KU; kt < KT; ++kt, As += S::STEP) {
      if (g.k - kt * BK < BK) {
        zero_tail(As, As + S::A_BYTES, g.k - kt * BK);
        __syncthreads();
      }
#pragma unroll
      for (int h = 0; h < HPS; ++h) {
        load_frag(f[0], As, h);
        mma_frag(f[0]);
      }
    }
  }

  if constexpr (KS == 2) {
    // k group 1 hands its sums to group 0 through LDS (the ring is free once
    // every wave is past its last step); group 0 adds them and stores.
    constexpr int NA = sizeof(Acc) / sizeof(T);
    T *red = reinterpret_cast<T *>(lds) + (size_t)sw * S::FM * S::FN * NA * 64 + lane;
    __syncthreads();
    if (kg == 1) {
#pragma unroll
      for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
#pragma unroll
          for (int e = 0; e < NA; ++e) red[((i * S::FN + j) * NA + e) * 64] = acc[i][j][e];
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
      for (int j = 0; j < S::FN; ++j)
#pragma unroll
        for (int e = 0; e < NA; ++e) acc[i][j][e] += red[((i * S::FN + j) * NA + e) * 64];
  }

  if constexpr (PAIR)
    store_paired_f64<S::FM, S::FN, S::FM, S::FN, PAIRA>(g, acc, m0 + wm0, n0 + wn0, lane);
  else if constexpr (ESZ == 8)
    Epilogue<T>::template store<S::FM, S::FN, S::FM, S::FN, PAIRA>(g, acc, m0 + wm0,
                                                                    n0 + wn0, lane);
  else
    Epilogue<T>::template store<S::FM, S::FN>(g, acc, m0 + wm0, n0 + wn0, lane);
}

}  // namespace mg
