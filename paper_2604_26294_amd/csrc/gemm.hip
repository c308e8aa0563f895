// bf16 MFMA GEMM family for the TSP shard products (gfx950).
//
//   gate+up+SwiGLU  Hs = bf16( SiLU(X W1^T) * (X W3^T) )          Algorithm 2, gate/up
//   down / O-proj   Y (+)= Hs W2   or   Y (+)= Flatten(A) W_O^T    Algorithm 2 / 1, "+="
//                   (over up to eight operand pairs at once: the contraction then runs
//                   over [A A' ..] and [B; B'; ..], held in separate buffers)
//   SwiGLU backward G = X W1^T, U = X W3^T, dHs = dY W2^T in one pass; dG, dU and the
//                   transposes of dG, dU, Hs for the weight-gradient products
//   Q/K/V proj      Q = X W_Q^T (times a factor, then rounded) -> workspace, K, V ->
//                   full-sequence buffers at the rows' sequence positions (zigzag
//                   reorder folded in)  Algorithm 1
//
// One workgroup = WGM x WGN wavefronts (8 by default: two per SIMD); each wavefront owns
// a (BM/WGM) x (BN/WGN) block of C.  K advances in steps of 64.  Operand panels go from HBM
// straight into LDS (buffer loads with an LDS destination, no register staging).  Two main
// loops: PpTile, 256 x 256 accumulators of 16 x 16 x 32 MFMAs with the two wavefronts of a
// SIMD alternating between MFMAs and memory (products that fill the chip with such tiles),
// and gemm_tile, smaller tiles with a ring of STAGES slots: while the MFMAs consume step k
// the loads fill the steps up to k + STAGES - 1.  Both use the 16 x 16 x 32 MFMA, whose
// accumulator traffic per product is half that of 32 x 32 x 16: on real data these kernels
// run at the chip's power limit (see PpTile).
//
// LDS layouts.  LDS has 64 banks of 4 bytes, so a byte address maps to bank window
// position (address mod 256).  A [M, K] and "NT" B [N, K] panels are rows of 64 bf16
// (128 bytes, eight 16-byte chunks); an MFMA operand is one 16-byte read, 16 lanes of
// which read 16 consecutive rows at one logical chunk, so the physical chunk is the
// logical one XOR ((row / 2) mod 8) and those 16 reads hit 16 distinct windows.
// "NN" B panels ([K, N] operands: W2 and W_O^(r)^T) keep their natural [64][columns] layout
// and are read with the gfx950 LDS transpose read ds_read_b64_tr_b16: in each 16-lane
// group, source lane s points at row kbase + s/4, columns base + 4 (s % 4), and lane t
// receives column base + t of rows kbase..kbase+3, i.e. four consecutive contraction indices
// of one output column -- no transpose pass over HBM and no register shuffles.  A half-wave
// reads rows r .. r + 3 and r + 8 .. r + 11 of 16 columns, 8 x 32 bytes, which the chunk XOR
// of those row bits (nn_swz) spreads over all 64 banks.  Every LDS address is a per-lane base
// XOR a wave-uniform constant plus an immediate offset.
//
// Tails.  Rows or columns past M / N are clamped to the last valid one on load (finite
// values, results never stored).  K must be a multiple of 64: the gated product Hs is
// stored with its width padded to a multiple of 64 with zero columns (written by the
// SwiGLU epilogue), and the matching W2 rows past F/D are clamped, so padded terms
// contribute exact zeros.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "lds_dma.h"

namespace tsp {
namespace {

constexpr int BK = 64;
template <int N>
using Ic = std::integral_constant<int, N>;
enum { EPI_SWIGLU = 0, EPI_ACC = 1, EPI_QKV = 2, EPI_SWIGLU_BWD = 3 };

// Wait until at most N of this wavefront's operand loads are still in flight (loads
// complete in issue order).
template <int N>
__device__ __forceinline__ void wait_dma() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Wait for the stage that a step is about to read, with up to AHEAD later stages of LOADS
// loads each (`issued` of them, if fewer) left in flight.
template <int AHEAD, int LOADS>
__device__ __forceinline__ void wait_ahead(int issued) {
  if constexpr (AHEAD == 0) {
    wait_dma<0>();
  } else {
    if (issued >= AHEAD) wait_dma<AHEAD * LOADS>();
    else wait_ahead<AHEAD - 1, LOADS>(issued);
  }
}

template <int BM, int BN, int WGM, int WGN, bool NN, int EPI, int STAGES>
struct Cfg {
  static constexpr int WAVES = WGM * WGN, THREADS = kWave * WAVES;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int TM = WM / 32, TN = WN / 16;  // 32-row, 16-column blocks
  // Output columns of a wavefront: 32-column block j starts at wn COL_WN + j COL_BLK.
  static constexpr int COL_WN = WN, COL_BLK = 32;
  static constexpr int NBP = EPI == EPI_SWIGLU ? 2 : 1;       // B panels
  static constexpr int TNB = NBP * TN;
  static constexpr int NB = NBP * BN;                         // B rows of an NT panel
  static constexpr int A_BYTES = BM * BK * 2;
  static constexpr int B_BYTES = NB * BK * 2;                  // NT [NB][64] or NN [64][BN]
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = STAGES * STAGE;
  // Operand load instructions one wavefront issues per stage.
  // [N, K]-operand tiles: only the first half of the wavefronts (one per SIMD) load, each
  // its own share of a stage and that of the other wavefront of its SIMD; [K, N] tiles:
  // every wavefront loads its share.
  static constexpr bool HALF_LOADERS = !NN && WAVES == 8;
  static constexpr int LOADS = (HALF_LOADERS ? 2 : 1) *
      (BM / 8 / WAVES + (NN ? BK * (BN * 2) / 1024 / WAVES : NB / 8 / WAVES));
  static_assert(STAGES >= 2 && LDS_BYTES <= 160 * 1024, "LDS ring");
  static_assert(LOADS * (STAGES - 2) < 64, "vmcnt range");
  static constexpr int NN_RB = BN * 2;                         // NN panel row bytes
  static_assert(!(NN && EPI == EPI_SWIGLU), "SwiGLU operands are [N, K]");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile");
  static_assert(!NN || BN == 64 || BN == 128, "NN panel swizzle");
  static_assert((BM / 8) % WAVES == 0 && (NB / 8) % WAVES == 0, "NT DMA cover");
  static_assert(!NN || (BK * NN_RB / 1024) % WAVES == 0, "NN DMA cover");
};

// Output tile t of a tiles_m x tiles_n grid in the work order: blocks of kTileGroupM
// consecutive row tiles, column tiles in order within a block and the rows of a block
// fastest, so that the 32 consecutive tiles an XCD runs at a time span about as many row
// as column tiles and its L2 serves each operand panel to several of them.
constexpr int kTileGroupM = 4;
__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int* tm, int* tn) {
  const int blk = t / (kTileGroupM * tiles_n), in = t - blk * kTileGroupM * tiles_n;
  const int rows = min(kTileGroupM, tiles_m - blk * kTileGroupM);
  *tm = blk * kTileGroupM + in % rows;
  *tn = in / rows;
}

// Chunk swizzles of the NT and NN panels (physical chunk = logical chunk XOR swz(row)).
__device__ __forceinline__ int nt_swz(int row) { return (row >> 1) & 7; }
// Panels of 128 columns (256-byte rows) and of 64 (128-byte rows, two per bank window).
template <int COLS>
__device__ __forceinline__ int nn_swz(int row) {
  static_assert(COLS == 64 || COLS == 128, "panel width");
  return COLS == 128 ? 4 * (row & 3) + 2 * ((row >> 3) & 1)
                     : 4 * ((row >> 3) & 1) + 2 * ((row >> 1) & 1);
}

// Operand panels go HBM -> LDS through buffer loads with an LDS destination (lds_dma.h):
// address = resource base (the matrix) + scalar offset (the stage's K position) + a
// per-lane offset.  The per-lane offsets only depend on the tile and the lane, so they
// are formed once per tile and a stage is issued without vector arithmetic.  The byte
// extent of every operand must stay below 4 GiB (checked at launch).
//
// NT panel rows [row0, row0 + ROWS) x k [k0, k0 + 64) of a row-major [nrows, ld] matrix
// (128-byte LDS rows): instruction i of wave w fills rows 8 (i W + w) .. +7, lane l row
// 8 (i W + w) + l / 8, physical chunk l % 8 (logical chunk XOR nt_swz(row)); rows past
// nrows are clamped to the last one.  Stage offset: 2 k0 bytes.
template <int ROWS, int WAVES>
struct NtRows {
  static constexpr int NI = ROWS / 8 / WAVES;
  uint32_t off[NI];
  __device__ __forceinline__ void init(int ld, int row0, int nrows, int wave, int lane) {
    const int rsub = lane >> 3, pc = lane & 7;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = 8 * (i * WAVES + wave) + rsub;
      const uint32_t grow = (uint32_t)min(row0 + r, nrows - 1);
      off[i] = 2u * (grow * (uint32_t)ld + 8u * (uint32_t)(pc ^ nt_swz(r)));
    }
  }
  __device__ __forceinline__ void issue(lds_char* dst, const rsrc_t& rs, uint32_t k0,
                                        int wave) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) dma16(rs, off[i], 2u * k0, dst + (i * WAVES + wave) * 1024);
  }
};

// NN panel: k rows [k0, k0 + 64) x n [n0, n0 + BN) of a row-major [krows, ld] matrix
// (natural layout, BN * 2-byte LDS rows, chunk XOR nn_swz(row)); instruction i of wave w
// fills rows RPI (i W + w) .. +RPI-1.  Columns past ncols are clamped (in the per-lane
// offsets) and rows past krows too (only in a stage that reaches past them).
template <int BN, int WAVES>
struct NnRows {
  static constexpr int CH = BN / 8, RPI = kWave / CH, NI = BK / RPI / WAVES;
  uint32_t off[NI];  // 2 (r ld + gn): row r of the stage, column gn
  int r0;            // this lane's row in instruction 0 (instruction i: r0 + i RPI W)
  __device__ __forceinline__ void init(int ld, int n0, int ncols, int wave, int lane) {
    const int rsub = lane / CH, pc = lane % CH;
    r0 = RPI * wave + rsub;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = r0 + i * RPI * WAVES;
      const uint32_t gn = (uint32_t)min(n0 + 8 * (pc ^ nn_swz<BN>(r)), ncols - 8);
      off[i] = 2u * ((uint32_t)r * (uint32_t)ld + gn);
    }
  }
  __device__ __forceinline__ void issue(lds_char* dst, const rsrc_t& rs, int k0, int krows,
                                        int ld, int wave) const {
    if (k0 + BK <= krows) {
      const uint32_t soff = 2u * (uint32_t)k0 * (uint32_t)ld;
#pragma unroll
      for (int i = 0; i < NI; ++i) dma16(rs, off[i], soff, dst + (i * WAVES + wave) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int r = r0 + i * RPI * WAVES;
        const int gk = min(k0 + r, krows - 1);
        const uint32_t voff = off[i] + 2u * (uint32_t)(gk - r) * (uint32_t)ld;
        dma16(rs, voff, 0u, dst + (i * WAVES + wave) * 1024);
      }
    }
  }
};

// Orders this wavefront's LDS writes before its later LDS reads (and those reads before
// its next writes) without a workgroup barrier: every wavefront stages its blocks in an
// LDS region of its own, and LDS operations of one wavefront complete in issue order, so
// only the compiler must be kept from moving them across each other.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Epilogue of one C tile (configuration C: WAVES, WM, WN, TM, TN, COL_WN, COL_BLK, LDS_BYTES)
// from the accumulators of each wavefront, staged through the workgroup's LDS (free:
// every operand read has completed).
template <class C, int EPI, class Acc>
__device__ __forceinline__ void gemm_epilogue(const GemmParams& P, Acc& acc, char* L, const int wave, const int lane,
                                              const int m0, const int n0, const int wm,
                                              const int wn, const int split = 0) {
  constexpr int TM = C::TM, TN = C::TN;
  // Each wavefront stages one 32-row block of its C tile in LDS as fp32, then writes it
  // out in 4-column chunks: consecutive lanes cover consecutive columns, every global
  // access is 16 bytes (fp32) or 8 bytes (bf16), and all loads of a block are in flight
  // before the first store.
  constexpr int EST = C::WN + 4;  // staging row stride in floats
  constexpr int CPR = C::WN / 4;  // 4-column chunks per row
  constexpr int PER_LANE = 32 * CPR / kWave;
  static_assert(C::WAVES * 32 * EST * 4 <= C::LDS_BYTES, "epilogue staging fits");
  float* E = reinterpret_cast<float*>(L) + wave * 32 * EST;
  // Element e of accumulator block [row block 2 i + q][column block j] of 32-row block i.
  auto staged = [&](int q, int j, int e) __attribute__((always_inline)) -> float& {
    return E[(16 * q + 4 * (lane >> 4) + e) * EST + 16 * j + (lane & 15)];
  };
  const int ncol0 = n0 + wn * C::COL_WN;
  if constexpr (EPI == EPI_SWIGLU_BWD) {
    // SwiGLU backward.  Per 32-row block: dG, dU and Hs replace G, U and dHs in the
    // accumulators, then each is staged once in LDS as bf16, transposed (a lane holds four
    // consecutive rows of a column: one 8-byte write), [column][32 rows].  The transposed
    // outputs are 16-byte reads of that, the row-major ones (dG, dU) transpose reads of 4
    // columns of a row.  (Staged in fp32 and read back column by column this epilogue took
    // 17 % of the launch, 180 of 1045 us at 7B, S_loc = 8192, 4 shards.)
    constexpr int TST = 32 * 2 + 16;  // staging stride of a column, in bytes
    lds_char* T = (lds_char*)L + wave * (C::WN * TST);
    const int l16 = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = acc[2 * i + r][j][e], u = acc[2 * i + r][j + TN][e];
            const float dh = acc[2 * i + r][j + 2 * TN][e];
            const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-g));
            const float sl = g * sg;
            acc[2 * i + r][j][e] = dh * u * (sg * (1.f + g * (1.f - sg)));  // dG
            acc[2 * i + r][j + TN][e] = dh * sl;                           // dU
            acc[2 * i + r][j + 2 * TN][e] = sl * u;                        // Hs
          }
      const int mrow0 = m0 + wm * C::WM + 32 * i;
      if (mrow0 + 32 > P.M) {  // rows M..ldt of the transposes: zero padding
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int j = 0; j < 3 * TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (mrow0 + 16 * r + 4 * lg + e >= P.M) acc[2 * i + r][j][e] = 0.f;
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const f32x4& v = acc[2 * i + r][q * TN + j];
            *reinterpret_cast<__attribute__((address_space(3))) u32x2*>(
                T + (16 * j + l16) * TST + 2 * (16 * r + 4 * lg)) =
                u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
          }
        wave_lds_sync();
        if (q < 2) {
          // Lane group lg takes columns 16 c + 4 lg .. +3 of rows 16 r + l16.
          uint16_t* H = q == 0 ? P.H : P.H2;
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < TN; ++c) {
              const u32x2 v = lds_read_tr(T + (16 * c + 4 * lg + (l16 >> 2)) * TST +
                                          2 * (16 * r + 4 * (l16 & 3)));
              const int mm = mrow0 + 16 * r + l16, nn = ncol0 + 16 * c + 4 * lg;
              if (mm < P.M && nn < P.h_cols)  // columns N..h_cols: zero padding
                *reinterpret_cast<u32x2*>(H + (size_t)mm * P.ldh + nn) = nn < P.N ? v : u32x2{0u, 0u};
            }
        }
        uint16_t* Tg = q == 0 ? P.T0 : (q == 1 ? P.T1 : P.T2);
#pragma unroll
        for (int k = 0; k < C::WN / 16; ++k) {
          const int c = 16 * k + (lane >> 2), r0 = 8 * (lane & 3);
          const u32x4 v = lds_read16(T + c * TST + 2 * r0);
          const int nn = ncol0 + c, mm = mrow0 + r0;
          if (nn < P.N && mm < P.ldt) st16(Tg + (size_t)nn * P.ldt + mm, v);
        }
        wave_lds_sync();
      }
    }
    return;
  }
  auto value = [](float v, float up) __attribute__((always_inline)) {
    if constexpr (EPI == EPI_SWIGLU) v = v * __builtin_amdgcn_rcpf(1.f + __expf(-v)) * up;
    return v;
  };
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          staged(q, j, e) =
              value(acc[2 * i + q][j][e], EPI == EPI_SWIGLU ? acc[2 * i + q][j + TN][e] : 0.f);
    wave_lds_sync();
    const int mrow0 = m0 + wm * C::WM + 32 * i;
    // Q/K/V scatter: batch entry and token of the block's first row, once per block (a row
    // r of the block is then token t0 + r of entry b0, or of the next entry past its end).
    int b0 = 0, t0 = 0;
    if constexpr (EPI == EPI_QKV) {
      b0 = mrow0 / P.rows_per_batch;
      t0 = mrow0 - b0 * P.rows_per_batch;
    }
    f32x4 v[PER_LANE];
    int mm[PER_LANE], nn[PER_LANE];
    bool ok[PER_LANE];
#pragma unroll
    for (int q = 0; q < PER_LANE; ++q) {
      const int idx = q * kWave + lane, row = idx / CPR, c4 = idx % CPR;
      v[q] = *reinterpret_cast<const f32x4*>(E + row * EST + 4 * c4);
      mm[q] = mrow0 + row;
      nn[q] = ncol0 + (c4 / 8) * C::COL_BLK + 4 * (c4 % 8);
      ok[q] = mm[q] < P.M && nn[q] < P.N;
    }
    if constexpr (EPI == EPI_ACC) {
      if (P.k_splits > 1) {  // a partial product of one contraction range
        float* dst = P.part + (size_t)split * P.M * P.N;
#pragma unroll
        for (int q = 0; q < PER_LANE; ++q)
          if (ok[q]) *reinterpret_cast<f32x4*>(dst + (size_t)mm[q] * P.N + nn[q]) = v[q];
        wave_lds_sync();
        continue;
      }
      // The base values of the block: every lane loads (chunks outside the product read
      // an in-range element instead and are not stored), so that all loads of the block
      // are issued before the first wait rather than one load and one wait per chunk.
      f32x4 base[PER_LANE];
      if (P.R) {
        u32x2 r[PER_LANE];
#pragma unroll
        for (int q = 0; q < PER_LANE; ++q)
          r[q] = *reinterpret_cast<const u32x2*>(P.R + (size_t)min(mm[q], P.M - 1) * P.ldr +
                                                 min(nn[q], P.N - 4));
#pragma unroll
        for (int q = 0; q < PER_LANE; ++q)
          base[q] = f32x4{bf16_bits_to_f32(r[q][0] & 0xffffu), bf16_bits_to_f32(r[q][0] >> 16),
                          bf16_bits_to_f32(r[q][1] & 0xffffu), bf16_bits_to_f32(r[q][1] >> 16)};
      } else if (P.accumulate) {
#pragma unroll
        for (int q = 0; q < PER_LANE; ++q)
          base[q] = *reinterpret_cast<const f32x4*>(P.Y + (size_t)min(mm[q], P.M - 1) * P.ldy +
                                                    min(nn[q], P.N - 4));
      } else {
#pragma unroll
        for (int q = 0; q < PER_LANE; ++q) base[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int q = 0; q < PER_LANE; ++q) {
        if (!ok[q]) continue;
        const f32x4 out = v[q] + base[q];
        *reinterpret_cast<f32x4*>(P.Y + (size_t)mm[q] * P.ldy + nn[q]) = out;
        if (P.U)
          *reinterpret_cast<u32x2*>(P.U + (size_t)mm[q] * P.ldu + nn[q]) =
              u32x2{pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3])};
      }
    } else {
#pragma unroll
      for (int q = 0; q < PER_LANE; ++q) {
        if constexpr (EPI == EPI_SWIGLU) {
          // Columns [N, h_cols) are the zero padding of the gated product.
          if (mm[q] >= P.M || nn[q] >= (P.h_cols > 0 ? P.h_cols : P.ldh)) continue;
          const u32x2 bits = nn[q] < P.N ? u32x2{pack_bf16x2(v[q][0], v[q][1]),
                                                 pack_bf16x2(v[q][2], v[q][3])}
                                         : u32x2{0u, 0u};
          *reinterpret_cast<u32x2*>(P.H + (size_t)mm[q] * P.ldh + nn[q]) = bits;
        } else {
          if (!ok[q]) continue;
          const int n = nn[q], m = mm[q];
          const float f = n < P.nq ? P.q_scale : 1.f;  // the Q block is scaled, then rounded
          const u32x2 bits{pack_bf16x2(f * v[q][0], f * v[q][1]),
                           pack_bf16x2(f * v[q][2], f * v[q][3])};
          uint16_t* dst;
          if (n < P.nq) {
            dst = P.Q + (size_t)m * P.ldq + n;
          } else {
            int b = b0, t = t0 + (m - mrow0);
            while (t >= P.rows_per_batch) {  // once at most when entries hold >= 32 rows
              t -= P.rows_per_batch;
              ++b;
            }
            const long long pos = t < P.kv_seg ? P.kv_pos0 + t : P.kv_pos1 + (t - P.kv_seg);
            const size_t row = (size_t)b * P.kv_batch_stride +
                               (size_t)pos * P.kv_row_stride + P.kv_col0;
            dst = n < P.nq + P.nkv ? P.Kb + row + (n - P.nq) : P.Vb + row + (n - P.nq - P.nkv);
          }
          *reinterpret_cast<u32x2*>(dst) = bits;
        }
      }
    }
    wave_lds_sync();
  }
}

// The output tile at (m0, n0) of the product P (its contraction range `split`), in the
// workgroup's LDS L.
template <int BM, int BN, int WGM, int WGN, bool NN, int EPI, int STAGES>
__device__ __forceinline__ void gemm_tile(const GemmParams& P, const int m0, const int n0,
                                          const int split, char* L) {
  using C = Cfg<BM, BN, WGM, WGN, NN, EPI, STAGES>;
  constexpr int TM = 2 * C::TM, TN = C::TN, TNB = C::TNB;  // 16 x 16 blocks
  lds_char* Ls = (lds_char*)L;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int l16 = lane & 15, lg = lane >> 4;

  f32x4 acc[TM][TNB];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TNB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // The operand pairs of a multi-part contraction, read once into scalar registers (the
  // asm keeps them there: the per-stage choice is then a chain of scalar selects, not an
  // indexed access, which would put the parameters in scratch memory).
  const uint16_t* ap[kGemmPartsMax];
  const uint16_t* bp[kGemmPartsMax];
  int k_part = INT_MAX;
  if constexpr (NN) {
    const bool multi = P.n_parts > 1;
#pragma unroll
    for (int i = 0; i < kGemmPartsMax; ++i) {
      ap[i] = multi && i < P.n_parts ? P.A_part[i] : P.A;
      bp[i] = multi && i < P.n_parts ? P.B_part[i] : P.B;
      asm volatile("" : "+s"(ap[i]), "+s"(bp[i]));
    }
    if (multi) k_part = P.k_part;
    asm volatile("" : "+s"(k_part));
  }
  // Per-lane DMA offsets of this tile (the NT B panels share rows and stride), and the
  // operands' buffer resources.
  // With HALF_LOADERS only the first half of the wavefronts (one per SIMD: wavefronts are
  // placed on the SIMDs round-robin) issue loads, each its own share and that of
  // wavefront wave + W/2 (the other wavefront of its SIMD): a CU's load path takes a
  // stage's 64 KB at about 60 bytes per cycle, so a wavefront that issues loads stalls
  // for hundreds of cycles, and this way one wavefront of every SIMD never does and keeps
  // the matrix pipe fed meanwhile.
  constexpr int HW = C::WAVES / 2;
  const bool loader = !C::HALF_LOADERS || wave < HW;
  const int wave2 = wave + HW;
  NtRows<BM, C::WAVES> rows_a, rows_a_hi;
  rows_a.init(P.lda, m0, P.M, wave, lane);
  if constexpr (C::HALF_LOADERS) rows_a_hi.init(P.lda, m0, P.M, wave2, lane);
  NtRows<NN ? 8 * C::WAVES : BN, C::WAVES> rows_b, rows_b_hi;  // (unused for NN)
  NnRows<BN, C::WAVES> rows_nn, rows_nn_hi;                     // (unused for NT)
  if constexpr (NN) {
    rows_nn.init(P.ldb, n0, P.N, wave, lane);
    if constexpr (C::HALF_LOADERS) rows_nn_hi.init(P.ldb, n0, P.N, wave2, lane);
  } else {
    rows_b.init(P.ldb, n0, P.N, wave, lane);
    if constexpr (C::HALF_LOADERS) rows_b_hi.init(P.ldb, n0, P.N, wave2, lane);
  }
  const rsrc_t rs_a = make_rsrc(P.A);
  const rsrc_t rs_b = make_rsrc(P.B);
  const rsrc_t rs_b2 = make_rsrc(EPI == EPI_SWIGLU ? P.B2 : P.B);
  auto dma_stage = [&](int stage, int k0) __attribute__((always_inline)) {
    if (!loader) return;
    lds_char* S = Ls + stage * C::STAGE;
    if constexpr (NN) {
      // (k0 is uniform: the part is chosen per stage, from scalar values)
      const int part = k0 / k_part, kk = k0 - part * k_part;
      const uint16_t* a = ap[0];
      const uint16_t* b = bp[0];
#pragma unroll
      for (int i = 1; i < kGemmPartsMax; ++i) {
        a = part == i ? ap[i] : a;
        b = part == i ? bp[i] : b;
      }
      const rsrc_t ra = make_rsrc(a), rb = make_rsrc(b);
      rows_a.issue(S, ra, (uint32_t)kk, wave);
      if constexpr (C::HALF_LOADERS) rows_a_hi.issue(S, ra, (uint32_t)kk, wave2);
      rows_nn.issue(S + C::A_BYTES, rb, kk, P.Kb_rows, P.ldb, wave);
      if constexpr (C::HALF_LOADERS)
        rows_nn_hi.issue(S + C::A_BYTES, rb, kk, P.Kb_rows, P.ldb, wave2);
      return;
    }
    rows_a.issue(S, rs_a, (uint32_t)k0, wave);
    if constexpr (C::HALF_LOADERS) rows_a_hi.issue(S, rs_a, (uint32_t)k0, wave2);
    rows_b.issue(S + C::A_BYTES, rs_b, (uint32_t)k0, wave);
    if constexpr (C::HALF_LOADERS) rows_b_hi.issue(S + C::A_BYTES, rs_b, (uint32_t)k0, wave2);
    if constexpr (EPI == EPI_SWIGLU) {
      rows_b.issue(S + C::A_BYTES + BN * BK * 2, rs_b2, (uint32_t)k0, wave);
      if constexpr (C::HALF_LOADERS)
        rows_b_hi.issue(S + C::A_BYTES + BN * BK * 2, rs_b2, (uint32_t)k0, wave2);
    }
  };

  // Operand addressing (see the header), substep s of 32 contraction indices: A / NT-B row R
  // + l16, chunk 4 s + lg  ->  R * 128 + (opa ^ 64 s),  opa = l16 * 128 + 16 (lg ^ nt_swz(l16)).
  const int opa = l16 * 128 + 16 * (lg ^ nt_swz(l16));
  // NN-B transpose reads for output column block j: rows 32 s + 8 lg + l16 / 4 (+4), columns
  // wn WN + 16 j + 4 (l16 mod 4)  ->  32 s NN_RB + (nb ^ 2 (wn WN + 16 j)).
  int nb_lo = 0, nb_hi = 0;
  if constexpr (NN) {
    const int cl = (l16 & 3) >> 1, half8 = 8 * (l16 & 1);
    const int r_lo = 8 * lg + (l16 >> 2), r_hi = r_lo + 4;
    nb_lo = r_lo * C::NN_RB + 16 * (cl ^ nn_swz<BN>(r_lo)) + half8;
    nb_hi = r_hi * C::NN_RB + 16 * (cl ^ nn_swz<BN>(r_hi)) + half8;
  }

  // STAGES-deep ring: stage k lives in slot k mod STAGES.  Step kt waits for stage kt
  // (the loads of up to STAGES - 2 later stages stay in flight), then refills the slot
  // that step kt - 1 read with stage kt + STAGES - 1.
  // Contraction steps [kb, kb + nk) (all of them unless the contraction is split); step
  // kb + kt lives in ring slot kt mod STAGES.
  int kb = 0, nk = P.K / BK;
  if (EPI == EPI_ACC && P.k_splits > 1) {
    const int all = nk;
    kb = split * all / P.k_splits;
    nk = (split + 1) * all / P.k_splits - kb;
  }
#pragma unroll
  for (int st = 0; st < STAGES - 1; ++st)
    if (st < nk) dma_stage(st, (kb + st) * BK);
  for (int kt = 0; kt < nk; ++kt) {
    wait_ahead<STAGES - 2, C::LOADS>(nk - 1 - kt);  // (later stages stay in flight)
    __syncthreads();  // stage kt resident; every wave is past step kt-1
    const lds_char* SA = Ls + (kt % STAGES) * C::STAGE;
    const lds_char* SB = SA + C::A_BYTES;
    // Operands of substep s into set s % 2.
    u32x4 a[2][TM], b[2][TNB];
    auto read_sub = [&](int s) __attribute__((always_inline)) {
      const int xo = opa ^ (64 * s), q = s & 1;
#pragma unroll
      for (int i = 0; i < TM; ++i) a[q][i] = lds_read16(SA + (wm * C::WM + 16 * i) * 128 + xo);
#pragma unroll
      for (int j = 0; j < TNB; ++j) {
        if constexpr (NN) {
          const int cx = 2 * (wn * C::WN + 16 * j);
          const u32x2 lo = lds_read_tr(SB + 32 * s * C::NN_RB + (nb_lo ^ cx));
          const u32x2 hi = lds_read_tr(SB + 32 * s * C::NN_RB + (nb_hi ^ cx));
          b[q][j] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        } else {
          const int brow = (j / TN) * BN + wn * C::WN + 16 * (j % TN);  // panel j / TN
          b[q][j] = lds_read16(SB + brow * 128 + xo);
        }
      }
    };
    // The first substep's operand reads go out before the refill, so their LDS latency
    // overlaps the issue of the next stage's loads.
    read_sub(0);
    if (kt + STAGES - 1 < nk)
      dma_stage((kt + STAGES - 1) % STAGES, (kb + kt + STAGES - 1) * BK);
#pragma unroll
    for (int s = 0; s < BK / 32; ++s) {
      if (s + 1 < BK / 32) read_sub(s + 1);
      const int q = s & 1;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
          acc[i][j] = mfma16(a[q][i], b[q][j], acc[i][j]);
    }
    // Issue order: the operand reads of k-substep s+1 are spread between the MFMAs of
    // substep s (R / M per MFMA, one more for the first R mod M), so LDS latency hides
    // behind matrix work.
    {
      constexpr int R = TM + (NN ? 2 : 1) * TNB;  // LDS reads per substep
      constexpr int M = TM * TNB;                          // MFMAs per substep
      constexpr int RM = R / M;
      __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
#pragma unroll
      for (int s = 0; s < BK / 32; ++s)
#pragma unroll
        for (int i = 0; i < M; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (s + 1 < BK / 32) {
            if (i < R % M) __builtin_amdgcn_sched_group_barrier(0x100, RM + 1, 0);
            else if (RM > 0) __builtin_amdgcn_sched_group_barrier(0x100, RM, 0);
          }
        }
    }
  }
  __syncthreads();  // operand stages are free for the epilogue

  gemm_epilogue<C, EPI>(P, acc, L, wave, lane, m0, n0, wm, wn, split);
}

// Work index w of a product P on tiles of K -> output tile and contraction range (ranges
// outermost).
template <class K>
__device__ __forceinline__ void work_tile(const GemmParams& P, const int w, int* m0, int* n0,
                                          int* split) {
  const int tiles_m = (P.M + K::BM - 1) / K::BM, tiles_n = (P.N + K::BN - 1) / K::BN;
  int wt = w, tm, tn;
  *split = 0;
  if (K::EPI == EPI_ACC && P.k_splits > 1) {
    *split = w / (tiles_m * tiles_n);
    wt = w - *split * tiles_m * tiles_n;
  }
  tile_coords(wt, tiles_m, tiles_n, &tm, &tn);
  *m0 = tm * K::BM;
  *n0 = tn * K::BN;
}

// The tiles of gemm_tile as a kernel configuration.
template <int BM_, int BN_, int WGM, int WGN, bool NN_, int EPI_, int STAGES>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, EPI = EPI_, THREADS = kWave * WGM * WGN;
  static constexpr bool NN = NN_;
  static constexpr int LDS_BYTES = Cfg<BM_, BN_, WGM, WGN, NN_, EPI_, STAGES>::LDS_BYTES;
  static __device__ __forceinline__ void run(const GemmParams& P, int m0, int n0, int split,
                                             char* L) {
    gemm_tile<BM, BN, WGM, WGN, NN, EPI, STAGES>(P, m0, n0, split, L);
  }
};

// ------------------------------------------------------------------ alternating tiles
// The barrier that ends a slot of both tiles below: nothing moves across it.
__device__ __forceinline__ void swap_slot() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// 256 x 256 accumulators (SwiGLU: 256 x 128 gate and as many up) on 8 wavefronts, each
// 128 x 64, in which the two wavefronts of a SIMD take turns: while one issues the MFMAs
// of a quarter of its K step (64 x 32 of its output, 256 matrix cycles), the other reads
// the operands of its next quarter and issues loads, and a barrier swaps the roles.  With
// both free to run (gemm_tile) they stop together at the step's barrier, at its wait for
// the next stage and at its first operand reads, and the matrix pipe stops with them.
//
// What bounds it: on operands of zeros it is the issue schedule (gate+up 4096 x 57344 x
// 8192: 1674 TFLOP/s with gemm_tile, 1979 with this schedule on 32 x 32 x 16 MFMAs, 1941 on
// 16 x 16 x 32), on real data the power limit, which lowers the clock: there the schedule
// alone gained nothing (1309 and 1310) and the MFMA shape decides.  A 16 x 16 x 32 MFMA
// reads and writes half the accumulator bytes per product of a 32 x 32 x 16 one: 1458
// TFLOP/s.  Same for the [K, N] operand (down, 4096 x 8192 x 28672): 1148, 1278, 1325.
//
// LDS: every operand panel of a 64-deep stage is two units of 16 KB (A0, A1: the first and
// second 64 rows of each wavefront row's 128; B0, B1: each wavefront's first and second 32
// columns), two stages of each.  A unit is refilled as soon as both wavefront groups
// hold it in registers, one unit per quarter, so a load has five quarters (1.25 steps,
// about 2600 cycles) to arrive and the CU's load path is asked for 16 KB at a time instead
// of a whole stage at once.
//
// Quarters of step k, with F = B(k mod 2) and S the other B unit (alternating, so that the
// F of the next step can be read into registers while the last quarter still uses S's
// successor):
//            operands   MEM reads   MEM loads (unit of stage)
//   Q0       A0 x F     A0          A1 of k + 1
//   Q1       A0 x S     S           F  of k + 2
//   Q2       A1 x S     A1          A0 of k + 2
//   Q3       A1 x F     F' of k+1   S  of k + 2
// where F' = B((k + 1) mod 2).  Order of the slots (X: wavefronts 0-3, Y: 4-7, one of each
// per SIMD): X MEM(Q0) | X MFMA(Q0), Y MEM(Q0) | X MEM(Q1), Y MFMA(Q0) | ...  A unit read
// in X's slot t and Y's slot t + 1 is in registers by the barrier that ends slot t + 2 (both
// wait for their LDS reads before their MFMAs), and its refill is issued in slot t + 4 at
// the earliest.  B0 of the first step, read before slot 0 by both and refilled in slot 2, has a
// wait of its own in Y.  A unit read in slot t (X) was waited for by every wavefront in its MEM
// slot before, i.e. ahead of the barrier that ends slot t - 1: five units are issued after
// it by then, two loads each per wavefront, hence vmcnt(10).
// MULTI: the contraction may have several parts or be split into ranges ([K, N] operands,
// accumulate epilogue).
template <bool NN_, int EPI_, bool MULTI = false>
struct PpTile {
  static constexpr bool NN = NN_;
  static constexpr int EPI = EPI_;
  static constexpr bool SW = EPI == EPI_SWIGLU;
  static constexpr int BM = 256, BN = SW ? 128 : 256, WGM = 2, WGN = 4;
  static constexpr int WAVES = 8, THREADS = kWave * WAVES;
  static constexpr int WM = 128, WN = SW ? 32 : 64, TM = 4, TN = WN / 16;
  // NN units are 128 consecutive columns, so a wavefront's second 32 columns are 128 on.
  static constexpr int COL_WN = NN ? 32 : WN, COL_BLK = NN ? 128 : 32;
  static_assert(!MULTI || (NN && EPI == EPI_ACC), "multi-part contractions");
  static constexpr int UNIT = 128 * BK * 2;
  static constexpr int LDS_BYTES = 8 * UNIT;  // A units [stage parity][half], then B units
  static __device__ __forceinline__ void run(const GemmParams& P, int m0, int n0, int split,
                                             char* L);
};

template <bool NN_, int EPI_, bool MULTI>
__device__ __forceinline__ void PpTile<NN_, EPI_, MULTI>::run(const GemmParams& P, const int m0,
                                                              const int n0, const int split,
                                                              char* L) {
  using C = PpTile<NN_, EPI_, MULTI>;
  lds_char* Ls = (lds_char*)L;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  // Contraction steps [kb, kb + nk); step kt of the tile lives in slot kt mod 2.
  int kb = 0, nk = P.K / BK;
  if (MULTI && P.k_splits > 1) {
    const int all = nk;
    kb = split * all / P.k_splits;
    nk = (split + 1) * all / P.k_splits - kb;
  }

  // Per-lane load offsets.  Load i (of two) of a unit: LDS rows 8 (8 i + wave) + lane / 8
  // for 128-byte rows, 4 (8 i + wave) + lane / 16 for the 256-byte rows of an NN unit.
  uint32_t off_a[2][2], off_b[2][2];
  int kr[2];  // NN: this lane's k row in the unit
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = 8 * (8 * i + wave) + (lane >> 3), pc = (lane & 7) ^ nt_swz(r);
    const int rn = 4 * (8 * i + wave) + (lane >> 4), pn = (lane & 15) ^ nn_swz<128>(rn);
    kr[i] = rn;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t ga = (uint32_t)min(m0 + (r >> 6) * 128 + u * 64 + (r & 63), P.M - 1);
      off_a[u][i] = 2u * (ga * (uint32_t)P.lda + 8u * (uint32_t)pc);
      if constexpr (NN) {
        const uint32_t gn = (uint32_t)min(n0 + 128 * u + 8 * pn, P.N - 8);
        off_b[u][i] = 2u * ((uint32_t)rn * (uint32_t)P.ldb + gn);
      } else {
        const int col = SW ? r : (r >> 5) * 64 + u * 32 + (r & 31);
        const uint32_t gb = (uint32_t)min(n0 + col, P.N - 1);
        off_b[u][i] = 2u * (gb * (uint32_t)P.ldb + 8u * (uint32_t)pc);
      }
    }
  }
  // The stages in load order: a cursor over the parts of a multi-part contraction (operand
  // pair and column within it), whose operands are chosen from scalar registers whenever a
  // part ends.  A1 of a stage is loaded after the cursor has moved on for the other units,
  // so the stage's A resource and column are kept for it.
  int k_part = INT_MAX, cur_part = 0, cur_k = kb * BK;
  rsrc_t rs_a = make_rsrc(P.A), rs_b = make_rsrc(P.B);
  const rsrc_t rs_b2 = make_rsrc(SW ? P.B2 : P.B);
  rsrc_t cur_a = rs_a;
  uint32_t a_k0 = 0;
  int b_k0 = 0;
  auto set_part = [&]() __attribute__((always_inline)) {
    if constexpr (MULTI) {
      const uint16_t* pa = P.A_part[0];
      const uint16_t* pb = P.B_part[0];
#pragma unroll
      for (int i = 1; i < kGemmPartsMax; ++i) {
        pa = cur_part == i ? P.A_part[i] : pa;
        pb = cur_part == i ? P.B_part[i] : pb;
      }
      cur_a = make_rsrc(pa);
      rs_b = make_rsrc(pb);
    }
  };
  if (MULTI && P.n_parts > 1) {
    k_part = P.k_part;
    cur_part = cur_k / k_part;
    cur_k -= cur_part * k_part;
    set_part();
  }
  auto next_stage = [&]() __attribute__((always_inline)) {
    if (MULTI && cur_k >= k_part) {
      cur_k = 0;
      ++cur_part;
      set_part();
    }
    rs_a = cur_a;
    a_k0 = (uint32_t)cur_k;
    b_k0 = cur_k;
    cur_k += BK;
  };
  // Unit u of the stage into slot S.
  auto load_a = [&](auto slot, auto half) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value, U = decltype(half)::value;
    lds_char* dst = Ls + (2 * S + U) * UNIT + wave * 1024;
#pragma unroll
    for (int i = 0; i < 2; ++i) dma16(rs_a, off_a[U][i], 2u * a_k0, dst + i * 8192);
  };
  auto load_b = [&](auto slot, auto half) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value, U = decltype(half)::value;
    lds_char* dst = Ls + (4 + 2 * S + U) * UNIT + wave * 1024;
    if constexpr (NN) {
      if (b_k0 + BK <= P.Kb_rows) {
        const uint32_t soff = 2u * (uint32_t)b_k0 * (uint32_t)P.ldb;
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16(rs_b, off_b[U][i], soff, dst + i * 8192);
      } else {  // rows past Kb_rows repeat the last one
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int gk = min(b_k0 + kr[i], P.Kb_rows - 1);
          dma16(rs_b, off_b[U][i] + 2u * (uint32_t)(gk - kr[i]) * (uint32_t)P.ldb, 0u,
                dst + i * 8192);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        dma16(SW && U == 1 ? rs_b2 : rs_b, off_b[U][i], 2u * (uint32_t)b_k0, dst + i * 8192);
    }
  };

  // Operand reads (slots and units are immediates).  A and NT B: row 16 x + lane % 16 of a
  // unit, chunk 4 t + lane / 16 of contraction step t (32 indices).  NN B: transpose reads
  // of k rows 32 t + 8 (lane / 16) + .. at 16 columns.
  int ra[2], rb[2], nb[2][2];
  {
    const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int op = l16 * 128 + 16 * ((4 * t + g) ^ nt_swz(l16));
      ra[t] = wm * 64 * 128 + op;
      rb[t] = 4 * UNIT + wn * 32 * 128 + op;
    }
    if constexpr (NN) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = 8 * g + 4 * h + (l16 >> 2), cl = (l16 & 3) >> 1;
#pragma unroll
        for (int j = 0; j < 2; ++j)
          nb[j][h] = 4 * UNIT + r * 256 + 16 * ((4 * wn + 2 * j + cl) ^ nn_swz<128>(r)) + 8 * (l16 & 1);
      }
    }
  }
  u32x4 a[2][4][2], b[2][2][2];  // [unit][16-row / column block][contraction step]
  auto read_a = [&](auto slot, auto half) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value, U = decltype(half)::value;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[U][i][t] = lds_read16(Ls + ra[t] + ((2 * S + U) * UNIT + i * 16 * 128));
  };
  auto read_b = [&](auto slot, auto half) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value, U = decltype(half)::value;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if constexpr (NN) {
          const u32x2 lo = lds_read_tr(Ls + nb[j][0] + ((2 * S + U) * UNIT + t * 32 * 256));
          const u32x2 hi = lds_read_tr(Ls + nb[j][1] + ((2 * S + U) * UNIT + t * 32 * 256));
          b[U][j][t] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        } else {
          b[U][j][t] = lds_read16(Ls + rb[t] + ((2 * S + U) * UNIT + j * 16 * 128));
        }
      }
  };
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // Ends a MEM slot, issues the quarter's MFMAs and ends their slot.  The wait for the LDS
  // reads comes before the MFMAs in every quarter, also where they are for the next step:
  // the units' refills rely on it.
  auto quarter = [&](auto half_a, auto half_b) __attribute__((always_inline)) {
    constexpr int UA = decltype(half_a)::value, UB = decltype(half_b)::value;
    swap_slot();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[4 * UA + i][2 * UB + j] =
              mfma16(a[UA][i][t], b[UB][j][t], acc[4 * UA + i][2 * UB + j]);
    __builtin_amdgcn_s_setprio(0);
    swap_slot();
  };
  // Step in slot S (F = B unit S) with `left` steps left, this one included: the last two
  // have nothing (or only A1 of the last) to load and wait for what is still in flight.
  auto step = [&](auto slot, const int left) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value;
    constexpr Ic<S> s{};
    constexpr Ic<1 - S> o{};
    constexpr Ic<0> i0{};
    constexpr Ic<1> i1{};
    read_a(s, i0);
    if (left >= 2) {
      load_a(o, i1);
      wait_dma<10>();
    } else {
      wait_dma<0>();
    }
    quarter(i0, s);
    read_b(s, o);
    if (left >= 3) {
      next_stage();
      load_b(s, s);
      wait_dma<10>();
    } else if (left == 2) {
      wait_dma<8>();
    }
    quarter(i0, o);
    read_a(s, i1);
    if (left >= 3) {
      load_a(s, i0);
      wait_dma<10>();
    } else if (left == 2) {
      wait_dma<6>();
    }
    quarter(i1, o);
    read_b(o, o);  // (the last step reads a unit it does not use)
    if (left >= 3) {
      load_b(s, o);
      wait_dma<10>();
    } else if (left == 2) {
      wait_dma<4>();
    }
    quarter(i1, s);
  };

  constexpr Ic<0> s0{};
  constexpr Ic<1> s1{};
  next_stage();
  load_b(s0, s0);
  load_a(s0, s0);
  load_b(s0, s1);
  load_a(s0, s1);
  if (nk > 1) {
    next_stage();
    load_b(s1, s1);
    load_a(s1, s0);
    load_b(s1, s0);
    wait_dma<10>();
  } else {
    wait_dma<4>();
  }
  swap_slot();  // B0 and A0 of step 0 resident
  read_b(s0, s0);
  if (wave >= 4) {
    // Y runs one slot behind X, so its first MFMA slot's wait for LDS reads lies behind two
    // barriers, and X refills B0 right after the second.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    swap_slot();
  }
  for (int left = nk; left > 0; left -= 2) {
    step(s0, left);
    if (left > 1) step(s1, left - 1);
  }
  if (wave < 4) swap_slot();
  __syncthreads();  // operand units are free for the epilogue

  gemm_epilogue<C, EPI>(P, acc, L, wave, lane, m0, n0, wm, wn, split);
}

// SwiGLU backward on the alternating schedule: 128 x 128 tiles of G = X W1^T, U = X W3^T and
// dHs = dY W2^T on 8 wavefronts, each 64 x 32 of all three.  A 64-deep stage is five units
// (X, dY, W1, W3, W2: 128 rows each), two stages of each fill the LDS; a step has one slot per
// product, X staying in registers for two of them:
//            operands    MEM reads   MEM loads (unit of stage)
//   Q0       dY x W2     dY, W2      W1, X of k + 1
//   Q1       X x W1      X, W1       W3    of k + 1
//   Q2       X x W3      W3          dY, W2 of k + 2
// with the slot order, the refill rule and the wait of PpTile (five units are issued after
// the one that the next quarter reads: vmcnt(10), a lead of four quarters).  It is bound by
// the CU's load path (80 KB per 1536 matrix cycles: 5 units per 3 blocks of 128 x 128, where
// PpTile loads 4 per 4): with the waits loosened it runs as long, without the loads 30 %
// less.  7B, S_loc = 8192, 4 shards a launch: 1060 us against 1207 for a two-slot ring with a
// barrier per step, which asked for a whole stage at once.
struct PpBwdTile {
  static constexpr bool NN = false;
  static constexpr int EPI = EPI_SWIGLU_BWD;
  static constexpr int BM = 128, BN = 128, WGM = 2, WGN = 4, WAVES = 8, THREADS = kWave * WAVES;
  static constexpr int WM = 64, WN = 32, TM = 2, TN = WN / 16;
  static constexpr int COL_WN = WN, COL_BLK = 32;
  static constexpr int UNIT = 128 * BK * 2;
  static constexpr int LDS_BYTES = 10 * UNIT;  // [X, dY, W1, W3, W2][stage parity]
  static __device__ __forceinline__ void run(const GemmParams& P, int m0, int n0, int split,
                                             char* L);
};

__device__ __forceinline__ void PpBwdTile::run(const GemmParams& P, const int m0, const int n0, int,
                                               char* L) {
  using C = PpBwdTile;
  lds_char* Ls = (lds_char*)L;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int nk = P.K / BK;

  enum { X = 0, Y = 1, W1 = 2, W3 = 3, W2 = 4 };
  // Load i (of two) of a unit: LDS rows 8 (8 i + wave) + lane / 8.
  uint32_t off_a[2], off_b[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = 8 * (8 * i + wave) + (lane >> 3), pc = (lane & 7) ^ nt_swz(r);
    off_a[i] = 2u * ((uint32_t)min(m0 + r, P.M - 1) * (uint32_t)P.lda + 8u * (uint32_t)pc);
    off_b[i] = 2u * ((uint32_t)min(n0 + r, P.N - 1) * (uint32_t)P.ldb + 8u * (uint32_t)pc);
  }
  const rsrc_t rs[5] = {make_rsrc(P.A), make_rsrc(P.A2), make_rsrc(P.B), make_rsrc(P.B2),
                        make_rsrc(P.B3)};
  // Unit u of stage k into slot S.
  auto load = [&](auto unit, auto slot, int k) __attribute__((always_inline)) {
    constexpr int U = decltype(unit)::value, S = decltype(slot)::value;
    lds_char* dst = Ls + (2 * U + S) * UNIT + wave * 1024;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      dma16(rs[U], U == X || U == Y ? off_a[i] : off_b[i], 2u * (uint32_t)(k * BK),
            dst + i * 8192);
  };
  // Operand reads as in PpTile; W2's units are out of reach of the 16-bit immediate offset.
  int ra[2], rb[2], rb2[2];
  {
    const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int op = l16 * 128 + 16 * ((4 * t + g) ^ nt_swz(l16));
      ra[t] = wm * 64 * 128 + op;
      rb[t] = 2 * W1 * UNIT + wn * 32 * 128 + op;
      rb2[t] = 2 * W2 * UNIT + wn * 32 * 128 + op;
    }
  }
  u32x4 ax[4][2], ay[4][2], b1[2][2], b3[2][2], b2[2][2];
  auto read_a = [&](auto unit, auto slot, u32x4 (&a)[4][2]) __attribute__((always_inline)) {
    constexpr int U = decltype(unit)::value, S = decltype(slot)::value;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[i][t] = lds_read16(Ls + ra[t] + ((2 * U + S) * UNIT + i * 16 * 128));
  };
  auto read_b = [&](auto unit, auto slot, u32x4 (&b)[2][2]) __attribute__((always_inline)) {
    constexpr int U = decltype(unit)::value, S = decltype(slot)::value;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        b[j][t] = U == W2 ? lds_read16(Ls + rb2[t] + (S * UNIT + j * 16 * 128))
                          : lds_read16(Ls + rb[t] + ((2 * (U - W1) + S) * UNIT + j * 16 * 128));
  };
  f32x4 acc[4][6];  // [16-row block][G, U, dHs x 16-column block]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 6; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Ends a MEM slot, issues product `panel`'s MFMAs and ends their slot.
  auto quarter = [&](auto panel, u32x4 (&a)[4][2], u32x4 (&b)[2][2]) __attribute__((always_inline)) {
    constexpr int PN = decltype(panel)::value;
    swap_slot();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][2 * PN + j] = mfma16(a[i][t], b[j][t], acc[i][2 * PN + j]);
    __builtin_amdgcn_s_setprio(0);
    swap_slot();
  };
  // Step k in slot S = k mod 2, `left` steps left, this one included.
  auto step = [&](auto slot, const int k, const int left) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value;
    constexpr Ic<S> s{};
    constexpr Ic<1 - S> o{};
    read_a(Ic<Y>{}, s, ay);
    read_b(Ic<W2>{}, s, b2);
    if (left >= 2) {
      load(Ic<W1>{}, o, k + 1);
      load(Ic<X>{}, o, k + 1);
      wait_dma<10>();
    } else {
      wait_dma<2>();
    }
    quarter(Ic<2>{}, ay, b2);
    read_a(Ic<X>{}, s, ax);
    read_b(Ic<W1>{}, s, b1);
    if (left >= 2) {
      load(Ic<W3>{}, o, k + 1);
      wait_dma<10>();
    } else {
      wait_dma<0>();
    }
    quarter(Ic<0>{}, ax, b1);
    read_b(Ic<W3>{}, s, b3);
    if (left >= 3) {
      load(Ic<Y>{}, s, k + 2);
      load(Ic<W2>{}, s, k + 2);
      wait_dma<10>();
    } else if (left == 2) {
      wait_dma<6>();
    }
    quarter(Ic<1>{}, ax, b3);
  };

  constexpr Ic<0> s0{};
  constexpr Ic<1> s1{};
  load(Ic<Y>{}, s0, 0);
  load(Ic<W2>{}, s0, 0);
  load(Ic<W1>{}, s0, 0);
  load(Ic<X>{}, s0, 0);
  load(Ic<W3>{}, s0, 0);
  if (nk > 1) {
    load(Ic<Y>{}, s1, 1);
    load(Ic<W2>{}, s1, 1);
    wait_dma<10>();
  } else {
    wait_dma<6>();
  }
  swap_slot();                  // dY and W2 of step 0 resident
  if (wave >= 4) swap_slot();  // wavefronts 4-7 run one slot behind
  for (int k = 0; k < nk; k += 2) {
    step(s0, k, nk - k);
    if (k + 1 < nk) step(s1, k + 1, nk - k - 1);
  }
  if (wave < 4) swap_slot();
  __syncthreads();  // operand units are free for the epilogue

  gemm_epilogue<C, EPI>(P, acc, L, wave, lane, m0, n0, wm, wn);
}

template <class K>
__global__ __launch_bounds__(K::THREADS) void gemm_kernel(const GemmParams P) {
  const int tiles = ((P.M + K::BM - 1) / K::BM) * ((P.N + K::BN - 1) / K::BN);
  const int items = K::EPI == EPI_ACC && P.k_splits > 1 ? tiles * P.k_splits : tiles;
  __shared__ __attribute__((aligned(1024))) char L[K::LDS_BYTES];
  int m0, n0, split;
  work_tile<K>(P, xcd_work_index(blockIdx.x, items), &m0, &n0, &split);
  K::run(P, m0, n0, split, L);
}

// Y = base + sum of the k_splits partial products in range order (base and U as in the
// accumulate epilogue); 4 consecutive columns per thread.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmParams P) {
  const int c4 = P.N / 4;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)P.M * c4) return;
  const int m = (int)(i / c4), n = 4 * (int)(i - (long long)m * c4);
  const size_t mn = (size_t)P.M * P.N, at = (size_t)m * P.N + n;
  f32x4 sum = *reinterpret_cast<const f32x4*>(P.part + at);
  for (int c = 1; c < P.k_splits; ++c) sum += *reinterpret_cast<const f32x4*>(P.part + c * mn + at);
  f32x4 base = f32x4{0.f, 0.f, 0.f, 0.f};
  if (P.R) {
    const u32x2 r = *reinterpret_cast<const u32x2*>(P.R + (size_t)m * P.ldr + n);
    base = f32x4{bf16_bits_to_f32(r[0] & 0xffffu), bf16_bits_to_f32(r[0] >> 16),
                 bf16_bits_to_f32(r[1] & 0xffffu), bf16_bits_to_f32(r[1] >> 16)};
  } else if (P.accumulate) {
    base = *reinterpret_cast<const f32x4*>(P.Y + (size_t)m * P.ldy + n);
  }
  const f32x4 out = sum + base;
  *reinterpret_cast<f32x4*>(P.Y + (size_t)m * P.ldy + n) = out;
  if (P.U)
    *reinterpret_cast<u32x2*>(P.U + (size_t)m * P.ldu + n) =
        u32x2{pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3])};
}

// Up to kGemmGroupMax independent products of one configuration in one launch: the tiles of
// product i follow those of the products before it, so small products that would each
// leave CUs idle fill the chip together.
struct GemmGroup {
  GemmParams p[kGemmGroupMax];
  int n;
};
static_assert(sizeof(GemmGroup) <= 4096, "kernel argument size limit");
// Tiles of K in each product of G; returns their total.
template <class K>
__device__ __forceinline__ int group_tiles(const GemmGroup& G, int (&tiles)[kGemmGroupMax]) {
  int total = 0;
#pragma unroll
  for (int i = 0; i < kGemmGroupMax; ++i) {
    tiles[i] = i < G.n ? ((G.p[i].M + K::BM - 1) / K::BM) * ((G.p[i].N + K::BN - 1) / K::BN) : 0;
    total += tiles[i];
  }
  return total;
}

template <class K>
__global__ __launch_bounds__(K::THREADS) void gemm_group_kernel(const GemmGroup G) {
  __shared__ __attribute__((aligned(1024))) char L[K::LDS_BYTES];
  int tiles[kGemmGroupMax];
  const int total = group_tiles<K>(G, tiles);
  int w = xcd_work_index(blockIdx.x, total), i = 0;
  while (i + 1 < G.n && w >= tiles[i]) w -= tiles[i++];  // uniform per workgroup
  // A copy of the product's parameters: read through G.p[i] (an index into the kernel
  // arguments), the compiler reloads every field after each global store of the epilogue
  // (it cannot rule out aliasing), hundreds of serialized scalar loads per tile.
  const GemmParams P = G.p[i];
  int m0, n0, split;
  work_tile<K>(P, w, &m0, &n0, &split);
  K::run(P, m0, n0, split, L);
}

// The same with the tiles from n_big on cut in two row halves of Small tiles, which follow the
// others in dispatch order: the last, partly filled round of the chip then costs a round of
// the smaller tiles.
template <class Big, class Small>
__global__ __launch_bounds__(Big::THREADS) void gemm_mixed_group_kernel(const GemmGroup G,
                                                                        const int n_big) {
  static_assert(Big::THREADS == Small::THREADS && Big::BM == 2 * Small::BM &&
                    Big::BN == Small::BN, "halves");
  constexpr int kLds = Big::LDS_BYTES > Small::LDS_BYTES ? Big::LDS_BYTES : Small::LDS_BYTES;
  __shared__ __attribute__((aligned(1024))) char L[kLds];
  int tiles[kGemmGroupMax];
  const int total = group_tiles<Big>(G, tiles);
  const int b = blockIdx.x;
  const bool big = b < n_big;
  const int q = big ? 0 : xcd_work_index(b - n_big, 2 * (total - n_big));
  int w = big ? xcd_work_index(b, n_big) : n_big + (q >> 1), i = 0;
  while (i + 1 < G.n && w >= tiles[i]) w -= tiles[i++];
  const GemmParams P = G.p[i];
  int m0, n0, split;
  work_tile<Big>(P, w, &m0, &n0, &split);
  if (big) {
    Big::run(P, m0, n0, split, L);
    return;
  }
  m0 += (q & 1) * Small::BM;
  if (m0 < P.M) Small::run(P, m0, n0, split, L);
}

template <class K>
hipError_t check_params(const GemmParams& p) {
  if (p.K <= 0 || p.K % BK != 0) return hipErrorInvalidValue;
  // The operand loads address each operand with 32-bit byte offsets from its base.
  constexpr long long kMaxBytes = 1LL << 32;
  const long long b_rows = K::NN ? (long long)p.Kb_rows : (long long)p.N;
  if ((long long)p.M * p.lda * 2 >= kMaxBytes || b_rows * p.ldb * 2 >= kMaxBytes)
    return hipErrorInvalidValue;
  if (p.k_splits > 1 && (K::EPI != EPI_ACC || !p.part || p.N % 4 != 0 || p.k_splits > p.K / BK))
    return hipErrorInvalidValue;
  if (p.n_parts > 1) {
    if (!K::NN || p.n_parts > kGemmPartsMax || p.k_part <= 0 || p.k_part % BK != 0 ||
        (long long)p.n_parts * p.k_part != p.K)
      return hipErrorInvalidValue;
    for (int i = 0; i < p.n_parts; ++i)
      if (!p.A_part[i] || !p.B_part[i]) return hipErrorInvalidValue;
  }
  return hipSuccess;
}

// The products of one grouped launch, and the number of their tiles.  A grouped product has one
// part and one contraction range (the grouped tiles read neither).
template <class K>
hipError_t fill_group(const GemmParams* ps, int n, GemmGroup* g, long long* tiles) {
  if (n < 1 || n > kGemmGroupMax) return hipErrorInvalidValue;
  *tiles = 0;
  for (int i = 0; i < n; ++i) {
    const GemmParams& p = ps[i];
    if (p.M <= 0 || p.N <= 0 || p.n_parts > 1 || p.k_splits > 1) return hipErrorInvalidValue;
    const hipError_t e = check_params<K>(p);
    if (e != hipSuccess) return e;
    g->p[i] = p;
    *tiles += (long long)((p.M + K::BM - 1) / K::BM) * ((p.N + K::BN - 1) / K::BN);
  }
  g->n = n;
  return *tiles > INT32_MAX / 2 ? hipErrorInvalidValue : hipSuccess;
}

template <class K>
hipError_t launch_group(const GemmParams* ps, int n, hipStream_t s) {
  GemmGroup g = {};
  long long total = 0;
  const hipError_t e = fill_group<K>(ps, n, &g, &total);
  if (e != hipSuccess) return e;
  void* args[] = {&g};
  return hipLaunchKernel(reinterpret_cast<const void*>(&gemm_group_kernel<K>),
                         dim3((unsigned)total), dim3(K::THREADS), args, 0, s);
}

// n_big tiles of Big, the rest halved (gemm_mixed_group_kernel).
template <class Big, class Small>
hipError_t launch_mixed_group(const GemmParams* ps, int n, long long n_big, hipStream_t s) {
  GemmGroup g = {};
  long long total = 0;
  const hipError_t e = fill_group<Big>(ps, n, &g, &total);
  if (e != hipSuccess) return e;
  if (n_big > total) return hipErrorInvalidValue;
  int nb = (int)n_big;
  void* args[] = {&g, &nb};
  return hipLaunchKernel(reinterpret_cast<const void*>(&gemm_mixed_group_kernel<Big, Small>),
                         dim3((unsigned)(n_big + 2 * (total - n_big))), dim3(Big::THREADS), args,
                         0, s);
}

template <class K>
hipError_t launch(const GemmParams& p, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  const hipError_t e = check_params<K>(p);
  if (e != hipSuccess) return e;
  long long tiles = (long long)((p.M + K::BM - 1) / K::BM) * ((p.N + K::BN - 1) / K::BN);
  if (K::EPI == EPI_ACC && p.k_splits > 1) tiles *= p.k_splits;
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  // hipLaunchKernel returns the status of this launch only (not an earlier error).
  void* args[] = {const_cast<GemmParams*>(&p)};
  return hipLaunchKernel(reinterpret_cast<const void*>(&gemm_kernel<K>),
                         dim3((unsigned)tiles), dim3(K::THREADS), args, 0, s);
}

long long tiles_of(const GemmParams* ps, int n, int bm, int bn) {
  long long t = 0;
  for (int i = 0; i < n && i < kGemmGroupMax; ++i)
    t += (long long)((ps[i].M + bm - 1) / bm) * ((ps[i].N + bn - 1) / bn);
  return t;
}

}  // namespace

// Tile choice.  The alternating 256 x 256 tiles have the best rate once they fill the chip;
// smaller ones spread a product over more CUs.  A launch's time goes in rounds of one
// workgroup per CU, so the alternating tiles are taken when their rounds cost no more than
// those of the 128 x 128 tiles, with the measured ratio of one round to the other:
//   gate+up (K = 4096): 86-89 and 55-57 us, 1.55 (S_loc = 2048: 268 us against 329; 1024: 173
//     and 171; M = 1024 rows of one 7B shard leave the last of 1.4 rounds 60 % empty)
//   Q/K/V and weight gradients, whose 128 x 128 tiles run two to a CU: 90-104 and 33-42 us,
//     2.7 (Q/K/V at S_loc = 1024, 192 tiles of 256: 97 us against 127; two thirds of it, 128
//     tiles: 86 against 72)
constexpr long long kCus = 256;

long long rounds(long long tiles) { return (tiles + kCus - 1) / kCus; }

// Up to 64 tiles of 128 x 128 the 64 x 64 ones still fit the chip in one round and quarter
// the work of each CU, with a five-stage ring in place of two stages: a small product is
// bound by the latency of its chain of loads (S_loc = 128, h = 256: down projection, 12
// steps on one 256 x 256 tile 24 us, on 64 x 64 tiles 9.7).  From 65 to 256 tiles of 128 x 128 a
// CU holds one, and gives it a four-stage ring (Q of 8 shards, 1024 x 512 x 4096 each: 69 us
// with two stages, 50 with four); above, two per CU hide each other's waits.
constexpr long long kSmallTiles = 64;

hipError_t launch_gemm_swiglu_group(const GemmParams* ps, int n, hipStream_t s) {
  const long long big = tiles_of(ps, n, 256, 128), t128 = tiles_of(ps, n, 128, 128);
  if (t128 <= kSmallTiles)
    return launch_group<Tile<64, 64, 2, 2, false, EPI_SWIGLU, 3>>(ps, n, s);
  // Whole rounds of the alternating tiles with the last, partial one on halved tiles, when
  // that makes one round (7B, S_loc = 1024: 352 tiles, 176 -> 157 us; 700: 264 tiles, 179 -> 156).
  const long long full = big / kCus, rest = big - full * kCus;
  if (full > 0 && rest > 0 && 2 * rest <= kCus &&
      155 * full + 100 < std::min(155 * rounds(big), 100 * rounds(t128)))
    return launch_mixed_group<PpTile<false, EPI_SWIGLU>,
                              Tile<128, 128, 2, 4, false, EPI_SWIGLU, 3>>(ps, n, full * kCus, s);
  if (155 * rounds(big) <= 100 * rounds(t128))
    return launch_group<PpTile<false, EPI_SWIGLU>>(ps, n, s);
  return launch_group<Tile<128, 128, 2, 4, false, EPI_SWIGLU, 3>>(ps, n, s);
}

namespace {

// Accumulate products with few output tiles: the tile and the number of contraction ranges
// (through fp32 partial products and a second kernel) that together take the least time,
// from the measured time of a 64-deep step on each tile and of moving the partials.
enum NnTile { kNn256, kNn128, kNn64 };
struct NnPlan {
  NnTile tile;
  int splits;
};
NnPlan nn_acc_plan(int M, int N, int K, bool may_split = true) {
  const long long t256 = (long long)((M + 255) / 256) * ((N + 255) / 256);
  if (t256 <= 0 || t256 >= kCus || N % 4 != 0) return {kNn256, 1};
  // Most ranges: enough (tile, range) items of 256 x 256 for every CU with at least 16 steps
  // per range (the partials' workspace is sized by the choice, so it is bounded by that too).
  const int steps = K / BK;
  const int most = may_split ? std::max(1, (int)std::min((kCus + t256 - 1) / t256,
                                                         (long long)(steps / 16)))
                             : 1;
  // us of a step with one workgroup on every CU, and with two where they fit (64 x 64).
  constexpr struct {
    NnTile tile;
    int bm;
    double step_us;
  } kTiles[] = {{kNn256, 256, 1.5}, {kNn128, 128, 0.75}, {kNn64, 64, 0.42}};
  NnPlan best = {kNn256, 1};
  double best_us = -1.0;
  for (const auto& t : kTiles) {
    const long long tiles = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bm - 1) / t.bm);
    for (int n = 1; n <= most; ++n) {
      const long long items = tiles * n, per_cu = t.tile == kNn64 ? 2 : 1;
      // full rounds of per_cu workgroups (two take 1.5 times one's time), then what is left
      const long long full = items / (kCus * per_cu), rest = items - full * kCus * per_cu;
      const double passes = full * (per_cu == 2 ? 1.5 : 1.0) +
                            (rest == 0 ? 0.0 : (rest > kCus ? 1.5 : 1.0));
      const double us = passes * ((steps + n - 1) / n * t.step_us + 2.0) +
                        (n > 1 ? 5.0 + 2.0 * n * M * N * 4 / 4.5e6 : 0.0);
      if (best_us < 0 || us < best_us) {
        best_us = us;
        best = {t.tile, n};
      }
    }
  }
  return best;
}

}  // namespace

int gemm_nn_acc_splits(int M, int N, int K) { return nn_acc_plan(M, N, K).splits; }

hipError_t launch_gemm_nn_acc(const GemmParams& p, float* part, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  const NnPlan plan = nn_acc_plan(p.M, p.N, p.K, part != nullptr);
  GemmParams q = p;
  q.k_splits = plan.splits;
  q.part = part;
  hipError_t e;
  if (plan.tile == kNn256)
    e = launch<PpTile<true, EPI_ACC, true>>(q, s);
  else if (plan.tile == kNn128)
    e = launch<Tile<128, 128, 2, 4, true, EPI_ACC, 4>>(q, s);
  else
    e = launch<Tile<64, 64, 2, 2, true, EPI_ACC, 5>>(q, s);
  if (e != hipSuccess || plan.splits == 1) return e;
  const long long threads = (long long)p.M * (p.N / 4);
  void* args[] = {&q};
  return hipLaunchKernel(reinterpret_cast<const void*>(&splitk_reduce_kernel),
                         dim3((unsigned)((threads + 255) / 256)), dim3(256), args, 0, s);
}

// SwiGLU backward (M = S_loc, N = F/D).  Long launches are cut in two: over many rounds the
// workgroups of an XCD drift apart and share fewer operand panels in its L2, while short ones
// need all products to fill the chip (S_loc = 1024: 704 tiles, 332 us).  One launch of 8
// products against two of 4, us, by the rounds of the one (a card, two runs within 1 %):
//   7B   5.5: 695, 665   8.3: 964, 971   11: 1219, 1192   12.4: 1374, 1287   13.8: 1449, 1373
//        16.5: 1796, 1721   19.3: 2088, 1942   22: 2350, 2140
//   13B  7: 1043, 1071   14: 2023, 1899   21: 3001, 2861
//   70B  7: 1429, 1533   10.5: 2167, 2334   14: 2819, 2723   21: 4216, 4192
// so beyond 12 rounds two win everywhere (1 to 9 %); up to 11 it depends on how full each half's
// last round is.
int gemm_swiglu_bwd_per_launch(const GemmParams* ps, int n) {
  return n > 4 && rounds(tiles_of(ps, n, 128, 128)) > 12 ? (n + 1) / 2 : n;
}

hipError_t launch_gemm_swiglu_bwd_group(const GemmParams* ps, int n, hipStream_t s) {
  for (int i = 0; i < n; ++i)
    if (ps[i].ldt % 8 != 0 || ps[i].ldt < ps[i].M) return hipErrorInvalidValue;
  return launch_group<PpBwdTile>(ps, n, s);
}

// Weight gradients (M = F/D or H_s d, N = h, K = tokens), several products in one launch.
hipError_t launch_gemm_nn_acc_group(const GemmParams* ps, int n, hipStream_t s) {
  const long long big = tiles_of(ps, n, 256, 256), t128 = tiles_of(ps, n, 128, 128);
  if (t128 <= kSmallTiles) return launch_group<Tile<64, 64, 2, 2, true, EPI_ACC, 5>>(ps, n, s);
  if (27 * rounds(big) <= 10 * rounds(t128)) return launch_group<PpTile<true, EPI_ACC>>(ps, n, s);
  if (t128 <= kCus) return launch_group<Tile<128, 128, 2, 4, true, EPI_ACC, 4>>(ps, n, s);
  return launch_group<Tile<128, 128, 2, 4, true, EPI_ACC, 2>>(ps, n, s);
}

hipError_t launch_gemm_qkv_group(const GemmParams* ps, int n, hipStream_t s) {
  const long long big = tiles_of(ps, n, 256, 256), t128 = tiles_of(ps, n, 128, 128);
  if (t128 <= kSmallTiles) return launch_group<Tile<64, 64, 2, 2, false, EPI_QKV, 5>>(ps, n, s);
  if (27 * rounds(big) <= 10 * rounds(t128)) return launch_group<PpTile<false, EPI_QKV>>(ps, n, s);
  if (t128 <= kCus) return launch_group<Tile<128, 128, 2, 4, false, EPI_QKV, 4>>(ps, n, s);
  return launch_group<Tile<128, 128, 2, 4, false, EPI_QKV, 2>>(ps, n, s);
}

}  // namespace tsp
