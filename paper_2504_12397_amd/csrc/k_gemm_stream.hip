// Products of few rows with large weights: C[M,N] = A[M,K] W[N,K]^T, the weights streamed past all rows once -- gate/up with
// SwiGLU, W_down (up to 32 rows), the output head, the adapters' down-projections of a layer's tail.  (The QKV projection has
// k_qkv_stream.hip, which keeps one running sum over K.)
//
// What bounds it: reading the weights.  A read-only walk of this kind reads 235 MB in 38 us (6.1 TB/s) when a workgroup per compute
// unit keeps about 128 KB of its rows on the way into LDS and takes them in runs of 256 bytes of many rows or 1 KB of few; all
// workgroups at one offset of their rows costs a fifth of that (they hit the same channels), so a tile starts its walk over K at an
// offset of its own.  (128-byte runs: 4.9 TB/s; through registers, 32 KB on the way per compute unit: 4.1.)
// Four waves move weights (load_to_lds), the others multiply: RW row blocks of 32 x CWV column groups of CB blocks of 32 x
// KW parts of a stage's k.  Their rows come from memory (L2) in operand order, XB - 1 stages ahead.  A tile has as many columns as
// one compute unit has to read, so that there is one round of tiles: 56 pairs of gate and up columns at the 8B-class shape.
//
// us before (k_gemm_mfma.hip: 128 x 128 blocks, weights through registers) -> now, 8B-class shape: gate/up with SwiGLU 49 -> 42 (1 to 32 rows),
// 55 -> 48 (128), 73 -> 60 (160); W_down and its residual 22 and a kernel of 4.7 -> 25.6 (1 to 32 rows); output head of 128256 columns
// 206 -> 177.  Not taken, with the old kernel as quick: W_o (1 row 9.1 there, 9.5 here; 128 rows 13.4 both), W_down of more than 32 rows
// (128 rows 28.7 there, 30.5 here): partial sums either way, and those bound them.
//
// LDS: DEPTH stages of SR rows x RUN bytes; chunk c (16 bytes) of row r of a stage lies at c ^ (r & 15).
#include <algorithm>

#include "lds_dma.h"

namespace alora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// PW: KB of a stage that each of the four loading waves moves
template <int RW_, int CWV_, int KW_, int CB_, int PW_, int EPI_>
struct StreamCfg {
  static constexpr int RW = RW_, CWV = CWV_, KW = KW_, CB = CB_, PW = PW_, EPI = EPI_;
  static constexpr bool PAIRS = EPI == GEMM_EPI_SWIGLU;
  static constexpr int RUN = 256 * KW;                                 // bytes of a row in a stage: 128 values of k per part
  static constexpr int STAGE = PW * 4096, SR = STAGE / RUN, COLS = PAIRS ? SR / 2 : SR;
  static constexpr int DEPTH = 36 / PW < 8 ? 36 / PW : 8;
  static constexpr int NC = RW * CWV * KW, THREADS = 64 * (NC + 4);
  static constexpr int SLOTS = CWV * CB * 32;                          // columns that the matrix instructions cover (the last block may be part of one)
  static constexpr int SLACK = CB == 1 ? 0 : (SLOTS / (PAIRS ? 2 : 1) - COLS) * RUN;      // ... what lies behind the last stage is read for the others
  static constexpr int JOIN = DEPTH * STAGE + SLACK;                   // sums of the parts of k
  static constexpr int LDS = JOIN + (KW - 1) * RW * CWV * CB * 4096;
  static constexpr int XB = RW == 8 ? 2 : (CB > 2 ? 3 : 4);            // operand buffers (registers: 12 waves leave 168 each, 8 leave 256)
  static_assert(SLACK >= 0 && LDS <= 160 * 1024 && DEPTH >= 3, "");
};

// units: tile * segs + segment; a workgroup takes every gridDim.x-th
template <typename X>
__global__ __launch_bounds__(X::THREADS) void gemm_stream_kernel(GemmArgs g, int units, int segs) {
  constexpr int RUN = X::RUN, PW = X::PW, DEPTH = X::DEPTH, CB = X::CB, KW = X::KW, RW = X::RW, COLS = X::COLS, XB = X::XB;
  constexpr bool PAIRS = X::PAIRS;
  extern __shared__ u32x4 smem[];
  char *lds = reinterpret_cast<char *>(smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int M = g.M, K = g.K, n_cols = PAIRS ? g.N >> 1 : g.N, n_k = K * 2 / RUN;
  struct Unit { int tile, seg, s0, n, rot; };      // stages s0 .. s0 + n - 1 of K, from s0 + rot on and round
  auto unit_of = [&](int u) {
    Unit t{u, 0, 0, n_k, 0};
    if (segs > 1) {
      t.tile = (int)((unsigned)u / (unsigned)segs); t.seg = u - t.tile * segs;
      t.s0 = (int)((unsigned)(n_k * t.seg) / (unsigned)segs);
      t.n = (int)((unsigned)(n_k * (t.seg + 1)) / (unsigned)segs) - t.s0;
    }
    t.rot = (int)((unsigned)t.tile % (unsigned)t.n);
    return t;
  };
  auto stage_of = [&](const Unit &t, int i) { const int s = i + t.rot; return t.s0 + (s >= t.n ? s - t.n : s); };

  if (wave >= X::NC) {
    // ---- loading waves ------------------------------------------------------------------------------------------------
    constexpr int LPR = RUN / 16, RPQ = 64 / LPR;      // lanes of a row, rows of a request
    const int lw = wave - X::NC;
    const bool second = PAIRS && lw >= 2;              // rows of a stage: gate columns, then up columns
    const i32x4 r = make_rsrc(second ? g.B2 : g.B, (uint64_t)n_cols * g.ldb * 2);
    int vo[PW], ru = blockIdx.x, ri = 0, slot = 0;
    Unit rt{};
    auto begin = [&] {
      rt = unit_of(ru);
#pragma unroll
      for (int j = 0; j < PW; ++j) {
        const int row = (lw * PW + j) * RPQ + lane / LPR;
        const int col = min(rt.tile * COLS + row - (second ? COLS : 0), n_cols - 1);
        vo[j] = col * g.ldb * 2 + ((lane % LPR) ^ (row & 15)) * 16;
      }
    };
    auto req = [&] {
      const int so = stage_of(rt, ri) * RUN, dst = slot * X::STAGE + lw * (PW * 1024);
#pragma unroll
      for (int j = 0; j < PW; ++j) load_to_lds(r, vo[j], so, dst + j * 1024);
      slot = slot + 1 == DEPTH ? 0 : slot + 1;
      if (ri + 1 < rt.n) ++ri;
      else if (ru + (int)gridDim.x < units) { ru += gridDim.x; ri = 0; begin(); }
      // (past the end: the last stage again, which nobody reads)
    };
    begin();
    for (int s = 0; s < DEPTH - 1; ++s) req();
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
      const int n = unit_of(u).n;
      for (int s = 0; s < n; ++s) {
        wait_vm<(DEPTH - 2) * PW>();      // the stage is there (as far as this wave moves it)
        wave_barrier();                   // ... and the one before it is used up
        req();
      }
      if (KW > 1) wave_barrier();
    }
    wait_vm<0>();
    return;
  }

  // ---- multiplying waves ----------------------------------------------------------------------------------------------
  const int l32 = lane & 31, lhi = lane >> 5;
  const int rw = wave % RW, cc = wave / RW % X::CWV, kw = wave / (RW * X::CWV);
  const int row0 = rw * 32, row = row0 + l32, rc = min(row, M - 1);
  // slot l32 of block b: a column, or gate (0 .. 15) and up (16 .. 31) columns of 16 pairs
  const int first = PAIRS ? cc * CB * 16 + (l32 & 15) : cc * CB * 32 + l32;
  const int srow = (CB == 1 ? min(first, COLS - 1) : first) + (PAIRS ? (l32 >> 4) * COLS : 0);
  constexpr int BLOCK = (PAIRS ? 16 : 32) * RUN;
  // where the slot's operand of step k is: chunks 2 k and 2 k + 1 of the row, so k is bits 5 to 7 of the address.  An offset per step is kept where there
  // are registers; eight row blocks leave none (6 and 4 of them went to scratch, gate/up of 139 rows 62.7 us) and compute it, anew in every stage
  // (61.3; two registers of the tile of 56 pairs still wait in scratch, from one tile to the next).
  int off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) off[i] = srow * RUN + kw * 256 + ((i * 2 + lhi) ^ (srow & 15)) * 16;
  // the row's operands: 16 bytes per 16 values of k, where the matrix instruction wants them (GemmArgs::packed: lane after lane) or in rows
  const u32x4 *ap = reinterpret_cast<const u32x4 *>(g.A) + (g.packed & 1 ? (int64_t)(rc >> 5) * (K / 16) * 64 + (rc & 31) + 32 * lhi : 0);
  const bf16 *ar = g.A + (int64_t)rc * g.lda + lhi * 8;
  const bool idle = RW > 1 && row0 >= M;      // (comes to the barriers only)
  int slot = 0;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const Unit t = unit_of(u);
    u32x4 xr[XB][8];
    auto fetch = [&](int i, u32x4 (&f)[8]) {
      const int k0 = (stage_of(t, min(i, t.n - 1)) * KW + kw) * 8;
      if (g.packed & 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) f[k] = ap[(k0 + k) * 64];
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) f[k] = *reinterpret_cast<const u32x4 *>(ar + (k0 + k) * 16);
      }
    };
#pragma unroll
    for (int i = 0; i < XB - 1; ++i) fetch(i, xr[i]);
    f32x16 acc[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;

    // gated low-rank term (Eq.6): t of the row against the columns of the tile, adapter by adapter; rows of others get exact zeros
    if (g.tlow != nullptr && kw == 0 && t.seg == 0 && row0 < M) {
      const int r = g.rank, a_row = row < M ? g.row_adapter[rc] : -1;
      unsigned long long present = lane == l32 && a_row >= 0 ? 1ull << a_row : 0ull;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1)
        present |= ((unsigned long long)__shfl_xor((int)(present >> 32), o, 64) << 32) | (uint32_t)__shfl_xor((int)present, o, 64);
      const int kind = PAIRS ? l32 >> 4 : 0;
      const bf16 *Bk = kind ? g.Bk : g.Bq;
      int64_t brow[CB];
#pragma unroll
      for (int b = 0; b < CB; ++b) {
        const int c = PAIRS ? (cc * CB + b) * 16 + (l32 & 15) : (cc * CB + b) * 32 + l32;
        brow[b] = (int64_t)min(t.tile * COLS + c, n_cols - 1) * r;
      }
      for (int part = 0; part < (PAIRS ? 2 : 1); ++part)
        for (int ks = 0; ks < r; ks += 16) {
          const int k = min(ks + lhi * 8, r - 8);
          const bool beyond = ks + lhi * 8 >= r;      // (ranks that are not a multiple of 16)
          const bf16 *tp = g.tlow + ((int64_t)rc * g.lr_parts + part) * 2 * r + k;
          const u32x4 none = {0, 0, 0, 0}, th = *reinterpret_cast<const u32x4 *>(tp), tl = *reinterpret_cast<const u32x4 *>(tp + r);
          for (unsigned long long left = present; left; left &= left - 1) {
            const int a = (int)__builtin_ctzll(left);
            const bf16x8 mh = __builtin_bit_cast(bf16x8, a_row == a ? th : none), ml = __builtin_bit_cast(bf16x8, a_row == a ? tl : none);
            u32x4 w[CB];
#pragma unroll
            for (int b = 0; b < CB; ++b) w[b] = *reinterpret_cast<const u32x4 *>(Bk + (int64_t)a * n_cols * r + brow[b] + k);
#pragma unroll
            for (int b = 0; b < CB; ++b) {
              if (kind != part || beyond) w[b] = none;
              acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[b]), mh, acc[b], 0, 0, 0);
              acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[b]), ml, acc[b], 0, 0, 0);
            }
          }
        }
    }

    for (int i0 = 0; i0 < t.n; i0 += XB) {
#pragma unroll
      for (int j = 0; j < XB; ++j) {
        if (i0 + j >= t.n) break;
        fetch(i0 + j + XB - 1, xr[(j + XB - 1) % XB]);
        wave_barrier();
        if (!idle) {
        int at = slot * X::STAGE + off[0];
        if constexpr (RW == 8) asm("" : "+v"(at));      // (not kept from one stage to the next)
        auto of_step = [&](int k) { return lds + (RW == 8 ? at ^ (k * 32) : slot * X::STAGE + off[k]); };
        // (the reads run a step ahead: a wave that multiplies is alone on its SIMD, or has one neighbour)
        bf16x8 f[2][CB];
#pragma unroll
        for (int b = 0; b < CB; ++b) f[0][b] = *reinterpret_cast<const bf16x8 *>(of_step(0) + b * BLOCK);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (k < 7)
#pragma unroll
            for (int b = 0; b < CB; ++b) f[(k + 1) & 1][b] = *reinterpret_cast<const bf16x8 *>(of_step(k + 1) + b * BLOCK);
          if (RW < 8) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < CB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[k & 1][b], __builtin_bit_cast(bf16x8, xr[j][k]), acc[b], 0, 0, 0);
          if (RW < 8) __builtin_amdgcn_sched_barrier(0);
        }
        }
        slot = slot + 1 == DEPTH ? 0 : slot + 1;
        wait_lds();      // the reads are done before the next barrier hands the stage back to the loading waves
      }
    }
    if constexpr (KW > 1) {
      float4 *join = reinterpret_cast<float4 *>(lds + X::JOIN);
      auto at = [&](int p, int b, int q) { return (((p * RW * X::CWV + cc * RW + rw) * CB + b) * 4 + q) * 64 + lane; };
      if (kw > 0) {
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) join[at(kw - 1, b, q)] = make_float4(acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]);
        wait_lds();
      }
      wave_barrier();
#pragma unroll
      for (int p = 0; p < KW - 1; ++p)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {      // (the other parts' waves add too; only part 0 keeps it)
            const float4 v = join[at(p, b, q)];
            acc[b][4 * q] += v.x; acc[b][4 * q + 1] += v.y; acc[b][4 * q + 2] += v.z; acc[b][4 * q + 3] += v.w;
          }
    }
    // lane l32 is a row, register 4 q + i of block b the slot 8 q + 4 lhi + i
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
      for (int q = 0; q < (PAIRS ? 2 : 4); ++q) {
        const int c = (PAIRS ? (cc * CB + b) * 16 : (cc * CB + b) * 32) + 8 * q + 4 * lhi, col = t.tile * COLS + c;
        if (kw > 0 || row >= M || c >= COLS || col >= n_cols) continue;      // (columns come in fours)
        if constexpr (X::EPI == GEMM_EPI_SWIGLU) {
          bf16x4 v;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float gv = acc[b][4 * q + i], uv = acc[b][8 + 4 * q + i];
            v[i] = (bf16)(gv / (1.0f + __expf(-gv)) * uv);
          }
          if (g.packed & 2) *reinterpret_cast<bf16x4 *>(g.C + xh_chunk(row, col >> 3, n_cols, 1) * 8 + (col & 7)) = v;
          else *reinterpret_cast<bf16x4 *>(g.C + (int64_t)row * g.ldc + col) = v;
        } else if constexpr (X::EPI == GEMM_EPI_BF16) {
          bf16x4 v, res{};
          if (g.R != nullptr) res = *reinterpret_cast<const bf16x4 *>(g.R + (int64_t)row * g.ldc + col);
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = (bf16)(acc[b][4 * q + i] + (float)res[i]);
          *reinterpret_cast<bf16x4 *>(g.C + (int64_t)row * g.ldc + col) = v;
        } else {
          *reinterpret_cast<float4 *>(g.Cpart + ((int64_t)t.seg * M + row) * g.N + col) =
              make_float4(acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]);
        }
      }
  }
}

template <typename X>
static void launch_cfg(const GemmArgs &g, int segs, int n_cu, hipStream_t s) {
  const int n_cols = X::PAIRS ? g.N >> 1 : g.N, units = (n_cols + X::COLS - 1) / X::COLS * segs;
  auto kern = gemm_stream_kernel<X>;
  (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, X::LDS);
  hipLaunchKernelGGL(kern, dim3(std::min(units, n_cu)), dim3(X::THREADS), X::LDS, s, g, units, segs);
}

// gate/up: BL = blocks of 16 pairs of a tile of 8 PW pairs
template <int PW, int BL>
static void launch_swiglu(const GemmArgs &g, int n_cu, hipStream_t s) {
  constexpr int C2 = BL % 2 == 0 ? 2 : 1;
  if (g.M <= 32) launch_cfg<StreamCfg<1, BL, 1, 1, PW, GEMM_EPI_SWIGLU>>(g, 1, n_cu, s);
  else if (g.M <= 64) launch_cfg<StreamCfg<2, C2, 1, BL / C2, PW, GEMM_EPI_SWIGLU>>(g, 1, n_cu, s);
  else if (g.M <= 128) launch_cfg<StreamCfg<4, 1, 1, BL, PW, GEMM_EPI_SWIGLU>>(g, 1, n_cu, s);
  else launch_cfg<StreamCfg<8, 1, 1, BL, PW, GEMM_EPI_SWIGLU>>(g, 1, n_cu, s);
}

// The tile height (of `n` choices, in columns) whose rounds over the chip read the fewest columns one after the other; the largest among equals.
static int best_tile(int n_cols, int n_cu, const int *choice, int n) {
  int best = choice[0], least = 0x7fffffff;
  for (int i = 0; i < n; ++i) {
    const int rounds = ((n_cols + choice[i] - 1) / choice[i] + n_cu - 1) / n_cu, cost = rounds * choice[i];
    if (cost <= least) { least = cost; best = choice[i]; }
  }
  return best;
}

// W_down only up to 32 rows and where the reduction comes in whole kilobytes (see above).  gate/up of more than 192 rows where its tiles are one round of more than the smallest:
// us, here / in tiles of 128 rows, 193 rows and 256: 2 x 14336 x 4096 65.7 / 68.5 and 71.8 / 72.7, 2 x 13824 x 5120 78.2 / 96.2 and 84.9 / 101.2, 2 x 6912 x 2560 29.8 / 33.0 and 31.4 / 35.9,
// 2 x 8192 x 2048 27.1 / 26.9 and 29.1 / 29.5; several rounds, 2 x 28672 x 8192: 242 / 236 and 265 / 234 (160 rows 212 / 214); the smallest tiles, 2 x 4096 x 1024: 13.3 / 11.8 and 14.2 / 13.1.
bool gemm_stream_supported(const GemmArgs &g, int epi, int n_cu) {
  const int n_cols = epi == GEMM_EPI_SWIGLU ? g.N >> 1 : g.N;
  const int rows = epi == GEMM_EPI_BF16 ? 32 : epi == GEMM_EPI_SWIGLU && (n_cols <= 16 * n_cu || n_cols > 64 * n_cu) ? 192 : STREAM_ROWS;
  return g.M >= 1 && g.M <= rows && g.K % (epi == GEMM_EPI_BF16 ? 512 : 128) == 0 && n_cols % 4 == 0 &&
         g.rank % 8 == 0 && lds_aligned(g.B) && (epi != GEMM_EPI_SWIGLU || lds_aligned(g.B2)) && g.ldb == g.K &&
         (uint64_t)n_cols * g.K * 2 < (1ull << 31);
}

// segments of a product whose sums leave as fp32 partials: tiles of 64 columns, one round of workgroups
int gemm_stream_segments(const GemmArgs &g, int n_cu, int most) {
  const int tiles = (g.N + 63) / 64, n_k = g.K / 128;
  return std::max(1, std::min(std::min(most, n_k / 4), n_cu / std::max(tiles, 1)));
}

void launch_gemm_stream(const GemmArgs &g, int epi, int n_cu, hipStream_t s) {
  if (epi == GEMM_EPI_SWIGLU) {
    static const int tiles[] = {16, 32, 48, 56, 64};
    switch (best_tile(g.N >> 1, n_cu, tiles, 5)) {
      case 16: launch_swiglu<2, 1>(g, n_cu, s); break;
      case 32: launch_swiglu<4, 2>(g, n_cu, s); break;
      case 48: launch_swiglu<6, 3>(g, n_cu, s); break;
      case 56: launch_swiglu<7, 4>(g, n_cu, s); break;
      default: launch_swiglu<8, 4>(g, n_cu, s); break;
    }
  } else if (epi == GEMM_EPI_BF16) {
    static const int tiles[] = {8, 12, 16, 20, 24, 32};
    switch (best_tile(g.N, n_cu, tiles, 6)) {
      case 8: launch_cfg<StreamCfg<1, 1, 4, 1, 2, GEMM_EPI_BF16>>(g, 1, n_cu, s); break;
      case 12: launch_cfg<StreamCfg<1, 1, 4, 1, 3, GEMM_EPI_BF16>>(g, 1, n_cu, s); break;
      case 16: launch_cfg<StreamCfg<1, 1, 4, 1, 4, GEMM_EPI_BF16>>(g, 1, n_cu, s); break;
      case 20: launch_cfg<StreamCfg<1, 1, 4, 1, 5, GEMM_EPI_BF16>>(g, 1, n_cu, s); break;
      case 24: launch_cfg<StreamCfg<1, 1, 4, 1, 6, GEMM_EPI_BF16>>(g, 1, n_cu, s); break;
      default: launch_cfg<StreamCfg<1, 1, 4, 1, 8, GEMM_EPI_BF16>>(g, 1, n_cu, s); break;
    }
  } else if (g.k_splits == 1 && g.M <= 32) {      // the output head
    launch_cfg<StreamCfg<1, 4, 1, 1, 8, GEMM_EPI_PARTIAL>>(g, 1, n_cu, s);
  } else if (g.M <= 32) {
    launch_cfg<StreamCfg<1, 2, 1, 1, 4, GEMM_EPI_PARTIAL>>(g, g.k_splits, n_cu, s);
  } else if (g.M <= 64) {
    launch_cfg<StreamCfg<2, 2, 1, 1, 4, GEMM_EPI_PARTIAL>>(g, g.k_splits, n_cu, s);
  } else if (g.M <= 128) {
    launch_cfg<StreamCfg<4, 1, 1, 2, 4, GEMM_EPI_PARTIAL>>(g, g.k_splits, n_cu, s);
  } else {
    launch_cfg<StreamCfg<8, 1, 1, 2, 4, GEMM_EPI_PARTIAL>>(g, g.k_splits, n_cu, s);
  }
}

}  // namespace alora
