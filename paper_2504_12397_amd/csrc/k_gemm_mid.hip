// bf16 MFMA GEMM of 128-row tiles:  C[M,N] = A[M,K] B[N,K]^T for calls whose 256 x 256 tiles (k_gemm_large.hip) would leave much of
// the chip idle, or all but a little of a further round.  Tiles of 128 x 64, 96, 128, 192 or 256, one running sum over K (or over a segment of it): every accumulator starts
// from the gated low-rank term and adds its k-steps of 16 in ascending order, as the other projection kernels do.  A workgroup walks its tiles one after the other.
//
// What bounds it: LDS.  Four waves multiply, one per SIMD, a wave 64 x 64, 96 or 128 (32 x 64 and 32 x 96 in the tiles of 64 and 96): 96 KB of fragments for a
// k-tile (64 wide) of 128 x 256 where eight waves of 64 x 64 read 128, at about 140 bytes per clock and compute unit.  A wave is alone on its SIMD, so
// the reads of a k-step run beside the matrix instructions of the one before, over the barrier too: a k-tile's last fragments are in registers
// when its buffer is handed back, and the next one's first are read under the last products.  Four more waves only move tiles from memory to LDS
// (buffer_load ... lds), two (256 columns) to five (64) k-tiles ahead.  Apart, because a wave's loads complete in order: the low-rank term's loads would wait for
// the tiles.  (Lines of k-tiles further ahead asked for by a wave of their own, for the L2: up to 1.5 x slower, its scattered requests cost more
// than the misses.)
// Against the tiles of eight waves of 128 x 128 and 128 x 256 that it replaces (kernel trace, us): QKV with rotation and append, 1024 rows of eight rank-64 adapters
// 78 -> 62 (256 tiles of 192 columns where 192 of 256 left a quarter of the chip idle), 1024 rows of four rank-32 adapters in turn 90 -> 71, 512 rows 54 -> 43;
// W_o of 1024 rows 43 both.  Against the kernels of few rows: 139 rows of QKV 33 -> 25; W_o and W_down in as many segments: see gemm_few_plan.
//
// LDS: rows of 128 bytes (8 chunks of 16), chunk c of row i at position c ^ ((i >> 1) & 7): the rows that a fragment read serves together lie in
// different banks.
#include "lds_dma.h"

namespace alora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// BN columns; NB blocks of 32 columns and MB of 32 rows per wave
template <int BN_> struct MidTile {
  static constexpr int BM = 128, BN = BN_, WN = BN < 128 ? 1 : 2, NB = BN / 32 / WN, MB = BN < 128 ? 1 : 2;
  static constexpr int STAGE = (BM + BN) * 128, NBUF = 160 * 1024 / STAGE;
  static constexpr int NL = 4, R = (BM + BN) / 8 / NL;      // loading waves, their requests for a k-tile
};

template <typename X, int EPI>
__global__ __launch_bounds__(512) void gemm_mid_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int BM = X::BM, BN = X::BN, NB = X::NB, MB = X::MB, NBUF = X::NBUF, R = X::R, STAGE = X::STAGE;
  extern __shared__ u32x4 smem[];
  char *lds = reinterpret_cast<char *>(smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int M = g.M, N = g.N;
  const int nk = g.K / 64 / g.k_splits;
  const int n_out = tiles_m * tiles_n, n_tiles = n_out * g.k_splits;      // (PARTIAL only: several workgroups per output tile)
  // As in k_gemm_large.hip: an XCD takes a contiguous run of tiles, in patches of eight row tiles (1024 rows, as there) by all column tiles.  Every patch reads the weights, which from
  // about 240 MB on no cache holds until the next one does: gate/up of 513 rows in patches of four / so, us: 2 x 13824 x 5120 203 / 174, 2 x 28672 x 8192 595 / 523, 2 x 14336 x 4096 152 / 135.
  const int xcd = blockIdx.x & 7, per_xcd = gridDim.x >> 3;
  const int run0 = xcd * (n_tiles >> 3) + min(xcd, n_tiles & 7), run_n = (n_tiles >> 3) + (xcd < (n_tiles & 7) ? 1 : 0);
  const int in_run = blockIdx.x >> 3;
  if (in_run >= run_n) return;
  struct At { int m0, n0, split; };
  auto tile_at = [&](int i) {
    constexpr int GM = 8;
    const int split = EPI == GEMM_EPI_PARTIAL ? (run0 + i) / n_out : 0, t = run0 + i - split * n_out;
    const int patch = t / (GM * tiles_n), first = patch * GM, gm = min(GM, tiles_m - first), in = t - patch * GM * tiles_n;
    return At{(first + in % gm) * BM, (in / gm) * BN, split};
  };
  // Row of the weights (of gate or of up) that slot `slot` of the block at column n is.  Where columns come in pairs (c and c + 64 of a head, gate and
  // up) a block is 16 of them, first columns in slots 0 to 15 and their partners behind them.
  auto weight_row = [&](int n, int slot) {
    if (EPI == GEMM_EPI_ROPE) { const int p = (n >> 1) + (slot & 15); return min(p + (p & ~63) + (slot >> 4) * 64, N - 1); }
    if (EPI == GEMM_EPI_SWIGLU) return min((n >> 1) + (slot & 15), (N >> 1) - 1);
    return min(n + slot, N - 1);
  };

  if (wave >= 4) {
    // ---- loading waves: every fourth request of 8 rows -----------------------------------------------------------------
    const int lw = wave - 4;
    const i32x4 rA = make_rsrc(g.A, (uint64_t)M * g.lda * 2);
    const i32x4 rB0 = make_rsrc(g.B, (uint64_t)(EPI == GEMM_EPI_SWIGLU ? N >> 1 : N) * g.ldb * 2);
    const i32x4 rB1 = EPI == GEMM_EPI_SWIGLU ? make_rsrc(g.B2, (uint64_t)(N >> 1) * g.ldb * 2) : rB0;
    int vo[R], k0, ti = in_run, t = 0, buf = 0;
    auto aim = [&] {
      const At at = tile_at(ti);
      k0 = at.split * nk * 128;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int i = 8 * (lw + 4 * j) + (lane >> 3), c = (lane & 7) ^ ((i >> 1) & 7), ib = i - BM;      // (a request is of A or of B)
        if (8 * 4 * j < BM) vo[j] = (min(at.m0 + i, M - 1) * g.lda + c * 8) * 2;
        else vo[j] = (weight_row(at.n0 + (ib & ~31), ib & 31) * g.ldb + c * 8) * 2;
      }
    };
    auto req = [&] {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int q = lw + 4 * j;
        load_to_lds(8 * 4 * j < BM ? rA : (EPI == GEMM_EPI_SWIGLU && ((8 * q - BM) & 16)) ? rB1 : rB0, vo[j], k0 + t * 128, buf * STAGE + q * 1024);
      }
      buf = buf + 1 == NBUF ? 0 : buf + 1;
      if (++t == nk) {      // (behind the last tile its first k-tiles again, which nobody reads)
        t = 0;
        if (ti + per_xcd < run_n) { ti += per_xcd; aim(); }
      }
    };
    aim();
    for (int s = 0; s < NBUF - 1; ++s) req();
    for (int i = in_run; i < run_n; i += per_xcd)
      for (int s = 0; s < nk; ++s) {
        wait_vm<(NBUF - 2) * R>();      // the k-tile is there (as far as this wave moves it)
        wave_barrier();                 // ... and the one before it is used up
        req();
      }
    wait_vm<0>();
    return;
  }

  // ---- multiplying waves ----------------------------------------------------------------------------------------------
  const int wm = wave / X::WN, wn = wave % X::WN;
  int ra[4], rb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int pos = ((2 * ks + lhi) ^ ((l32 >> 1) & 7)) * 16;
    ra[ks] = (wm * MB * 32 + l32) * 128 + pos;
    rb[ks] = (BM + wn * NB * 32 + l32) * 128 + pos;
  }
  int buf = 0;
  struct Frag { bf16x8 a[MB], b[NB]; };
  auto read = [&](int ks, Frag &f) {
    const char *p = lds + buf * STAGE;
#pragma unroll
    for (int i = 0; i < MB; ++i) f.a[i] = *reinterpret_cast<const bf16x8 *>(p + ra[ks] + i * 4096);
#pragma unroll
    for (int j = 0; j < NB; ++j) f.b[j] = *reinterpret_cast<const bf16x8 *>(p + rb[ks] + j * 4096);
  };
  for (int it = in_run; it < run_n; it += per_xcd) {
    const At at = tile_at(it);
    const int row0 = at.m0 + wm * MB * 32, col0 = at.n0 + wn * NB * 32;      // of this wave
    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // ---- gated low-rank term (Eq.6), under the first tiles' way from memory --------------------------------------------
    // A step is LS slices of 16 values of k, of t_hi and of t_lo, against B of one adapter (other adapters' rows zeroed); the adapters of this
    // wave's rows pass slice by slice, so that t is fetched once.  What counts is the number of requests: a lane's 16 bytes lie in a row of
    // their own, and a request of 64 of them keeps the unit that looks up addresses for 64 clocks.  B of AHEAD - 1 steps is on its way.
    if (g.tlow != nullptr && (EPI != GEMM_EPI_PARTIAL || at.split == 0) && row0 < M) {
      constexpr int LS = MB * NB > 4 ? 1 : 2, AHEAD = NB == 4 ? 2 : 3;      // (registers)
      const int row_end = min(M, row0 + 32 * MB);
      unsigned long long present = 0ull;
      if (g.present16 != nullptr) {
        for (int t = row0 / 16; t < (row_end + 15) / 16; ++t) present |= g.present16[t];
      } else {
        const int a = row0 + lane < row_end ? g.row_adapter[row0 + lane] : -1;
        present = a >= 0 ? 1ull << a : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
          present |= ((unsigned long long)__shfl_xor((int)(present >> 32), o, 64) << 32) | (uint32_t)__shfl_xor((int)present, o, 64);
      }
      const int r = g.rank;
      int a_row[MB], kind[NB];      // part of a block's columns (gate and up share a block: of a lane's)
      const bf16 *trow[MB], *brow[NB];
      int64_t a_stride[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int row = row0 + i * 32 + l32, rc = min(row, M - 1);
        a_row[i] = row < M ? g.row_adapter[rc] : -1;
        trow[i] = g.tlow + (int64_t)rc * g.lr_parts * 2 * r;
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int w = weight_row(col0 + 32 * j, l32);
        if (EPI == GEMM_EPI_SWIGLU) {
          kind[j] = l32 >> 4;
          brow[j] = (kind[j] ? g.Bk : g.Bq) + (int64_t)w * r;
          a_stride[j] = (int64_t)(N >> 1) * r;
        } else {
          kind[j] = __builtin_amdgcn_readfirstlane(w < g.n_q ? 0 : (w < g.n_q + g.n_kv ? 1 : 2));
          brow[j] = kind[j] == 0 ? g.Bq + (int64_t)w * r : (kind[j] == 1 ? g.Bk + (int64_t)(w - g.n_q) * r : g.Bv + (int64_t)(w - g.n_q - g.n_kv) * r);
          a_stride[j] = (int64_t)(kind[j] == 0 ? g.n_q : g.n_kv) * r;
        }
      }
      const int part_end = !present ? 0 : EPI == GEMM_EPI_SWIGLU ? 2 : kind[NB - 1] + 1;
      for (int part = EPI == GEMM_EPI_SWIGLU ? 0 : kind[0]; part < part_end; ++part) {
        u32x4 t[LS][2][MB], b[AHEAD][LS][NB];
        auto at_k = [&](int ks, int i) { return min(ks + 16 * i + lhi * 8, r - 8); };
        auto fetch_t = [&](int ks) {
#pragma unroll
          for (int i = 0; i < LS; ++i)
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
#pragma unroll
              for (int m = 0; m < MB; ++m) t[i][hl][m] = *reinterpret_cast<const u32x4 *>(trow[m] + (part * 2 + hl) * r + at_k(ks, i));
        };
        auto fetch_b = [&](unsigned long long left, int ks, u32x4 (&f)[LS][NB]) {
#pragma unroll
          for (int i = 0; i < LS; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              f[i][j] = *reinterpret_cast<const u32x4 *>(brow[j] + (int64_t)__builtin_ctzll(left) * a_stride[j] + at_k(ks, i));
        };
        auto apply = [&](unsigned long long left, int ks, u32x4 (&f)[LS][NB]) {
          const int a = (int)__builtin_ctzll(left);
#pragma unroll
          for (int i = 0; i < LS; ++i) {
            if (ks + 16 * i >= r) continue;
#pragma unroll
            for (int j = 0; j < NB; ++j)
              if (kind[j] != part || ks + 16 * i + lhi * 8 >= r) f[i][j] = u32x4{0, 0, 0, 0};      // (ranks that are not a multiple of 16)
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
#pragma unroll
              for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                  acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                      __builtin_bit_cast(bf16x8, f[i][j]), __builtin_bit_cast(bf16x8, a_row[m] == a ? t[i][hl][m] : u32x4{0, 0, 0, 0}), acc[m][j], 0, 0, 0);
          }
        };
        auto advance = [&](unsigned long long &left, int &ks) {      // (behind the last step nothing is left)
          left &= left - 1;
          if (!left) { ks += 16 * LS; left = ks < r ? present : 0ull; }
        };
        unsigned long long left = present, ask = present;      // to multiply, to ask for
        int ks = 0, ask_ks = 0;
        fetch_t(0);
#pragma unroll
        for (int i = 0; i < AHEAD - 1; ++i)
          if (ask) { fetch_b(ask, ask_ks, b[i]); advance(ask, ask_ks); }
        while (left) {
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) {
            if (!left) break;
            if (ask) { fetch_b(ask, ask_ks, b[(i + AHEAD - 1) % AHEAD]); advance(ask, ask_ks); }
            apply(left, ks, b[i]);
            const int was = ks;
            advance(left, ks);
            if (left && ks != was) fetch_t(ks);
          }
        }
      }
    }

    // ---- main loop ------------------------------------------------------------------------------------------------------
    auto mma = [&](const Frag &f) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    Frag f0, f1;
    wave_barrier();
    read(0, f0);
    for (int s = 0; s < nk; ++s) {
      read(1, f1);
      mma(f0);
      read(2, f0);
      mma(f1);
      read(3, f1);
      mma(f0);
      buf = buf + 1 == NBUF ? 0 : buf + 1;
      wait_lds();      // the reads are done before the barrier hands the k-tile back to the loading waves
      if (s + 1 < nk) {
        wave_barrier();
        read(0, f0);
      }
      mma(f1);
    }

    // ---- epilogues --------------------------------------------------------------------------------------------------------
    // Lane l32 is a row, register 4 q + i of block j its slot 8 q + 4 lhi + i.  Two lanes trade half of two groups of four 16-bit values, so that each
    // has eight neighbours (16 bytes) to store: of groups q and q + 1, columns 8 q + 8 lhi.
    auto join = [&](uint2 q0, uint2 q1) {
      const uint2 give = lhi ? q0 : q1;
      uint2 got;
      got.x = (uint32_t)__shfl_xor((int)give.x, 32, 64);
      got.y = (uint32_t)__shfl_xor((int)give.y, 32, 64);
      return lhi ? u32x4{got.x, got.y, q1.x, q1.y} : u32x4{q0.x, q0.y, got.x, got.y};
    };
    auto pack = [&](const float (&y)[4], bool half) {
      if (half) {
        half4 a;
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = (_Float16)y[i];
        return __builtin_bit_cast(uint2, a);
      }
      bf16x4 a;
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = (bf16)y[i];
      return __builtin_bit_cast(uint2, a);
    };
    int pos[MB];
    int64_t slot[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
      if constexpr (EPI == GEMM_EPI_ROPE) {
        const int rc = min(row0 + m * 32 + l32, M - 1);
        pos[m] = g.rope_pos[rc];
        slot[m] = g.rope_slot[rc];
      }
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const int row = row0 + m * 32 + l32, rc = min(row, M - 1);
      if (row0 + m * 32 >= M) break;
      if constexpr (EPI == GEMM_EPI_ROPE) {
        const float2 *line = g.rope_table + (int64_t)pos[m] * 64 + 4 * lhi;
        float4 cs[NB][2][2];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i) cs[j][q][i] = reinterpret_cast<const float4 *>(line + ((((col0 >> 1) + 16 * j) & 63) + 8 * q))[i];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int p = (col0 >> 1) + 16 * j, col = p + (p & ~63);      // the block's first column
          const int kind = col < g.n_q ? 0 : (col < g.n_q + g.n_kv ? 1 : 2);
          const float qs = kind == 0 ? g.q_scale : 1.0f;
          uint2 lo[2], hi[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float u = acc[m][j][4 * q + i], w = acc[m][j][8 + 4 * q + i];
              const float c = i & 1 ? cs[j][q][i >> 1].z : cs[j][q][i >> 1].x, sn = i & 1 ? cs[j][q][i >> 1].w : cs[j][q][i >> 1].y;
              a[i] = kind == 2 ? u : rope_lo(u, w, c, sn) * qs;
              b[i] = kind == 2 ? w : rope_hi(u, w, c, sn) * qs;
            }
            lo[q] = pack(a, kind == 0);      // queries as fp16 for the MFMA attention kernels
            hi[q] = pack(b, kind == 0);
          }
          const u32x4 l = join(lo[0], lo[1]), h = join(hi[0], hi[1]);
          bf16 *dst = kind == 0 ? g.Qout + (int64_t)row * g.n_q + col
                                : (kind == 1 ? g.cacheK + slot[m] * g.n_kv + col - g.n_q : g.cacheV + slot[m] * g.n_kv + col - g.n_q - g.n_kv);
          if (row < M && col < N) {
            *reinterpret_cast<u32x4 *>(dst + 8 * lhi) = l;
            *reinterpret_cast<u32x4 *>(dst + 8 * lhi + 64) = h;
          }
        }
      } else if constexpr (EPI == GEMM_EPI_SWIGLU) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          uint2 y[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float gv = acc[m][j][4 * q + i], uv = acc[m][j][8 + 4 * q + i];
              v[i] = gv / (1.0f + __expf(-gv)) * uv;
            }
            y[q] = pack(v, false);
          }
          const u32x4 w = join(y[0], y[1]);
          const int col = (col0 >> 1) + 16 * j + 8 * lhi;
          if (row < M && col < (N >> 1)) *reinterpret_cast<u32x4 *>(g.C + (int64_t)row * g.ldc + col) = w;
        }
      } else if constexpr (EPI == GEMM_EPI_PARTIAL) {
        float *dst = g.Cpart + ((int64_t)at.split * M + row) * N + col0 + 4 * lhi;
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (row < M && col0 + 32 * j < N)
              *reinterpret_cast<float4 *>(dst + 32 * j + 8 * q) =
                  make_float4(acc[m][j][4 * q], acc[m][j][4 * q + 1], acc[m][j][4 * q + 2], acc[m][j][4 * q + 3]);
      } else {
        bf16x4 res[NB][4] = {};
        if (g.R != nullptr) {
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              res[j][q] = *reinterpret_cast<const bf16x4 *>(g.R + (int64_t)rc * g.ldc + min(col0 + 32 * j, N - 32) + 8 * q + 4 * lhi);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          uint2 y[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = acc[m][j][4 * q + i] + (float)res[j][q][i];
            y[q] = pack(v, false);
          }
#pragma unroll
          for (int q = 0; q < 4; q += 2) {
            const u32x4 w = join(y[q], y[q + 1]);
            if (row < M && col0 + 32 * j < N) *reinterpret_cast<u32x4 *>(g.C + (int64_t)row * g.ldc + col0 + 32 * j + 8 * q + 8 * lhi) = w;
          }
        }
      }
    }
  }
}

template <int BN, int EPI>
static void launch_cfg(const GemmArgs &g, hipStream_t s) {
  typedef MidTile<BN> X;
  const int tiles_m = (g.M + X::BM - 1) / X::BM, tiles_n = (g.N + BN - 1) / BN;
  const int all = (tiles_m * tiles_n * g.k_splits + 7) & ~7, grid = all < 256 ? all : 256;      // a workgroup per compute unit walks its tiles
  auto kern = gemm_mid_kernel<X, EPI>;
  (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, X::NBUF * X::STAGE);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), X::NBUF * X::STAGE, s, g, tiles_m, tiles_n);
}
template <int BN>
static void launch_epi(const GemmArgs &g, int epi, hipStream_t s) {
  if (epi == GEMM_EPI_ROPE) launch_cfg<BN, GEMM_EPI_ROPE>(g, s);
  else if (epi == GEMM_EPI_SWIGLU) launch_cfg<BN, GEMM_EPI_SWIGLU>(g, s);
  else if (epi == GEMM_EPI_PARTIAL) launch_cfg<BN, GEMM_EPI_PARTIAL>(g, s);
  else launch_cfg<BN, GEMM_EPI_BF16>(g, s);
}

void launch_gemm_mid(const GemmArgs &g, int epi, int cols, hipStream_t s) {
  if (cols == 64) launch_epi<64>(g, epi, s);
  else if (cols == 96) launch_epi<96>(g, epi, s);
  else if (cols == 128) launch_epi<128>(g, epi, s);
  else if (cols == 192) launch_epi<192>(g, epi, s);
  else launch_epi<256>(g, epi, s);
}

}  // namespace alora
