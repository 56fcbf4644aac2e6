// bf16 MFMA GEMM for many rows:  C[M,N] = A[M,K] B[N,K]^T, one workgroup per output tile and ONE running sum over K (every
// accumulator adds its k-steps of 16 in ascending order, starting from the gated low-rank term).
//
// What bounds it: matrix issue.  A 256 x 256 tile on eight waves of 128 x 64 reads 12 fragments of 16 bytes per lane for 16
// v_mfma_f32_32x32x16_bf16, 0.75 of the LDS time that the 128 x 128 block of four 64 x 64 waves needs, and the tiles go from
// memory to LDS without passing through registers (buffer_load ... lds), which leaves 256 registers per wave to the
// accumulators (128) and to fragments (96).
//
// Pipeline.  A k-tile (64 wide) is four half-tiles of 16 KB: the upper / lower 64 rows of every wave (A0, A1) and its two
// 32-column blocks (B0, B1).  It is consumed in four phases of eight MFMAs per wave, A0B0, A0B1, A1B1, A1B0, so that each phase
// needs one new half (B0, B1, A1, and in the last one the next tile's A0) and every half-tile is dead after one phase: its
// successor of two tiles later is requested in the next phase, six phases (about 3000 clocks) before it is needed.
// The waves form two groups of four, one wave per SIMD each; the second group runs one barrier behind the first, so
// that one group's fragment reads and requests run under the other group's matrix instructions.
//
// LDS: rows of 128 bytes (8 chunks of 16), chunk c of row i at position c ^ ((i >> 1) & 7): 16 consecutive rows of one chunk
// (fragment reads) hit 64 distinct banks.  The requests write LDS linearly, lane after lane, so the permutation is applied to
// the addresses they read from.
#include "lds_dma.h"

namespace alora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int EPI>
__global__ __launch_bounds__(512, 2) void gemm_large_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int BM = 256, BN = 256, BK = 64;
  constexpr int A_HALF = 16384, B_HALF = 16384;      // bytes of a half-tile
  constexpr int BUF = 2 * A_HALF + 2 * B_HALF, NBUF = 2;
  constexpr int NMI = 4;      // 32-row blocks of a wave
  extern __shared__ u32x4 smem[];
  char *lds = reinterpret_cast<char *>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int wm = wave >> 2, wn = wave & 3;
  const int M = g.M, N = g.N, K = g.K;

  const int nk = K / BK / g.k_splits;
  const int n_out = tiles_m * tiles_n, n_tiles = n_out * g.k_splits;      // (PARTIAL only: several workgroups per output tile)
  // Workgroups go round-robin to the 8 XCDs.  An XCD takes a contiguous run of tiles, walked in patches of GM row tiles by all
  // column tiles, so that the workgroups running on it share rows and columns in its L2.  A workgroup takes every
  // (gridDim / 8)-th tile of its XCD's run.
  const int xcd = blockIdx.x & 7, per_xcd = gridDim.x >> 3;
  const int run0 = xcd * (n_tiles >> 3) + min(xcd, n_tiles & 7), run_n = (n_tiles >> 3) + (xcd < (n_tiles & 7) ? 1 : 0);
  int in_run = blockIdx.x >> 3;
  if (in_run >= run_n) return;

  auto tile_at = [&](int i, int &m0, int &n0, int &k0) {
    constexpr int GM = 4;
    const int split = EPI == GEMM_EPI_PARTIAL ? (run0 + i) / n_out : 0, t = run0 + i - split * n_out;
    k0 = split * nk * (BK * 2);
    const int patch = t / (GM * tiles_n), first = patch * GM, gm = min(GM, tiles_m - first), in = t - patch * GM * tiles_n;
    m0 = (first + in % gm) * BM;
    n0 = (in / gm) * BN;
  };

  // ---- requests: wave w moves rows 16 w .. of a half of A and of a half of B -------------------------
  // LDS row i of a half of A is row (i / 64) * 128 + h * 64 + i % 64 of the tile; LDS row i of a half of
  // B is a weight row: plain n0 + 64 (i / 32) + 32 h + i % 32; rotary: the partner column c + 64 of column c in the other half;
  // SwiGLU: half 0 the gate row, half 1 the up row of the same output column.
  const i32x4 rA = make_rsrc(g.A, (uint64_t)M * g.lda * 2);
  const i32x4 rB0 = make_rsrc(g.B, (uint64_t)(EPI == GEMM_EPI_SWIGLU ? N >> 1 : N) * g.ldb * 2);
  const i32x4 rB1 = EPI == GEMM_EPI_SWIGLU ? make_rsrc(g.B2, (uint64_t)(N >> 1) * g.ldb * 2) : rB0;
  // byte offsets of a lane's rows (the k-tile is the scalar offset, so that a row past the end is out of range by its lane
  // offset alone); they move to the next output tile when the last requests of the current one are out
  int va[2][2], vb[2][2], ka[2], kb;      // ka, kb: byte offset of the first k-tile
  auto aim_a = [&](int m0, int k0, int h) {
    ka[h] = k0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = 8 * (2 * wave + j) + (lane >> 3), c = (lane & 7) ^ ((i >> 1) & 7);
      const int r = (i >> 6) * 128 + h * 64 + (i & 63);
      va[h][j] = ((m0 + r) * g.lda + c * 8) * 2;
    }
  };
  auto aim_b = [&](int n0, int k0) {
    kb = k0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = 8 * (2 * wave + j) + (lane >> 3), c = (lane & 7) ^ ((i >> 1) & 7);
      const int row = EPI == GEMM_EPI_SWIGLU ? (n0 >> 1) + i
                      : EPI == GEMM_EPI_ROPE ? n0 + (i >> 6) * 128 + (i & 63)
                                             : n0 + (i >> 5) * 64 + (i & 31);
      vb[0][j] = (row * g.ldb + c * 8) * 2;
      vb[1][j] = vb[0][j] + (EPI == GEMM_EPI_SWIGLU ? 0 : EPI == GEMM_EPI_ROPE ? 64 : 32) * g.ldb * 2;
    }
  };
  // half h of k-tile t (of the output tile aimed at) into the buffer at LDS byte `buf`
  auto req_a = [&](int t, int buf, int h) {
    const int dst = buf + h * A_HALF + wave * 2048;
#pragma unroll
    for (int j = 0; j < 2; ++j) load_to_lds(rA, va[h][j], ka[h] + t * (BK * 2), dst + j * 1024);
  };
  auto req_b = [&](int t, int buf, int h) {
    const int dst = buf + 2 * A_HALF + h * B_HALF + wave * 2048;
#pragma unroll
    for (int j = 0; j < 2; ++j) load_to_lds(h ? rB1 : rB0, vb[h][j], kb + t * (BK * 2), dst + j * 1024);
  };
  int m0, n0, k0;
  tile_at(in_run, m0, n0, k0);
  aim_a(m0, k0, 0);
  aim_a(m0, k0, 1);
  aim_b(n0, k0);
  for (int t = 0; t < NBUF; ++t) {      // in the order of the main loop
    req_a(t, t * BUF, 0);
    req_b(t, t * BUF, 0);
    req_b(t, t * BUF, 1);
    if (t < NBUF - 1) req_a(t, t * BUF, 1);
  }

  int ra[4], rb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int pos = ((2 * ks + lhi) ^ ((l32 >> 1) & 7)) * 16;
    ra[ks] = (wm * 64 + l32) * 128 + pos;
    rb[ks] = 2 * A_HALF + (wn * 32 + l32) * 128 + pos;
  }

  for (;;) {
  f32x16 acc[NMI][2];
#pragma unroll
  for (int i = 0; i < NMI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // first column of the 32-column accumulator block `nb` of this wave, in the weight matrix's rows
  auto col_of = [&](int nb) -> int {
    if (EPI == GEMM_EPI_SWIGLU) return (n0 >> 1) + 32 * wn;
    if (EPI == GEMM_EPI_ROPE) return n0 + (wn >> 1) * 128 + (wn & 1) * 32 + nb * 64;
    return n0 + wn * 64 + nb * 32;
  };
  const int row_base = m0 + wm * (32 * NMI);

  // ---- gated low-rank term (Eq.6), under the first tiles' way from memory ------------------------------------------
  if (g.tlow != nullptr && (EPI != GEMM_EPI_PARTIAL || k0 == 0)) {      // (split 0 carries it)
    unsigned long long present = 0ull;      // of this wave's rows
    const int row_end = min(M, row_base + 32 * NMI);
    if (g.present16 != nullptr) {
      for (int t = row_base / 16; t < (row_end + 15) / 16; ++t) present |= g.present16[t];
    } else {
      for (int r = row_base; r < row_end; r += 64) {
        const int a = r + lane < row_end ? g.row_adapter[r + lane] : -1;
        unsigned long long mine = a >= 0 ? 1ull << a : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
          mine |= ((unsigned long long)__shfl_xor((int)(mine >> 32), o, 64) << 32) | (uint32_t)__shfl_xor((int)mine, o, 64);
        present |= mine;
      }
    }
    const int r = g.rank, parts = g.lr_parts;
    int p_of[2];
    const bf16 *brow[2];
    int64_t a_stride[2];
    bool col_ok[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int colb = col_of(nb), col = colb + l32;
      if (EPI == GEMM_EPI_SWIGLU) {
        p_of[nb] = nb;
        col_ok[nb] = col < (N >> 1);
        brow[nb] = (nb ? g.Bk : g.Bq) + (int64_t)(col_ok[nb] ? col : 0) * r;
        a_stride[nb] = (int64_t)(N >> 1) * r;
      } else {
        p_of[nb] = colb < g.n_q ? 0 : (colb < g.n_q + g.n_kv ? 1 : 2);
        col_ok[nb] = col < N;
        const int cc = col < N ? col : N - 1;
        if (cc < g.n_q) brow[nb] = g.Bq + (int64_t)cc * r;
        else if (cc < g.n_q + g.n_kv) brow[nb] = g.Bk + (int64_t)(cc - g.n_q) * r;
        else brow[nb] = g.Bv + (int64_t)(cc - g.n_q - g.n_kv) * r;
        a_stride[nb] = (int64_t)(p_of[nb] == 0 ? g.n_q : g.n_kv) * r;
      }
    }
    int a_row[NMI];
    const bf16 *trow[NMI];
#pragma unroll
    for (int mi = 0; mi < NMI; ++mi) {
      const int row = row_base + mi * 32 + l32, rc = min(row, M - 1);
      a_row[mi] = row < M ? g.row_adapter[rc] : -1;
      trow[mi] = g.tlow + (int64_t)rc * parts * 2 * r;
    }
    // A step is 16 values of k of t_hi and of t_lo against the same 16 columns of B.  The requests of the next step go out before
    // the matrix instructions of the running one; other adapters' rows are zeroed afterwards.
    constexpr int NP = EPI == GEMM_EPI_SWIGLU ? 2 : 1;      // both blocks of a wave belong to one part, except gate | up
    struct Step { u32x4 b[2], t[2][NMI][NP]; };
    auto fetch = [&](unsigned long long left, int ks, Step &st) {
      const int a = left ? __builtin_ctzll(left) : 0, kk = min(ks + lhi * 8, r - 8);
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) st.b[nb] = *reinterpret_cast<const u32x4 *>(brow[nb] + (int64_t)a * a_stride[nb] + kk);
#pragma unroll
      for (int hl = 0; hl < 2; ++hl)
#pragma unroll
        for (int mi = 0; mi < NMI; ++mi)
#pragma unroll
          for (int p = 0; p < NP; ++p)
            st.t[hl][mi][p] = *reinterpret_cast<const u32x4 *>(trow[mi] + (p_of[p] * 2 + hl) * r + kk);
    };
    auto apply = [&](unsigned long long left, int ks, Step &st) {
      const int a = __builtin_ctzll(left);
      const bool live = ks + lhi * 8 < r;      // (ranks that are not a multiple of 16)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
        if (!col_ok[nb] || !live) st.b[nb] = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int hl = 0; hl < 2; ++hl)
#pragma unroll
        for (int mi = 0; mi < NMI; ++mi) {
#pragma unroll
          for (int p = 0; p < NP; ++p)
            if (a_row[mi] != a) st.t[hl][mi][p] = u32x4{0, 0, 0, 0};
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            acc[mi][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, st.b[nb]),
                                                                  __builtin_bit_cast(bf16x8, st.t[hl][mi][NP == 2 ? nb : 0]), acc[mi][nb], 0, 0, 0);
        }
    };
    auto advance = [&](unsigned long long &left, int &ks) {
      ks += 16;
      if (ks >= r) { ks = 0; left &= left - 1; }
    };
    if (present) {
      Step s0;
      int ks = 0;
      fetch(present, ks, s0);
      if constexpr (NP == 1) {
        Step s1;
        for (;;) {
          unsigned long long left = present;
          int kn = ks;
          advance(left, kn);
          fetch(left, kn, s1);
          apply(present, ks, s0);
          if (!left) break;
          present = left; ks = kn;
          advance(left, kn);
          fetch(left, kn, s0);
          apply(present, ks, s1);
          if (!left) break;
          present = left; ks = kn;
        }
      } else {
        while (present) {
          apply(present, ks, s0);
          advance(present, ks);
          fetch(present, ks, s0);
        }
      }
    }
  }

  // ---- main loop -----------------------------------------------------------------------------------------------
  constexpr int AR = 2;
  bf16x8 fa0[AR][4], fa1[AR][4], fb0[4], fb1[4];
  auto read_a = [&](int buf, int h, bf16x8 (&f)[AR][4]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < AR; ++i)
        f[i][ks] = *reinterpret_cast<const bf16x8 *>(lds + buf + ra[ks] + h * A_HALF + i * 4096);
  };
  auto read_b = [&](int buf, int h, bf16x8 (&f)[4]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) f[ks] = *reinterpret_cast<const bf16x8 *>(lds + buf + rb[ks] + h * B_HALF);
  };
  auto mma = [&](const bf16x8 (&a)[AR][4], const bf16x8 (&b)[4], int mh, int nb) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < AR; ++i)
        acc[mh * AR + i][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[ks], a[i][ks], acc[mh * AR + i][nb], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // end of a memory part: what the next phase reads has arrived as far as this wave's own requests go.  (Its own reads may still
  // be on their way: the matrix part waits for them one by one.)
#define ALORA_TURN(KEEP)                 \
  wait_vm<KEEP>();                       \
  __builtin_amdgcn_sched_barrier(0);     \
  wave_barrier();                        \
  __builtin_amdgcn_sched_barrier(0)
#define ALORA_TURN2()                    \
  __builtin_amdgcn_sched_barrier(0);     \
  wave_barrier();                        \
  __builtin_amdgcn_sched_barrier(0)

  const bool more = in_run + per_xcd < run_n;
  int m_next = m0, n_next = n0, k_next = k0;
  if (more) tile_at(in_run + per_xcd, m_next, n_next, k_next);
  wait_vm<10>();        // A0 and B0 of k-tile 0 are there
  wave_barrier();
  read_a(0, 0, fa0);
  wait_lds();
  if (wm == 1) wave_barrier();      // the second group runs one barrier behind
  wave_barrier();
  // The last k-tiles request the first ones of the workgroup's next output tile, which then arrive under the epilogue; behind the
  // last output tile they request its own first ones again, into buffers that nobody reads any more, so that the count
  // of requests in flight is the same everywhere.
  {
    auto tile = [&](int b, int t1, int t0) {      // buffer b; requests: A1 of k-tile t1, the rest of k-tile t0
      const int buf = b * BUF;
      read_b(buf, 0, fb0);
      req_a(t1, BUF - buf, 1);
      ALORA_TURN(10);
      mma(fa0, fb0, 0, 0);
      ALORA_TURN2();
      read_b(buf, 1, fb1);
      req_a(t0, buf, 0);
      ALORA_TURN(10);
      mma(fa0, fb1, 0, 1);
      ALORA_TURN2();
      read_a(buf, 1, fa1);
      req_b(t0, buf, 0);
      ALORA_TURN(10);
      mma(fa1, fb1, 1, 1);
      ALORA_TURN2();
      read_a(BUF - buf, 0, fa0);
      req_b(t0, buf, 1);
      ALORA_TURN(10);
      mma(fa1, fb0, 1, 0);
      ALORA_TURN2();
    };
    for (int t = 2; t < nk; t += 2) {
      tile(0, t - 1, t);
      tile(1, t, t + 1);
    }
    aim_a(m_next, k_next, 0);
    aim_b(n_next, k_next);
    tile(0, nk - 1, 0);
    aim_a(m_next, k_next, 1);
    tile(1, 0, 1);
  }
  if (wm == 0) wave_barrier();


  // ---- epilogues -------------------------------------------------------------------------------------------------
  // Weights were the first operand: accumulator register v of lane l is row l % 32 of the 32 x 32 block, column
  // 8 (v / 4) + 4 (l / 32) + v % 4.  A lane packs its four neighbouring columns, and each wave turns 32 rows x 64 bytes at a time
  // through 2 KB of LDS of its own into 16-byte accesses to memory: two-byte accesses of the registers as they are took
  // 40 us of a 140 us tile (8131 x 4096 x 4096).
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
  typedef _Float16 half4 __attribute__((ext_vector_type(4)));
  char *st = lds + NBUF * BUF + wave * 2048;
  auto st_at = [&](int i, int chunk) { return st + i * 64 + ((chunk ^ ((i >> 2) & 3)) * 16); };
  auto put = [&](int q, uint2 w) { *reinterpret_cast<uint2 *>(st_at(l32, q) + 8 * lhi) = w; };      // columns 8 q + 4 lhi ..
  const int io_chunk = lane & 3, io_row = lane >> 2;      // the lane's 16 bytes on the way from and to memory: rows io_row, + 16
  auto take = [&](int half) { return *reinterpret_cast<const u32x4 *>(st_at(16 * half + io_row, io_chunk)); };
  const int n_cols = EPI == GEMM_EPI_SWIGLU ? N >> 1 : N;
#pragma unroll
  for (int mi = 0; mi < NMI; ++mi) {
    const int rows0 = row_base + mi * 32;
    if (rows0 >= M) break;
    if constexpr (EPI == GEMM_EPI_ROPE) {
      // block 0 holds column c of a head, block 1 its rotation partner c + 64
      const int colb = n0 + (wn >> 1) * 128;
      const int kind = colb < g.n_q ? 0 : (colb < g.n_q + g.n_kv ? 1 : 2);
      const int row = min(rows0 + l32, M - 1);
      const float4 *tab = reinterpret_cast<const float4 *>(g.rope_table + (int64_t)(kind == 2 ? 0 : g.rope_pos[row]) * 64 +
                                                           (wn & 1) * 32 + 4 * lhi);
      float4 cs[4][2];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i) cs[q][i] = kind == 2 ? make_float4(1.f, 0.f, 1.f, 0.f) : tab[q * 4 + i];
      int64_t slot[2];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int orow = min(rows0 + 16 * half + io_row, M - 1);
        slot[half] = kind == 0 ? orow : g.rope_slot[orow];
      }
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float y[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float u = acc[mi][nb][4 * q + i], w = acc[mi][nb ^ 1][4 * q + i];
            const float c = i & 1 ? cs[q][i >> 1].z : cs[q][i >> 1].x, sn = i & 1 ? cs[q][i >> 1].w : cs[q][i >> 1].y;
            y[i] = kind == 2 ? u : (nb ? rope_hi(w, u, c, sn) : rope_lo(u, w, c, sn)) * (kind == 0 ? g.q_scale : 1.0f);
          }
          if (kind == 0) {      // queries as fp16 for the MFMA attention kernels
            half4 a;
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = (_Float16)y[i];
            put(q, __builtin_bit_cast(uint2, a));
          } else {
            bf16x4 a;
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = (bf16)y[i];
            put(q, __builtin_bit_cast(uint2, a));
          }
        }
        const int hcol = col_of(nb) + io_chunk * 8 - (kind == 0 ? 0 : (kind == 1 ? g.n_q : g.n_q + g.n_kv));
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const u32x4 w = take(half);
          bf16 *dst = kind == 0 ? g.Qout + slot[half] * g.n_q : (kind == 1 ? g.cacheK : g.cacheV) + slot[half] * g.n_kv;
          if (rows0 + 16 * half + io_row < M && colb < N) *reinterpret_cast<u32x4 *>(dst + hcol) = w;
        }
      }
    } else if constexpr (EPI == GEMM_EPI_PARTIAL) {
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {      // 16 columns of fp32
#pragma unroll
          for (int q = 0; q < 2; ++q)
            *reinterpret_cast<float4 *>(st_at(l32, 2 * q + lhi)) =
                make_float4(acc[mi][nb][8 * ch + 4 * q], acc[mi][nb][8 * ch + 4 * q + 1], acc[mi][nb][8 * ch + 4 * q + 2],
                            acc[mi][nb][8 * ch + 4 * q + 3]);
          const int col = col_of(nb) + ch * 16 + io_chunk * 4;
          float *dst = g.Cpart + (int64_t)(k0 / (nk * (BK * 2))) * M * N + col;
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const u32x4 w = take(half);
            const int orow = rows0 + 16 * half + io_row;
            if (orow < M && col < N) *reinterpret_cast<u32x4 *>(dst + (int64_t)orow * N) = w;
          }
        }
    } else {
#pragma unroll
      for (int nb = 0; nb < (EPI == GEMM_EPI_SWIGLU ? 1 : 2); ++nb) {
        const int col = col_of(nb) + io_chunk * 8;
        bf16x4 res[4] = {};
        if (EPI == GEMM_EPI_BF16 && g.R) {      // the residual comes in by the same route and joins the fp32 sum before the one rounding
          u32x4 w[2];
#pragma unroll
          for (int half = 0; half < 2; ++half)
            w[half] = *reinterpret_cast<const u32x4 *>(g.R + (int64_t)min(rows0 + 16 * half + io_row, M - 1) * g.ldc + min(col, N - 8));
#pragma unroll
          for (int half = 0; half < 2; ++half) *reinterpret_cast<u32x4 *>(st_at(16 * half + io_row, io_chunk)) = w[half];
#pragma unroll
          for (int q = 0; q < 4; ++q) res[q] = *reinterpret_cast<const bf16x4 *>(st_at(l32, q) + 8 * lhi);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bf16x4 a;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (EPI == GEMM_EPI_SWIGLU) {
              const float gv = acc[mi][0][4 * q + i], uv = acc[mi][1][4 * q + i];
              a[i] = (bf16)(gv / (1.0f + __expf(-gv)) * uv);
            } else {
              a[i] = (bf16)(acc[mi][nb][4 * q + i] + (float)res[q][i]);
            }
          }
          put(q, __builtin_bit_cast(uint2, a));
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const u32x4 w = take(half);
          const int orow = rows0 + 16 * half + io_row;
          if (orow < M && col < n_cols) *reinterpret_cast<u32x4 *>(g.C + (int64_t)orow * g.ldc + col) = w;
        }
      }
    }
  }
  if (!more) break;
  in_run += per_xcd;
  m0 = m_next;
  n0 = n_next;
  k0 = k_next;
  }
  wait_vm<0>();
}

template <int EPI>
static void launch_cfg(const GemmArgs &g, hipStream_t s) {
  constexpr int BM = 256, BN = 256;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const size_t smem = 2 * (BM + BN) * 128 + 8 * 2048;
  const int all = (tiles_m * tiles_n * g.k_splits + 7) & ~7, grid = all < 256 ? all : 256;      // a workgroup per compute unit walks its tiles
  auto kern = gemm_large_kernel<EPI>;
  (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), smem, s, g, tiles_m, tiles_n);
}

// Rows of A that one launch takes: their byte offsets are 32 bits wide, tiles past the end included.
int gemm_large_slice_rows(int lda) { return (int)(((int64_t)((1ull << 31) / ((uint64_t)lda * 2)) - 512) & ~(int64_t)255); }

// (32-bit byte offsets into both operands; at least four k-tiles per split, in the tiles of 256 rows in pairs; partial sums of one launch only: a
// second one would put its rows where the first one's are)
bool gemm_large_supported(const GemmArgs &g, int epi, int tile_rows) {
  const uint64_t b_rows = epi == GEMM_EPI_SWIGLU ? g.N / 2 : g.N;
  const int slice = gemm_large_slice_rows(g.lda);
  if (!lds_aligned(g.A) || !lds_aligned(g.B) || (epi == GEMM_EPI_SWIGLU && !lds_aligned(g.B2)) || g.lda % 8 != 0 || g.ldb % 8 != 0) return false;
  if (slice < 256 || (epi == GEMM_EPI_PARTIAL && (g.lora_split || g.M > slice))) return false;
  return g.K % ((tile_rows == 128 ? 64 : 128) * g.k_splits) == 0 && g.K >= 256 * g.k_splits && g.N % 32 == 0 && b_rows * g.ldb * 2 < (1ull << 31);
}

// Measured times of the tiles, us: a k-tile with most of the chip idle and with all of it at work (the clock gives way: 1.6 GHz at 0.83 matrix
// utilisation); a tile's prologue and epilogue take about 6.
struct LargeTile { int rows, cols; double idle, busy; };
static const LargeTile large_tiles[] = {
    {128, 64, 0.24, 0.34}, {128, 96, 0.38, 0.48}, {128, 128, 0.44, 0.53}, {128, 192, 0.62, 0.70}, {128, 256, 0.74, 0.86}, {256, 256, 1.1, 1.48}};
static double tile_us(const LargeTile &t, const GemmArgs &g, int sp, int n_cu) {
  const int n = (g.M + t.rows - 1) / t.rows * ((g.N + t.cols - 1) / t.cols) * sp, rounds = (n + n_cu - 1) / n_cu;
  const double load = n < n_cu ? (double)n / n_cu : 1.0;
  return rounds * ((t.idle + (t.busy - t.idle) * load) * (g.K / 64 / sp) + 6.0);
}

// Segments of the reduction (workgroups per output tile) of a product of more than 256 rows.  They are part of what a call returns -- the order in which a row's
// products are added -- so they do not follow the tiles' times when those change: they are the cheapest by the times of `tiles` here, those of when the
// rule was made.  Partial sums cost their bytes there and back and the launch that adds them.
// With the best tile for them W_o (its norm included) and W_down of 257 to 5000 rows are 2.7 % above the best of all cuts and tiles (159 of each, d = 512 to 5120); cut by the times above
// 5.8 % (us, so and as here: 512 rows of 4096 x 4096 39.2 and 36.3, its reduction normalises too; 640 rows of 4096 x 14336 99.5 and 90.0; but 4200 rows 490 and 517).
static int large_segments(int hint, const GemmArgs &g, int n_cu, int most) {
  static const LargeTile tiles[] = {{128, 128, 0.55, 0.60}, {128, 256, 0.65, 1.0}, {256, 256, 1.1, 1.5}};
  int best = 1;
  double best_us = 1e30;
  for (const auto &t : tiles)
    for (int sp = 1; sp <= most; sp *= 2) {
      if ((hint == 2 && (t.rows != 128 || t.cols != 256)) || (hint == 3 && t.rows != 256) || g.K % (128 * sp) != 0 || g.K < 512 * sp) continue;
      double us = tile_us(t, g, sp, n_cu);
      if (sp > 1) us += 5.0 + (double)sp * g.M * g.N * 8.0 / 4.5e6;
      if (us < best_us) { best_us = us; best = sp; }
    }
  return best;
}

// Tile and segments for a product of M rows: for those segments the cheapest tile by its times, with 4 % on those of 128 rows where there are several rounds of them (near a
// tie they lose: gate/up of 1200 rows, 2 x 13824 x 5120, 379 us in tiles of 128 x 192, 353 in 256 x 256).  Over 206 products of QKV and gate/up, 257 to 4300 rows, eight layer shapes: 0.5 % above
// the best tile on average, 12 % at most.
GemmLargePlan gemm_large_plan(int hint, const GemmArgs &g, int n_cu, int max_splits) {
  const int sp = max_splits > 1 ? large_segments(hint, g, n_cu, max_splits) : 1;
  GemmLargePlan best{256, 256, sp};
  double best_us = 1e30;
  for (const auto &t : large_tiles) {
    if ((hint == 2 && (t.rows != 128 || t.cols != 256)) || (hint == 3 && t.rows != 256) || g.K % (128 * sp) != 0 || g.K < 512 * sp) continue;
    double us = tile_us(t, g, sp, n_cu);
    if (t.rows == 128 && (g.M + 127) / 128 * ((g.N + t.cols - 1) / t.cols) * sp > n_cu) us *= 1.04;
    if (us < best_us) { best_us = us; best = GemmLargePlan{t.rows, t.cols, sp}; }
  }
  return best;
}

// The same for 33 to 256 rows; splits = 0: not here.  The segments are those that calls of these rows are cut in whichever kernel takes them
// (gemm_mfma_fixed_segments), so only the tile is chosen: over 220 products of 33 to 256 rows (d = 512 to 8192) 0.4 % above the best tile on average, 10 % at most.
// Up to 64 rows and in two row tiles the tiles of 128 rows are the quicker ones, us between events, k_gemm_mfma.hip and here, with the reduction:
//   N x K           33 rows        64             128            129            256
//   4096 x 4096     19.0 / 17.3    19.7 / 18.5    22.3 / 22.6    25.9 / 25.5    30.9 / 29.6
//   4096 x 14336    29.2 / 29.0    31.9 / 31.4    38.5 / 39.7    46.6 / 43.6    55.5 / 50.9
//   4096 x 11008    35.1 / 26.5    36.6 / 27.4    40.8 / 33.5    38.7 / 33.6    42.9 / 42.4
//   5120 x 13824    42.0 / 34.0    47.3 / 39.9    57.9 / 47.2    59.3 / 52.5    72.6 / 67.3
//   2048 x 8192     18.6 / 14.3    19.9 / 15.6    22.1 / 18.8    21.7 / 20.7    24.6 / 24.9
// One row tile of more than 64 rows stays with the 128 x 128 tiles of k_gemm_mfma.hip where they and their segments are nearly one round.
GemmLargePlan gemm_few_plan(const GemmArgs &g, int n_cu) {
  const int sp = gemm_mfma_fixed_segments(g.N, g.K, n_cu), there = (g.N + 127) / 128 * sp;
  if (g.M > 64 && g.M <= 128 && there <= n_cu && 3 * there > 2 * n_cu) return GemmLargePlan{0, 0, 0};
  GemmLargePlan best{0, 0, 0};
  double best_us = 1e30;
  for (const auto &t : large_tiles) {
    if (t.rows != 128) continue;
    const double us = tile_us(t, g, sp, n_cu);
    if (us < best_us) { best_us = us; best = GemmLargePlan{t.rows, t.cols, sp}; }
  }
  return best;
}

void launch_gemm_large(GemmArgs g, int epi, const GemmLargePlan &plan, hipStream_t s) {
  if (epi != GEMM_EPI_PARTIAL) g.k_splits = 1;
  const int slice = gemm_large_slice_rows(g.lda), M = g.M;
  for (int m = 0; m < M; m += slice) {
    GemmArgs q = g;
    q.M = M - m < slice ? M - m : slice;
    q.A += (int64_t)m * g.lda;
    if (q.C) q.C += (int64_t)m * g.ldc;
    if (q.R) q.R += (int64_t)m * g.ldc;
    if (q.tlow) q.tlow += (int64_t)m * g.lr_parts * 2 * g.rank;
    if (q.row_adapter) q.row_adapter += m;
    if (q.present16) q.present16 += m / 16;
    if (epi == GEMM_EPI_ROPE) { q.rope_pos += m; q.rope_slot += m; q.Qout += (int64_t)m * g.n_q; }
    if (plan.rows == 128) launch_gemm_mid(q, epi, plan.cols, s);
    else if (epi == GEMM_EPI_ROPE) launch_cfg<GEMM_EPI_ROPE>(q, s);
    else if (epi == GEMM_EPI_SWIGLU) launch_cfg<GEMM_EPI_SWIGLU>(q, s);
    else if (epi == GEMM_EPI_PARTIAL) launch_cfg<GEMM_EPI_PARTIAL>(q, s);
    else launch_cfg<GEMM_EPI_BF16>(q, s);
  }
}

}  // namespace alora
