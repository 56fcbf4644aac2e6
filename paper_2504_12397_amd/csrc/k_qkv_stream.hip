// QKV projection of a call with few rows (up to 32 CW per row tile): y = W x_hat + gated low-rank term (Eq.6), rotated and
// appended (Eq.3) in the epilogue, ONE running sum over K per output -- the same sums in the same order as the projection of
// many rows (k_gemm_mid.hip, k_gemm_large.hip), so a base row's keys and values are the same bits whatever call it came in, and an adapted
// row's where t is (the two kernels that compute t add its products over different slices of d).
//
// Any head size that is a multiple of 8, any reduction length that is a multiple of 128.
//
// What bounds it: streaming the weights (50 MB at the 8B-class shape), and from about 64 rows on the rows, which every workgroup
// reads whole.  The reduction is not split, so the chip is filled over the columns alone: a tile is PP <= 16 rotation pairs
// (c, c + h / 2), chosen so that there is about one tile per compute unit (N = 6144: 12 pairs, 256 tiles), and a workgroup keeps
// up to 112 KB of its weight rows on the way.  Four waves do nothing but move weights into an LDS ring (stages of 512
// bytes of every row); CW waves multiply, 32 rows each, and take their rows from memory (L2) in the order of the matrix operand --
// row preparation writes x_hat that way (PrepArgs::packed), 1 KB per operand.  The two kinds of waves are apart because a wave's
// loads complete in order: behind the weights' requests every operand would wait for memory.  (Rows through LDS as well:
// the same up to 128 rows, a quarter slower at 256.)  One row 14.4 us, 64 rows 17 us, 128 rows 23 us, plus 2 us with adapters;
// the weights alone 11.5 us.
//
// LDS ring: weight row r of a stage has 32 chunks of 16 bytes, chunk c at c ^ (r & 15).
#include "lds_dma.h"

namespace alora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

constexpr int QS_DEPTH = 8, QS_K = 256;      // stages in the ring, values of k per stage

// PW: requests of a loading wave per stage (4 waves x PW KB; PP = 4 PW pairs)
template <int CW, int PW>
__global__ __launch_bounds__(64 * (CW + 4)) void qkv_stream_kernel(GemmArgs g, int tiles_m) {
  constexpr int PP = 4 * PW, STAGE = 2 * PP * QS_K * 2;
  extern __shared__ u32x4 smem[];
  char *lds = reinterpret_cast<char *>(smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int M = g.M, K = g.K, n_pairs = g.N >> 1;
  // the row tiles of one column tile follow each other at a distance of 8: same XCD, one copy of the weights in its L2
  const int x = blockIdx.x & 7, q0 = blockIdx.x >> 3, tm = q0 % tiles_m, pair0 = ((q0 / tiles_m) * 8 + x) * PP;
  if (pair0 >= n_pairs) return;
  const int n_stages = (K + QS_K - 1) / QS_K, n_full = K / QS_K;      // (the last stage may be half a one: what it holds beyond K is not used)
  // pair p of a head of 2 h2: columns (p / h2) * 2 h2 + p % h2 and h2 more
  const int h2 = g.head_dim >> 1;
  auto col_of = [&](int p) { const int hd = p / h2; return p + hd * h2; };

  if (wave >= CW) {
    // ---- loading waves: PW KB of every stage each ---------------------------------------------------------------------
    const i32x4 r = make_rsrc(g.B, (uint64_t)g.N * g.ldb * 2);
    int vo[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int row = ((wave - CW) * PW + j) * 2 + lhi;      // row of the stage: first columns, then their partners
      const int p = min(pair0 + row % PP, n_pairs - 1);
      vo[j] = (col_of(p) + (row / PP) * h2) * g.ldb * 2 + ((lane & 31) ^ (row & 15)) * 16;
    }
    auto req = [&](int s) {
      const int so = min(s, n_stages - 1) * (QS_K * 2), dst = (s % QS_DEPTH) * STAGE + (wave - CW) * (PW * 1024);
#pragma unroll
      for (int j = 0; j < PW; ++j) load_to_lds(r, vo[j], so, dst + j * 1024);
    };
    for (int s = 0; s < QS_DEPTH - 1; ++s) req(s);
    for (int s = 0; s < n_stages; ++s) {
      wait_vm<(QS_DEPTH - 2) * PW>();      // stage s is there (as far as this wave moves it)
      wave_barrier();                      // ... and stage s - 1 is used up
      req(s + QS_DEPTH - 1);               // (past the end: the last stage again, which nobody reads)
    }
    wait_vm<0>();
    return;
  }

  // ---- multiplying waves --------------------------------------------------------------------------------------------
  const int row0 = (tm * CW + wave) * 32, row = row0 + l32, rc = min(row, M - 1);
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  // what the epilogue needs of this row
  const int pos = g.rope_pos[rc];
  const int64_t slot = g.rope_slot[rc];
  // column slot l32 of the accumulator: slots 0 .. 15 the first columns of the pairs, 16 .. 31 their partners
  const int my_pair = min(pair0 + min(l32 & 15, PP - 1), n_pairs - 1);
  const int lds_row = min(l32 & 15, PP - 1) + (l32 >> 4) * PP;
  // Operands on their way: XB buffers of eight, half a stage each, three halves ahead (their way takes about a microsecond).  Lanes past
  // the last row ask for that row again: with one row in the call a request is 32 bytes.
  const u32x4 *xp = reinterpret_cast<const u32x4 *>(g.A) + (int64_t)(rc >> 5) * (K / 16) * 64 + (rc & 31) + 32 * lhi;
  constexpr int XB = CW == 8 ? 2 : 4;
  u32x4 xr[XB][8];
  auto fetch = [&](int u, u32x4 (&f)[8]) {
    const u32x4 *p = xp + (int64_t)min(u, K / 128 - 1) * (8 * 64);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = p[i * 64];
  };
#pragma unroll
  for (int u = 0; u < XB - 1; ++u) fetch(u, xr[u]);

  if (g.tlow != nullptr && row0 < M) {
    unsigned long long present = 0ull;
    if (g.present16 != nullptr) {
      for (int t = row0 / 16; t < min(row0 / 16 + 2, (M + 15) / 16); ++t) present |= g.present16[t];
    } else {
      const int a = l32 == lane && row < M ? g.row_adapter[rc] : -1;
      present = a >= 0 ? 1ull << a : 0ull;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1)
        present |= ((unsigned long long)__shfl_xor((int)(present >> 32), o, 64) << 32) | (uint32_t)__shfl_xor((int)present, o, 64);
    }
    const int r = g.rank, a_row = row < M ? g.row_adapter[rc] : -1;
    const int col = col_of(my_pair) + (l32 >> 4) * h2;
    const int kind = col < g.n_q ? 0 : (col < g.n_q + g.n_kv ? 1 : 2);      // q, k or v
    const bf16 *brow = (kind == 0 ? g.Bq + (int64_t)col * r
                                  : (kind == 1 ? g.Bk + (int64_t)(col - g.n_q) * r : g.Bv + (int64_t)(col - g.n_q - g.n_kv) * r));
    const int64_t a_stride = (int64_t)(kind == 0 ? g.n_q : g.n_kv) * r;
    // The columns of one tile may belong to two parts (q | k or k | v): t of every part is multiplied with the columns of that
    // part.  Per 16 values of k first t_hi, then t_lo, as in the other projection kernels; LS such slices at a time, the B of the next
    // AHEAD - 1 adapters asked for: a round trip per adapter would be most of this kernel's time when a decode step runs eight of them
    // (eight rows of eight rank-64 adapters: 25.0 -> 22.9 us with seven ahead instead of one).
    const int c_lo = col_of(pair0), c_hi = col_of(min(pair0 + PP, n_pairs) - 1);
    const int k_lo = c_lo < g.n_q ? 0 : (c_lo < g.n_q + g.n_kv ? 1 : 2), k_hi = c_hi < g.n_q ? 0 : (c_hi < g.n_q + g.n_kv ? 1 : 2);
    // t of a row is the same whatever adapter is multiplied (the others' rows are zeroed): it stays in registers.
    constexpr int LS = 2, AHEAD = CW == 8 ? 2 : 8;
    auto fetch_b = [&](unsigned long long left, int ks0, u32x4 (&b)[LS]) {
      if (!left) return;
      const bf16 *bp = brow + __builtin_ctzll(left) * a_stride;
#pragma unroll
      for (int i = 0; i < LS; ++i) b[i] = *reinterpret_cast<const u32x4 *>(bp + min(ks0 + 16 * i + lhi * 8, r - 8));
    };
    for (int part = k_lo; part <= k_hi; ++part)
      for (int ks0 = 0; ks0 < r; ks0 += 16 * LS) {
        const bf16 *tp = g.tlow + ((int64_t)rc * 3 + part) * 2 * r;
        u32x4 t[LS][2], b[AHEAD][LS];
#pragma unroll
        for (int i = 0; i < LS; ++i)
#pragma unroll
          for (int hl = 0; hl < 2; ++hl) t[i][hl] = *reinterpret_cast<const u32x4 *>(tp + hl * r + min(ks0 + 16 * i + lhi * 8, r - 8));
        auto apply = [&](unsigned long long left, u32x4 (&b)[LS]) {
          const bool mine = a_row == (int)__builtin_ctzll(left);
#pragma unroll
          for (int i = 0; i < LS; ++i) {
            if (ks0 + 16 * i >= r) continue;
            if (kind != part || ks0 + 16 * i + lhi * 8 >= r) b[i] = u32x4{0, 0, 0, 0};      // (ranks that are not a multiple of 16)
#pragma unroll
            for (int hl = 0; hl < 2; ++hl) {
              const u32x4 tm = mine ? t[i][hl] : u32x4{0, 0, 0, 0};
              acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[i]), __builtin_bit_cast(bf16x8, tm), acc, 0, 0, 0);
            }
          }
        };
        unsigned long long left = present, ask = present;      // to multiply, to ask for
#pragma unroll
        for (int i = 0; i < AHEAD - 1; ++i) { fetch_b(ask, ks0, b[i]); ask &= ask - 1; }
        while (left) {
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) {
            if (!left) break;
            fetch_b(ask, ks0, b[(i + AHEAD - 1) % AHEAD]);
            ask &= ask - 1;
            apply(left, b[i]);
            left &= left - 1;
          }
        }
      }
  }

  float2 rot[2][4];
  {
    const float2 *table = g.rope_table + (int64_t)(g.rope_by_row ? rc : pos) * h2;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) rot[q][i] = table[min(pair0 + 8 * q + 4 * lhi, n_pairs - 4) % h2 + i];
  }
  auto multiply = [&](int s, const u32x4 (&x0)[8], const u32x4 (&x1)[8], auto between) {      // stage s
    const char *w = lds + (s % QS_DEPTH) * STAGE + lds_row * (QS_K * 2);
    bf16x8 f[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) f[i] = *reinterpret_cast<const bf16x8 *>(w + ((i * 2 + lhi) ^ (lds_row & 15)) * 16);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], __builtin_bit_cast(bf16x8, x0[i]), acc, 0, 0, 0);
    between();
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[8 + i], __builtin_bit_cast(bf16x8, x1[i]), acc, 0, 0, 0);
  };
  // (XB / 2 stages to a round, so that the buffers' numbers are constants)
  for (int s0 = 0; s0 < n_full; s0 += XB / 2) {
#pragma unroll
    for (int j = 0; j < XB / 2; ++j) {
      const int s = s0 + j;
      if (j > 0 && s >= n_full) break;
      fetch(2 * s + XB - 1, xr[(2 * j + XB - 1) % XB]);
      wave_barrier();
      multiply(s, xr[2 * j], xr[2 * j + 1], [&] { fetch(2 * s + XB, xr[2 * j]); });
      wait_lds();      // the reads are done before the next barrier hands the stage back to the loading waves
    }
  }
  if (n_full < n_stages) {
    fetch(2 * n_full, xr[0]);
    wave_barrier();
    const char *w = lds + (n_full % QS_DEPTH) * STAGE + lds_row * (QS_K * 2);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(w + ((i * 2 + lhi) ^ (lds_row & 15)) * 16),
                                                    __builtin_bit_cast(bf16x8, xr[0][i]), acc, 0, 0, 0);
  }

  // ---- rotation and append: lane l32 is a row, register 4 q + i the slot 8 q + 4 lhi + i -------------------------------
  if (row >= M) return;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int pl = 8 * q + 4 * lhi, p = pair0 + pl;
    if (pl >= PP || p >= n_pairs) continue;      // (pairs come in fours: same head, same kind)
    const int col = col_of(p), kind = col < g.n_q ? 0 : (col < g.n_q + g.n_kv ? 1 : 2);
    const int hcol = kind == 0 ? col : (kind == 1 ? col - g.n_q : col - g.n_q - g.n_kv);
    float lo[4], hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float u = acc[4 * q + i], w = acc[8 + 4 * q + i];
      const float2 cs = kind == 2 ? make_float2(1.f, 0.f) : rot[q][i];
      const float qs = kind == 0 ? g.q_scale : 1.0f;
      lo[i] = kind == 2 ? u : rope_lo(u, w, cs.x, cs.y) * qs;
      hi[i] = kind == 2 ? w : rope_hi(u, w, cs.x, cs.y) * qs;
    }
    if (kind == 0 && g.q_f32) {      // queries for the plain attention kernel
      float *dst = reinterpret_cast<float *>(g.Qout) + (int64_t)row * g.n_q + hcol;
      *reinterpret_cast<float4 *>(dst) = make_float4(lo[0], lo[1], lo[2], lo[3]);
      *reinterpret_cast<float4 *>(dst + h2) = make_float4(hi[0], hi[1], hi[2], hi[3]);
    } else if (kind == 0) {      // queries as fp16 for the MFMA attention kernels
      half4 a, b;
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = (_Float16)lo[i]; b[i] = (_Float16)hi[i]; }
      _Float16 *dst = reinterpret_cast<_Float16 *>(g.Qout) + (int64_t)row * g.n_q + hcol;
      *reinterpret_cast<half4 *>(dst) = a;
      *reinterpret_cast<half4 *>(dst + h2) = b;
    } else {
      bf16x4 a, b;
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = (bf16)lo[i]; b[i] = (bf16)hi[i]; }
      bf16 *dst = (kind == 1 ? g.cacheK : g.cacheV) + slot * g.n_kv + hcol;
      *reinterpret_cast<bf16x4 *>(dst) = a;
      *reinterpret_cast<bf16x4 *>(dst + h2) = b;
    }
  }
}

// A matter of the weights alone, never of the number of rows.  (Pairs are stored in fours, which must not straddle two heads.)
bool qkv_stream_supported(const void *W, int N, int K, int head_dim) {
  return lds_aligned(W) && head_dim % 8 == 0 && K % 128 == 0 && K >= QS_K && (uint64_t)N * K * 2 < (1ull << 31);
}

// Weights of more than one round of the widest tiles (8192 x 10240: 427 tiles of 12 pairs, every one with all of the rows): from 129 rows
// on the 128 x 128 tiles, or the kernel without rotation, are quicker (256 rows: 111 us here, 79 and 93 there; 128 rows: 71 here, 90 there).
int qkv_stream_rows(int N, int n_cu) { return N / 2 > 16 * n_cu ? QKV_STREAM_ROWS / 2 : QKV_STREAM_ROWS; }

template <int CW, int PW>
static void launch_cfg(const GemmArgs &g, hipStream_t s) {
  const int tiles_m = (g.M + 32 * CW - 1) / (32 * CW), tiles_n = (g.N / 2 + 4 * PW - 1) / (4 * PW);
  const size_t smem = (size_t)QS_DEPTH * 2 * (4 * PW) * QS_K * 2;
  auto kern = qkv_stream_kernel<CW, PW>;
  (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  hipLaunchKernelGGL(kern, dim3(8 * ((tiles_n + 7) / 8) * tiles_m), dim3(64 * (CW + 4)), smem, s, g, tiles_m);
}
template <int CW>
static void launch_cw(const GemmArgs &g, int n_cu, hipStream_t s) {
  // pairs per tile: the one of 8, 12, 16 whose rounds of a tile per compute unit move the fewest weights one after the other
  const int pairs = g.N / 2;
  int pw = 4, least = 0;
  for (int p = 4; p >= 2; --p) {
    const int t = ((pairs + 4 * p - 1) / (4 * p) + n_cu - 1) / n_cu * p;
    if (p == 4 || t < least) { least = t; pw = p; }
  }
  if (pw == 2) launch_cfg<CW, 2>(g, s);
  else if (pw == 3) launch_cfg<CW, 3>(g, s);
  else launch_cfg<CW, 4>(g, s);
}

void launch_qkv_stream(const GemmArgs &g, int n_cu, hipStream_t s) {
  if (g.M <= 32) launch_cw<1>(g, n_cu, s);
  else if (g.M <= 64) launch_cw<2>(g, n_cu, s);
  else if (g.M <= 128) launch_cw<4>(g, n_cu, s);
  else launch_cw<8>(g, n_cu, s);
}

}  // namespace alora
