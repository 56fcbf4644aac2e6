// Plain kernels: every step of the path in straightforward fp32-FMA HIP, for any dtype and
// any shape.  They are the fp32 path (small single-block configuration) and the fallback
// for shapes the MFMA kernels do not cover.
#include "lds_dma.h"

namespace alora {

// ---------------------------------------------------------------------------------------
// rotary table: table[pos * half + c] = (cos, sin)(pos * theta^(-2c/h)), evaluated in
// double so that positions in the tens of thousands keep full fp32 accuracy.
// ---------------------------------------------------------------------------------------
__global__ void rope_table_kernel(float2 *table, int n_pos, int half, double log2_theta) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)n_pos * half) return;
  int pos = (int)(i / half), c = (int)(i % half);
  double inv = exp2(-(double)c / (double)half * log2_theta);   // theta^(-2c/h), h = 2*half
  double ang = (double)pos * inv;
  double sn, cs;
  sincos(ang, &sn, &cs);
  table[i] = make_float2((float)cs, (float)sn);
}

// The same entries for the positions of given rows only: table[row * half + c] for position pos[row] (callers
// that may not allocate a table of all positions keep one line per row).  Same arithmetic, same bits.
__global__ void rope_rows_kernel(float2 *table, const int32_t *__restrict__ pos, int n_rows, int half, double log2_theta) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)n_rows * half) return;
  int row = (int)(i / half), c = (int)(i % half);
  double inv = exp2(-(double)c / (double)half * log2_theta);
  double ang = (double)pos[row] * inv;
  double sn, cs;
  sincos(ang, &sn, &cs);
  table[i] = make_float2((float)cs, (float)sn);
}

void launch_rope_rows(float2 *table, const int32_t *pos, int n_rows, int half_dim, float theta, hipStream_t s) {
  int64_t n = (int64_t)n_rows * half_dim;
  if (n == 0) return;
  hipLaunchKernelGGL(rope_rows_kernel, dim3((int)((n + 255) / 256)), dim3(256), 0, s, table, pos, n_rows, half_dim,
                     log2((double)theta));
}

void launch_rope_table(float2 *table, int n_pos, int half_dim, float theta, hipStream_t s) {
  int64_t n = (int64_t)n_pos * half_dim;
  if (n == 0) return;
  int grid = (int)((n + 255) / 256);
  hipLaunchKernelGGL(rope_table_kernel, dim3(grid), dim3(256), 0, s, table, n_pos, half_dim,
                     log2((double)theta));
}

// ---------------------------------------------------------------------------------------
// row preparation: per-row metadata, RMSNorm, and the low-rank down projection
// t = s_a * A_a x_hat for adapted rows (Eq.6's Delta applied right to left).
// One workgroup per packed row.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void prep_rows_kernel(const T *__restrict__ x, const T *__restrict__ gain,
                                                        float eps, int d, const SeqMeta *__restrict__ seqs,
                                                        int n_seqs, int pos_shift, const T *__restrict__ A, int rank,
                                                        int write_meta, T *__restrict__ xh,
                                                        float *__restrict__ tlow, bf16 *__restrict__ tlow16,
                                                        RowMeta rm, StagedCall st, int packed) {
  extern __shared__ float xs[];
  __shared__ float red[4];
  __shared__ int s_adapter;
  __shared__ float s_scale;
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  Carried<256> staged;
  staged.load(st, tid, row == 0);
  if (tid == 0) {
    int adapter = -1;
    float scale = 0.f;
    if (seqs != nullptr) {
      int lo = 0, hi = n_seqs - 1;   // last sequence whose first row is <= row
      if (st.n_few) {
        while (lo < hi && st.few[lo + 1].row_start <= row) ++lo;
      } else {
        while (lo < hi) {
          int mid = (lo + hi + 1) >> 1;
          if (seqs[mid].row_start <= row) lo = mid; else hi = mid - 1;
        }
      }
      SeqMeta sm = st.n_few ? st.few[lo] : seqs[lo];
      int pos = sm.P + pos_shift + (row - sm.row_start);
      if (sm.adapter >= 0 && pos >= sm.k) { adapter = sm.adapter; scale = sm.scale; }
      if (write_meta) {
        rm.seq[row] = lo;
        rm.pos[row] = pos;
        rm.adapter[row] = adapter;
        rm.slot[row] = sm.pool_off + pos;
      }
    }
    s_adapter = adapter;
    s_scale = scale;
  }
  const T *xr = x + (int64_t)row * d;
  float ssq = 0.f;
  for (int c = tid; c < d; c += 256) {
    float v = to_f32<T>(xr[c]);
    xs[c] = v;
    ssq += v * v;
  }
  ssq = wave_sum(ssq);
  if (lane == 0) red[wave] = ssq;
  __syncthreads();
  float rinv = 1.f;
  if (gain != nullptr) rinv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
  for (int c = tid; c < d; c += 256) {
    float v = xs[c];
    if (gain != nullptr) v = v * to_f32<T>(gain[c]) * rinv;
    T stored = from_f32<T>(v);
    xh[packed ? xh_chunk(row, c >> 3, d, 1) * 8 + (c & 7) : (int64_t)row * d + c] = stored;
    xs[c] = to_f32<T>(stored);      // the projections consume the stored (rounded) value
  }
  staged.store(st, tid, row == 0);
  __syncthreads();
  const int a = s_adapter;
  if (a < 0 || rank == 0) return;
  const float scale = s_scale;
  // eight columns of t at a time, their loads together: one after the other, the round trips were most of a small call's first kernel
  // (16 rows of rank 8, d = 256: 9.6 -> 6.1 us)
  constexpr int U = 8;
  for (int j0 = wave; j0 < 3 * rank; j0 += 4 * U) {
    const T *ar = A + (int64_t)a * 3 * rank * d;
    int64_t at[U];
    float sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { at[u] = (int64_t)min(j0 + 4 * u, 3 * rank - 1) * d; sum[u] = 0.f; }
#pragma unroll 4
    for (int c = lane; c < d; c += 64)
#pragma unroll
      for (int u = 0; u < U; ++u) sum[u] += to_f32<T>(ar[at[u] + c]) * xs[c];
#pragma unroll
    for (int u = 0; u < U; ++u) sum[u] = wave_sum(sum[u]);
    if (lane < U && j0 + 4 * lane < 3 * rank) {
      const int j = j0 + 4 * lane;
      float acc = sum[0];
#pragma unroll
      for (int u = 1; u < U; ++u) acc = lane == u ? sum[u] : acc;
      const float t = scale * acc;
      if (tlow16) {
        // bf16 pair (hi, lo) with hi + lo = t to ~2^-17: the MFMA path feeds both as extra k-steps,
        // so the low-rank term keeps fp32-level accuracy.  Layout [row][p][hi|lo][rank].
        const int p = j / rank, jj = j % rank;
        const bf16 hi = (bf16)t;
        bf16 *dst = tlow16 + (((int64_t)row * 3 + p) * 2) * rank + jj;
        dst[0] = hi;
        dst[rank] = (bf16)(t - (float)hi);
      } else {
        tlow[(int64_t)row * 3 * rank + j] = t;
      }
    }
  }
}

template <typename T>
void launch_prep_rows(const T *x, const T *gain, float eps, int T_rows, int d, const SeqMeta *seqs,
                      int n_seqs, int pos_shift, const T *A, int rank, bool write_meta, T *xh, float *tlow,
                      bf16 *tlow16, RowMeta rm, const StagedCall &st, bool packed, hipStream_t s) {
  if (T_rows == 0) return;
  hipLaunchKernelGGL((prep_rows_kernel<T>), dim3(T_rows), dim3(256), (size_t)d * sizeof(float), s, x, gain,
                     eps, d, seqs, n_seqs, pos_shift, A, rank, write_meta ? 1 : 0, xh, tlow, tlow16, rm, st, packed ? 1 : 0);
}
template void launch_prep_rows<float>(const float *, const float *, float, int, int, const SeqMeta *, int, int,
                                      const float *, int, bool, float *, float *, bf16 *, RowMeta, const StagedCall &, bool, hipStream_t);
template void launch_prep_rows<bf16>(const bf16 *, const bf16 *, float, int, int, const SeqMeta *, int, int,
                                     const bf16 *, int, bool, bf16 *, float *, bf16 *, RowMeta, const StagedCall &, bool, hipStream_t);

// ---------------------------------------------------------------------------------------
// plain tiled GEMM  C[M,N] = A[M,K] B[N,K]^T, 64x64 tile, 16-deep, 4x4 outputs per thread
// ---------------------------------------------------------------------------------------
struct LoraEpi {
  const float *tlow;
  const void *Bq, *Bk, *Bv;
  const int32_t *row_adapter;
  int rank, n_q, n_kv;
};

template <typename T, int MODE>
__global__ __launch_bounds__(256) void gemm_plain_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                         const T *__restrict__ R, void *__restrict__ Cv,
                                                         int M, int N, int K, LoraEpi epi) {
  __shared__ float As[16][68];
  __shared__ float Bs[16][68];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int lr = tid >> 2, lk = (tid & 3) * 4;
  const int ty = tid >> 4, tx = tid & 15;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int kk = k0 + lk + i;
      int ar = m0 + lr, br = n0 + lr;
      As[lk + i][lr] = (ar < M && kk < K) ? to_f32<T>(A[(int64_t)ar * K + kk]) : 0.f;
      Bs[lk + i][lr] = (br < N && kk < K) ? to_f32<T>(B[(int64_t)br * K + kk]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Bs[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int row = m0 + ty * 4 + i;
    if (row >= M) continue;
    int a = -1;
    if (MODE == EPI_F32_LORA) a = epi.row_adapter[row];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int col = n0 + tx * 4 + j;
      if (col >= N) continue;
      float v = acc[i][j];
      if (MODE == EPI_F32_LORA) {
        if (a >= 0) {     // adapted row: add s * B (A x); other rows get nothing added
          const int r = epi.rank;
          const T *bp;
          int p;
          if (col < epi.n_q) { p = 0; bp = (const T *)epi.Bq + ((int64_t)a * epi.n_q + col) * r; }
          else if (col < epi.n_q + epi.n_kv) { p = 1; bp = (const T *)epi.Bk + ((int64_t)a * epi.n_kv + (col - epi.n_q)) * r; }
          else { p = 2; bp = (const T *)epi.Bv + ((int64_t)a * epi.n_kv + (col - epi.n_q - epi.n_kv)) * r; }
          const float *t = epi.tlow + (int64_t)row * 3 * r + p * r;
          float lo = 0.f;
          for (int jj = 0; jj < r; ++jj) lo += t[jj] * to_f32<T>(bp[jj]);
          v += lo;
        }
        ((float *)Cv)[(int64_t)row * N + col] = v;
      } else if (MODE == EPI_STORE_F32) {
        ((float *)Cv)[(int64_t)row * N + col] = v;
      } else {
        if (MODE == EPI_STORE_RESIDUAL) v += to_f32<T>(R[(int64_t)row * N + col]);
        ((T *)Cv)[(int64_t)row * N + col] = from_f32<T>(v);
      }
    }
  }
}

// The QKV projection of a call too small to fill the chip with 64 x 64 tiles, rotated and appended where it is computed: 16 rows x 8
// rotation pairs (c, c + h/2) per workgroup, a thread per output, 256 values of k at a time through LDS with the next 256 on their
// way.  A thread adds its products in ascending k, as the tiled kernel does (same bits).  16 rows x 768 columns x 256: 40 us in
// 12 workgroups of 16 dependent k-steps each, plus the rotation's own launch.
template <typename T>
__global__ __launch_bounds__(256) void qkv_small_plain_kernel(const T *__restrict__ X, const T *__restrict__ W, LayerDims L, int M,
                                                              LoraEpi epi, const int32_t *__restrict__ pos,
                                                              const int64_t *__restrict__ slot, const float2 *__restrict__ table,
                                                              int table_by_row, float q_scale, int q_mode, void *__restrict__ Q,
                                                              T *__restrict__ cacheK, T *__restrict__ cacheV) {
  constexpr int KC = 256, LD = KC + 4;
  __shared__ float xs[16][LD], ws[16][LD];
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  const int h = L.head_dim, h2 = h >> 1, n_pairs = L.n_qkv >> 1, K = L.d;
  const int m0 = blockIdx.y * 16, p0 = blockIdx.x * 8;
  auto col_of = [&](int i) {      // column i of the tile: the pairs' first columns, then their partners
    const int p = min(p0 + (i & 7), n_pairs - 1);
    return (p / h2) * h + p % h2 + (i >> 3) * h2;
  };
  const int row = m0 + r, rc = min(row, M - 1), col = col_of(c);
  const int kind = col < L.n_q ? 0 : (col < L.n_q + L.n_kv ? 1 : 2);
  const int a = epi.row_adapter[rc];
  const int64_t sl = slot[rc];
  const float2 cs = table[(int64_t)(table_by_row ? rc : pos[rc]) * h2 + (col % h) % h2];
  const T *xrow = X + (int64_t)rc * K, *wrow = W + (int64_t)col_of(r) * K;      // (thread r, c loads row r of both, k from 16 c)
  float xv[16], wv[16];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int k = k0 + c + 16 * i;
      xv[i] = k < K ? to_f32<T>(xrow[k]) : 0.f;
      wv[i] = k < K ? to_f32<T>(wrow[k]) : 0.f;
    }
  };
  float acc = 0.f;
  fetch(0);
  // the low-rank term's operands, eight ranks ahead of their use, the first ones before the product
  constexpr int RA = 8;
  const int rk = a >= 0 ? epi.rank : 0;
  const T *bp = (const T *)epi.Bq;
  const float *tp = epi.tlow;
  if (rk > 0) {
    bp = kind == 0 ? (const T *)epi.Bq + ((int64_t)a * L.n_q + col) * rk
                   : (kind == 1 ? (const T *)epi.Bk + ((int64_t)a * L.n_kv + col - L.n_q) * rk
                                : (const T *)epi.Bv + ((int64_t)a * L.n_kv + col - L.n_q - L.n_kv) * rk);
    tp = epi.tlow + (int64_t)rc * 3 * rk + kind * rk;
  }
  float tv[RA];
  T bv[RA];
  auto fetch_low = [&](int j0) {
#pragma unroll
    for (int i = 0; i < RA; ++i) { tv[i] = tp[min(j0 + i, rk - 1)]; bv[i] = bp[min(j0 + i, rk - 1)]; }
  };
  if (rk > 0) fetch_low(0);
  for (int k0 = 0; k0 < K; k0 += KC) {
#pragma unroll
    for (int i = 0; i < 16; ++i) { xs[r][c + 16 * i] = xv[i]; ws[r][c + 16 * i] = wv[i]; }
    __syncthreads();
    if (k0 + KC < K) fetch(k0 + KC);
#pragma unroll 8
    for (int k = 0; k < KC; k += 4) {
      const float4 x4 = *reinterpret_cast<const float4 *>(&xs[r][k]), w4 = *reinterpret_cast<const float4 *>(&ws[c][k]);
      acc = __builtin_fmaf(x4.x, w4.x, acc);
      acc = __builtin_fmaf(x4.y, w4.y, acc);
      acc = __builtin_fmaf(x4.z, w4.z, acc);
      acc = __builtin_fmaf(x4.w, w4.w, acc);
    }
    __syncthreads();
  }
  if (rk > 0) {
    float lo = 0.f;
    for (int j0 = 0; j0 < rk; j0 += RA) {
      if (j0 > 0) fetch_low(j0);
#pragma unroll
      for (int i = 0; i < RA; ++i)
        if (j0 + i < rk) lo += tv[i] * to_f32<T>(bv[i]);
    }
    acc += lo;
  }
  const float other = __shfl_xor(acc, 8, 64);      // the rotation partner
  if (row >= M || p0 + (c & 7) >= n_pairs) return;
  const float u = c < 8 ? acc : other, w = c < 8 ? other : acc;
  const int hcol = kind == 0 ? col : (kind == 1 ? col - L.n_q : col - L.n_q - L.n_kv);
  if (kind == 2) { cacheV[sl * L.n_kv + hcol] = from_f32<T>(acc); return; }
  const float y = (c < 8 ? rope_lo(u, w, cs.x, cs.y) : rope_hi(u, w, cs.x, cs.y)) * (kind == 0 ? q_scale : 1.0f);
  if (kind == 1) cacheK[sl * L.n_kv + hcol] = from_f32<T>(y);
  else if (q_mode == 1) reinterpret_cast<_Float16 *>(Q)[(int64_t)row * L.n_q + hcol] = (_Float16)y;
  else reinterpret_cast<float *>(Q)[(int64_t)row * L.n_q + hcol] = y;
}

// Where the 64 x 64 tiles of the projection would leave half of the chip idle or more.  Projection and rotation in fp32, us, here / tiled:
// 12 tiles (16 x 768 x 256) 8 / 49, 64 (64 x 4096 x 1024) 30 / 144, at the line 120 (640 x 768 x 256) 21 / 57 and 128 (64 x 8192 x 4096) 170 / 518.
// Beyond it the distance shrinks with the reuse that 16 x 16 outputs lack: 192 tiles (192 x 4096 x 1024) 68 / 145, 384 (192 x 8192 x 4096)
// 465 / 681, 480 (640 x 3072 x 4096) 571 / 690.
bool qkv_small_plain_wanted(int T_rows, int n_qkv, int n_cu) { return ((T_rows + 63) / 64) * ((n_qkv + 63) / 64) * 2 <= n_cu; }

template <typename T>
void launch_qkv_small_plain(const T *xh, const T *W, const float *tlow, const T *Bq, const T *Bk, const T *Bv, const LayerDims &L,
                            RowMeta rm, int T_rows, const float2 *table, bool by_row, float q_scale, int q_mode, void *Q, T *cacheK,
                            T *cacheV, hipStream_t s) {
  if (T_rows == 0) return;
  LoraEpi epi{tlow, Bq, Bk, Bv, rm.adapter, L.rank, L.n_q, L.n_kv};
  dim3 grid((L.n_qkv / 2 + 7) / 8, (T_rows + 15) / 16);
  hipLaunchKernelGGL((qkv_small_plain_kernel<T>), grid, dim3(256), 0, s, xh, W, L, T_rows, epi, rm.pos, rm.slot, table, by_row ? 1 : 0,
                     q_scale, q_mode, Q, cacheK, cacheV);
}
template void launch_qkv_small_plain<float>(const float *, const float *, const float *, const float *, const float *, const float *,
                                            const LayerDims &, RowMeta, int, const float2 *, bool, float, int, void *, float *, float *, hipStream_t);
template void launch_qkv_small_plain<bf16>(const bf16 *, const bf16 *, const float *, const bf16 *, const bf16 *, const bf16 *,
                                           const LayerDims &, RowMeta, int, const float2 *, bool, float, int, void *, bf16 *, bf16 *, hipStream_t);

template <typename T>
void launch_qkv_gemm_plain(const T *xh, const T *W, const float *tlow, const T *Bq, const T *Bk,
                           const T *Bv, const LayerDims &L, RowMeta rm, int T_rows, float *Y,
                           hipStream_t s) {
  if (T_rows == 0) return;
  LoraEpi epi{tlow, Bq, Bk, Bv, rm.adapter, L.rank, L.n_q, L.n_kv};
  dim3 grid((L.n_qkv + 63) / 64, (T_rows + 63) / 64);
  hipLaunchKernelGGL((gemm_plain_kernel<T, EPI_F32_LORA>), grid, dim3(256), 0, s, xh, W, (const T *)nullptr,
                     (void *)Y, T_rows, L.n_qkv, L.d, epi);
}
template void launch_qkv_gemm_plain<float>(const float *, const float *, const float *, const float *,
                                           const float *, const float *, const LayerDims &, RowMeta, int,
                                           float *, hipStream_t);
template void launch_qkv_gemm_plain<bf16>(const bf16 *, const bf16 *, const float *, const bf16 *,
                                          const bf16 *, const bf16 *, const LayerDims &, RowMeta, int,
                                          float *, hipStream_t);

template <typename T>
void launch_gemm_plain(const T *A, const T *B, const T *R, T *C, int M, int N, int K, hipStream_t s) {
  if (M == 0 || N == 0) return;
  LoraEpi epi{};
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  if (R)
    hipLaunchKernelGGL((gemm_plain_kernel<T, EPI_STORE_RESIDUAL>), grid, dim3(256), 0, s, A, B, R, (void *)C,
                       M, N, K, epi);
  else
    hipLaunchKernelGGL((gemm_plain_kernel<T, EPI_STORE>), grid, dim3(256), 0, s, A, B, R, (void *)C, M, N, K,
                       epi);
}
template <typename T>
void launch_gemm_plain_f32(const T *A, const T *B, float *C, int M, int N, int K, hipStream_t s) {
  if (M == 0 || N == 0) return;
  LoraEpi epi{};
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  hipLaunchKernelGGL((gemm_plain_kernel<T, EPI_STORE_F32>), grid, dim3(256), 0, s, A, B, (const T *)nullptr, (void *)C, M,
                     N, K, epi);
}
template void launch_gemm_plain_f32<float>(const float *, const float *, float *, int, int, int, hipStream_t);
template void launch_gemm_plain_f32<bf16>(const bf16 *, const bf16 *, float *, int, int, int, hipStream_t);
template void launch_gemm_plain<float>(const float *, const float *, const float *, float *, int, int, int,
                                       hipStream_t);
template void launch_gemm_plain<bf16>(const bf16 *, const bf16 *, const bf16 *, bf16 *, int, int, int,
                                      hipStream_t);

// ---------------------------------------------------------------------------------------
// rotary embedding + cache append (Eq.3: K_{1:t} = [K_{1:t-1}; K_t]).
// ---------------------------------------------------------------------------------------
// One wave per (row, head slot), four slots per workgroup: slots 0..Hq-1 are query heads, then the
// key heads, then the value heads.  Every lane handles whole rotation pairs, all loads are
// independent.
template <typename T, bool MULTI>      // MULTI: Y arrives as several partial sums
__global__ __launch_bounds__(256) void rope_append_kernel(const float *__restrict__ Y, int n_parts,
                                                         int64_t part_stride, LayerDims L, RowMeta rm,
                                                         const float2 *__restrict__ table, int table_by_row,
                                                         float q_scale, int q_half, T *__restrict__ Q,
                                                         T *__restrict__ cacheK,
                                                         T *__restrict__ cacheV) {
  const int row = blockIdx.x, slot_id = blockIdx.y * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int h = L.head_dim, h2 = h >> 1;
  if (slot_id >= L.n_q_heads + 2 * L.n_kv_heads) return;
  const float *y = Y + (int64_t)row * L.n_qkv;
  // Y may arrive as n_parts partial sums over the reduction axis: add them in a fixed order
  // (the first eight are requested together: a loop over the run-time count costs a memory round trip per part)
  auto ysum = [&](const float *p) {
    if constexpr (!MULTI) return p[0];
    float t[8];
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (s < n_parts) t[s] = p[(int64_t)s * part_stride];
    float v = t[0];
#pragma unroll
    for (int s = 1; s < 8; ++s)
      if (s < n_parts) v += t[s];
    for (int s = 8; s < n_parts; ++s) v += p[(int64_t)s * part_stride];
    return v;
  };
  if (slot_id < L.n_q_heads + L.n_kv_heads) {
    const bool is_q = slot_id < L.n_q_heads;
    const int head = is_q ? slot_id : slot_id - L.n_q_heads;
    const int base = (is_q ? 0 : L.n_q) + head * h;
    const float2 *tab = table + (int64_t)(table_by_row ? row : rm.pos[row]) * h2;
    T *dst = is_q ? Q + (int64_t)row * L.n_q + head * h : cacheK + rm.slot[row] * L.n_kv + head * h;
    // q_scale: the attention kernel that follows may want its queries premultiplied (softmax scale and
    // log2 e, so that its scores come out of the MFMA ready for exp2); keys are never scaled
    const float qs = is_q ? q_scale : 1.0f;
    for (int c = lane; c < h2; c += 64) {
      const float u = ysum(y + base + c), w = ysum(y + base + c + h2);
      const float2 cs = tab[c];
      const float lo = rope_lo(u, w, cs.x, cs.y) * qs, hi = rope_hi(u, w, cs.x, cs.y) * qs;
      if (is_q && q_half == 1) {
        // the MFMA attention kernels want their queries as fp16
        _Float16 *dq = reinterpret_cast<_Float16 *>(Q) + (int64_t)row * L.n_q + head * h;
        dq[c] = (_Float16)lo;
        dq[c + h2] = (_Float16)hi;
      } else if (is_q && q_half == 2) {
        // the plain attention kernel keeps them in fp32
        float *dq = reinterpret_cast<float *>(Q) + (int64_t)row * L.n_q + head * h;
        dq[c] = lo;
        dq[c + h2] = hi;
      } else {
        dst[c] = from_f32<T>(lo);
        dst[c + h2] = from_f32<T>(hi);
      }
    }
  } else {
    const int head = slot_id - L.n_q_heads - L.n_kv_heads;
    const float *yv = y + L.n_q + L.n_kv + head * h;
    T *dst = cacheV + rm.slot[row] * L.n_kv + head * h;
    for (int c = lane; c < h; c += 64) dst[c] = from_f32<T>(ysum(yv + c));
  }
}

template <typename T>
void launch_rope_append(const float *Y, int n_parts, const LayerDims &L, RowMeta rm, int T_rows,
                        const float2 *rope_table, bool table_by_row, float q_scale, int q_half, void *Q, T *cacheK,
                        T *cacheV, hipStream_t s) {
  if (T_rows == 0) return;
  dim3 grid(T_rows, (L.n_q_heads + 2 * L.n_kv_heads + 3) / 4);
  if (n_parts > 1)
    hipLaunchKernelGGL((rope_append_kernel<T, true>), grid, dim3(256), 0, s, Y, n_parts, (int64_t)T_rows * L.n_qkv, L, rm,
                       rope_table, table_by_row ? 1 : 0, q_scale, q_half, (T *)Q, cacheK, cacheV);
  else
    hipLaunchKernelGGL((rope_append_kernel<T, false>), grid, dim3(256), 0, s, Y, n_parts, (int64_t)T_rows * L.n_qkv, L, rm,
                       rope_table, table_by_row ? 1 : 0, q_scale, q_half, (T *)Q, cacheK, cacheV);
}
template void launch_rope_append<float>(const float *, int, const LayerDims &, RowMeta, int, const float2 *, bool, float, int,
                                        void *, float *, float *, hipStream_t);
template void launch_rope_append<bf16>(const float *, int, const LayerDims &, RowMeta, int, const float2 *, bool, float, int,
                                       void *, bf16 *, bf16 *, hipStream_t);

// ---------------------------------------------------------------------------------------
// plain split-KV attention (Eq.1 / Eq.4, causal, GQA).  One workgroup of four waves per (row, kv head, chunk of
// up to 8 query heads, key split), 64 keys at a time: four threads to a key for the scores, a wave to a head for the
// softmax, every fourth key to a wave for the values (lanes across head_dim), the four waves' sums added at the end.  Latency is
// what it costs (16 rows over 80 keys: one wave per workgroup with a key per lane took 44 us), so every phase has its loads
// together.  out != nullptr (one split): the result itself; otherwise
// partial layout: part[(((row*Hq + hq) * n_splits) + split) * (h + 2)] = acc[h], m, l.
// ---------------------------------------------------------------------------------------
#define ATT_GMAX 8
#define ATT_DMAX 4     // head_dim <= 256

// four neighbouring elements and one, as they lie in memory
template <typename T> struct Raw;
template <> struct Raw<float> { typedef float4 Four; static __device__ __forceinline__ float4 f4(float4 v) { return v; } };
template <> struct Raw<bf16> {
  typedef uint2 Four;
  static __device__ __forceinline__ float4 f4(uint2 w) {
    return make_float4(__builtin_bit_cast(float, w.x << 16), __builtin_bit_cast(float, w.x & 0xffff0000u),
                       __builtin_bit_cast(float, w.y << 16), __builtin_bit_cast(float, w.y & 0xffff0000u));
  }
};

// GM: most query heads of a workgroup (G = 1: a third of the code).  DD: 64-column pieces of a head that is a multiple of 16, 0: any head size (column by column, nothing asked for ahead).  A tile's keys
// are asked for while the tile before it is multiplied with its values, its values while its own scores are computed: a small call has
// one or two tiles, and every round trip was waited for on its own (16 rows, 80 keys of 64: 14.1 -> 7.5 us).
template <typename T, int DD, int GM>
__global__ __launch_bounds__(256) void attn_partial_kernel(const float *__restrict__ Q, const T *__restrict__ cacheK,
                                                          const T *__restrict__ cacheV,
                                                          const SeqMeta *__restrict__ seqs, RowMeta rm,
                                                          LayerDims L, int n_splits, float *__restrict__ part,
                                                          T *__restrict__ out) {
  extern __shared__ float smem[];       // qs[GMAX][h], ps[GMAX][64]; the waves' sums at the end: [4][GMAX][h]
  __shared__ float s_corr[ATT_GMAX], s_m[ATT_GMAX], s_l[ATT_GMAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = L.head_dim;
  const int G = L.n_q_heads / L.n_kv_heads;
  const int row = blockIdx.x / L.n_kv_heads, g = blockIdx.x % L.n_kv_heads;
  const int split = blockIdx.y;
  const int g0 = blockIdx.z * ATT_GMAX;
  const int ng = min(ATT_GMAX, G - g0);
  float *qs = smem, *ps = smem + ATT_GMAX * h;
  const SeqMeta sm = seqs[rm.seq[row]];
  const int n_keys = rm.pos[row] + 1;
  int chunk = (n_keys + n_splits - 1) / n_splits;
  chunk = (chunk + 63) & ~63;
  const int begin = split * chunk, end = min(n_keys, begin + chunk);
  const float sm_scale = 1.0f / sqrtf((float)h);
  for (int i = tid; i < ng * h; i += 256) qs[i] = Q[(int64_t)row * L.n_q + (g * G + g0) * h + i] * sm_scale;
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};      // of heads wave and wave + 4
  constexpr int D1 = DD > 0 ? DD : 1, DA = DD > 0 ? DD : ATT_DMAX;
  float acc[GM][DA];
#pragma unroll
  for (int gi = 0; gi < GM; ++gi)
#pragma unroll
    for (int dd = 0; dd < DA; ++dd) acc[gi][dd] = 0.f;
  typename Raw<T>::Four kf[4 * D1];
  T vf[16][D1];
  auto ask_k = [&](int t0) {
    const T *kr = cacheK + seq_pool_row(sm, min(t0 + (tid >> 2), end - 1)) * L.n_kv + g * h + 4 * (tid & 3);
#pragma unroll
    for (int i = 0; i < 4 * D1; ++i)
      if (16 * i < h) kf[i] = *reinterpret_cast<const typename Raw<T>::Four *>(kr + 16 * i);
  };
  auto ask_v = [&](int t0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const T *vr = cacheV + seq_pool_row(sm, min(t0 + wave + 4 * i, end - 1)) * L.n_kv + g * h;
#pragma unroll
      for (int dd = 0; dd < D1; ++dd)
        if (lane + 64 * dd < h) vf[i][dd] = vr[lane + 64 * dd];
    }
  };
  if constexpr (DD > 0) {
    if (begin < end) { ask_k(begin); ask_v(begin); }
  }
  __syncthreads();
  for (int t0 = begin; t0 < end; t0 += 64) {
    {
      const int key = t0 + (tid >> 2), q4 = tid & 3;
      float sc[GM];
#pragma unroll
      for (int gi = 0; gi < GM; ++gi) sc[gi] = 0.f;
      if constexpr (DD > 0) {
#pragma unroll
        for (int i = 0; i < 4 * D1; ++i) {
          if (16 * i >= h) break;
          const float4 kv = Raw<T>::f4(kf[i]);
#pragma unroll
          for (int gi = 0; gi < GM; ++gi)
            if (GM == 1 || gi < ng) {
              const float4 qv = *reinterpret_cast<const float4 *>(qs + gi * h + 4 * q4 + 16 * i);
              sc[gi] += qv.x * kv.x + qv.y * kv.y + qv.z * kv.z + qv.w * kv.w;
            }
        }
        if (t0 + 64 < end) ask_k(t0 + 64);
      } else {
        const T *kr = cacheK + seq_pool_row(sm, min(key, end - 1)) * L.n_kv + g * h;
        for (int c = q4; c < h; c += 4) {
          const float kv = to_f32<T>(kr[c]);
#pragma unroll
          for (int gi = 0; gi < GM; ++gi)
            if (GM == 1 || gi < ng) sc[gi] += qs[gi * h + c] * kv;
        }
      }
#pragma unroll
      for (int gi = 0; gi < GM; ++gi)
        if (GM == 1 || gi < ng) {
          float v = sc[gi] + __shfl_xor(sc[gi], 1, 64);
          v += __shfl_xor(v, 2, 64);
          if (q4 == 0) ps[gi * 64 + (tid >> 2)] = key < end ? v : -INFINITY;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int gi = wave + 4 * u;
      if (gi < ng) {      // (with one head three waves have none: not a loop that GM bounds)
        const float s = ps[gi * 64 + lane];
        const float mn = fmaxf(m[u], wave_max(s));
        const float p = __expf(s - mn), corr = __expf(m[u] - mn);      // (every tile holds a valid key: mn is finite)
        l[u] = l[u] * corr + wave_sum(p);
        m[u] = mn;
        ps[gi * 64 + lane] = p;
        if (lane == 0) s_corr[gi] = corr;
      }
    }
    __syncthreads();
#pragma unroll
    for (int gi = 0; gi < GM; ++gi)
      if (GM == 1 || gi < ng)
#pragma unroll
        for (int dd = 0; dd < DA; ++dd) acc[gi][dd] *= s_corr[gi];
    const int nk = min(64, end - t0);
    if constexpr (DD > 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int j = wave + 4 * i;
        if (j >= nk) break;
#pragma unroll
        for (int dd = 0; dd < D1; ++dd)
          if (lane + 64 * dd < h) {
            const float vv = to_f32<T>(vf[i][dd]);
#pragma unroll
            for (int gi = 0; gi < GM; ++gi)
              if (GM == 1 || gi < ng) acc[gi][dd] += ps[gi * 64 + j] * vv;
          }
      }
      if (t0 + 64 < end) ask_v(t0 + 64);
    } else {
#pragma unroll 8
      for (int j = wave; j < nk; j += 4) {
        const T *vr = cacheV + seq_pool_row(sm, t0 + j) * L.n_kv + g * h;
#pragma unroll
        for (int dd = 0; dd < DA; ++dd) {
          const int c = lane + 64 * dd;
          if (c < h) {
            const float vv = to_f32<T>(vr[c]);
#pragma unroll
            for (int gi = 0; gi < GM; ++gi)
              if (GM == 1 || gi < ng) acc[gi][dd] += ps[gi * 64 + j] * vv;
          }
        }
      }
    }
    __syncthreads();      // the probabilities are used up
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (wave + 4 * u < ng && lane == 0) { s_m[wave + 4 * u] = m[u]; s_l[wave + 4 * u] = l[u]; }
#pragma unroll
  for (int gi = 0; gi < GM; ++gi)
    if (GM == 1 || gi < ng)
#pragma unroll
      for (int dd = 0; dd < DA; ++dd)
        if (lane + 64 * dd < h) smem[(wave * ng + gi) * h + lane + 64 * dd] = acc[gi][dd];
  __syncthreads();
  for (int i = tid; i < ng * h; i += 256) {
    const float v = ((smem[i] + smem[ng * h + i]) + smem[2 * ng * h + i]) + smem[3 * ng * h + i];
    const int gi = i / h, c = i - gi * h;
    const int64_t rh = (int64_t)row * L.n_q_heads + g * G + g0 + gi;
    if (out != nullptr) out[rh * h + c] = from_f32<T>(v * (1.0f / s_l[gi]));
    else part[(rh * n_splits + split) * (h + 2) + c] = v;
  }
  if (out == nullptr && tid < ng) {
    float *o = part + (((int64_t)row * L.n_q_heads + g * G + g0 + tid) * n_splits + split) * (h + 2);
    o[h] = s_m[tid];
    o[h + 1] = s_l[tid];
  }
}

// One wave per (row, query head), four per workgroup.  The per-split maxima are fetched by the
// first lanes in parallel, and the accumulators are read MU splits at a time (added in ascending order whatever
// MU is: a short batch over a long cache has few (row, head) pairs and a hundred records each, and every group
// of records is a memory round trip).
template <typename T, int MU>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float *__restrict__ part, LayerDims L, int n_parts, MergeCounts mc,
                                                         int64_t n_rh, T *__restrict__ out) {
  const int lane = threadIdx.x & 63, h = L.head_dim;
  const int64_t rh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);       // row * Hq + hq
  if (rh >= n_rh) return;
  const float *p0 = part + rh * n_parts * (h + 2);
  int own, n_splits;
  mc.of_row((int)(rh / L.n_q_heads), n_parts, own, n_splits);
  auto rec = [&](int s) { return p0 + (int64_t)(s < own ? s : s + mc.first_shared - own) * (h + 2); };
  float M = -INFINITY;
  for (int s0 = 0; s0 < n_splits; s0 += 64) {
    const int s = s0 + lane;
    M = fmaxf(M, s < n_splits ? rec(s)[h] : -INFINITY);
  }
  M = wave_max(M);
  float denom = 0.f;
  float acc[ATT_DMAX] = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < n_splits; s0 += MU) {
    float ms[MU], ls[MU], v[MU][ATT_DMAX];
#pragma unroll
    for (int u = 0; u < MU; ++u) {
      const float *ps = rec(min(s0 + u, n_splits - 1));
      ms[u] = ps[h];
      ls[u] = ps[h + 1];
#pragma unroll
      for (int dd = 0; dd < ATT_DMAX; ++dd) {
        const int c = lane + 64 * dd;
        v[u][dd] = c < h ? ps[c] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < MU; ++u) {
      const float w = (s0 + u >= n_splits || ms[u] == -INFINITY) ? 0.f : __expf(ms[u] - M);
      denom += w * ls[u];
#pragma unroll
      for (int dd = 0; dd < ATT_DMAX; ++dd) acc[dd] += w * v[u][dd];
    }
  }
  const float inv = 1.0f / denom;
#pragma unroll
  for (int dd = 0; dd < ATT_DMAX; ++dd) {
    int c = lane + 64 * dd;
    if (c < h) out[rh * h + c] = from_f32<T>(acc[dd] * inv);
  }
}

// The same merge for few (row, head) pairs with many records each (a handful of sequences decoding over long
// caches): one workgroup per pair, its four waves take the records w, w + 4, w + 8, ... (eight in flight each, two
// columns per lane and load), and their sums are added in wave order.  head_dim <= 128.
template <typename T>
__global__ __launch_bounds__(256) void attn_merge_wide_kernel(const float *__restrict__ part, LayerDims L, int n_parts, MergeCounts mc,
                                                              T *__restrict__ out) {
  __shared__ float s_acc[4][130];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = L.head_dim;
  const int64_t rh = blockIdx.x;
  const float *p0 = part + rh * n_parts * (h + 2);
  int own, n_splits;
  mc.of_row((int)(rh / L.n_q_heads), n_parts, own, n_splits);
  auto rec = [&](int s) { return p0 + (int64_t)(s < own ? s : s + mc.first_shared - own) * (h + 2); };
  float M = -INFINITY;
  for (int s0 = 0; s0 < n_splits; s0 += 64) {
    const int s = s0 + lane;
    M = fmaxf(M, s < n_splits ? rec(s)[h] : -INFINITY);
  }
  M = wave_max(M);
  float denom = 0.f;
  float2 acc = make_float2(0.f, 0.f);
  const bool col_ok = 2 * lane < h;
  constexpr int MU = 8;
  for (int s0 = wave; s0 < n_splits; s0 += 4 * MU) {
    float ms[MU], ls[MU];
    float2 v[MU];
#pragma unroll
    for (int u = 0; u < MU; ++u) {
      const float *ps = rec(min(s0 + 4 * u, n_splits - 1));
      ms[u] = ps[h];
      ls[u] = ps[h + 1];
      v[u] = col_ok ? *reinterpret_cast<const float2 *>(ps + 2 * lane) : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < MU; ++u) {
      const float w = (s0 + 4 * u >= n_splits || ms[u] == -INFINITY) ? 0.f : __expf(ms[u] - M);
      denom += w * ls[u];
      acc.x += w * v[u].x;
      acc.y += w * v[u].y;
    }
  }
  if (col_ok) { s_acc[wave][2 * lane] = acc.x; s_acc[wave][2 * lane + 1] = acc.y; }
  if (lane == 0) s_acc[wave][128] = denom;
  __syncthreads();
  if (wave == 0 && col_ok) {
    const float d = ((s_acc[0][128] + s_acc[1][128]) + s_acc[2][128]) + s_acc[3][128];
    const float inv = 1.0f / d;
    const float x = ((s_acc[0][2 * lane] + s_acc[1][2 * lane]) + s_acc[2][2 * lane]) + s_acc[3][2 * lane];
    const float y = ((s_acc[0][2 * lane + 1] + s_acc[1][2 * lane + 1]) + s_acc[2][2 * lane + 1]) + s_acc[3][2 * lane + 1];
    out[rh * h + 2 * lane] = from_f32<T>(x * inv);
    out[rh * h + 2 * lane + 1] = from_f32<T>(y * inv);
  }
}

size_t attn_plain_partial_floats(const LayerDims &L, int T_rows, int n_splits) {
  return (size_t)T_rows * L.n_q_heads * n_splits * (L.head_dim + 2);
}

template <typename T>
void launch_attn_plain(const float *Q, const T *cacheK, const T *cacheV, const SeqMeta *seqs, RowMeta rm,
                       const LayerDims &L, int T_rows, int n_splits, float *partials, T *out, hipStream_t s) {
  if (T_rows == 0) return;
  const int G = L.n_q_heads / L.n_kv_heads, ng = G < ATT_GMAX ? G : ATT_GMAX;
  dim3 grid(T_rows * L.n_kv_heads, n_splits, (G + ATT_GMAX - 1) / ATT_GMAX);
  const size_t tile = (size_t)(ATT_GMAX * L.head_dim + ATT_GMAX * 64), sums = (size_t)4 * ng * L.head_dim;
  const size_t smem = (tile > sums ? tile : sums) * sizeof(float);
  auto of_heads = [&](auto one, auto four, auto more) { return ng == 1 ? one : ng <= 4 ? four : more; };
  auto kern = L.head_dim % 16 != 0 ? attn_partial_kernel<T, 0, 8>
              : L.head_dim <= 64   ? of_heads(attn_partial_kernel<T, 1, 1>, attn_partial_kernel<T, 1, 4>, attn_partial_kernel<T, 1, 8>)
              : L.head_dim <= 128  ? of_heads(attn_partial_kernel<T, 2, 1>, attn_partial_kernel<T, 2, 4>, attn_partial_kernel<T, 2, 8>)
                                   : of_heads(attn_partial_kernel<T, 4, 1>, attn_partial_kernel<T, 4, 4>, attn_partial_kernel<T, 4, 8>);
  hipLaunchKernelGGL(kern, grid, dim3(256), smem, s, Q, cacheK, cacheV, seqs, rm, L, n_splits, partials, out);
}
template void launch_attn_plain<float>(const float *, const float *, const float *, const SeqMeta *, RowMeta,
                                       const LayerDims &, int, int, float *, float *, hipStream_t);
template void launch_attn_plain<bf16>(const float *, const bf16 *, const bf16 *, const SeqMeta *, RowMeta,
                                      const LayerDims &, int, int, float *, bf16 *, hipStream_t);

// Two to eight records of heads of 128, the same number in every row: all of them in one round trip, the maximum from what came with them (the same sums in
// the same order).  1024 rows of 32 heads, four records: 23.2 -> 11.7 us.
template <int N>
__global__ __launch_bounds__(256) void attn_merge_few_kernel(const float *__restrict__ part, int64_t n_rh, bf16 *__restrict__ out) {
  constexpr int h = 128;
  const int lane = threadIdx.x & 63;
  const int64_t rh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (rh >= n_rh) return;
  const float *p = part + rh * N * (h + 2);
  float2 v[N], t[N];      // maximum, row sum
#pragma unroll
  for (int i = 0; i < N; ++i) {
    v[i] = *reinterpret_cast<const float2 *>(p + i * (h + 2) + 2 * lane);
    t[i] = *reinterpret_cast<const float2 *>(p + i * (h + 2) + h);
  }
  float M = t[0].x;
#pragma unroll
  for (int i = 1; i < N; ++i) M = fmaxf(M, t[i].x);
  float denom = 0.f;
  float2 acc = make_float2(0.f, 0.f);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float w = t[i].x == -INFINITY ? 0.f : __expf(t[i].x - M);
    denom += w * t[i].y;
    acc.x += w * v[i].x;
    acc.y += w * v[i].y;
  }
  const float inv = 1.0f / denom;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
  bf16x2_t ov;
  ov[0] = (bf16)(acc.x * inv);
  ov[1] = (bf16)(acc.y * inv);
  *reinterpret_cast<bf16x2_t *>(out + rh * h + lane * 2) = ov;
}

template <typename T>
void launch_attn_merge(const float *partials, const LayerDims &L, int T_rows, int n_splits, MergeCounts mc, T *out, hipStream_t s) {
  if (T_rows == 0) return;
  const int64_t n_rh = (int64_t)T_rows * L.n_q_heads;
  if constexpr (std::is_same<T, bf16>::value) {
    if (mc.counts == nullptr && L.head_dim == 128 && n_splits >= 2 && n_splits <= 8) {
      const dim3 grid((unsigned)((n_rh + 3) / 4));
      switch (n_splits) {
        case 2: hipLaunchKernelGGL(attn_merge_few_kernel<2>, grid, dim3(256), 0, s, partials, n_rh, out); break;
        case 3: hipLaunchKernelGGL(attn_merge_few_kernel<3>, grid, dim3(256), 0, s, partials, n_rh, out); break;
        case 4: hipLaunchKernelGGL(attn_merge_few_kernel<4>, grid, dim3(256), 0, s, partials, n_rh, out); break;
        case 5: hipLaunchKernelGGL(attn_merge_few_kernel<5>, grid, dim3(256), 0, s, partials, n_rh, out); break;
        case 6: hipLaunchKernelGGL(attn_merge_few_kernel<6>, grid, dim3(256), 0, s, partials, n_rh, out); break;
        case 7: hipLaunchKernelGGL(attn_merge_few_kernel<7>, grid, dim3(256), 0, s, partials, n_rh, out); break;
        default: hipLaunchKernelGGL(attn_merge_few_kernel<8>, grid, dim3(256), 0, s, partials, n_rh, out);
      }
      return;
    }
  }
  if (n_splits >= 16 && n_rh <= 512 && L.head_dim <= 128 && L.head_dim % 2 == 0)
    hipLaunchKernelGGL((attn_merge_wide_kernel<T>), dim3((unsigned)n_rh), dim3(256), 0, s, partials, L, n_splits, mc, out);
  else if (n_splits > 16)
    hipLaunchKernelGGL((attn_merge_kernel<T, 32>), dim3((unsigned)((n_rh + 3) / 4)), dim3(256), 0, s, partials, L, n_splits, mc,
                       n_rh, out);
  else
    hipLaunchKernelGGL((attn_merge_kernel<T, 8>), dim3((unsigned)((n_rh + 3) / 4)), dim3(256), 0, s, partials, L, n_splits, mc,
                       n_rh, out);
}
template void launch_attn_merge<float>(const float *, const LayerDims &, int, int, MergeCounts, float *, hipStream_t);
template void launch_attn_merge<bf16>(const float *, const LayerDims &, int, int, MergeCounts, bf16 *, hipStream_t);

// ---------------------------------------------------------------------------------------
template <typename T>
__global__ void silu_mul_kernel(const T *__restrict__ gate, const T *__restrict__ up, T *__restrict__ out,
                                int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    float gv = to_f32<T>(gate[i]);
    float uv = to_f32<T>(up[i]);
    out[i] = from_f32<T>(gv / (1.0f + __expf(-gv)) * uv);
  }
}

template <typename T>
void launch_silu_mul(const T *gate, const T *up, T *out, int64_t n, hipStream_t s) {
  if (n == 0) return;
  int grid = (int)((n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536);
  hipLaunchKernelGGL((silu_mul_kernel<T>), dim3(grid), dim3(256), 0, s, gate, up, out, n);
}
template <typename T>
__global__ void silu_mul_f32_kernel(const float *__restrict__ gate, const float *__restrict__ up, T *__restrict__ out,
                                    int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    const float gv = gate[i];
    out[i] = from_f32<T>(gv / (1.0f + __expf(-gv)) * up[i]);
  }
}
template <typename T>
void launch_silu_mul_f32(const float *gate, const float *up, T *out, int64_t n, hipStream_t s) {
  if (n == 0) return;
  int grid = (int)((n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536);
  hipLaunchKernelGGL((silu_mul_f32_kernel<T>), dim3(grid), dim3(256), 0, s, gate, up, out, n);
}
template void launch_silu_mul_f32<float>(const float *, const float *, float *, int64_t, hipStream_t);
template void launch_silu_mul_f32<bf16>(const float *, const float *, bf16 *, int64_t, hipStream_t);

template <typename T>
__global__ void residual_store_kernel(const float *__restrict__ C, const T *__restrict__ R, T *__restrict__ out,
                                      int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) out[i] = from_f32<T>(C[i] + (R != nullptr ? to_f32<T>(R[i]) : 0.f));
}
template <typename T>
void launch_residual_store(const float *C, const T *R, T *out, int64_t n, hipStream_t s) {
  if (n == 0) return;
  int grid = (int)((n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536);
  hipLaunchKernelGGL((residual_store_kernel<T>), dim3(grid), dim3(256), 0, s, C, R, out, n);
}
template void launch_residual_store<float>(const float *, const float *, float *, int64_t, hipStream_t);
template void launch_residual_store<bf16>(const float *, const bf16 *, bf16 *, int64_t, hipStream_t);
template void launch_silu_mul<float>(const float *, const float *, float *, int64_t, hipStream_t);
template void launch_silu_mul<bf16>(const bf16 *, const bf16 *, bf16 *, int64_t, hipStream_t);

// Gated low-rank term of Eq.6 added to an already computed linear, any shape and dtype:
// C[row, :] += s_a * B_a (A_{a,part} x[row]) for adapted rows (a = row_adapter[row] >= 0).  One workgroup per row.
template <typename T, typename TC>
__global__ __launch_bounds__(256) void lowrank_add_plain_kernel(const T *__restrict__ x, int K, const T *__restrict__ A,
                                                                int parts, int part, const T *__restrict__ B, int N,
                                                                int rank, const int32_t *__restrict__ row_adapter,
                                                                const float *__restrict__ scale, TC *__restrict__ C) {
  __shared__ float t[256];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int a = row_adapter[row];
  if (a < 0) return;
  const T *xr = x + (int64_t)row * K;
  const float sc = scale[a];
  for (int j = wave; j < rank; j += 4) {
    const T *ar = A + (((int64_t)a * parts + part) * rank + j) * K;
    float acc = 0.f;
    for (int c = lane; c < K; c += 64) acc += to_f32<T>(ar[c]) * to_f32<T>(xr[c]);
    acc = wave_sum(acc);
    if (lane == 0) t[j] = acc * sc;
  }
  __syncthreads();
  for (int col = tid; col < N; col += 256) {
    const T *br = B + ((int64_t)a * N + col) * rank;
    float acc = 0.f;
    for (int j = 0; j < rank; ++j) acc += to_f32<T>(br[j]) * t[j];
    const int64_t o = (int64_t)row * N + col;
    C[o] = from_f32<TC>(to_f32<TC>(C[o]) + acc);
  }
}

template <typename T, typename TC>
void launch_lowrank_add_plain(const T *x, int K, const T *A, int parts, int part, const T *B, int N, int rank,
                              const int32_t *row_adapter, const float *scale, TC *C, int M, hipStream_t s) {
  if (M == 0) return;
  hipLaunchKernelGGL((lowrank_add_plain_kernel<T, TC>), dim3(M), dim3(256), 0, s, x, K, A, parts, part, B, N, rank,
                     row_adapter, scale, C);
}
template void launch_lowrank_add_plain<float, float>(const float *, int, const float *, int, int, const float *, int, int,
                                                     const int32_t *, const float *, float *, int, hipStream_t);
template void launch_lowrank_add_plain<bf16, bf16>(const bf16 *, int, const bf16 *, int, int, const bf16 *, int, int,
                                                   const int32_t *, const float *, bf16 *, int, hipStream_t);
template void launch_lowrank_add_plain<bf16, float>(const bf16 *, int, const bf16 *, int, int, const bf16 *, int, int,
                                                    const int32_t *, const float *, float *, int, hipStream_t);

}  // namespace alora
