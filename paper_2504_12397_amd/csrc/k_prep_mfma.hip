// Row preparation (bf16): per-row metadata, RMSNorm, and the low-rank down projection t = s_a * A_a x_hat (Eq.6, Delta applied
// right to left).
//
// Three kernels.  norm_rows: metadata and RMSNorm, a wave per row (or four), for calls without adapters and for many
// rows.  t_rows: t for many rows, from the normalised rows (which the caches still hold).  prep_few: both in one launch for few
// rows, where every round trip and every launch counts: the workgroups of a row tile each normalise it again (registers
// to matrix operand, no memory between) and compute 16 columns of one adapter's t.
// With T rows of four rank-32 adapters at d = 4096 the one kernel that used to do it all (16 rows per workgroup, all columns)
// took 41 us at T = 512 and 81 us at T = 4458.
#include "lds_dma.h"

namespace alora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int PREP_ROWS = 16;
constexpr int PREP_WAVES = 8;
constexpr int PREP_FEW = 512;      // workgroups
constexpr int T_NARROW = 220;      // workgroups, up to which t_rows takes 32 columns each instead of 96 (launch_t_rows_mfma)
constexpr int PREP_NARROW = 128;      // up to so many of 16 columns (half of the compute units) they take 8 columns instead

// Sum of squares of a row, in ONE order for every kernel that normalises rows (a row's x_hat must not depend on
// which of them ran -- the base rows of a long prefill and of a decode step are compared bit for bit): the
// row is cut into 16-byte chunks, chunk index c = 4 CH w + 4 u + g (w < 8, u < CH = d / 256, g < 4); a chunk's eight
// squares are added in order starting from zero; the chunk sums of one (w, g) go through a balanced tree over u
// (neighbours first), the four g of a w through a tree (g ^ 1, then g ^ 2), the eight w are added in order.
__device__ __forceinline__ float chunk_ssq(u32x4 c) {
  const bf16x8 v = __builtin_bit_cast(bf16x8, c);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) { const float f = (float)v[e]; s = __builtin_fmaf(f, f, s); }
  return s;
}
__device__ __forceinline__ float row_rinv(float ssq, int d, float eps) { return 1.0f / sqrtf(ssq / (float)d + eps); }
__device__ __forceinline__ u32x4 norm_chunk(u32x4 x, u32x4 g, float rinv) {
  const bf16x8 xv = __builtin_bit_cast(bf16x8, x), gv = __builtin_bit_cast(bf16x8, g);
  bf16x8 xh;
#pragma unroll
  for (int e = 0; e < 8; ++e) xh[e] = (bf16)((float)xv[e] * (float)gv[e] * rinv);
  return __builtin_bit_cast(u32x4, xh);
}
// Metadata of the rows [row0, tile_end) of one tile: a thread takes a sequence, fetches its record once and fills
// in the rows of the tile that belong to it -- one memory round trip, where a search over the sequence table
// per row costs log2(n_seqs) dependent ones.  s_adapter / s_scale may be nullptr.
__device__ __forceinline__ void fill_row_meta(const PrepArgs &a, const SeqMeta &sm, int sq, int mrow, int row0, bool write,
                                              int *s_adapter, float *s_scale, unsigned long long *s_present) {
  const int pos = sm.P + a.pos_shift + (mrow - sm.row_start);
  int adapter = -1;
  float scale = 0.f;
  if (sm.adapter >= 0 && pos >= sm.k) { adapter = sm.adapter; scale = sm.scale; }
  if (write) {
    a.rm.seq[mrow] = sq;
    a.rm.pos[mrow] = pos;
    a.rm.adapter[mrow] = adapter;
    a.rm.slot[mrow] = sm.pool_off + pos;
  }
  if (s_adapter != nullptr) { s_adapter[mrow - row0] = adapter; s_scale[mrow - row0] = scale; }
  if (adapter >= 0) atomicOr(s_present, 1ull << adapter);
}

// Few rows with adapters (up to PREP_FEW workgroups): workgroup (x, y) takes row tile x % tiles (16 rows), columns NC (x / tiles) .. of the 3 * rank
// columns of t and adapter used[y]; the first of a tile also writes x_hat and the row metadata.  Where there is staged metadata, x begins at 1 and workgroup (0, 0) carries it: in the first
// tile's workgroup its registers left one workgroup a compute unit of d = 2048 instead of two (300 rows of four rank-32 adapters 17 us, before that and so 14.5 and 15; 16 rows of eight rank-64 adapters of d = 4096 13.7, so 11.6).  Eight waves split the hidden dimension; a lane
// owns 8 consecutive elements of one row at a time, which is both the 16-byte global access and the operand layout of
// v_mfma_f32_16x16x32_bf16 (lane l: row l % 16, k = 8 * (l / 16) ..).  CH = d / 256: chunks of its row a lane holds.
// The kernel is memory round trips and little else, so everything is requested at once: x, the gain, the sequences' records (in the kernel arguments when they are few)
// and this adapter's down matrix, before anybody knows whether a row of the tile uses it.
// No load stands behind a branch of its own or is a generic one (the compiler waits for all that was asked for there), and the arguments arrive
// together: as it was compiled before, records, x with the gain, one chunk of A and the rest of A were a round trip each.  One row of one rank-64 adapter
// 10.2 -> 9.0 us, eight rows of eight 11.4 -> 10.5, five rows of rank-8 adapters 10.1 -> 9.2.
// NC = 8: half the columns of the matrix operand, for calls whose 16-column workgroups would leave half of the chip idle: a compute
// unit takes operands in this order at 28 bytes per ns, so it is
// done sooner with half the 128 KB of 16 columns.  A one-row token step of 16 layers at rank 64 2615 -> 2589 us (1.6 a layer), five rows of
// rank-8 adapters 50.7 -> 49.4, 128 rows through 16 layers 4083 -> 4063.  With more workgroups than units the rows would be read twice.
template <int CH, int NC>
__global__ __launch_bounds__(512, 2) void prep_few_kernel(PrepArgs a) {
  __shared__ float s_ssq[PREP_WAVES][PREP_ROWS];
  __shared__ int s_adapter[PREP_ROWS];
  __shared__ float s_scale[PREP_ROWS];
  __shared__ unsigned long long s_present;
  __shared__ u32x4 s_gain[CH * 32];          // d / 8 chunks of the gain
  __shared__ float s_part[PREP_WAVES][PREP_ROWS][17];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kg = lane >> 4;
  const int carries = a.st.src != nullptr ? 1 : 0;
  if (carries && blockIdx.x == 0) {      // (one of each adapter's)
    if (blockIdx.y == 0) {
      Carried<512> staged;
      staged.load(a.st, tid, true);
      staged.store(a.st, tid, true);
    }
    return;
  }
  const int tiles = (a.T + PREP_ROWS - 1) / PREP_ROWS;
  int tile = 0, part = (int)blockIdx.x - carries;      // row tile, columns
  if (tiles > 1) {
    const int at = part;
    part = at / tiles;
    tile = at - part * tiles;
  }
  const int row0 = tile * PREP_ROWS;
  constexpr int d = CH * 256;
  const int rank = a.rank, col0 = part * NC;
  const int ad = (reinterpret_cast<const uint32_t *>(a.used)[blockIdx.y >> 2] >> (8 * (blockIdx.y & 3))) & 255;      // (a scalar load)
  // all arguments in one round trip, not where they are used
  asm volatile("" ::"s"(a.rm.seq), "s"(a.rm.pos), "s"(a.rm.adapter), "s"(a.rm.slot), "s"(a.rm.present16), "s"(a.xh), "s"(a.tlow16), "s"(a.gain),
               "s"(a.packed), "s"(a.eps), "s"(a.write_meta), "s"(a.pos_shift), "s"(a.n_seqs), "s"(ad),
               "s"(a.x), "s"(a.A), "s"(a.rank), "s"(a.T), "s"(a.st.src), "s"(a.st.dst), "s"(a.st.n16));
  const bool lead = part == 0 && blockIdx.y == 0;
  const int row = min(row0 + r16, a.T - 1);
  const bool row_ok = row0 + r16 < a.T;
  const int k_lo = wave * (CH * 32) + kg * 8;  // this lane's first element; chunk u is at k_lo + 32 u

  // this thread's sequence (the first half of its record); of a few sequences, from the kernel arguments
  typedef uint32_t rec16 __attribute__((ext_vector_type(4), aligned(8)));
  const uint64_t recs = a.st.n_few ? (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PrepArgs, st.few) : (uint64_t)a.seqs;
  const auto *rec = reinterpret_cast<const __attribute__((address_space(1))) rec16 *>(recs + (uint64_t)min(tid, a.n_seqs - 1) * sizeof(SeqMeta));
  const u32x4 rec0 = rec[0], rec1 = rec[1];
  u32x4 xr[CH], br[CH];
  const bf16 *xrow = a.x + (int64_t)row * d + k_lo;
#pragma unroll
  for (int u = 0; u < CH; ++u) xr[u] = *reinterpret_cast<const u32x4 *>(xrow + 32 * u);
  // (the gain goes through LDS: one 16-byte chunk per thread instead of CH of them in every lane's registers)
  // (no branch around these loads: behind one the compiler waits for everything that was asked for before)
  const u32x4 gown = *reinterpret_cast<const u32x4 *>((a.gain != nullptr ? a.gain : a.x) + min(tid, d / 8 - 1) * 8);
  const int my_col = min(col0 + r16, 3 * rank - 1);      // (3 * rank need not be a multiple of 16)
  const auto A_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.A + (int64_t)ad * 3 * rank * d), 0, 3 * rank * d * 2, 0x00020000);
  const int A_off = NC == 16 || r16 < NC ? (my_col * d + k_lo) * 2 : 0x7fff0000;      // (lanes without a column: out of range, they read zeros)
#pragma unroll
  for (int u = 0; u < CH; ++u) br[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(A_rsrc, A_off, 64 * u, 0));

  if (tid == 0) s_present = 0ull;
  if (tid < PREP_ROWS) { s_adapter[tid] = -1; s_scale[tid] = 0.f; }
  __syncthreads();
  const int tile_end = min(row0 + PREP_ROWS, a.T);
  auto fill_row = [&](const SeqMeta &sm, int sq, int mrow) {
    fill_row_meta(a, sm, sq, mrow, row0, a.write_meta && lead, s_adapter, s_scale, &s_present);
  };
  auto fill = [&](const SeqMeta &sm, int sq) {
    const int lo = max(sm.row_start, row0), hi = min(sm.row_start + sm.n_new, tile_end);
    for (int mrow = lo; mrow < hi; ++mrow) fill_row(sm, sq, mrow);
  };
  if (tid < a.n_seqs) {
    SeqMeta sm{};
    sm.row_start = (int)rec0[0]; sm.n_new = (int)rec0[1]; sm.P = (int)rec0[2]; sm.k = (int)rec0[3];
    sm.adapter = (int)rec1[0]; sm.scale = __uint_as_float(rec1[1]); sm.pool_off = (int64_t)((uint64_t)rec1[3] << 32 | rec1[2]);
    fill(sm, tid);
  }
  for (int sq = tid + 512; sq < a.n_seqs; sq += 512) fill(a.seqs[sq], sq);      // (a few have fewer)

  if (a.gain != nullptr) {
    float cs[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) cs[u] = chunk_ssq(xr[u]);
#pragma unroll
    for (int st = 1; st < CH; st *= 2)
#pragma unroll
      for (int u = 0; u < CH; u += 2 * st) cs[u] += cs[u + st];
    float ssq = cs[0];
    ssq += __shfl_xor(ssq, 16, 64);
    ssq += __shfl_xor(ssq, 32, 64);
    if (kg == 0) s_ssq[wave][r16] = ssq;
    if (tid < d / 8) s_gain[tid] = gown;
  }
  __syncthreads();
  if (lead && tid == 0 && a.rm.present16 != nullptr) a.rm.present16[tile] = s_present;
  if (a.gain != nullptr) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < PREP_WAVES; ++w) t += s_ssq[w][r16];
    const float rinv = row_rinv(t, d, a.eps);
#pragma unroll
    for (int u = 0; u < CH; ++u) xr[u] = norm_chunk(xr[u], s_gain[(k_lo >> 3) + 4 * u], rinv);
  }
  if (lead && row_ok) {
    u32x4 *dst = reinterpret_cast<u32x4 *>(a.xh);
#pragma unroll
    for (int u = 0; u < CH; ++u) dst[xh_chunk(row, (k_lo >> 3) + 4 * u, d, a.packed)] = xr[u];
  }
  if (!((s_present >> ad) & 1)) return;

  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool mine = s_adapter[r16] == ad;
#pragma unroll
  for (int u = 0; u < CH; ++u) {
    const u32x4 au = mine ? xr[u] : u32x4{0, 0, 0, 0};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, au), __builtin_bit_cast(bf16x8, br[u]), acc, 0, 0, 0);
  }
  // accumulator register v of lane l is T[row 4*(l/16) + v][column l%16]
#pragma unroll
  for (int v = 0; v < 4; ++v) s_part[wave][4 * kg + v][r16] = acc[v];
  __syncthreads();
  if (tid < PREP_ROWS * 16) {
    const int lr = tid >> 4, col = tid & 15, orow = row0 + lr;
    if (orow < a.T && s_adapter[lr] == ad && col < NC && col0 + col < 3 * rank) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < PREP_WAVES; ++w) t += s_part[w][lr][col];
      t *= s_scale[lr];
      const int p = (col0 + col) / rank, jj = (col0 + col) % rank;
      const bf16 hi = (bf16)t;
      bf16 *dst = a.tlow16 + (((int64_t)orow * 3 + p) * 2) * rank + jj;
      dst[0] = hi;
      dst[rank] = (bf16)(t - (float)hi);
    }
  }
}

// Tree over u, neighbours first, for N rows at once: while there are several a lane keeps half of them and gives the other half for its partner's.
template <int N, int O, int GL> __device__ __forceinline__ float tree_of_rows(const float (&v)[N], int lane, int &row) {
  if constexpr (O >= GL) {
    return v[0];
  } else if constexpr (N > 1) {
    const bool high = lane & O;
    float k[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) k[i] = (high ? v[N / 2 + i] : v[i]) + __shfl_xor(high ? v[i] : v[N / 2 + i], O, 64);
    row = row * 2 + (high ? 1 : 0);
    return tree_of_rows<N / 2, O * 2, GL>(k, lane, row);
  } else {
    const float k[1] = {v[0] + __shfl_xor(v[0], O, 64)};
    return tree_of_rows<1, O * 2, GL>(k, lane, row);
  }
}
// The same for at most RT rows (RT = 2, 4, 8): a thread has one chunk of each of them, not a lane sixteen of one row, of which lanes without a row repeat the last
// one.  With one row that was 128 elements per lane to square, scale and convert, sixteen times over; now it is 8.  x_hat goes through LDS, chunk c of row r
// at c ^ r, to become the matrix operand.  Sums as above, bit for bit.
// The kernel, us, sixteen rows a tile -> so: one row of a rank-64 adapter 9.6 -> 6.6, four rows of four 9.8 -> 7.4, five of five 9.8 -> 8.6, eight of eight 10.3 -> 9.2; five
// rows of four rank-8 adapters 9.7 -> 8.8.
template <int CH, int NC, int RT>
__global__ __launch_bounds__(512, 2) void prep_few_rows_kernel(PrepArgs a) {
  constexpr int d = CH * 256, NCHUNK = d / 8, GL = 4 * CH;      // GL: chunks (neighbouring lanes) of one w
  static_assert(4 * RT <= GL, "");
  __shared__ float s_ssq[RT][PREP_WAVES];
  __shared__ int s_adapter[PREP_ROWS];
  __shared__ float s_scale[PREP_ROWS];
  __shared__ unsigned long long s_present;
  __shared__ u32x4 s_x[RT * NCHUNK];
  __shared__ float s_part[PREP_WAVES][PREP_ROWS][17];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kg = lane >> 4;
  const int rank = a.rank, col0 = blockIdx.y * NC;
  const int ad = (reinterpret_cast<const uint32_t *>(a.used)[blockIdx.z >> 2] >> (8 * (blockIdx.z & 3))) & 255;      // (a scalar load)
  // all arguments in one round trip, not where they are used
  asm volatile("" ::"s"(a.rm.seq), "s"(a.rm.pos), "s"(a.rm.adapter), "s"(a.rm.slot), "s"(a.rm.present16), "s"(a.xh), "s"(a.tlow16), "s"(a.gain),
               "s"(a.packed), "s"(a.eps), "s"(a.write_meta), "s"(a.pos_shift), "s"(a.n_seqs), "s"(ad),
               "s"(a.x), "s"(a.A), "s"(a.rank), "s"(a.T), "s"(a.st.src), "s"(a.st.dst), "s"(a.st.n16));
  const bool lead = blockIdx.y == 0 && blockIdx.z == 0;
  const int c = min(tid, NCHUNK - 1);

  // (requests as in the kernel above: none behind a branch)
  typedef uint32_t rec16 __attribute__((ext_vector_type(4), aligned(8)));
  const uint64_t recs = a.st.n_few ? (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PrepArgs, st.few) : (uint64_t)a.seqs;
  const auto *rec = reinterpret_cast<const __attribute__((address_space(1))) rec16 *>(recs + (uint64_t)min(tid, a.n_seqs - 1) * sizeof(SeqMeta));
  const u32x4 rec0 = rec[0], rec1 = rec[1];
  u32x4 xr[RT], br[CH];
#pragma unroll
  for (int r = 0; r < RT; ++r) xr[r] = *reinterpret_cast<const u32x4 *>(a.x + (int64_t)min(r, a.T - 1) * d + c * 8);
  const u32x4 gain = *reinterpret_cast<const u32x4 *>((a.gain != nullptr ? a.gain : a.x) + c * 8);
  const int my_col = min(col0 + r16, 3 * rank - 1), k_lo = wave * (CH * 32) + kg * 8;
  const auto A_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.A + (int64_t)ad * 3 * rank * d), 0, 3 * rank * d * 2, 0x00020000);
  const int A_off = NC == 16 || r16 < NC ? (my_col * d + k_lo) * 2 : 0x7fff0000;
#pragma unroll
  for (int u = 0; u < CH; ++u) br[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(A_rsrc, A_off, 64 * u, 0));
  Carried<512> staged;
  staged.load(a.st, tid, lead);      // (host memory: behind what everybody waits for)

  if (tid == 0) s_present = 0ull;
  if (tid < PREP_ROWS) { s_adapter[tid] = -1; s_scale[tid] = 0.f; }
  __syncthreads();
  auto fill = [&](const SeqMeta &sm, int sq) {
    for (int mrow = sm.row_start; mrow < min(sm.row_start + sm.n_new, a.T); ++mrow)
      fill_row_meta(a, sm, sq, mrow, 0, a.write_meta && lead, s_adapter, s_scale, &s_present);
  };
  if (tid < a.n_seqs) {
    SeqMeta sm{};
    sm.row_start = (int)rec0[0]; sm.n_new = (int)rec0[1]; sm.P = (int)rec0[2]; sm.k = (int)rec0[3];
    sm.adapter = (int)rec1[0]; sm.scale = __uint_as_float(rec1[1]); sm.pool_off = (int64_t)((uint64_t)rec1[3] << 32 | rec1[2]);
    fill(sm, tid);
  }
  for (int sq = tid + 512; sq < a.n_seqs; sq += 512) fill(a.seqs[sq], sq);

  if (a.gain != nullptr) {
    float v[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) v[r] = chunk_ssq(xr[r]);
    int row = 0;
    float sum = tree_of_rows<RT, 4, GL>(v, lane, row);
    sum += __shfl_xor(sum, 1, 64);      // tree over g
    sum += __shfl_xor(sum, 2, 64);
    if (tid < NCHUNK && (lane % GL & ~(4 * (RT - 1))) == 0) s_ssq[row][tid / GL] = sum;
  }
  __syncthreads();
  if (lead && tid == 0 && a.rm.present16 != nullptr) a.rm.present16[0] = s_present;
  if (a.gain != nullptr) {
    float t = 0.f;      // of row lane % RT
#pragma unroll
    for (int w = 0; w < PREP_WAVES; ++w) t += s_ssq[lane % RT][w];
    const float rinv = row_rinv(t, d, a.eps);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      xr[r] = norm_chunk(xr[r], gain, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rinv), r)));
    }
  }
  if (tid < NCHUNK) {
#pragma unroll
    for (int r = 0; r < RT; ++r) s_x[r * NCHUNK + (tid ^ r)] = xr[r];
    if (lead) {
      u32x4 *dst = reinterpret_cast<u32x4 *>(a.xh) + xh_chunk(0, tid, d, a.packed);
      const int step = a.packed ? 1 : NCHUNK;      // (all rows are in the first block of 32)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        if (r < a.T) dst[r * step] = xr[r];
    }
  }
  staged.store(a.st, tid, lead);
  if (!((s_present >> ad) & 1)) return;
  __syncthreads();

  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool mine = s_adapter[r16] == ad;      // (no row: -1)
  const u32x4 *xa = s_x + (r16 % RT) * NCHUNK;
#pragma unroll
  for (int u = 0; u < CH; ++u) {
    const u32x4 au = mine ? xa[((k_lo >> 3) + 4 * u) ^ (r16 % RT)] : u32x4{0, 0, 0, 0};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, au), __builtin_bit_cast(bf16x8, br[u]), acc, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) s_part[wave][4 * kg + v][r16] = acc[v];
  __syncthreads();
  if (tid < RT * 16) {
    const int row = tid >> 4, col = tid & 15;
    if (row < a.T && s_adapter[row] == ad && col < NC && col0 + col < 3 * rank) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < PREP_WAVES; ++w) t += s_part[w][row][col];
      t *= s_scale[row];
      const int p = (col0 + col) / rank, jj = (col0 + col) % rank;
      const bf16 hi = (bf16)t;
      bf16 *dst = a.tlow16 + (((int64_t)row * 3 + p) * 2) * rank + jj;
      dst[0] = hi;
      dst[rank] = (bf16)(t - (float)hi);
    }
  }
}

// Metadata and RMSNorm, four waves per workgroup, RW rows per wave.  A wave takes its rows whole -- every load and
// store instruction covers 1 KB of one row -- and the only wait besides the rows themselves is the sequences' records.  One row
// per wave (four per workgroup, so that a few hundred rows reach every compute unit: 512 rows 12 -> 8.4 us against 16 rows per workgroup), four
// rows (32 KB in flight) for long calls.  Memory-bound: 21 us at 4096 rows of 4096.  The first workgroup of 16 rows sees to their metadata.
// Lane l holds the chunks c = l + 64 j: in the terms of chunk_ssq's order, a lane group of 4 CH lanes is one w.
template <int CH, int RW>
__global__ __launch_bounds__(256) void norm_rows_kernel(PrepArgs a) {
  __shared__ unsigned long long s_present;
  constexpr int NT = 256;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Staged metadata comes from host memory: a workgroup of its own, the first, carries it beside the others' rows (one row of 4096 6.7 -> 4.7 us against the rows' first workgroup doing
  // so behind them; of 512 4.2 -> 3.3, with 9 KB 7.8 -> 3.4).
  const int carries = a.st.src != nullptr ? 1 : 0;
  if (carries && blockIdx.x == 0) {
    Carried<NT> staged;
    staged.load(a.st, tid, true);
    staged.store(a.st, tid, true);
    return;
  }
  const int row0 = ((int)blockIdx.x - carries) * (4 * RW);
  constexpr int D = CH * 256, NJ = D / 512;
  const int wrow0 = row0 + wave * RW;
  u32x4 xr[RW][NJ], gr[NJ];
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int row = min(wrow0 + i, a.T - 1);      // rows past the end repeat the last one and are not stored
    const bf16 *xrow = a.x + (int64_t)row * D + lane * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) xr[i][j] = *reinterpret_cast<const u32x4 *>(xrow + 512 * j);
  }
  if (a.gain != nullptr) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) gr[j] = *reinterpret_cast<const u32x4 *>(a.gain + lane * 8 + 512 * j);
  }
  if (a.seqs != nullptr && a.write_meta && row0 % PREP_ROWS == 0) {
    if (tid == 0) s_present = 0ull;
    __syncthreads();
    const int tile_end = min(row0 + PREP_ROWS, a.T);
    for (int sq = tid; sq < a.n_seqs; sq += NT) {
      const SeqMeta sm = a.st.n_few ? a.st.few[sq] : a.seqs[sq];
      const int lo = max(sm.row_start, row0), hi = min(sm.row_start + sm.n_new, tile_end);
      for (int mrow = lo; mrow < hi; ++mrow) fill_row_meta(a, sm, sq, mrow, row0, true, nullptr, nullptr, &s_present);
    }
    __syncthreads();
    if (tid == 0 && a.rm.present16 != nullptr) a.rm.present16[row0 / PREP_ROWS] = s_present;
  }
  constexpr int GL = 4 * CH, GW = 64 / GL;      // lanes of one w, and how many w a chunk row j of the wave covers
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    if (a.gain != nullptr) {
      float t = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float v = chunk_ssq(xr[i][j]);
#pragma unroll
        for (int o = 4; o < GL; o *= 2) v += __shfl_xor(v, o, 64);      // tree over u, neighbours first
        v += __shfl_xor(v, 1, 64);                                     // tree over g
        v += __shfl_xor(v, 2, 64);
#pragma unroll
        for (int w = 0; w < GW; ++w) t += GW == 1 ? v : __shfl(v, w * GL, 64);      // the eight w in order
      }
      const float rinv = row_rinv(t, D, a.eps);
#pragma unroll
      for (int j = 0; j < NJ; ++j) xr[i][j] = norm_chunk(xr[i][j], gr[j], rinv);
    }
    if (wrow0 + i < a.T) {
      u32x4 *dst = reinterpret_cast<u32x4 *>(a.xh);
#pragma unroll
      for (int j = 0; j < NJ; ++j) dst[xh_chunk(wrow0 + i, lane + 64 * j, D, a.packed)] = xr[i][j];
    }
  }
}

// t of many rows from x_hat (or from the input of another linear with `parts` down-matrices): workgroup (x, y, z) takes 32 rows, columns 32 NB y .. of the parts * rank and adapter used[z]; it leaves at
// once when no row of its tile uses that adapter.  What bounds it: down matrix and rows through one compute unit, which
// loads to registers in operand order brought in at 28 bytes per ns; requests to LDS arrive at 50 to 130.  So 96 columns per workgroup
// (1 MB) only where 32 columns (0.5 MB) would make more workgroups than the chip takes at once: 512 rows of four
// adapters 20.5 -> 11.3 us, 1024 rows at rank 64 23 -> 17, 8131 rows of which 127 are adapted 20.5 -> 11.6; 4458 rows 24.6 with 96, 31.7 with 32.  128 values of k per
// step, RING steps on their way; wave w multiplies the 16 values 16 w .. of a step, the eight sums are added in wave order.
// LDS rows are 256 bytes, chunk c of row i at c ^ (i & 15); x_hat in operand order needs no rows (1 KB per 16 values of k).
template <int NB> struct TRows { static constexpr int STEP = (1 + NB) * 8192, RING = NB == 1 ? 8 : 4, LDS = RING * STEP > 8 * 32 * 100 * 4 ? RING * STEP : 8 * 32 * 100 * 4; };
template <int NB>
__global__ __launch_bounds__(512) void t_rows_kernel(PrepArgs a) {
  constexpr int T_STEP = TRows<NB>::STEP, RING = TRows<NB>::RING;
  extern __shared__ u32x4 smem[];
  char *lds = reinterpret_cast<char *>(smem);
  typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int row0 = blockIdx.x * 32, ad = a.used[blockIdx.z], cols = a.parts * a.rank, d = a.d;
  const int col0 = blockIdx.y * (32 * NB), nb = min(NB, (cols - col0 + 31) / 32);
  const int my_row = row0 + (tid >> 4), mine = a.rm.adapter[min(my_row, a.T - 1)];      // (of the row this thread finishes)
  const int g0 = row0 / 16, g1 = min(g0 + 1, (a.T - 1) / 16);
  if (!(((a.rm.present16[g0] | a.rm.present16[g1]) >> ad) & 1)) return;

  const i32x4 rx = make_rsrc(a.xh + (int64_t)row0 * d, (uint64_t)32 * d * 2);      // (this tile's rows: offsets are 32 bits wide)
  const i32x4 rw = make_rsrc(a.A + ((int64_t)ad * cols + col0) * d, (uint64_t)(cols - col0) * d * 2);      // rows past the end: zeros
  const int r4 = lane >> 4, pos = lane & 15;
  int vx, vw[NB];
  if (a.packed) vx = wave * 1024 + lane * 16;
  else vx = min(4 * wave + r4, a.T - 1 - row0) * d * 2 + (pos ^ ((4 * wave + r4) & 15)) * 16;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int i = 4 * (NB * wave + j) + r4;
    vw[j] = i * d * 2 + (pos ^ (i & 15)) * 16;
  }
  const int steps = d / 128, x_step = a.packed ? 8 * 1024 : 256;
  auto req = [&](int s) {
    const int t = min(s, steps - 1), dst = (s & (RING - 1)) * T_STEP;      // (past the end: the last step again, which nobody reads)
    load_to_lds(rx, vx, t * x_step, dst + wave * 1024);
#pragma unroll
    for (int j = 0; j < NB; ++j) load_to_lds(rw, vw[j], t * 256, dst + 8192 + (NB * wave + j) * 1024);
  };
  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
  const int at = ((2 * wave + lhi) ^ (l32 & 15)) * 16, xa = a.packed ? wave * 1024 + lane * 16 : l32 * 256 + at;
  for (int s = 0; s < RING - 1; ++s) req(s);
  for (int s = 0; s < steps; ++s) {
    wait_vm<(RING - 2) * (1 + NB)>();
    wave_barrier();      // step s is there, step s - 1 used up
    const char *b = lds + (s & (RING - 1)) * T_STEP;
    const bf16x8 x = *reinterpret_cast<const bf16x8 *>(b + xa);
    bf16x8 w[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) w[j] = *reinterpret_cast<const bf16x8 *>(b + 8192 + (32 * j + l32) * 256 + at);
    req(s + RING - 1);
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[j], x, acc[j], 0, 0, 0);
  }
  wait_vm<0>();
  wave_barrier();      // the ring becomes the place of the eight sums: [wave][row][100]
  // weights first: register v of lane l is column 8 (v / 4) + 4 (l / 32) + v % 4 of row l % 32
  float *part = reinterpret_cast<float *>(lds);
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4 *>(part + (wave * 32 + l32) * 100 + 32 * j + 8 * q + 4 * lhi) =
          make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
  __syncthreads();
  const float scale = a.used_scale[blockIdx.z];
  const int rank = a.rank;
  for (int i = 0; i < 2 * nb; ++i) {
    const int lc = 16 * i + (tid & 15), col = col0 + lc;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < PREP_WAVES; ++w) t += part[(w * 32 + (tid >> 4)) * 100 + lc];
    t *= scale;
    if (my_row < a.T && col < cols && mine == ad) {
      const int p = col / rank, jj = col % rank;
      const bf16 hi = (bf16)t;
      bf16 *dst = a.tlow16 + (((int64_t)my_row * a.parts + p) * 2) * rank + jj;
      dst[0] = hi;
      dst[rank] = (bf16)(t - (float)hi);
    }
  }
}

bool prep_rows_mfma_supported(int d, int rank) {
  return (d == 4096 || d == 2048 || d == 1024 || d == 512) && rank % 8 == 0;
}

template <int CH>
static void launch_norm(const PrepArgs &a, hipStream_t s) {
  // (us, one row a wave / four: d = 4096: 2500 rows 17.2 / 21.6, 4458 17.3 / 21.6, 6000 25.8 / 23.7, 8131 33 / 30; 2049 and 5000 rows of d = 2048 7.7 / 9.9 and 10.3 / 13.3, of 1024 6.6 / 7.3 and 7.5 / 9.2, of 512 alike)
  const int carries = a.st.src != nullptr ? 1 : 0;
  if (a.T <= 5000) hipLaunchKernelGGL((norm_rows_kernel<CH, 1>), dim3((a.T + 3) / 4 + carries), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((norm_rows_kernel<CH, 4>), dim3((a.T + 15) / 16 + carries), dim3(256), 0, s, a);
}

template <int NB>
static void launch_t_rows(const PrepArgs &a, hipStream_t s) {
  auto kern = t_rows_kernel<NB>;
  (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, TRows<NB>::LDS);
  hipLaunchKernelGGL(kern, dim3((a.T + 31) / 32, (a.parts * a.rank + 32 * NB - 1) / (32 * NB), a.n_used), dim3(512), TRows<NB>::LDS, s, a);
}

bool t_rows_mfma_supported(const PrepArgs &a) { return a.d % 128 == 0 && lds_aligned(a.A) && lds_aligned(a.xh); }

void launch_t_rows_mfma(const PrepArgs &a, hipStream_t s) {
  // Those with something to do, and a fiftieth of the others (each of them holds a compute unit's LDS for a moment): the least loss over 700 products of
  // 8 to 4458 rows, 1 to 16 adapters of rank 16 to 64, all or a tenth of the rows adapted, K 2048 to 8192: 0.3 % on average against the quicker
  // one of the two each time, 14 % at most.  Counting adapted rows instead 0.5 % and 73 %: 1000 rows of eight rank-64 adapters are 234 workgroups
  // with something to do and 1302 others, row preparation 33 us in 96 columns, 54 in 32.
  const int cols = (a.parts * a.rank + 31) / 32, busy = a.adapted_tiles * cols, all = (a.T + 31) / 32 * cols * a.n_used;
  if (busy + (all - busy) / 50 <= T_NARROW) launch_t_rows<1>(a, s);
  else launch_t_rows<3>(a, s);
}

template <int CH>
static void launch_prep_ch(const PrepArgs &a, hipStream_t s) {
  const int row_tiles = (a.T + PREP_ROWS - 1) / PREP_ROWS, cols16 = (3 * a.rank + 15) / 16;
  if (a.rank == 0 || a.A == nullptr || a.n_used == 0) {
    launch_norm<CH>(a, s);
  } else if (a.few == 2 || !lds_aligned(a.A) || (a.few == 1 && row_tiles * cols16 * a.n_used <= PREP_FEW)) {
    const int carries = a.st.src != nullptr ? 1 : 0;      // (prep_few_kernel only)
    const dim3 narrow(1, (3 * a.rank + 7) / 8, a.n_used);
    const bool rows = CH >= 8 && cols16 * a.n_used <= PREP_NARROW;
    if (rows && a.T <= 2)
      hipLaunchKernelGGL((prep_few_rows_kernel<CH < 8 ? 8 : CH, 8, 2>), narrow, dim3(512), 0, s, a);
    else if (rows && a.T <= 4)
      hipLaunchKernelGGL((prep_few_rows_kernel<CH < 8 ? 8 : CH, 8, 4>), narrow, dim3(512), 0, s, a);
    else if (rows && a.T <= 8)
      hipLaunchKernelGGL((prep_few_rows_kernel<CH < 8 ? 8 : CH, 8, 8>), narrow, dim3(512), 0, s, a);
    else if (row_tiles * cols16 * a.n_used <= PREP_NARROW)
      hipLaunchKernelGGL((prep_few_kernel<CH, 8>), dim3(row_tiles * ((3 * a.rank + 7) / 8) + carries, a.n_used), dim3(512), 0, s, a);
    else
      hipLaunchKernelGGL((prep_few_kernel<CH, 16>), dim3(row_tiles * cols16 + carries, a.n_used), dim3(512), 0, s, a);
  } else {
    launch_norm<CH>(a, s);
    launch_t_rows_mfma(a, s);
  }
}

void launch_prep_rows_mfma(const PrepArgs &a, hipStream_t s) {
  if (a.T == 0) return;
  switch (a.d) {
    case 4096: launch_prep_ch<16>(a, s); break;
    case 2048: launch_prep_ch<8>(a, s); break;
    case 1024: launch_prep_ch<4>(a, s); break;
    case 512: launch_prep_ch<2>(a, s); break;
    default: break;
  }
}

}  // namespace alora
