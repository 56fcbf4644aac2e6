// Decode attention (Eq.4: one new query per sequence over its whole cache), memory-bound:
// every cached key/value byte is read exactly once and everything else is kept out of the way.
//
// Work item: one workgroup of eight waves = (rows, range of keys), listed by the host with the pool rows it reads, so that a
// wave requests keys as soon as it has its item.  Wave w takes kv head g0 + w % HW and sub-range w / HW of the item's keys.
// HW = 8 kv heads side by side read whole 2 KB token rows of the token-major cache, and the waves never meet.  HW = 2 with four
// sub-ranges that join in LDS: every wave's chain of 32-key steps is a quarter as long and a head still has few partial records
// (one row of 16448 keys: 24 us, 27 with eight heads and 172 records).  The host cuts the keys and takes the form that is
// quicker for the call.  Normally an item is one row (one sequence's new token) over that sequence's own cache rows.  Sequences
// that name the same shared prefix (Section 2, "Cache reuse patterns": several adapters on one context) are packed 32 / G to an
// item for the prefix part: their heads fill the MFMA columns a single sequence leaves empty (NC blocks of 16), and the prefix
// is read from memory once for all of them.  A wave consumes 32 keys per step:
//   * K rows go from global memory straight into the A operand of v_mfma_f32_16x16x32_bf16
//     (lane l: key l%16, head-dim slice 8*(l/16)..+7 of the current 32-wide k-step), the G query
//     heads of the group are the (zero padded) 16 B-operand columns: S^T[key][head].
//   * Accumulator register v of lane l is S^T[key 4*(l/16)+v][head l%16]: a lane owns one head, so
//     max / sum / rescale are per-lane scalars, and the two key blocks' probabilities
//     p[16u + 4*(l/16) + v] are, as they sit, the B operand (k = 32 keys) of O^T += V^T P^T.
//   * V rows are loaded as 8 columns x 1 key per lane (16 B) for exactly those 8 keys and
//     transposed inside the lane with byte permutes: MFMA number c uses column 8*i + c of lane
//     row i, so O^T_c[i][head] = O[column 8*i + c][head].  No LDS, no cross-lane traffic.
// Every MFMA operand is fp16, as in the prefill kernel: the queries arrive as fp16, the bf16 cache rows are
// converted in registers on their way into the operands (exact; the V conversion packs two keys of one column into
// a word, which is the transposition) and the probabilities are packed to fp16.  The kernel waits for memory, the
// vector ALU has the time, and the rounding of bf16 queries and probabilities was most of the error.
// Partials (acc, max, sum) per (row, head, split) are merged by the log-sum-exp merge kernel.
#include "mfma_kernels.h"

namespace alora {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// two floats as an fp16 pair (round toward zero: finite stays finite; exact for bf16 values)
__device__ __forceinline__ uint32_t dec_pack2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}
__device__ __forceinline__ float dec_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float dec_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
__device__ __forceinline__ u32x4 dec_bf16x8_to_f16x8(u32x4 r) {
  return u32x4{dec_pack2(dec_lo(r.x), dec_hi(r.x)), dec_pack2(dec_lo(r.y), dec_hi(r.y)),
               dec_pack2(dec_lo(r.z), dec_hi(r.z)), dec_pack2(dec_lo(r.w), dec_hi(r.w))};
}

// acc + lo + hi of a packed fp16 pair
__device__ __forceinline__ float dec_sum2(uint32_t pair, float acc) {
  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, pair), __builtin_bit_cast(half2_t, 0x3c003c00u), acc, false);
}

constexpr float DEC_LOG2E = 1.4426950408889634f;
constexpr float DEC_LN2 = 0.6931471805599453f;

// SHORT: at most 32 keys an item (the own keys of a run of decode steps).  Nothing to ask for ahead: without the copies two workgroups share a
// compute unit.  1024 rows of 1 to 16 keys: 32 -> 19 us (of these 23 -> 19 for asking for the first 16 keys only).
template <int NC, bool SHORT = false>
__global__ __launch_bounds__(512, SHORT ? 4 : 2) void attn_decode_mfma_kernel(DecodeArgs a) {
  constexpr int H = 128;
  extern __shared__ float s_o[];           // [wave][column < cols_max][acc..., m, l], several sub-ranges only

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kg = lane >> 4;           // j: head column / key row / V row; kg: k group
  // The item in one round trip: as whole words, which are scalar loads (its 16-bit fields are not, and the first of them was waited for by itself).
  const int32_t *iw = reinterpret_cast<const int32_t *>(a.items + blockIdx.x);
  const int32_t w0 = iw[0], w1 = iw[1], w2 = iw[2], w3 = iw[3], w4 = iw[4], w5 = iw[5], w6 = iw[6], w7 = iw[7];
  static_assert(sizeof(DecItem) == 32 && offsetof(DecItem, n_rows) == 20 && offsetof(DecItem, shared) == 26 && offsetof(DecItem, n_keys) == 28, "");
  DecItem it;
  it.key_row0 = (int64_t)((uint64_t)(uint32_t)w1 << 32 | (uint32_t)w0);
  it.row = w2; it.kbeg = w3; it.kend = w4;
  it.n_rows = (int16_t)w5; it.g = (int16_t)(w5 >> 16); it.part = (int16_t)w6; it.shared = (int16_t)(w6 >> 16); it.n_keys = w7;
  // (and the arguments with it: a round trip less before the first keys are asked for.  0.2 to 0.4 us of every launch: five short rows 12.8 -> 12.6 us,
  // one row on 32896 keys 28.9 -> 28.6, eight on a context of 32768 39.3 -> 38.9)
  asm volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(w3), "s"(w4), "s"(w5), "s"(w6), "s"(w7), "s"(a.Q), "s"(a.K), "s"(a.V), "s"(a.rows), "s"(a.partials), "s"(a.n_q), "s"(a.n_kv),
               "s"(a.n_q_heads), "s"(a.n_kv_heads), "s"(a.heads_per_wg), "s"(a.ranges_per_wg), "s"(a.cols_max), "s"(a.pos_shift), "s"(a.n_parts));
  if (it.n_rows == 0) return;
  const int HW = a.heads_per_wg, KR = a.ranges_per_wg, CM = a.cols_max;
  const int hw = wave % HW, sub = wave / HW;
  const bool active = sub < KR && it.g + hw < a.n_kv_heads;      // (a workgroup may hold fewer than eight (head, range) pairs)
  const int g = min(it.g + hw, a.n_kv_heads - 1);
  const int G = a.n_q_heads / a.n_kv_heads;
  const int n_cols = it.n_rows * G;                 // MFMA columns in use: column = row index * G + head
  const int item_end = it.shared ? it.kend : min(it.kend, it.n_keys + a.pos_shift);
  // keys of this sub-range: contiguous, multiple of 32
  int per = (item_end - it.kbeg + KR - 1) / KR;
  per = (per + 31) & ~31;
  const int kbeg = it.kbeg + sub * per, kend = active ? min(item_end, kbeg + per) : kbeg;
  const bf16 *Kp = a.K + it.key_row0 * a.n_kv + g * H;
  const bf16 *Vp = a.V + it.key_row0 * a.n_kv + g * H;
  auto row_of = [&](int rj) { return it.shared ? a.rows[it.row + rj] : it.row; };

  u32x4 kr[2][4], vr[2][4];      // [key block u][k-step s] and [u][n]: key 16u + 4kg + n
  const bool one_block = SHORT && it.kend - it.kbeg <= 16;      // (the second 16 keys are then not asked for)
  auto load_k = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && one_block) {
#pragma unroll
        for (int s = 0; s < 4; ++s) kr[1][s] = u32x4{0, 0, 0, 0};
        break;
      }
      const int kk = min(k0 + 16 * u + j, item_end - 1);
#pragma unroll
      for (int s = 0; s < 4; ++s)
        kr[u][s] = *reinterpret_cast<const u32x4 *>(Kp + (int64_t)kk * a.n_kv + 32 * s + 8 * kg);
    }
  };
  auto load_v = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        if (u == 1 && one_block) { vr[1][n] = u32x4{0, 0, 0, 0}; continue; }
        const int kv = min(k0 + 16 * u + 4 * kg + n, item_end - 1);
        vr[u][n] = *reinterpret_cast<const u32x4 *>(Vp + (int64_t)kv * a.n_kv + 8 * j);
      }
  };
  if (kbeg < kend) { load_k(kbeg); load_v(kbeg); }

  // queries: B operand columns = (row, head of the group) pairs (zero for padding columns)
  u32x4 qf[NC][4];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    const int col = 16 * nc + j, rj = col / G, hj = col - rj * G;
    const int qrow = row_of(col < n_cols ? rj : 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      qf[nc][s] = u32x4{0, 0, 0, 0};
      if (col < n_cols) qf[nc][s] = *reinterpret_cast<const u32x4 *>(a.Q + (int64_t)qrow * a.n_q + (g * G + hj) * H + 32 * s + 8 * kg);
    }
  }

  f32x4 o[NC][8];
  float m_run[NC], l_run[NC];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
#pragma unroll
    for (int c = 0; c < 8; ++c) o[nc][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[nc] = -INFINITY;
    l_run[nc] = 0.f;
  }
  const float c_scale = a.sm_scale * DEC_LOG2E;

  for (int k0 = kbeg; k0 < kend; k0 += 32) {
    f32x4 sc[NC][2];
    u32x4 vc[2][4];
    if constexpr (NC == 1 && !SHORT) {
      // consume copies of this step's registers and refill them for the next step at once: 16 KB per wave on the way
      u32x4 kc[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int s = 0; s < 4; ++s) { kc[u][s] = kr[u][s]; vc[u][s] = vr[u][s]; }
      load_k(k0 + 32);      // unconditional: key indices are clamped to the last valid row
      load_v(k0 + 32);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        sc[0][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          sc[0][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, dec_bf16x8_to_f16x8(kc[u][s])),
                                                            __builtin_bit_cast(f16x8, qf[0][s]), sc[0][u], 0, 0, 0);
      }
    } else {
      // two blocks of columns leave no registers for copies: keys and values are refilled each after their own products
#pragma unroll
      for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) sc[nc][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f16x8 kf = __builtin_bit_cast(f16x8, dec_bf16x8_to_f16x8(kr[u][s]));
#pragma unroll
          for (int nc = 0; nc < NC; ++nc)
            sc[nc][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, __builtin_bit_cast(f16x8, qf[nc][s]), sc[nc][u], 0, 0, 0);
        }
      }
      if (!SHORT) load_k(k0 + 32);
    }
    u32x4 pf[NC];
    float alpha[NC];
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
      if (k0 + 32 > kend) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (k0 + 16 * u + 4 * kg + v >= kend) sc[nc][u][v] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) mx = fmaxf(mx, sc[nc][u][v]);
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run[nc], mx * c_scale);       // finite: every step has at least one valid key
      alpha[nc] = __builtin_amdgcn_exp2f(m_run[nc] - m_new);
      m_run[nc] = m_new;
      float p[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) p[u][v] = __builtin_amdgcn_exp2f(fmaf(sc[nc][u][v], c_scale, -m_new));
      const uint32_t d0 = dec_pack2(p[0][0], p[0][1]), d1 = dec_pack2(p[0][2], p[0][3]);
      const uint32_t d2 = dec_pack2(p[1][0], p[1][1]), d3 = dec_pack2(p[1][2], p[1][3]);
      // row sum from the rounded probabilities, so numerator and denominator carry the same rounding
      const float rs = dec_sum2(d3, dec_sum2(d2, dec_sum2(d1, dec_sum2(d0, 0.f))));
      pf[nc] = u32x4{d0, d1, d2, d3};
      l_run[nc] = l_run[nc] * alpha[nc] + rs;
    }
    u32x4 (&vs)[2][4] = NC == 1 && !SHORT ? vc : vr;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      // column 8*j + c of the 8 keys this lane loaded: element c of each 16-byte row
      const int w = c >> 1;
      auto el = [&](uint32_t word) { return (c & 1) ? dec_hi(word) : dec_lo(word); };
      const u32x4 vf = u32x4{dec_pack2(el(vs[0][0][w]), el(vs[0][1][w])), dec_pack2(el(vs[0][2][w]), el(vs[0][3][w])),
                             dec_pack2(el(vs[1][0][w]), el(vs[1][1][w])), dec_pack2(el(vs[1][2][w]), el(vs[1][3][w]))};
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) {
        f32x4 oc = o[nc][c];
#pragma unroll
        for (int v = 0; v < 4; ++v) oc[v] *= alpha[nc];
        o[nc][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, vf), __builtin_bit_cast(f16x8, pf[nc]), oc, 0, 0, 0);
      }
    }
    if constexpr (NC != 1 && !SHORT) load_v(k0 + 32);
    if constexpr (SHORT) break;
  }

  // o[c][v] of lane (j, kg) is O[column 8*(4*kg + v) + c][head j]
  if (KR == 1) {      // one range per head: the wave's registers are the record
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
      const float l_tot = l_run[nc] + __shfl_xor(l_run[nc], 16, 64) + __shfl_xor(l_run[nc], 32, 64) +
                          __shfl_xor(__shfl_xor(l_run[nc], 16, 64), 32, 64);
      const int col = 16 * nc + j, rj = col / G, hj = col - rj * G;
      if (!active || col >= n_cols) continue;
      float *pp = a.partials + (((int64_t)row_of(rj) * a.n_q_heads + g * G + hj) * a.n_parts + it.part) * (H + 2);
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < 8; c += 2)      // (a record has 8-byte alignment)
          *reinterpret_cast<float2 *>(pp + 8 * (4 * kg + v) + c) = make_float2(o[nc][c][v], o[nc][c + 1][v]);
      if (kg == 0) {
        pp[H] = (m_run[nc] == -INFINITY) ? -INFINITY : m_run[nc] * DEC_LN2;     // natural-log domain for the merge kernel
        pp[H + 1] = l_tot;
      }
    }
    return;
  }
  // ---- merge the sub-ranges of every head (fixed order) and write the partials ----------------------
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    const float l_tot = l_run[nc] + __shfl_xor(l_run[nc], 16, 64) + __shfl_xor(l_run[nc], 32, 64) +
                        __shfl_xor(__shfl_xor(l_run[nc], 16, 64), 32, 64);
    if (16 * nc + j < CM) {
      float *mine = s_o + ((size_t)wave * CM + 16 * nc + j) * (H + 2);
#pragma unroll
      for (int c = 0; c < 8; c += 2)
#pragma unroll
        for (int v = 0; v < 4; ++v) *reinterpret_cast<float2 *>(mine + 8 * (4 * kg + v) + c) = make_float2(o[nc][c][v], o[nc][c + 1][v]);
      if (kg == 0) { mine[H] = m_run[nc]; mine[H + 1] = l_tot; }
    }
  }
  __syncthreads();
  // eight waves, a (head, column) pair each at a time, two of its 128 columns per lane
  for (int i = wave; i < HW * n_cols; i += 8) {
    const int hwi = i / n_cols, hd = i - hwi * n_cols;
    const int gi = it.g + hwi;
    if (gi >= a.n_kv_heads) continue;
    const int rj = hd / G, hj = hd - rj * G;
    // wave kr2 * HW + hwi holds sub-range kr2 of this head
    const float *src = s_o + ((size_t)hwi * CM + hd) * (H + 2);
    const size_t step = (size_t)HW * CM * (H + 2);
    float M = -INFINITY;
    for (int kr2 = 0; kr2 < KR; ++kr2) M = fmaxf(M, src[kr2 * step + H]);
    float2 acc = make_float2(0.f, 0.f);
    float den = 0.f;
    for (int kr2 = 0; kr2 < KR; ++kr2) {
      const float mw = src[kr2 * step + H];
      const float wgt = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - M);
      const float2 v = *reinterpret_cast<const float2 *>(src + kr2 * step + 2 * lane);
      acc.x += wgt * v.x;
      acc.y += wgt * v.y;
      den += wgt * src[kr2 * step + H + 1];
    }
    float *pp = a.partials + (((int64_t)row_of(rj) * a.n_q_heads + gi * G + hj) * a.n_parts + it.part) * (H + 2);
    *reinterpret_cast<float2 *>(pp + 2 * lane) = acc;
    if (lane == 0) {
      pp[H] = (M == -INFINITY) ? -INFINITY : M * DEC_LN2;     // natural-log domain for the merge kernel
      pp[H + 1] = den;
    }
  }
}

bool attn_decode_mfma_supported(const LayerDims &L) {
  const int G = L.n_q_heads / L.n_kv_heads;
  return L.head_dim == 128 && G <= 16;
}

void decode_mfma_shape(int n_kv_heads, bool two_heads, int *heads_per_wg, int *ranges_per_wg) {
  const int most = two_heads ? 2 : 8, hw = n_kv_heads < most ? n_kv_heads : most;
  *heads_per_wg = hw;
  *ranges_per_wg = 8 / hw;
}

void launch_attn_decode_mfma(const DecodeArgs &a, int n_items, hipStream_t s) {
  if (n_items == 0) return;
  const size_t smem = a.ranges_per_wg == 1 ? 0 : (size_t)8 * a.cols_max * (128 + 2) * sizeof(float);
  auto kern = a.keys_max <= 32 && a.cols_max <= 16 ? attn_decode_mfma_kernel<1, true> : a.cols_max <= 16 ? attn_decode_mfma_kernel<1> : attn_decode_mfma_kernel<2>;
  // set on every launch that needs it: a host-side attribute write, safe from any thread and on any device
  if (smem > 48 * 1024)
    (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  hipLaunchKernelGGL(kern, dim3(n_items), dim3(512), smem, s, a);
}

}  // namespace alora
