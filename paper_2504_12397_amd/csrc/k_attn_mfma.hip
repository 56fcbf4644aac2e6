// Flash-style causal attention of new queries over [cached prefix ; new suffix] (Eq.1 with the
// causal mask, rows as in Eq.6) on the gfx950 matrix cores, head_dim 128, grouped-query sharing.
//
// Operand precision.  The cache holds bf16 keys and values (storage), but inside this kernel every MFMA
// operand is fp16: the queries arrive as fp16 from the rotation step, K/V tiles are converted bf16 -> fp16 on
// their way into LDS (exact: 8 significant bits fit in 11; magnitudes beyond 65504 saturate, values below
// 2^-24 vanish), and the probabilities are packed to fp16.  With bf16 operands the rounding of q (2^-9 per
// element, amplified through the exponential) and of p dominated the error against the float64 oracle --
// 1.5e-3 and 1.2e-3 rms of the row scale, with maxima of 1-2.3e-2 over 10^6 elements, right at the 2e-2
// bar; fp16 operands cut both by 8x at the price of ~40 conversion instructions per thread and tile.
//
// Work item: one workgroup = (q-tile of 256/G tokens of one sequence, kv head, key split).
// The G query heads of the kv group are packed next to the tokens into 256 "packed rows"
// (packed row = token * G + head), 32 per wave and eight waves per workgroup, so every K/V tile
// fetched from HBM serves all heads of the group.  Two kernels: attn_prefill_pipe_kernel (folded softmax, eight waves: what calls
// take by default) weaves the steps of consecutive key blocks together; attn_prefill_mfma_kernel does them one after the other and
// serves the options attn_fold = 0 and attn_waves = 4.
//
// Per 64-key tile, each wave computes S^T = K Q^T (keys are MFMA rows, packed query rows are
// MFMA columns).  In that orientation a lane owns one query row (column l%32) in every
// accumulator register, so the online-softmax state (running max, running sum, rescale
// factor) is one scalar per lane and the probabilities can be fed straight back, from
// registers, as the B operand of O^T += V^T P^T.  The only data that needs a transpose is V:
// the loader threads turn 4 keys x 8 columns into 8 columns x 4 keys in registers (byte
// permutes) and store V^T tiles to LDS in the exact k-order the P registers have.
//
// K tile in LDS: [64 keys][16 chunks of 16 B], chunk c of key r at c ^ (r & 15).
// V^T tile in LDS: [128 columns][8 chunks of 16 B]; chunk (2*s4 + kh) of a column holds keys
//   32*(s4/2) + 16*(s4%2) + {4kh..4kh+3, 8+4kh..8+4kh+3}  (s4 = k-step 0..3, kh = lane/32),
//   stored at chunk ^ v_swz(column).
#include <type_traits>

#include "mfma_kernels.h"

namespace alora {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f16x8 u4_as_f16x8(u32x4 u) { return __builtin_bit_cast(f16x8, u); }

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  bf16x2 p;
  p[0] = (bf16)a;
  p[1] = (bf16)b;
  return __builtin_bit_cast(uint32_t, p);
}

// two floats as an fp16 pair (v_cvt_pkrtz_f16_f32: one instruction, round toward zero, so a finite value
// never becomes infinite).  Used for the probabilities -- numerator and denominator of the softmax are both
// taken from the packed values, so the rounding direction cancels -- and for bf16 values, where it is exact.
__device__ __forceinline__ uint32_t pack_f16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}
// the two bf16 halves of a word as floats
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
// a word of two bf16 -> a word of two fp16
__device__ __forceinline__ uint32_t bf16x2_to_f16x2(uint32_t w) { return pack_f16x2(bf16_lo(w), bf16_hi(w)); }

// chunk swizzle of the V^T tile (128-byte rows).  LDS serves 16 lanes at a time over 64 banks:
// 16 consecutive columns of one chunk (operand reads) must land on 16 distinct 16-byte slots
// modulo 256 B, which (col >> 1) & 7 together with the row parity gives; the extra col >> 4 term
// spreads the transposing 8-byte stores (columns 4 apart) to a 2-way conflict at worst.
__device__ __forceinline__ int v_swz(int col) { return ((col >> 1) ^ (col >> 4)) & 7; }

// max of a value with the one held by the lane 32 away.  v_permlane32_swap trades lanes 32..63 of its
// first register with lanes 0..31 of its second; given two copies of x, the first then holds the low
// half's values in both halves and the second the high half's.  Written as inline assembly because
// the compiler builtin hands back its first result for both (the maximum then silently covers one
// half only); the s_nop's are the wait states between a vector write and this instruction's read.
__device__ __forceinline__ float max_with_other_half(float x) {
  float lo = x, hi = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1\n\tv_max_f32 %0, %0, %1" : "+v"(lo), "+v"(hi));
  return lo;
}

// acc + lo + hi of a packed fp16 pair (v_dot2_f32_f16 against (1, 1)): products and sum in fp32
__device__ __forceinline__ float sum_f16x2(uint32_t pair, float acc) {
  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, pair), __builtin_bit_cast(half2_t, 0x3c003c00u), acc, false);
}

// the same on one half of the pair at a time.  v_dot2 shares the matrix pipe: one of them between matrix instructions keeps that pipe for 16
// cycles more (32 -> 49 per v_mfma_f32_32x32x16 with one dot2, 33 with six of these); v_fma_mix_f32 runs beside them.
template <int HI> __device__ __forceinline__ void add_f16(uint32_t pair, float &acc) {
  if (HI) asm volatile("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(acc) : "v"(pair));
  else asm volatile("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel_hi:[1,0,0]" : "+v"(acc) : "v"(pair));
}

// Waits for every outstanding global load (s_waitcnt vmcnt(0); the other counters left alone).
// Used once before the key loops: the query fragments are loaded before a conditional prologue,
// and unless their loads are known to be complete on every path into the loop the compiler guards
// each use of them inside the loop with a vmcnt wait -- which, the counter being in-order, also
// drains the K/V prefetches that are supposed to stay in flight.
__device__ __forceinline__ void wait_all_global_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

constexpr int ATT_BN = 64;        // keys per tile
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// ---- write the partial (or final) result of a row: the lane's half of its columns -------------------------------------
__device__ __forceinline__ void write_result(const AttnArgs &a, int part, int64_t row, bool valid, int head, int kh, float m_ref,
                                             float l_run, const f32x16 (&o)[4]) {
  constexpr int H = 128;
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);      // the two halves of the wave hold disjoint keys
  if (!valid) return;
  if (a.out != nullptr) {
    const float inv = 1.0f / l_tot;
    bf16 *op = a.out + row * a.n_q + head * H;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int col = cb * 32 + 8 * v4 + 4 * kh;
        uint2 w;
        w.x = pack_bf16x2(o[cb][4 * v4] * inv, o[cb][4 * v4 + 1] * inv);
        w.y = pack_bf16x2(o[cb][4 * v4 + 2] * inv, o[cb][4 * v4 + 3] * inv);
        *reinterpret_cast<uint2 *>(op + col) = w;
      }
  } else if (a.compact) {
    // compact partial record (ATTN_REC16 bytes): the unnormalised accumulators of the row divided by their
    // largest magnitude, as 128 fp16 values (relative precision 2^-11, finer than the bf16 the merged result
    // is rounded to; no overflow whatever the values), then that magnitude, the reference and the row sum.
    // Half the bytes of the fp32 record -- and these records are most of what a short call writes and reads.
    float amax = 0.f;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 16; ++v) amax = fmaxf(amax, fabsf(o[cb][v]));
    amax = max_with_other_half(amax);
    const float rs = amax > 0.f ? 1.0f / amax : 0.f;
    char *rec = reinterpret_cast<char *>(a.partials) +
                ((row * a.n_q_heads + head) * a.n_parts + part) * (int64_t)ATTN_REC16;
    typedef __attribute__((__vector_size__(4 * sizeof(_Float16)))) _Float16 half4_t;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int col = cb * 32 + 8 * v4 + 4 * kh;
        half4_t hv;
#pragma unroll
        for (int i = 0; i < 4; ++i) hv[i] = (_Float16)(o[cb][4 * v4 + i] * rs);
        *reinterpret_cast<half4_t *>(rec + col * 2) = hv;
      }
    if (kh == 0) {
      float *tail = reinterpret_cast<float *>(rec + 2 * H);
      tail[0] = (l_tot == 0.f || m_ref == -INFINITY) ? -INFINITY : m_ref * LN2;
      tail[1] = l_tot;
      tail[2] = amax;
    }
  } else {
    float *pp = a.partials + ((row * a.n_q_heads + head) * a.n_parts + part) * (H + 2);
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int col = cb * 32 + 8 * v4 + 4 * kh;
        // (H + 2) floats per record keeps 8-byte, not 16-byte, alignment
        *reinterpret_cast<float2 *>(pp + col) = make_float2(o[cb][4 * v4], o[cb][4 * v4 + 1]);
        *reinterpret_cast<float2 *>(pp + col + 2) = make_float2(o[cb][4 * v4 + 2], o[cb][4 * v4 + 3]);
      }
    if (kh == 0) {
      // natural-log domain; a row that saw no key keeps -inf so that the merge gives it no weight
      pp[H] = (l_tot == 0.f || m_ref == -INFINITY) ? -INFINITY : m_ref * LN2;
      pp[H + 1] = l_tot;
    }
  }
}

// The same, whole pieces of 64 bytes of a row at a time: eight bytes of 32 rows a request are what the unit that looks up addresses takes longest for.  Each wave
// turns 32 rows x 64 bytes at a time through 2 KB of LDS of its own; there and on the way out a lane has rows lane / 4 and 16 more, 16 bytes lane % 4 of them.
// io_rh: (row, head) of those two rows, or -1.
__device__ __forceinline__ void write_result_staged(const AttnArgs &a, int part, char *st, const int64_t (&io_rh)[2], int lane, float m_ref, float l_run,
                                                    const f32x16 (&o)[4]) {
  constexpr int H = 128;
  typedef __attribute__((__vector_size__(4 * sizeof(_Float16)))) _Float16 half4_t;
  typedef uint32_t w16 __attribute__((ext_vector_type(4), aligned(8)));
  const int l32 = lane & 31, kh = lane >> 5, chunk = lane & 3;
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);      // the two halves of the wave hold disjoint keys
  auto at = [&](int r, int c) { return st + r * 64 + ((c ^ ((r >> 2) & 3)) * 16); };
  auto take = [&](int half) { return *reinterpret_cast<const u32x4 *>(at(16 * half + (lane >> 2), chunk)); };
  const bool direct = a.out != nullptr;
  if (direct || a.compact) {
    float rs, amax = 0.f;
    if (direct) {
      rs = 1.0f / l_tot;
    } else {      // (compact record: see write_result)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int v = 0; v < 16; ++v) amax = fmaxf(amax, fabsf(o[cb][v]));
      amax = max_with_other_half(amax);
      rs = amax > 0.f ? 1.0f / amax : 0.f;
    }
    const int64_t step = direct ? H * 2 : (int64_t)a.n_parts * ATTN_REC16;
    char *base = direct ? reinterpret_cast<char *>(a.out) : reinterpret_cast<char *>(a.partials) + part * ATTN_REC16;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        uint2 w;
        if (direct) {
          w.x = pack_bf16x2(o[cb][4 * v4] * rs, o[cb][4 * v4 + 1] * rs);
          w.y = pack_bf16x2(o[cb][4 * v4 + 2] * rs, o[cb][4 * v4 + 3] * rs);
        } else {
          half4_t hv;
#pragma unroll
          for (int i = 0; i < 4; ++i) hv[i] = (_Float16)(o[cb][4 * v4 + i] * rs);
          w = __builtin_bit_cast(uint2, hv);
        }
        *reinterpret_cast<uint2 *>(at(l32, v4) + 8 * kh) = w;
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const u32x4 w = take(half);
        if (io_rh[half] >= 0) *reinterpret_cast<u32x4 *>(base + io_rh[half] * step + cb * 64 + chunk * 16) = w;
      }
    }
    if (direct) return;
    // the three numbers of a record: row l32's, to the lanes that know where its record is
    if (kh == 0)
      *reinterpret_cast<float4 *>(at(l32, 0)) = make_float4((l_tot == 0.f || m_ref == -INFINITY) ? -INFINITY : m_ref * LN2, l_tot, amax, 0.f);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const float4 t = *reinterpret_cast<const float4 *>(at(16 * half + (lane >> 2), 0));
      if (chunk == 0 && io_rh[half] >= 0) *reinterpret_cast<float4 *>(base + io_rh[half] * step + 2 * H) = t;
    }
  } else {
    float *base = a.partials + (int64_t)part * (H + 2);
    const int64_t step = (int64_t)a.n_parts * (H + 2);
#pragma unroll
    for (int hc = 0; hc < 8; ++hc) {      // 16 columns
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int v = 8 * (hc & 1) + 4 * q;
        *reinterpret_cast<float4 *>(at(l32, 2 * q + kh)) = make_float4(o[hc >> 1][v], o[hc >> 1][v + 1], o[hc >> 1][v + 2], o[hc >> 1][v + 3]);
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const u32x4 w = take(half);
        // ((H + 2) floats per record keeps 8-byte, not 16-byte, alignment)
        if (io_rh[half] >= 0) *reinterpret_cast<w16 *>(base + io_rh[half] * step + hc * 16 + chunk * 4) = w;
      }
    }
    if (kh == 0) *reinterpret_cast<float2 *>(at(l32, 0)) = make_float2((l_tot == 0.f || m_ref == -INFINITY) ? -INFINITY : m_ref * LN2, l_tot);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const float2 t = *reinterpret_cast<const float2 *>(at(16 * half + (lane >> 2), 0));
      if (chunk == 0 && io_rh[half] >= 0) *reinterpret_cast<float2 *>(base + io_rh[half] * step + H) = t;
    }
  }
}

// PFX: tile loads with full 64-bit address arithmetic (items whose keys lie beyond 2 GB from their first row)
// instead of buffer loads with 32-bit offsets
//
// FOLD: the queries arrive premultiplied by sm_scale * log2(e) (the rotation kernel does it while it
// rounds them), and the softmax bookkeeping moves onto the matrix unit:
//   * the accumulator of the first K Q^T product starts at -m_ref (the row's reference exponent,
//     replicated over the lane's 16 registers), so the scores come out as s - m_ref, ready for exp2;
//   * the row sums are taken on the vector ALU from the packed probabilities (v_dot2_f32_f16 against (1, 1)),
//     so numerator and denominator see the same rounded values; each half of the wave sums the keys it holds and
//     the two halves are added once, at the end (they share the reference exponent);
//   * m_ref is set to the exact maximum of the first block in which the row sees a key, and later moves
//     only when a block's maximum exceeds it by more than `lazy`, in a branch that is rare.
// The softmax is the same function: numerator and denominator share the reference exponent.
template <int G, int NW, bool PFX, bool FOLD>      // NW waves per workgroup (8 or 4), 32 packed rows each
__global__ __launch_bounds__(64 * NW) void attn_prefill_mfma_kernel(AttnArgs a) {
  constexpr int H = 128;
  constexpr int NT = 64 * NW;
  __shared__ u32x4 Ks[2][ATT_BN * 16];
  __shared__ u32x4 Vs[2][H * 8];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, kh = lane >> 5;
  // work list built by the host: one item per workgroup -- up to TQ consecutive packed rows against one range of
  // key positions of one kv head -- ordered so that the items that stream the same keys and values sit on one XCD
  // (one L2) together.  The rows of an item belong to one sequence (the causal mask uses pos0 + token), or to
  // several consecutive sequences over the shared prefix they all name (no mask needed: pos0 is out of reach).
  const AttnItem wk = a.work[blockIdx.x];
  if (wk.ntok <= 0) return;
  const int g = wk.g, split = wk.part;
  const int ntok = wk.ntok;
  const int row0 = wk.row0;
  const int n_visible = wk.n_addr;                   // key positions addressable from key_row0
  const int kbeg = wk.kbeg, kend = wk.kend;
  const int ntiles = kend > kbeg ? (kend - kbeg + ATT_BN - 1) / ATT_BN : 0;
  const bf16 *Kp = a.K + wk.key_row0 * a.n_kv + g * H;
  const bf16 *Vp = a.V + wk.key_row0 * a.n_kv + g * H;
  const int first_pos = wk.pos0;                     // smallest query position in the tile

  // ---- this wave's queries as B operands: 2 column blocks x 8 k-steps ---------------------
  u32x4 qf[8];
  const int pr = wave * 32 + l32, tok = pr / G, head = g * G + pr % G;
  const int pos = tok < ntok ? first_pos + tok : -1;       // -1: padding row, sees nothing
  {
    const _Float16 *qp = a.Q + (int64_t)(row0 + min(tok, ntok - 1)) * a.n_q + head * H + kh * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = *reinterpret_cast<const u32x4 *>(qp + ks * 16);
  }

  f32x16 o[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[cb][v] = 0.f;
  const float c_scale = a.sm_scale * LOG2E;
  // softmax state of the lane's query row: the reference exponent m_ref (exp2 domain), the sum l_run of the
  // probabilities of the keys this half of the wave holds (for FOLD the score accumulators start at -m_ref)
  float m_ref = FOLD ? 0.f : -INFINITY;
  float l_run = 0.f;
  bool seen = false;        // the row has met a visible key (the same in both halves: derived from the shared maximum)

  // ---- tile loader: K rows as they are, V transposed in registers -------------------------
  // 512 threads: K = 1024 chunks of 16 B, two per thread; V = 16 key quads x 32 column groups of
  // 4, one (quad, group) per thread: four 8-byte loads become four columns x four keys.
  // Two tiles are kept in flight in registers (sets 0 and 1) on top of the one being consumed
  // from LDS: one tile of compute is shorter than the HBM latency.
  constexpr int KC = 1024 / NT;          // 16-byte K chunks per thread and tile
  constexpr int CW = 2048 / NT;          // V columns per thread (for 4 keys): 4 or 8
  constexpr int VW = CW / 2;             // 32-bit words per key
  typedef uint32_t vword __attribute__((ext_vector_type(VW)));
  u32x4 rk0[KC], rk1[KC];
  vword rv0[4], rv1[4];
  const int v_qd = tid / (H / CW), v_cg = tid % (H / CW);
  // Without shared prefixes the tile loads are buffer loads: a resource that covers exactly the rows
  // [0, n_visible) of this sequence and kv head, per-lane byte offsets that never change, and the tile's
  // first row as the scalar offset -- no address arithmetic per load, and rows past the end read as zero
  // (the range check of the buffer resource) instead of needing a clamp.  (The host takes the other path
  // when a sequence is too long for 32-bit byte offsets.)
  const uint32_t row_bytes = (uint32_t)a.n_kv * 2u;
  __amdgpu_buffer_rsrc_t k_rsrc, v_rsrc;
  uint32_t k_off[KC], v_off[4];
  if constexpr (!PFX) {
    const int n_rec = (int)(((uint32_t)max(n_visible, 1) - 1u) * row_bytes + H * 2u);
    k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)Kp, 0, n_rec, 0x00020000);
    v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)Vp, 0, n_rec, 0x00020000);
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const int q = tid + i * NT;
      k_off[i] = (uint32_t)(q >> 4) * row_bytes + (q & 15) * 16u;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v_off[i] = (uint32_t)(v_qd * 4 + i) * row_bytes + v_cg * (CW * 2u);
  }
  auto load_tile = [&](int t, u32x4 (&rk)[KC], vword (&rv)[4]) {
    const int k0 = kbeg + t * ATT_BN;
    if constexpr (!PFX) {
      const int s_off = __builtin_amdgcn_readfirstlane((int)((uint32_t)k0 * row_bytes));
#pragma unroll
      for (int i = 0; i < KC; ++i)
        rk[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, (int)k_off[i], s_off, 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (VW == 2) rv[i] = __builtin_bit_cast(vword, __builtin_amdgcn_raw_buffer_load_b64(v_rsrc, (int)v_off[i], s_off, 0));
        else rv[i] = __builtin_bit_cast(vword, __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, (int)v_off[i], s_off, 0));
      }
    } else {
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        const int q = tid + i * NT, key = q >> 4, c = q & 15;
        const int kidx = min(k0 + key, n_visible - 1);
        const int64_t e = (int64_t)kidx * a.n_kv + c * 8;
        rk[i] = *reinterpret_cast<const u32x4 *>(Kp + e);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kidx = min(k0 + v_qd * 4 + i, n_visible - 1);
        const int64_t e = (int64_t)kidx * a.n_kv + v_cg * CW;
        rv[i] = *reinterpret_cast<const vword *>(Vp + e);
      }
    }
  };
  auto store_k = [&](int buf, const u32x4 (&rk)[KC]) {
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const int q = tid + i * NT, key = q >> 4, c = q & 15;
      Ks[buf][key * 16 + (c ^ (key & 15))] = u32x4{bf16x2_to_f16x2(rk[i].x), bf16x2_to_f16x2(rk[i].y),
                                                   bf16x2_to_f16x2(rk[i].z), bf16x2_to_f16x2(rk[i].w)};
    }
  };
  auto store_v = [&](int buf, const vword (&rv)[4]) {
    // V: this thread holds keys 4*v_qd..+3 for columns CW*v_cg..+CW-1
    const int grp16 = v_qd >> 2, qi = v_qd & 3;
    const int vkh = qi & 1, halfpos = qi >> 1;
    const int vchunk = grp16 * 2 + vkh;
    u32x2 *vs2 = reinterpret_cast<u32x2 *>(Vs[buf]);
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      // even column 2j: low halves; odd column 2j+1: high halves.  The conversion to fp16 packs two keys of one
      // column into a word, which is the transposition.
      u32x2 ev, od;
      ev.x = pack_f16x2(bf16_lo(rv[0][j]), bf16_lo(rv[1][j]));
      ev.y = pack_f16x2(bf16_lo(rv[2][j]), bf16_lo(rv[3][j]));
      od.x = pack_f16x2(bf16_hi(rv[0][j]), bf16_hi(rv[1][j]));
      od.y = pack_f16x2(bf16_hi(rv[2][j]), bf16_hi(rv[3][j]));
      const int c0 = v_cg * CW + 2 * j, c1 = c0 + 1;
      vs2[(c0 * 8 + (vchunk ^ v_swz(c0))) * 2 + halfpos] = ev;
      vs2[(c1 * 8 + (vchunk ^ v_swz(c1))) * 2 + halfpos] = od;
    }
  };

  // A 64-key tile is consumed as two 32-key blocks, each with its own softmax update, so that only one
  // block of scores and probabilities is live at a time.  The three steps of a block:
  f32x16 sv;            // scores of the block in flight, then its probabilities
  u32x4 pf[2];          // the probabilities as fp16: [half of the block's keys] x 8
  // ---- S^T = K Q^T ------------------------------------------------------------------------------
  auto qk = [&](int buf, int kb) {
    // all eight K fragments of this key block are fetched from LDS first: with one MFMA per
    // fragment there is nothing else to hide the LDS latency behind
    f16x8 kf[8];
    const int key = kb * 32 + l32;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kf[ks] = u4_as_f16x8(Ks[buf][key * 16 + ((2 * ks + kh) ^ (key & 15))]);
    if constexpr (FOLD) {
      const float neg_m = -m_ref;
#pragma unroll
      for (int v = 0; v < 16; ++v) sv[v] = neg_m;
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) sv[v] = 0.f;
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) sv = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[ks], u4_as_f16x8(qf[ks]), sv, 0, 0, 0);
  };
  // ---- causal mask and online softmax (log2 domain), one query row per lane -----------------------
  auto softmax = [&](int t, int kb) {
    const int k0 = kbeg + t * ATT_BN;
    // only tiles that reach past the first query position or the split end need the mask
    if ((k0 + ATT_BN - 1 > first_pos) || (k0 + ATT_BN > kend)) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = k0 + kb * 32 + 8 * (v >> 2) + 4 * kh + (v & 3);
        if (key > pos || key >= kend) sv[v] = -INFINITY;
      }
    }
    float mx = sv[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, sv[v]);
    if constexpr (!FOLD) mx = max_with_other_half(mx);
    // The reference exponent of a row moves (and its 64 output accumulators and row sum are rescaled)
    // only in blocks where some row of the wave needs it -- a wave-uniform, rare branch: with random
    // scores a third of all blocks would otherwise move the maximum of some row.  The softmax is
    // mathematically unchanged (numerator and denominator share the reference); probabilities reach
    // 2^lazy instead of 1, with the same relative bf16 rounding.
    if constexpr (FOLD) {
      // sv holds s - m_ref.  A row's first keys set the reference to their exact maximum (the largest
      // probability is then exactly 1, which matters most for rows that see few keys).
      // mx covers the keys of this half of the wave.  Whether ANY row of the wave has to move is decided from the
      // half maxima (some half exceeds the threshold exactly when its row does); the exchange between the two
      // halves of a row is needed only inside the rare branch.  A row's `seen` flag changes only there too: a half
      // that meets its first key wants the branch, and both halves then take the row's maximum.
      if (__any(mx > a.lazy || (!seen && mx > -INFINITY))) {
        mx = max_with_other_half(mx);
        const bool fresh = !seen;              // nothing accumulated for this row yet
        const bool want = mx > a.lazy || (fresh && mx > -INFINITY);
        seen = seen || mx > -INFINITY;
        const float delta = want ? mx : 0.f;
        const float alpha = fresh ? 1.0f : __builtin_amdgcn_exp2f(-delta);
        m_ref += delta;
        l_run *= alpha;
#pragma unroll
        for (int v = 0; v < 16; ++v) sv[v] -= delta;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[cb][v] *= alpha;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) sv[v] = __builtin_amdgcn_exp2f(sv[v]);
    } else {
      // sv holds raw scores; m_ref is in the exp2 domain (score * sm_scale * log2 e)
      const float m_blk = mx * c_scale;
      const bool move = __any(m_blk > m_ref + a.lazy);
      const float m_new = move ? fmaxf(m_ref, m_blk) : m_ref;
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      if (move) {
        const float alpha = __builtin_amdgcn_exp2f(m_ref - m_safe);
        l_run *= alpha;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[cb][v] *= alpha;
      }
      m_ref = m_new;
#pragma unroll
      for (int v = 0; v < 16; ++v) sv[v] = __builtin_amdgcn_exp2f(fmaf(sv[v], c_scale, -m_safe));
    }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int e = 8 * hf;
      pf[hf] = u32x4{pack_f16x2(sv[e], sv[e + 1]), pack_f16x2(sv[e + 2], sv[e + 3]), pack_f16x2(sv[e + 4], sv[e + 5]),
                     pack_f16x2(sv[e + 6], sv[e + 7])};
      // row sum of the PACKED probabilities (the values the products below use)
      l_run = sum_f16x2(pf[hf].x, l_run);
      l_run = sum_f16x2(pf[hf].y, l_run);
      l_run = sum_f16x2(pf[hf].z, l_run);
      l_run = sum_f16x2(pf[hf].w, l_run);
    }
  };
  // ---- O^T += V^T P^T ----------------------------------------------------------------------------------
  auto pv = [&](int buf, int kb) {
    f16x8 vf[2][4];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int col = cb * 32 + l32, c = 2 * (kb * 2 + hf) + kh;
        vf[hf][cb] = u4_as_f16x8(Vs[buf][col * 8 + (c ^ v_swz(col))]);
      }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[hf][cb], u4_as_f16x8(pf[hf]), o[cb], 0, 0, 0);
  };

  {
    auto compute_tile = [&](int buf, int t) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        qk(buf, kb);
        softmax(t, kb);
        pv(buf, kb);
      }
    };
    // Loads and stores in the loop are unconditional (tile indices clamped) so that the compiler's
    // count of outstanding loads is exact and it waits only for the tile it is about to store.
    if (ntiles > 0) {
      load_tile(0, rk0, rv0);
      load_tile(min(1, ntiles - 1), rk1, rv1);
      store_k(0, rk0);
      store_v(0, rv0);
    }
    __syncthreads();
    wait_all_global_loads();
    for (int t = 0; t < ntiles; t += 2) {
      load_tile(min(t + 2, ntiles - 1), rk0, rv0);
      compute_tile(0, t);
      store_k(1, rk1);
      store_v(1, rv1);
      __syncthreads();
      load_tile(min(t + 3, ntiles - 1), rk1, rv1);
      if (t + 1 < ntiles) compute_tile(1, t + 1);
      store_k(0, rk0);
      store_v(0, rv0);
      __syncthreads();
    }
  }

  write_result(a, split, row0 + tok, tok < ntok, head, kh, m_ref, l_run, o);
}

// ---- folded softmax, eight waves: the steps of consecutive 32-key blocks woven together -----------------------------------
//
// While a block's probabilities are made and multiplied with V, the scores of the next block come out of the matrix unit: every one of a
// block's 16 matrix instructions (32 cycles each) carries one operand read from LDS and at most six vector instructions of another
// step beside it -- eight for K Q^T of the next block with the exponentials of this one, eight for P V with the row sums, the maximum
// of the next block's scores, and the conversion of the tile after next, a word at a time.  The order is fixed in the source
// (sched_barrier after every matrix instruction); in the compiler's own order LDS waits and softmax stand between the products.
// What it rests on (measured beside v_mfma_f32_32x32x16): six v_fma / v_cvt / v_max3 or two v_exp cost nothing; one v_dot2_f32_f16 costs 16 cycles
// of the matrix pipe, which is why the row sums are v_fma_mix; a branch on the mask between the two halves of a block costs 70
// register moves, so blocks that may need the mask run in a loop of their own, which puts -inf in the place of scores whose row does not see
// a key.
//
// 1024 rows x 32 heads over 32768 keys: 555 -> 497 us (0.99 -> 1.11 PFLOP/s), 4300 -> 3150 cycles per 256 x 64 tile, matrix pipes busy 0.48 ->
// 0.65 of the time; the power limit takes part of it back (1.97 -> 1.62 GHz).  Bound now: that limit -- the matrix work alone, without
// tiles, LDS reads and exponentials, takes 388 us at 0.84 busy and 1.6 GHz; without the tile traffic 430; without operand reads 470.
// No gain (within 1 %): operands requested 2 to 6 instructions ahead, two tiles in registers instead of one, other wave priorities.
template <int N> using ic = std::integral_constant<int, N>;
// one K tile (rows 16 bytes apart from a multiple of 256, so that 16 of them lie in different banks) and one V^T tile in LDS; four of each
constexpr int PIPE_AHEAD = 4;      // operand reads run this many matrix instructions ahead
constexpr int PIPE_KROW = 272, PIPE_K = ATT_BN * PIPE_KROW, PIPE_VT = ATT_BN * 256;
constexpr int PIPE_V = 4 * PIPE_K, PIPE_OUT = PIPE_V + 4 * PIPE_VT, PIPE_LDS = PIPE_OUT + 8 * 2048;      // (the last: results on their way out)
// a value that the compiler takes as computed here (and whose parts it does not look into)
__device__ __forceinline__ void pin(int &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(uint32_t &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(float &x) { asm volatile("" : "+v"(x)); }
// LDS by its byte address
template <typename V> __device__ __forceinline__ V lds_read(int at) {
  return *reinterpret_cast<const __attribute__((address_space(3))) V *>((uint32_t)at);
}
template <typename V> __device__ __forceinline__ void lds_write(int at, V v) {
  *reinterpret_cast<__attribute__((address_space(3))) V *>((uint32_t)at) = v;
}

__global__ __launch_bounds__(512) void attn_prefill_pipe_kernel(AttnArgs a, int g_log2) {
  constexpr int H = 128;
  extern __shared__ u32x4 pipe_lds[];
  const int lds = (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4 *)pipe_lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kh = lane >> 5;
  const AttnItem wk = a.work[blockIdx.x];
  if (wk.ntok <= 0) return;
  const int ntok = wk.ntok, row0 = wk.row0, n_visible = wk.n_addr, kbeg = wk.kbeg, kend = wk.kend, first_pos = wk.pos0;
  const int ntiles = kend > kbeg ? (kend - kbeg + ATT_BN - 1) / ATT_BN : 0;
  const bf16 *Kp = a.K + wk.key_row0 * a.n_kv + wk.g * H;
  const bf16 *Vp = a.V + wk.key_row0 * a.n_kv + wk.g * H;

  // this lane's packed row: its row of Q and the records (rows past the last repeat that one); other lanes' rows come from them
  const int tok = (wave * 32 + l32) >> g_log2, pos = tok < ntok ? first_pos + tok : -1;       // -1: padding row
  int my_row = row0 + min(tok, ntok - 1);
  if (a.steps > 0) {      // (a run has 1024 rows at most: its sequence is exact in floats)
    const int seq = (int)(((float)my_row + 0.5f) / (float)a.steps);
    my_row = (my_row - seq * a.steps) * a.seqs + (a.order != nullptr ? a.order[seq] : seq);
  }
  const int head0 = wk.g << g_log2, in_group = (1 << g_log2) - 1;
  auto rh_of = [&](int r) { return (int64_t)__shfl(my_row, r, 64) * a.n_q_heads + head0 + ((wave * 32 + r) & in_group); };      // (row, head) of the wave's row r
  // The wave's 32 query rows of 256 bytes come in whole, four a request, and through LDS (in the tile buffers that are filled last) into operand order: chunk
  // c of row r at c ^ (r & 15).  Asked for in operand order they are 32 bytes of 32 rows a request, and 64 such requests 2 us of a compute unit.
  u32x4 qf[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int r = 4 * j + (lane >> 4);
    qf[j] = *reinterpret_cast<const u32x4 *>(a.Q + rh_of(r) * H + ((lane & 15) ^ (r & 15)) * 8);
  }
  f32x16 o[4], negm;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    negm[v] = 0.f;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) o[cb][v] = 0.f;
  }
  float l_run = 0.f, thr = -INFINITY;      // thr: what a block's maximum (relative to m_ref) has to exceed to move m_ref

  // ---- tiles: memory -> registers (a tile's time before the store) -> LDS (two tiles ahead of the products) ----------------
  const int v_qd = tid >> 5, v_cg = tid & 31;
  const uint32_t row_bytes = (uint32_t)a.n_kv * 2u;
  const int k_off0 = (int)((uint32_t)(tid >> 4) * row_bytes + (tid & 15) * 16u), k_step = (int)(32u * row_bytes);
  const int v_off0 = (int)((uint32_t)(v_qd * 4) * row_bytes + v_cg * 8u);
  const int n_load = min(n_visible, kbeg + ntiles * ATT_BN);
  auto rsrc_of = [&](const bf16 *base, int t) {      // the rows of tile t that exist; the others read as zero
    const int k0 = kbeg + t * ATT_BN, n = min(n_load - k0, ATT_BN);
    const int bytes = max((n - 1) * (int)row_bytes + H * 2, 0);
    return __builtin_amdgcn_make_buffer_rsrc((void *)(base + (int64_t)k0 * a.n_kv), 0, bytes, 0x00020000);
  };
  u32x4 rk[2];
  u32x2 rv[4];
  auto load_k = [&](int t, int i, u32x4 (&r)[2]) {
    r[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_of(Kp, t), k_off0, i * k_step, 0));
  };
  auto load_v = [&](int t, int i, u32x2 (&r)[4]) {
    r[i] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc_of(Vp, t), v_off0, i * (int)row_bytes, 0));
  };
  auto load_tile = [&](int t, u32x4 (&k)[2], u32x2 (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) load_k(t, i, k);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_v(t, i, v);
  };
  int k_st = lds + 2 * PIPE_K + (tid >> 4) * PIPE_KROW + (tid & 15) * 16;
  uint32_t cv[4];      // what goes to LDS next, converted a word at a time
  auto cv_k = [&](int par, int n, const u32x4 (&r)[2]) {      // n = 0 .. 7: word n % 4 of chunk n / 4
    cv[n & 3] = bf16x2_to_f16x2(r[n >> 2][n & 3]);
    pin(cv[n & 3]);
    if ((n & 3) == 3) lds_write(k_st + par * PIPE_K + (n >> 2) * (32 * PIPE_KROW), u32x4{cv[0], cv[1], cv[2], cv[3]});
  };
  // column c = 4 v_cg + j of key quad v_qd: chunk ((v_qd / 4) * 2 + (v_qd & 1)) ^ v_swz(c), half (v_qd >> 1) & 1 of it; columns 2 j and 2 j + 1 share
  // their swizzle
  const int v_chunk = (v_qd >> 2) * 2 + (v_qd & 1), v_half = (v_qd >> 1) & 1;
  int v_st[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) v_st[j] = lds + PIPE_V + 2 * PIPE_VT + (v_cg * 4 + 2 * j) * 128 + (v_chunk ^ v_swz(v_cg * 4 + 2 * j)) * 16 + v_half * 8;
  auto cv_v = [&](int par, int n, const u32x2 (&r)[4]) {      // n = 0 .. 7: column n / 2, keys 2 (n % 2) and the next of the quad
    const int j = n >> 2, odd = (n >> 1) & 1, p = (n & 1) * 2;
    cv[n & 1] = odd ? pack_f16x2(bf16_hi(r[p][j]), bf16_hi(r[p + 1][j])) : pack_f16x2(bf16_lo(r[p][j]), bf16_lo(r[p + 1][j]));
    pin(cv[n & 1]);
    if (n & 1) lds_write(v_st[j] + par * PIPE_VT + odd * 128, u32x2{cv[0], cv[1]});
  };

  // ---- operands from LDS ---------------------------------------------------------------------------------------------------
  int ka = lds + l32 * PIPE_KROW + kh * 16, va[4];
  pin(ka);
#pragma unroll
  for (int x = 0; x < 4; ++x) { va[x] = lds + PIPE_V + l32 * 128 + (((2 * x + kh) ^ (((l32 >> 1) ^ (l32 >> 4)) & 7)) * 16); pin(va[x]); }
  pin(k_st); pin(v_st[0]); pin(v_st[1]);
  // operands on their way: PIPE_AHEAD matrix instructions before they are needed
  u32x4 fr[8];
  auto read_k = [&](int par, int kb, int ks) { fr[ks] = lds_read<u32x4>(ka + par * PIPE_K + kb * (32 * PIPE_KROW) + ks * 32); };
  auto read_v = [&](int par, int kb, int n) {      // n = 4 * (half of the block's keys) + column block
    const int s4 = kb * 2 + (n >> 2), cb = n & 3;
    fr[n] = lds_read<u32x4>(va[s4 ^ cb] + par * PIPE_VT + cb * 4096);
  };

  // Scores of keys that the row does not see become -inf once their product is there, not before: what lies behind the row may be Inf or NaN,
  // and -inf plus such a product is NaN.
  const int vis = min(pos, kend - 1) - 4 * kh;      // (of key block k0 .. k0 + 31, register v holds key k0 + 4 kh + 8 (v / 4) + v % 4)
  auto hide = [&](f32x16 &s, int v, int lim) { if (8 * (v >> 2) + (v & 3) > lim) s[v] = -INFINITY; };
  auto move_ref = [&](f32x16 &s, float mx) {
    mx = max_with_other_half(mx);
    const bool fresh = thr == -INFINITY;
    const float delta = mx > thr ? mx : 0.f;
    const float alpha = fresh ? 1.0f : __builtin_amdgcn_exp2f(-delta);
    if (mx > -INFINITY) thr = a.lazy;
    l_run *= alpha;
#pragma unroll
    for (int v = 0; v < 16; ++v) { s[v] -= delta; negm[v] -= delta; }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[cb][v] *= alpha;
  };

  // ---- one 32-key block: its probabilities and P V, woven with K Q^T and the maximum of the next ------------------------
  uint32_t pw[8];
  auto pf_of = [&](int hf) { return u4_as_f16x8(u32x4{pw[4 * hf], pw[4 * hf + 1], pw[4 * hf + 2], pw[4 * hf + 3]}); };
  int dk = 2 * PIPE_K, dv = 2 * PIPE_VT;      // to the other pair of buffers
  auto block = [&](auto par_c, auto kb_c, auto mask_c, f32x16 &sc, f32x16 &sn, int t) {
    constexpr int PAR = par_c, KB = kb_c, MASK = mask_c;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      sn = __builtin_amdgcn_mfma_f32_32x32x16_f16(u4_as_f16x8(fr[n]), u4_as_f16x8(qf[n]), n == 0 ? negm : sn, 0, 0, 0);
      if (n < 8 - PIPE_AHEAD) read_k(MASK ? 0 : PAR ^ KB, KB ^ 1, n + PIPE_AHEAD);
      else read_v(PAR, KB, n + PIPE_AHEAD - 8);
      // requests of the tile that takes the place of what the last block stored, a few at a time (all eight waves ask together)
      if (KB == 1 && (n & 3) == 1) load_k(t + 3, n >> 2, rk);
      if (KB == 0 && (n & 1) == 1) load_v(t + 2, n >> 1, rv);
      sc[2 * n] = __builtin_amdgcn_exp2f(sc[2 * n]);
      sc[2 * n + 1] = __builtin_amdgcn_exp2f(sc[2 * n + 1]);
      if (n >= 1) { pw[n - 1] = pack_f16x2(sc[2 * n - 2], sc[2 * n - 1]); pin(pw[n - 1]); }
      if (KB == 0 && n == 7) {
        // the stores of the tile before are done (the eight youngest LDS operations are this block's reads), in every wave
        asm volatile("s_waitcnt lgkmcnt(8)\n\ts_barrier" ::: "memory");
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (MASK && KB == 0) ka += (t & 3) == 3 ? -3 * PIPE_K : PIPE_K;
    if (!MASK && PAR == 1 && KB == 0) ka += dk;      // (the other pair of buffers)
    __builtin_amdgcn_s_setprio(1);
    float m0 = 0.f;
    int lim = vis - (kbeg + t * ATT_BN + (KB + 1) * 32);
    if constexpr (MASK) pin(lim);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      o[n & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(u4_as_f16x8(fr[n]), pf_of(n >> 2), o[n & 3], 0, 0, 0);
      if (n < 8 - PIPE_AHEAD) read_v(PAR, KB, n + PIPE_AHEAD);
      else read_k(MASK ? 0 : PAR ^ 1, KB, n + PIPE_AHEAD - 8);
      if (n == 0) { pw[7] = pack_f16x2(sc[14], sc[15]); pin(pw[7]); }
      add_f16<0>(pw[n], l_run);
      add_f16<1>(pw[n], l_run);
      // (the scores are there two matrix instructions after the last that made them)
      if constexpr (MASK) {
        if (n == 2) { hide(sn, 0, lim); hide(sn, 1, lim); hide(sn, 2, lim); }
        if (n >= 3) { hide(sn, 2 * n - 3, lim); hide(sn, 2 * n - 2, lim); }
        if (n == 6) { hide(sn, 13, lim); hide(sn, 14, lim); }
        if (n == 7) hide(sn, 15, lim);
      }
      if (n == 2) m0 = fmaxf(fmaxf(sn[0], sn[1]), sn[2]);
      if (n >= 3) m0 = fmaxf(fmaxf(m0, sn[2 * n - 3]), sn[2 * n - 2]);
      if (n == 6) m0 = fmaxf(fmaxf(m0, sn[13]), sn[14]);
      if (n == 7) m0 = __builtin_amdgcn_fmed3f(m0, sn[15], INFINITY);
      if (n >= 2) pin(m0);
      if constexpr (KB == 0) {
        cv_k(PAR, n, rk);
      } else {
        cv_v(PAR, n, rv);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    if (__any(m0 > thr)) move_ref(sn, m0);
  };
  // the other pair of buffers: reads of K; reads of V^T, and the stores
  auto other_v = [&] {
#pragma unroll
    for (int x = 0; x < 4; ++x) va[x] += dv;
    k_st -= dk; v_st[0] -= dv; v_st[1] -= dv;
    dk = -dk; dv = -dv;
  };

  if (ntiles > 0) {
    u32x4 rk1[2];
    u32x2 rv1[4];
    load_tile(0, rk, rv);
    load_tile(1, rk1, rv1);
    const int q_at = lds + (wave < 4 ? 2 * PIPE_K + wave * 8192 : PIPE_V + 2 * PIPE_VT + (wave - 4) * 8192);
#pragma unroll
    for (int j = 0; j < 8; ++j) lds_write(q_at + j * 1024 + lane * 16, qf[j]);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = lds_read<u32x4>(q_at + l32 * 256 + (((2 * ks + kh) ^ (l32 & 15)) * 16));
    wait_all_global_loads();
    k_st -= dk; v_st[0] -= dv; v_st[1] -= dv;
#pragma unroll
    for (int n = 0; n < 8; ++n) cv_k(0, n, rk);
    load_k(2, 0, rk); load_k(2, 1, rk);
#pragma unroll
    for (int n = 0; n < 8; ++n) cv_v(0, n, rv);
#pragma unroll
    for (int n = 0; n < 8; ++n) cv_k(1, n, rk1);
#pragma unroll
    for (int n = 0; n < 8; ++n) cv_v(1, n, rv1);
    k_st += dk; v_st[0] += dv; v_st[1] += dv;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f32x16 s0, s1;
#pragma unroll
    for (int n = 0; n < 8; ++n) read_k(0, 0, n);
#pragma unroll
    for (int n = 0; n < 8; ++n) s0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(u4_as_f16x8(fr[n]), u4_as_f16x8(qf[n]), n == 0 ? negm : s0, 0, 0, 0);
#pragma unroll
    for (int n = 0; n < PIPE_AHEAD; ++n) read_k(0, 1, n);
#pragma unroll
    for (int v = 0; v < 16; ++v) hide(s0, v, vis - kbeg);
    float m0 = s0[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m0 = fmaxf(m0, s0[v]);
    if (__any(m0 > thr)) move_ref(s0, m0);
    // tiles that every row of the item sees whole; a pair of tiles goes without the mask if they and the next are
    const int n_full = (min(first_pos + 1, kend) - kbeg) / ATT_BN;
    int t = 0;
    for (; t + 2 < n_full; t += 2) {
      block(ic<0>{}, ic<0>{}, ic<0>{}, s0, s1, t);
      block(ic<0>{}, ic<1>{}, ic<0>{}, s1, s0, t);
      block(ic<1>{}, ic<0>{}, ic<0>{}, s0, s1, t + 1);
      block(ic<1>{}, ic<1>{}, ic<0>{}, s1, s0, t + 1);
      other_v();
    }
    for (; t < ntiles; ++t) {      // (a tile at a time, round the four buffers)
      block(ic<0>{}, ic<0>{}, ic<1>{}, s0, s1, t);
      block(ic<0>{}, ic<1>{}, ic<1>{}, s1, s0, t);
      const int av = (t & 3) == 3 ? -3 * PIPE_VT : PIPE_VT, as = (t & 3) == 1 ? -3 : 1;
#pragma unroll
      for (int x = 0; x < 4; ++x) va[x] += av;
      k_st += as * PIPE_K; v_st[0] += as * PIPE_VT; v_st[1] += as * PIPE_VT;
    }
  }
  const float m_ref = -negm[0];
  if ((wave * 32 >> g_log2) >= ntok) return;      // (no row)
  // The rows of one wave: as they lie in its registers, without the way through LDS, which takes longer than one wave's requests.  One row on 40 keys, us, before results went
  // through LDS / all of them / so: 32 groups of one head 6.6 / 7.4 / 5.9, 4 of two 6.4 / 6.8 / 6.0, 8 of four 7.8 / 7.4 / 6.7; 64 x 16 rows of 32 groups of one 43.5 / 51.1 / 46.2.
  if ((ntok << g_log2) <= 32) {
    write_result(a, wk.part, my_row, tok < ntok, head0 + ((wave * 32 + l32) & in_group), kh, m_ref, l_run, o);
    return;
  }
  int64_t io_rh[2];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int r = 16 * half + (lane >> 2);
    const int64_t rh = rh_of(r);
    io_rh[half] = ((wave * 32 + r) >> g_log2) < ntok ? rh : -1;
  }
  write_result_staged(a, wk.part, reinterpret_cast<char *>(pipe_lds) + PIPE_OUT + wave * 2048, io_rh, lane, m_ref, l_run, o);
}

bool attn_prefill_mfma_supported(const LayerDims &L) {
  const int G = L.n_q_heads / L.n_kv_heads;
  return L.head_dim == 128 && (G == 1 || G == 2 || G == 4 || G == 8);
}

int attn_prefill_mfma_tokens_per_tile(const LayerDims &L, int waves) {
  return 32 * waves / (L.n_q_heads / L.n_kv_heads);
}

template <int NW, bool PFX, bool FOLD>
static void launch_attn_nw(const AttnArgs &a, int n_work, int G, hipStream_t s) {
  dim3 grid(n_work);
  switch (G) {
    case 1: hipLaunchKernelGGL((attn_prefill_mfma_kernel<1, NW, PFX, FOLD>), grid, dim3(64 * NW), 0, s, a); break;
    case 2: hipLaunchKernelGGL((attn_prefill_mfma_kernel<2, NW, PFX, FOLD>), grid, dim3(64 * NW), 0, s, a); break;
    case 4: hipLaunchKernelGGL((attn_prefill_mfma_kernel<4, NW, PFX, FOLD>), grid, dim3(64 * NW), 0, s, a); break;
    case 8: hipLaunchKernelGGL((attn_prefill_mfma_kernel<8, NW, PFX, FOLD>), grid, dim3(64 * NW), 0, s, a); break;
    default: break;
  }
}

template <int NW, bool FOLD>
static void launch_attn_nw_any(const AttnArgs &a, int n_work, int G, bool prefix, hipStream_t s) {
  if (prefix) launch_attn_nw<NW, true, FOLD>(a, n_work, G, s);
  else launch_attn_nw<NW, false, FOLD>(a, n_work, G, s);
}

// Log-sum-exp merge of the compact partial records (Eq.1 over the union of the key splits): one wave per
// (row, head), a lane two columns.  out = sum_i w_i amax_i u_i / sum_i w_i l_i with w_i = exp(m_i - max m).
__global__ __launch_bounds__(256) void attn_merge16_kernel(const char *__restrict__ part, int n_splits, int64_t n_rh,
                                                           bf16 *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t rh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (rh >= n_rh) return;
  const char *p = part + rh * n_splits * (int64_t)ATTN_REC16;
  typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 half2_t;
  float M = -INFINITY;
  for (int s0 = 0; s0 < n_splits; s0 += 64) {
    const int sp = s0 + lane;
    M = fmaxf(M, sp < n_splits ? *reinterpret_cast<const float *>(p + sp * (int64_t)ATTN_REC16 + 256) : -INFINITY);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
  float denom = 0.f, a0 = 0.f, a1 = 0.f;
  for (int s0 = 0; s0 < n_splits; s0 += 8) {       // eight records requested together
    float ms[8], ls[8], am[8];
    half2_t u[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const char *r = p + min(s0 + i, n_splits - 1) * (int64_t)ATTN_REC16;
      const float *tail = reinterpret_cast<const float *>(r + 256);
      ms[i] = tail[0]; ls[i] = tail[1]; am[i] = tail[2];
      u[i] = *reinterpret_cast<const half2_t *>(r + lane * 4);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float w = (s0 + i >= n_splits || ms[i] == -INFINITY) ? 0.f : __expf(ms[i] - M);
      denom += w * ls[i];
      a0 += w * am[i] * (float)u[i][0];
      a1 += w * am[i] * (float)u[i][1];
    }
  }
  const float inv = 1.0f / denom;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
  bf16x2_t ov;
  ov[0] = (bf16)(a0 * inv);
  ov[1] = (bf16)(a1 * inv);
  *reinterpret_cast<bf16x2_t *>(out + rh * 128 + lane * 2) = ov;
}

// Up to sixteen records: all of them in one round trip, the maximum from what came with them (the same sums in the same order).  1024 rows of 32 heads, three
// records: 15.8 -> 7.3 us (it asked for eight records' places whatever their number, and for the maxima first); 512 rows, five: 10.2 -> 5.6; 128 rows, sixteen: 5.8 -> 5.6.
template <int N>
__global__ __launch_bounds__(256) void attn_merge16_few_kernel(const char *__restrict__ part, int64_t n_rh, bf16 *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t rh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (rh >= n_rh) return;
  const char *p = part + rh * N * (int64_t)ATTN_REC16;
  typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 half2_t;
  float4 t[N];      // reference, row sum, magnitude
  half2_t u[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    t[i] = *reinterpret_cast<const float4 *>(p + i * ATTN_REC16 + 256);
    u[i] = *reinterpret_cast<const half2_t *>(p + i * ATTN_REC16 + lane * 4);
  }
  float M = t[0].x;
#pragma unroll
  for (int i = 1; i < N; ++i) M = fmaxf(M, t[i].x);
  float denom = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float w = t[i].x == -INFINITY ? 0.f : __expf(t[i].x - M);
    denom += w * t[i].y;
    a0 += w * t[i].z * (float)u[i][0];
    a1 += w * t[i].z * (float)u[i][1];
  }
  const float inv = 1.0f / denom;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
  bf16x2_t ov;
  ov[0] = (bf16)(a0 * inv);
  ov[1] = (bf16)(a1 * inv);
  *reinterpret_cast<bf16x2_t *>(out + rh * 128 + lane * 2) = ov;
}

void launch_attn_merge16(const float *partials, const LayerDims &L, int T_rows, int n_splits, bf16 *out, hipStream_t s) {
  if (T_rows == 0) return;
  const int64_t n_rh = (int64_t)T_rows * L.n_q_heads;
  const dim3 grid((unsigned)((n_rh + 3) / 4));
  const char *p = (const char *)partials;
  switch (n_splits) {
    case 2: hipLaunchKernelGGL(attn_merge16_few_kernel<2>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 3: hipLaunchKernelGGL(attn_merge16_few_kernel<3>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 4: hipLaunchKernelGGL(attn_merge16_few_kernel<4>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 5: hipLaunchKernelGGL(attn_merge16_few_kernel<5>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 6: hipLaunchKernelGGL(attn_merge16_few_kernel<6>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 7: hipLaunchKernelGGL(attn_merge16_few_kernel<7>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 8: hipLaunchKernelGGL(attn_merge16_few_kernel<8>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 9: hipLaunchKernelGGL(attn_merge16_few_kernel<9>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 10: hipLaunchKernelGGL(attn_merge16_few_kernel<10>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 11: hipLaunchKernelGGL(attn_merge16_few_kernel<11>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 12: hipLaunchKernelGGL(attn_merge16_few_kernel<12>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 13: hipLaunchKernelGGL(attn_merge16_few_kernel<13>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 14: hipLaunchKernelGGL(attn_merge16_few_kernel<14>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 15: hipLaunchKernelGGL(attn_merge16_few_kernel<15>, grid, dim3(256), 0, s, p, n_rh, out); break;
    case 16: hipLaunchKernelGGL(attn_merge16_few_kernel<16>, grid, dim3(256), 0, s, p, n_rh, out); break;
    default: hipLaunchKernelGGL(attn_merge16_kernel, grid, dim3(256), 0, s, p, n_splits, n_rh, out);
  }
}

void launch_attn_prefill_mfma(const AttnArgs &a, int n_work, int G, int waves, bool prefix, hipStream_t s) {
  if (n_work == 0) return;
  if (waves == 8 && a.q_prescaled) {
    auto kern = attn_prefill_pipe_kernel;
    (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, PIPE_LDS);
    hipLaunchKernelGGL(kern, dim3(n_work), dim3(512), PIPE_LDS, s, a, G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : 3);
  } else if (waves == 8) {
    launch_attn_nw_any<8, false>(a, n_work, G, prefix, s);
  } else if (a.q_prescaled) {
    launch_attn_nw_any<4, true>(a, n_work, G, prefix, s);
  } else {
    launch_attn_nw_any<4, false>(a, n_work, G, prefix, s);
  }
}

// What the rotation kernel multiplies the queries by: the folded softmax wants them in the exp2 domain,
// otherwise the kernel applies sm_scale itself.
float attn_prefill_mfma_q_scale(const LayerDims &L, bool fold) {
  return fold ? LOG2E / sqrtf((float)L.head_dim) : 1.0f;
}

}  // namespace alora
