// Host side of libalora: the C ABI of include/alora.h -- argument validation, staging of
// the small per-sequence arrays, workspace management and launch planning.  No arithmetic
// of the method happens here; every step runs in the kernels.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/alora.h"
#include "common.h"
#include "mfma_kernels.h"

using namespace alora;

// ---- scratch of the entry point that may not allocate (alora_decode_static) --------------------------------
// One array per GPU the library is loaded on, alive until the process ends.  Host code never uses this name as
// an address: alora_create asks the runtime for the array's device address once per context
// (hipGetSymbolAddress, with the context's device current) and everything below works with that pointer.
constexpr size_t SCRATCH_BYTES = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

namespace {

constexpr int N_SLOTS = 8;

// per-sequence records travel to the device as kernel arguments (no staging buffer, no copy from host memory)
constexpr int STAGE_SEQS = 32;
struct SeqChunk { SeqMeta m[STAGE_SEQS]; };
__global__ void stage_seqs_kernel(SeqChunk c, int n, SeqMeta *dst) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = c.m[threadIdx.x];
}
// the work list of the decode attention kernel for sequences without shared prefixes, from the sequences' records: item
// ((row * n_groups) + gb) * n_own + part covers range `part` of row `row`, kv heads gb * heads_per_wg ...  The ranges are the host
// list's (dec_cut); a row with fewer of them than n_own leaves empty items.  Every sequence has one new row here.
__global__ void make_decode_items_kernel(const SeqMeta *seqs, int n_seqs, DecItem *items, int32_t *counts, int n_groups, int heads_per_wg,
                                         int n_own, int range, int splits) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int row = i / (n_own * n_groups);
  if (row >= n_seqs) return;
  const SeqMeta sm = seqs[row];
  const int n_keys = sm.P + 1, part = i % n_own;
  const DecCut c = dec_cut(n_keys, splits > 0 ? max(1, (n_keys + splits - 1) / splits) : range);
  DecItem it{};
  it.key_row0 = sm.pool_off;
  it.row = row;
  it.kbeg = part * c.len;
  it.kend = min(n_keys, it.kbeg + c.len);
  it.n_rows = part < c.parts ? 1 : 0;
  it.g = (int16_t)(((i / n_own) % n_groups) * heads_per_wg);
  it.part = (int16_t)part;
  it.n_keys = n_keys;
  items[i] = it;
  if (i % (n_own * n_groups) == 0) { counts[2 * row] = c.parts; counts[2 * row + 1] = 0; }
}

// copies the staged metadata from the pinned host buffer (which the GPU can read directly) into device memory: as a
// kernel it is one more dispatch in the stream's queue, where a copy operation is a hand-over to another engine
__global__ void stage_meta_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int n16) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

struct MetaSlot {
  char *host = nullptr;      // pinned
  char *dev = nullptr;
  size_t cap = 0;            // bytes
  hipEvent_t ev = nullptr;
  bool in_flight = false;
};

}  // namespace

struct ProfEvent {
  hipEvent_t start, stop;
  int kernel;
};

static const char *const KERNEL_NAMES[] = {"prep_rows", "qkv_gemm", "rope_append", "attn_prefill", "attn_decode",
                                           "attn_merge", "o_proj", "mlp_norm", "gate_up", "silu_mul", "down_proj",
                                           "lm_head", "lm_argmax"};
enum KernelId { K_PREP = 0, K_QKV, K_ROPE, K_ATTN_PREFILL, K_ATTN_DECODE, K_ATTN_MERGE, K_OPROJ, K_MLPNORM,
                K_GATEUP, K_SILU, K_DOWN, K_LMHEAD, K_ARGMAX, K_COUNT };

struct alora_ctx {
  int opt_profile = 0;
  std::vector<ProfEvent> prof_pending;
  std::vector<hipEvent_t> prof_free;
  double prof_ms[K_COUNT] = {};
  int64_t prof_n[K_COUNT] = {};
  int device = 0;
  std::string err;
  char *ws = nullptr;
  size_t ws_cap = 0;
  unsigned char *scratch_dev = nullptr;      // device address of the static scratch array on this context's GPU
  float2 *rope = nullptr;
  int rope_pos = 0, rope_half = 0;
  float rope_theta = 0.f;
  MetaSlot slots[N_SLOTS];
  int next_slot = 0;
  int opt_kernels = 0;
  int opt_splits = 0;
  int opt_gemm_splits = 0;
  int opt_gemm_tile = 0;
  int opt_prep_split = 1;        // calls with adapters: RMSNorm and down projection in one kernel (1: few rows; 0: never; 2: always)
  int opt_attn_waves = 0;
  int opt_lora_split = 0;        // 0 = automatic, 1 = always, 2 = never: low-rank term in workgroups of its own
  int opt_stage_copy = 0;        // 1: the staged metadata travels by hipMemcpyAsync instead of a copy kernel
  int opt_attn_lazy = 3;         // lazy-maximum threshold of the prefill attention kernels, log2 units
  int opt_attn_partials16 = 1;   // split prefill attention (MFMA path): compact partial records
  int opt_rope_fuse = 1;         // rotation + cache append in the epilogue of the QKV projection where the shape allows
  int opt_attn_fold = 1;         // 1 = prefill attention takes prescaled queries and starts its score accumulators at -m_ref
  int n_cu = 256;
};

namespace {

alora_status fail(alora_ctx *ctx, alora_status st, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (ctx) ctx->err = buf;
  return st;
}

#define HIP_TRY(ctx, call)                                                                   \
  do {                                                                                       \
    hipError_t e_ = (call);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      return fail(ctx, ALORA_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));           \
  } while (0)

// Brackets one kernel launch with events when profiling is on.
struct ProfScope {
  alora_ctx *ctx;
  hipStream_t s;
  ProfEvent ev{};
  bool on;
  ProfScope(alora_ctx *c, int kernel, hipStream_t st) : ctx(c), s(st), on(c->opt_profile != 0) {
    if (!on) return;
    ev.kernel = kernel;
    for (hipEvent_t *e : {&ev.start, &ev.stop}) {
      if (!ctx->prof_free.empty()) { *e = ctx->prof_free.back(); ctx->prof_free.pop_back(); }
      else if (hipEventCreate(e) != hipSuccess) { on = false; return; }
    }
    (void)hipEventRecord(ev.start, s);
  }
  ~ProfScope() {
    if (!on) return;
    (void)hipEventRecord(ev.stop, s);
    ctx->prof_pending.push_back(ev);
  }
};

struct Bump {
  char *base;
  size_t off = 0;
  explicit Bump(char *b) : base(b) {}
  template <typename U> U *take(size_t n) {
    size_t bytes = (n * sizeof(U) + 255) & ~(size_t)255;
    U *p = base ? reinterpret_cast<U *>(base + off) : nullptr;
    off += bytes;
    return p;
  }
};

alora_status ensure_workspace(alora_ctx *ctx, size_t bytes) {
  if (bytes <= ctx->ws_cap) return ALORA_OK;
  HIP_TRY(ctx, hipDeviceSynchronize());        // earlier calls may still be using the old block
  if (ctx->ws) HIP_TRY(ctx, hipFree(ctx->ws));
  ctx->ws = nullptr;
  ctx->ws_cap = 0;
  size_t want = bytes + bytes / 8;
  HIP_TRY(ctx, hipMalloc((void **)&ctx->ws, want));
  ctx->ws_cap = want;
  return ALORA_OK;
}

alora_status ensure_rope(alora_ctx *ctx, int n_pos, int half, float theta, hipStream_t s) {
  if (ctx->rope && ctx->rope_pos >= n_pos && ctx->rope_half == half && ctx->rope_theta == theta)
    return ALORA_OK;
  HIP_TRY(ctx, hipDeviceSynchronize());
  if (ctx->rope) HIP_TRY(ctx, hipFree(ctx->rope));
  ctx->rope = nullptr;
  int want = std::max(n_pos + n_pos / 4, 4096);
  HIP_TRY(ctx, hipMalloc((void **)&ctx->rope, (size_t)want * half * sizeof(float2)));
  launch_rope_table(ctx->rope, want, half, theta, s);
  HIP_TRY(ctx, hipGetLastError());
  ctx->rope_pos = want;
  ctx->rope_half = half;
  ctx->rope_theta = theta;
  return ALORA_OK;
}

alora_status acquire_slot(alora_ctx *ctx, size_t bytes, MetaSlot **out) {
  MetaSlot &sl = ctx->slots[ctx->next_slot];
  ctx->next_slot = (ctx->next_slot + 1) % N_SLOTS;
  if (sl.in_flight) {
    HIP_TRY(ctx, hipEventSynchronize(sl.ev));
    sl.in_flight = false;
  }
  if (sl.cap < bytes) {
    // grow every slot of the ring now, not one per call: each growth is an allocation (and a wait for the slot's
    // last user), which belongs in the first call of a given size and not in the seven after it
    const size_t cap = (std::max<size_t>(4096, bytes + bytes / 2) + 15) & ~(size_t)15;
    for (MetaSlot &o : ctx->slots) {
      if (o.cap >= cap) continue;
      if (o.in_flight) {
        HIP_TRY(ctx, hipEventSynchronize(o.ev));
        o.in_flight = false;
      }
      if (o.host) HIP_TRY(ctx, hipHostFree(o.host));
      if (o.dev) HIP_TRY(ctx, hipFree(o.dev));
      o.host = nullptr; o.dev = nullptr; o.cap = 0;
      HIP_TRY(ctx, hipHostMalloc((void **)&o.host, cap, hipHostMallocDefault));
      HIP_TRY(ctx, hipMalloc((void **)&o.dev, cap));
      o.cap = cap;
      if (!o.ev) HIP_TRY(ctx, hipEventCreateWithFlags(&o.ev, hipEventDisableTiming));
    }
  }
  if (!sl.ev) HIP_TRY(ctx, hipEventCreateWithFlags(&sl.ev, hipEventDisableTiming));
  *out = &sl;
  return ALORA_OK;
}

struct Plan {
  LayerDims L;
  int T = 0, B = 0;
  int max_len = 0;        // max over sequences of P_b + S_b
  bool any_adapter = false;
  bool any_prefix = false;   // some sequence reads a shared prefix
  std::vector<SeqMeta> seqs;
  int n_used = 0;            // adapters that a row of the call may use (at most 64 listed), and their scales
  uint8_t used[64] = {};
  float used_scale[64] = {};
  int adapted_tiles = 0;     // pairs of 32 rows (of the last step) and an adapter that applies to one of them
  bool cached_only = false;  // prefill attention walks the keys that were cached before the call and no others
};

// of a call that ends `more` steps later than its records say
void count_adapted_tiles(Plan *pl, int more) {
  pl->adapted_tiles = 0;
  int last[64];
  std::fill(last, last + 64, -1);
  for (const SeqMeta &m : pl->seqs) {      // (in the order of their rows)
    const int rows = (int)std::min<int64_t>(m.n_new, (int64_t)m.P + m.n_new + more - m.k);
    if (m.adapter < 0 || m.adapter >= 64 || rows <= 0) continue;
    const int lo = std::max((m.row_start + m.n_new - rows) / 32, last[m.adapter] + 1), hi = (m.row_start + m.n_new - 1) / 32;
    pl->adapted_tiles += std::max(0, hi - lo + 1);
    last[m.adapter] = std::max(last[m.adapter], hi);
  }
}

alora_status check_layer(alora_ctx *ctx, const alora_layer_desc *ly, bool need_tail, LayerDims *L) {
  if (!ly) return fail(ctx, ALORA_EINVAL, "layer descriptor is NULL");
  if (ly->dtype != ALORA_F32 && ly->dtype != ALORA_BF16)
    return fail(ctx, ALORA_EDTYPE, "dtype %d is neither ALORA_F32 nor ALORA_BF16", ly->dtype);
  if (ly->d < 1 || ly->d > 16000) return fail(ctx, ALORA_ESHAPE, "d = %d outside [1, 16000]", ly->d);
  if (ly->n_q_heads < 1 || ly->n_kv_heads < 1 || ly->n_q_heads % ly->n_kv_heads != 0)
    return fail(ctx, ALORA_ESHAPE, "n_q_heads = %d must be a positive multiple of n_kv_heads = %d",
                ly->n_q_heads, ly->n_kv_heads);
  if (ly->head_dim < 2 || ly->head_dim > 256 || (ly->head_dim & 1))
    return fail(ctx, ALORA_ESHAPE, "head_dim = %d must be even and in [2, 256]", ly->head_dim);
  if (ly->n_adapters < 0) return fail(ctx, ALORA_ESHAPE, "n_adapters = %d is negative", ly->n_adapters);
  if (ly->rank < 0 || ly->rank > 256 || (ly->n_adapters > 0 && ly->rank < 1))
    return fail(ctx, ALORA_ESHAPE, "rank = %d outside [1, 256]", ly->rank);
  if (!ly->W_qkv) return fail(ctx, ALORA_EINVAL, "W_qkv is NULL");
  if (ly->n_adapters > 0 && (!ly->A || !ly->B_q || !ly->B_k || !ly->B_v || !ly->scale))
    return fail(ctx, ALORA_EINVAL, "adapter tensors (A, B_q, B_k, B_v, scale) must be given when n_adapters > 0");
  if (!(ly->rope_theta > 0.f)) return fail(ctx, ALORA_ESHAPE, "rope_theta must be positive");
  if (need_tail) {
    if (ly->intermediate < 1) return fail(ctx, ALORA_ESHAPE, "intermediate = %d must be positive", ly->intermediate);
    if (!ly->W_o || !ly->rms2_gain || !ly->W_gate || !ly->W_up || !ly->W_down)
      return fail(ctx, ALORA_EINVAL, "W_o, rms2_gain, W_gate, W_up and W_down are required for a layer stack");
    const bool any_rest = ly->A_o || ly->B_o || ly->A_gu || ly->B_gate || ly->B_up || ly->A_down || ly->B_down;
    if (any_rest && ly->n_adapters < 1)
      return fail(ctx, ALORA_EINVAL, "adapters of W_o / the MLP are given but n_adapters = 0");
    if ((ly->A_o != nullptr) != (ly->B_o != nullptr)) return fail(ctx, ALORA_EINVAL, "A_o and B_o go together");
    if ((ly->A_down != nullptr) != (ly->B_down != nullptr)) return fail(ctx, ALORA_EINVAL, "A_down and B_down go together");
    if ((ly->A_gu != nullptr) != (ly->B_gate != nullptr) || (ly->A_gu != nullptr) != (ly->B_up != nullptr))
      return fail(ctx, ALORA_EINVAL, "A_gu, B_gate and B_up go together");
  }
  L->d = ly->d; L->n_q_heads = ly->n_q_heads; L->n_kv_heads = ly->n_kv_heads; L->head_dim = ly->head_dim;
  L->rank = ly->rank; L->n_adapters = ly->n_adapters;
  L->n_q = ly->n_q_heads * ly->head_dim;
  L->n_kv = ly->n_kv_heads * ly->head_dim;
  L->n_qkv = L->n_q + 2 * L->n_kv;
  return ALORA_OK;
}

alora_status check_batch(alora_ctx *ctx, const alora_layer_desc *ly, const alora_kv_cache *cache,
                         const int32_t *cu, const int32_t *kps, const int32_t *aps, int B, int n_steps, Plan *pl) {
  if (!cache) return fail(ctx, ALORA_EINVAL, "cache is NULL");
  if (B < 1) return fail(ctx, ALORA_EINVAL, "B = %d must be at least 1", B);
  if (!cu || !kps || !aps) return fail(ctx, ALORA_EINVAL, "cu_seqlens / k_per_seq / adapter_per_seq is NULL");
  if (!cache->seq_offset || !cache->seq_capacity || !cache->seq_len)
    return fail(ctx, ALORA_EINVAL, "cache seq_offset / seq_capacity / seq_len is NULL");
  if (!cache->k || !cache->v) return fail(ctx, ALORA_EINVAL, "cache k / v is NULL");
  if (cache->prefix_len && !cache->prefix_offset)
    return fail(ctx, ALORA_EINVAL, "cache prefix_len is given without prefix_offset");
  if (cu[0] != 0) return fail(ctx, ALORA_EINVAL, "cu_seqlens[0] = %d must be 0", cu[0]);
  pl->B = B;
  pl->seqs.resize(B);
  pl->max_len = 0;
  pl->any_adapter = false;
  pl->any_prefix = false;
  pl->n_used = 0;
  uint64_t listed = 0;
  for (int b = 0; b < B; ++b) {
    const int S = cu[b + 1] - cu[b];
    if (S < 0) return fail(ctx, ALORA_EINVAL, "cu_seqlens decreases at sequence %d", b);
    const int P = cache->seq_len[b];
    const int cap = cache->seq_capacity[b];
    const int64_t off = cache->seq_offset[b];
    if (P < 0) return fail(ctx, ALORA_EINVAL, "seq_len[%d] = %d is negative", b, P);
    if (kps[b] < 0) return fail(ctx, ALORA_EINVAL, "k_per_seq[%d] = %d is negative", b, kps[b]);
    if (aps[b] < -1 || aps[b] >= ly->n_adapters)
      return fail(ctx, ALORA_EADAPTER, "adapter_per_seq[%d] = %d outside [-1, %d)", b, aps[b], ly->n_adapters);
    if (cap < 0 || off < 0 || off + cap > cache->pool_tokens)
      return fail(ctx, ALORA_ECAPACITY, "sequence %d: rows [%lld, %lld) lie outside the pool of %lld tokens", b,
                  (long long)off, (long long)(off + cap), (long long)cache->pool_tokens);
    const int plen = cache->prefix_len ? cache->prefix_len[b] : 0;
    const int64_t poff = plen > 0 ? cache->prefix_offset[b] : 0;
    if (plen < 0 || plen > P)
      return fail(ctx, ALORA_EINVAL, "sequence %d: prefix_len = %d outside [0, seq_len = %d]", b, plen, P);
    if (plen > 0 && (poff < 0 || poff + plen > cache->pool_tokens))
      return fail(ctx, ALORA_ECAPACITY, "sequence %d: shared prefix rows [%lld, %lld) lie outside the pool of %lld tokens",
                  b, (long long)poff, (long long)(poff + plen), (long long)cache->pool_tokens);
    const int64_t grown = (int64_t)P + (int64_t)S * n_steps;      // cached length after the call
    if (grown - plen > cap)
      return fail(ctx, ALORA_ECAPACITY, "sequence %d: %d cached + %lld new tokens exceed its capacity %d", b, P - plen,
                  (long long)S * n_steps, cap);
    if (grown > (1 << 24))
      return fail(ctx, ALORA_ECAPACITY, "sequence %d: position %lld beyond the supported 2^24", b, (long long)grown);
    SeqMeta &m = pl->seqs[b];
    m.row_start = cu[b]; m.n_new = S; m.P = P; m.k = kps[b]; m.adapter = aps[b];
    m.scale = aps[b] >= 0 ? ly->scale[aps[b]] : 0.f;
    m.pool_off = off - plen;
    m.prefix_off = poff;
    m.prefix_len = plen;
    m.pad_ = 0;
    if (plen > 0) pl->any_prefix = true;
    if (aps[b] >= 0 && S > 0 && grown > kps[b]) {
      pl->any_adapter = true;
      if (aps[b] < 64 && !((listed >> aps[b]) & 1)) {
        listed |= 1ull << aps[b];
        pl->used[pl->n_used] = (uint8_t)aps[b];
        pl->used_scale[pl->n_used++] = m.scale;
      }
    }
    pl->max_len = std::max(pl->max_len, (int)grown);
  }
  pl->T = cu[B];
  count_adapted_tiles(pl, n_steps - 1);
  // The regions the sequences own must be disjoint, and nobody may write where somebody reads a shared prefix:
  // the kernels would write those cache rows concurrently, silently.
  {
    struct Iv { int64_t lo, hi; int b; };
    std::vector<Iv> own, wr, pf;
    for (int b = 0; b < B; ++b) {
      const SeqMeta &m = pl->seqs[b];
      const int64_t off = cache->seq_offset[b];
      if (cache->seq_capacity[b] > 0) own.push_back(Iv{off, off + cache->seq_capacity[b], b});
      if (m.n_new > 0) {
        const int64_t w0 = off + (m.P - m.prefix_len);
        wr.push_back(Iv{w0, w0 + (int64_t)m.n_new * n_steps, b});
      }
      if (m.prefix_len > 0) pf.push_back(Iv{m.prefix_off, m.prefix_off + m.prefix_len, b});
    }
    auto by_lo = [](const Iv &x, const Iv &y) { return x.lo < y.lo; };
    std::sort(own.begin(), own.end(), by_lo);
    for (size_t i = 1; i < own.size(); ++i)
      if (own[i].lo < own[i - 1].hi)
        return fail(ctx, ALORA_ECAPACITY, "sequences %d and %d own overlapping cache rows [%lld, %lld) and [%lld, %lld)",
                    own[i - 1].b, own[i].b, (long long)own[i - 1].lo, (long long)own[i - 1].hi, (long long)own[i].lo,
                    (long long)own[i].hi);
    if (!pf.empty() && !wr.empty()) {
      std::sort(wr.begin(), wr.end(), by_lo);       // disjoint (inside disjoint regions), so sorted by hi as well
      std::sort(pf.begin(), pf.end(), by_lo);
      size_t j = 0;
      for (const Iv &p : pf) {
        while (j < wr.size() && wr[j].hi <= p.lo) ++j;     // prefixes come in ascending lo: skipped writes end before all later ones too
        for (size_t q = j; q < wr.size() && wr[q].lo < p.hi; ++q)
          if (wr[q].hi > p.lo)
            return fail(ctx, ALORA_ECAPACITY, "sequence %d would write rows [%lld, %lld) that sequence %d reads as its shared prefix",
                        wr[q].b, (long long)wr[q].lo, (long long)wr[q].hi, p.b);
      }
    }
  }
  return ALORA_OK;
}

struct Workspace {
  RowMeta rm;
  void *xh;        // [T, d]
  float *tlow;     // [T, 3r]
  float *Y;        // [k_splits, T, n_qkv] fp32 projection partials; also split-K scratch of the dense layers
  size_t y_floats;
  void *Q;         // [T, n_q]
  float *partials;
  // layer-stack buffers
  void *attn, *h1, *hn, *gate, *up, *xa, *xb;
  int dec_hw = 1, dec_kr = 1, dec_cols_max = 1;      // shape of the decode attention workgroups
  float *f0 = nullptr, *f1 = nullptr;      // plain bf16 stack: sums of a linear before their one rounding
  size_t bytes;
  bool mfma = false;
  int k_splits = 1;                  // workgroups per output tile along the reduction axis of the QKV projection
  int k_segments = 1;                // its fixed reduction segments (from the weight shape alone)
  int lora_split = 0;                // the low-rank term of the QKV projection has a partial of its own
  bool attn_mfma = false;
  bool decode_mfma = false;
  int attn_waves = 8;
  int run_steps = 0, run_seqs = 0;   // a run of decode steps whose attention is prefill attention (AttnArgs::steps, order)
  const int32_t *run_order = nullptr;
  const AttnItem *qtiles = nullptr;
  int n_qtiles = 0;
  const DecItem *ditems = nullptr;   // work list of the MFMA decode kernel
  int n_ditems = 0;
  const int32_t *drows = nullptr;    // rows of its shared items
  MergeCounts merge{nullptr, 0};     // records per row (decode)
  const float *scale_dev = nullptr;  // [n_adapters] s_a on the device (adapters of W_o / the MLP)
  const uint4 *stage_src = nullptr;  // staged metadata that the first kernel of the call carries to the device (n16 > 0)
  uint4 *stage_dst = nullptr;
  int stage_n16 = 0;
  bool any_adapter = false;
  const Plan *pl = nullptr;
  const float2 *rope = nullptr;      // rotary table: one line per position, or (rope_by_row) one per packed row
  bool rope_by_row = false;
  float2 *rope_rows = nullptr;       // where the per-row table is built after row preparation
};

int pick_splits(const alora_ctx *ctx, int T, int n_kv_heads, int max_len) {
  if (ctx->opt_splits > 0) return ctx->opt_splits;
  // enough (row, kv head, split) work items to fill the chip, chunks of at least 256 keys
  int64_t items = (int64_t)T * n_kv_heads;
  int want = (int)std::min<int64_t>(64, std::max<int64_t>(1, (4 * ctx->n_cu + items - 1) / std::max<int64_t>(items, 1)));
  int max_by_len = std::max(1, max_len / 256);
  return std::max(1, std::min(want, max_by_len));
}

// (T_attn: rows that attend together, where that is fewer than are projected together)
Workspace layout_workspace(char *base, const LayerDims &L, int T, size_t esz, int n_splits, int k_splits,
                           int intermediate, bool stack, bool f32_tail = false, int T_attn = 0) {
  Bump b(base);
  Workspace w{};
  w.rm.seq = b.take<int32_t>(T);
  w.rm.pos = b.take<int32_t>(T);
  w.rm.adapter = b.take<int32_t>(T);
  w.rm.slot = b.take<int64_t>(T);
  w.rm.present16 = b.take<unsigned long long>((T + 15) / 16);
  w.xh = b.take<char>((size_t)(T <= QKV_STREAM_ROWS ? (T + 31) & ~31 : T) * L.d * esz);      // (operand order: blocks of 32 rows)
  w.tlow = b.take<float>((size_t)T * 3 * std::max(L.rank, 1));
  w.y_floats = (size_t)T * L.n_qkv * (std::max(k_splits, 1) + 1);
  if (stack) {      // split-K partials of W_o / W_down and of the down-projections of their adapters
    w.y_floats = std::max(w.y_floats, (size_t)8 * T * L.d);
    w.y_floats = std::max(w.y_floats, (size_t)8 * T * std::max(L.n_adapters, 1) * 2 * std::max(L.rank, 1));
  }
  w.Y = b.take<float>(w.y_floats);
  w.Q = b.take<char>((size_t)T * L.n_q * 4);      // fp16 for the MFMA attention kernels, fp32 for the plain one
  w.partials = b.take<float>(attn_plain_partial_floats(L, T_attn > 0 ? T_attn : T, n_splits));
  if (stack) {
    w.attn = b.take<char>((size_t)T * L.n_q * esz);
    w.h1 = b.take<char>((size_t)T * L.d * esz);
    const size_t rows = T <= STREAM_ROWS ? (T + 31) & ~31 : T;      // (operand order: blocks of 32 rows)
    w.hn = b.take<char>(rows * L.d * esz);
    w.gate = b.take<char>(rows * intermediate * esz);
    w.up = b.take<char>((size_t)T * intermediate * esz);
    w.xa = b.take<char>((size_t)T * L.d * esz);
    w.xb = b.take<char>((size_t)T * L.d * esz);
    if (f32_tail) {
      w.f0 = b.take<float>((size_t)T * std::max(intermediate, L.d));
      w.f1 = b.take<float>((size_t)T * std::max(intermediate, L.d));
    }
  }
  w.bytes = b.off;
  return w;
}

// How the queries are stored between projection and attention.
// The MFMA attention kernels (prefill and decode) take them as fp16 (every operand of their matrix products is fp16), prefill
// in its folded-softmax form premultiplied by sm_scale * log2(e); the plain attention kernel reads them as fp32 (the Q buffer holds
// four bytes per element).
struct QueryForm { bool half; float scale; };
template <typename T> QueryForm query_form(const alora_ctx *ctx, const LayerDims &L, const Workspace &w) {
  const bool half = (w.attn_mfma || w.decode_mfma) && std::is_same<T, bf16>::value;
  return QueryForm{half, (w.attn_mfma && half) ? attn_prefill_mfma_q_scale(L, ctx->opt_attn_fold != 0) : 1.0f};
}

// The first half of an attention block on already-staged metadata: rows -> projections -> rotation/append.
// write_meta is false for layers after the first of a stack (same rows).
template <typename T>
void project_rows(alora_ctx *ctx, const alora_layer_desc *ly, const LayerDims &L, const alora_kv_cache *cache,
                  const T *x, const Plan &pl, const SeqMeta *seqs_dev, const Workspace &w, bool write_meta,
                  int pos_shift, hipStream_t s) {
  const bool mfma = w.mfma && std::is_same<T, bf16>::value;
  const int rank_used = pl.any_adapter ? L.rank : 0;
  const bool prep_mfma = mfma && prep_rows_mfma_supported(L.d, rank_used);      // it also leaves the adapter masks
  const QueryForm qf = query_form<T>(ctx, L, w);
  const bool q_half = qf.half;
  const int q_mode = q_half ? 1 : 2;
  const float q_scale = qf.scale;
  // The projection rotates and appends by itself: up to stream_rows rows in the kernel that streams the weights past all rows,
  // beyond that, where a head is 128 columns, in tiles of 128 or 256 rows (all add in one order), or in the
  // 128 x 128 block of four waves, which also adds segments.
  const bool fuse = mfma && ctx->opt_rope_fuse && ctx->opt_gemm_tile < 4 && ctx->opt_gemm_tile != 1;
  const bool lora_split = pl.any_adapter && w.lora_split;      // (in a kernel that takes partial sums)
  GemmArgs g{};
  if (mfma) {
    g.A = (const bf16 *)w.xh; g.lda = L.d;
    g.B = (const bf16 *)ly->W_qkv; g.ldb = L.d;
    g.M = pl.T; g.N = L.n_qkv; g.K = L.d;
    g.k_splits = w.k_splits;
    g.k_segments = w.k_segments;
    g.lora_split = lora_split ? 1 : 0;
    g.tile_hint = ctx->opt_gemm_tile;
    g.Cpart = w.Y;
    g.tlow = pl.any_adapter ? (const bf16 *)w.tlow : nullptr;
    g.rank = L.rank;
    g.lr_parts = 3;
    g.Bq = (const bf16 *)ly->B_q; g.Bk = (const bf16 *)ly->B_k; g.Bv = (const bf16 *)ly->B_v;
    g.n_q = L.n_q; g.n_kv = L.n_kv;
    g.row_adapter = w.rm.adapter;
    g.present16 = prep_mfma ? w.rm.present16 : nullptr;
    g.rope_pos = w.rm.pos; g.rope_slot = w.rm.slot; g.rope_table = w.rope; g.q_scale = q_scale;
    g.rope_by_row = w.rope_by_row ? 1 : 0;
    g.head_dim = L.head_dim; g.q_f32 = q_half ? 0 : 1;
    g.Qout = (bf16 *)w.Q; g.cacheK = (bf16 *)cache->k; g.cacheV = (bf16 *)cache->v;
  }
  // The tiles are the quicker way from 129 rows on, unless even those of 64 columns leave more than three fifths of the chip idle: preparation and projection, us, streamed / in
  // tiles, 129 rows and 256: N x K 6144 x 4096 50.9 / 45.6 and 64.8 / 60.0, 7680 x 5120 102.6 / 93.1 and 105.9 / 103.0, 3840 x 2560 56.1 / 54.7 and 59.5 / 60.5,
  // 3072 x 2048 29.1 / 28.9 and 37.1 / 37.5 (224 rows 30.3 / 32.0), 1536 x 1024 21.0 / 22.0 and 24.0 / 25.3.  (128 rows of 6144 x 4096: 22.7 / 28.9, the projection alone.)
  const bool tiles = fuse && q_half && !w.rope_by_row && w.k_segments == 1 && gemm_mfma_rope_supported(g, L.head_dim) && gemm_large_supported(g, GEMM_EPI_ROPE);
  const bool tiles_fill = 5 * ((L.n_qkv + 63) / 64) >= ctx->n_cu;
  const int stream_rows = tiles && tiles_fill ? std::min(128, qkv_stream_rows(L.n_qkv, ctx->n_cu)) : qkv_stream_rows(L.n_qkv, ctx->n_cu);
  const bool stream = fuse && !lora_split && w.k_segments == 1 && ctx->opt_gemm_tile == 0 && pl.T <= stream_rows && qkv_stream_supported(ly->W_qkv, L.n_qkv, L.d, L.head_dim);
  auto stage_of = [&](bool first) {
    StagedCall st{};
    if (w.stage_n16 > 0) {
      st.n_few = pl.B;
      memcpy(st.few, pl.seqs.data(), (size_t)pl.B * sizeof(SeqMeta));
      if (first) { st.src = w.stage_src; st.dst = w.stage_dst; st.n16 = w.stage_n16; }
    }
    return st;
  };
  {
    ProfScope p(ctx, K_PREP, s);
    if (prep_mfma) {
      PrepArgs pa{};
      pa.x = (const bf16 *)x; pa.gain = (const bf16 *)ly->rms_gain; pa.eps = ly->rms_eps;
      pa.T = pl.T; pa.d = L.d; pa.seqs = seqs_dev; pa.n_seqs = pl.B; pa.pos_shift = pos_shift;
      pa.st = stage_of(write_meta && pos_shift == 0);
      pa.A = rank_used ? (const bf16 *)ly->A : nullptr; pa.rank = rank_used;
      if (rank_used) {
        pa.parts = 3;
        pa.n_used = pl.n_used;
        pa.adapted_tiles = pl.adapted_tiles;
        memcpy(pa.used, pl.used, sizeof pa.used);
        memcpy(pa.used_scale, pl.used_scale, sizeof pa.used_scale);
      }
      pa.few = ctx->opt_prep_split;
      pa.write_meta = write_meta ? 1 : 0;
      pa.xh = (bf16 *)w.xh; pa.packed = stream ? 1 : 0; pa.tlow16 = (bf16 *)w.tlow; pa.rm = w.rm;
      launch_prep_rows_mfma(pa, s);
    } else {
      launch_prep_rows<T>(x, (const T *)ly->rms_gain, ly->rms_eps, pl.T, L.d, seqs_dev, pl.B, pos_shift,
                          (const T *)ly->A, rank_used, write_meta, (T *)w.xh, w.tlow, mfma ? (bf16 *)w.tlow : nullptr, w.rm, stage_of(write_meta && pos_shift == 0), stream, s);
    }
  }
  if (w.rope_by_row) launch_rope_rows(w.rope_rows, w.rm.pos, pl.T, L.head_dim / 2, ly->rope_theta, s);
  bool rope_fused = false;
  {
    ProfScope p(ctx, K_QKV, s);
    if (mfma) {
      if (stream) {
        launch_qkv_stream(g, ctx->n_cu, s);
        rope_fused = true;
      } else if (tiles && pl.T > stream_rows) {
        launch_gemm_large(g, GEMM_EPI_ROPE, gemm_large_plan(ctx->opt_gemm_tile, g, ctx->n_cu, 1), s);
        rope_fused = true;
      } else if (fuse && q_half && !w.rope_by_row && ctx->opt_gemm_tile == 0 && pl.T > 256 && gemm_mfma_rope_supported(g, L.head_dim)) {
        launch_gemm_mfma(g, GEMM_EPI_ROPE, ctx->n_cu, s);
        rope_fused = true;
      } else {
        launch_gemm_mfma(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
      }
    } else if (qkv_small_plain_wanted(pl.T, L.n_qkv, ctx->n_cu)) {
      launch_qkv_small_plain<T>((const T *)w.xh, (const T *)ly->W_qkv, w.tlow, (const T *)ly->B_q, (const T *)ly->B_k, (const T *)ly->B_v,
                                L, w.rm, pl.T, w.rope, w.rope_by_row, q_scale, q_mode, w.Q, (T *)cache->k, (T *)cache->v, s);
      rope_fused = true;
    } else {
      launch_qkv_gemm_plain<T>((const T *)w.xh, (const T *)ly->W_qkv, w.tlow, (const T *)ly->B_q,
                               (const T *)ly->B_k, (const T *)ly->B_v, L, w.rm, pl.T, w.Y, s);
    }
  }
  if (!rope_fused) {
    ProfScope p(ctx, K_ROPE, s);
    launch_rope_append<T>(w.Y, mfma ? w.k_splits + (lora_split ? 1 : 0) : 1, L, w.rm, pl.T, w.rope, w.rope_by_row, q_scale, q_mode, w.Q,
                          (T *)cache->k, (T *)cache->v, s);
  }
}

// The second half: attention of pl's rows, whose queries and metadata begin at row `row0` of the workspace's.
template <typename T>
void attend_rows(alora_ctx *ctx, const LayerDims &L, const alora_kv_cache *cache, const Plan &pl, const SeqMeta *seqs_dev, const Workspace &w,
                 int n_splits, bool decode, int pos_shift, int row0, T *out, hipStream_t s) {
  const QueryForm qf = query_form<T>(ctx, L, w);
  const void *Q = (const char *)w.Q + (size_t)row0 * L.n_q * (qf.half ? 2 : 4);
  const bool mfma_attn = std::is_same<T, bf16>::value && (w.attn_mfma || w.decode_mfma);
  const bool direct = n_splits == 1 && (mfma_attn ? w.attn_mfma && w.run_steps == 0 : true);
  // split prefill attention on the MFMA path: partial results travel in the compact record
  // (the records of decode steps stay in fp32)
  const bool compact16 = w.attn_mfma && std::is_same<T, bf16>::value && !direct && ctx->opt_attn_partials16 && w.run_steps == 0;
  // `folded`: the queries carry the softmax scale and log2(e) already
  auto decode_items = [&](bool folded) {
    ProfScope p(ctx, K_ATTN_DECODE, s);
    DecodeArgs a{};
    a.Q = (const _Float16 *)Q; a.K = (const bf16 *)cache->k; a.V = (const bf16 *)cache->v;
    a.n_q = L.n_q; a.n_kv = L.n_kv; a.n_q_heads = L.n_q_heads; a.n_kv_heads = L.n_kv_heads;
    a.items = w.ditems; a.rows = w.drows; a.pos_shift = pos_shift;
    a.n_parts = n_splits;
    a.heads_per_wg = w.dec_hw; a.ranges_per_wg = w.dec_kr; a.cols_max = w.dec_cols_max;
    a.sm_scale = folded ? 0.6931471805599453f : 1.0f / sqrtf((float)L.head_dim);
    a.partials = w.partials;
    a.keys_max = w.run_steps > 0 ? w.run_steps : pl.max_len;
    launch_attn_decode_mfma(a, w.n_ditems, s);
  };
  if (w.attn_mfma && std::is_same<T, bf16>::value) {
    ProfScope p(ctx, K_ATTN_PREFILL, s);
    AttnArgs a{};
    a.Q = (const _Float16 *)Q; a.K = (const bf16 *)cache->k; a.V = (const bf16 *)cache->v;
    a.work = w.qtiles;
    a.n_q = L.n_q; a.n_kv = L.n_kv; a.n_q_heads = L.n_q_heads; a.n_kv_heads = L.n_kv_heads;
    a.n_parts = n_splits;
    a.sm_scale = 1.0f / sqrtf((float)L.head_dim);
    a.lazy = (float)ctx->opt_attn_lazy;
    a.steps = w.run_steps; a.seqs = w.run_seqs; a.order = w.run_order;
    a.q_prescaled = qf.scale != 1.0f;
    a.partials = direct ? nullptr : w.partials;
    a.compact = compact16 ? 1 : 0;
    a.out = direct ? (bf16 *)out : nullptr;
    // the kernels' fast tile loads use 32-bit byte offsets from an item's first key row; (absurdly) long
    // sequences take the variant with full address arithmetic
    bool generic_addr = false;
    for (const SeqMeta &q : pl.seqs)
      if ((uint64_t)(q.P + q.n_new) * (uint64_t)L.n_kv * 2u >= (1ull << 31)) generic_addr = true;
    launch_attn_prefill_mfma(a, w.n_qtiles, L.n_q_heads / L.n_kv_heads, w.attn_waves, generic_addr, s);
  } else if (w.decode_mfma && std::is_same<T, bf16>::value) {
    decode_items(false);
  } else {
    ProfScope p(ctx, decode ? K_ATTN_DECODE : K_ATTN_PREFILL, s);
    RowMeta rm = w.rm;
    rm.seq += row0; rm.pos += row0;      // (all it reads of them)
    launch_attn_plain<T>((const float *)Q, (const T *)cache->k, (const T *)cache->v, seqs_dev, rm, L, pl.T,
                         n_splits, w.partials, direct ? out : nullptr, s);
  }
  if (w.run_steps > 0) decode_items(true);      // (a run of decode steps: its own keys)
  if (!direct) {
    ProfScope p(ctx, K_ATTN_MERGE, s);
    if (compact16) launch_attn_merge16(w.partials, L, pl.T, n_splits, (bf16 *)out, s);
    else launch_attn_merge<T>(w.partials, L, pl.T, n_splits, w.merge, out, s);
  }
}

template <typename T>
void attention_block(alora_ctx *ctx, const alora_layer_desc *ly, const LayerDims &L, const alora_kv_cache *cache,
                     const T *x, const Plan &pl, const SeqMeta *seqs_dev, const Workspace &w, bool write_meta,
                     int n_splits, bool decode, int pos_shift, T *out, hipStream_t s) {
  project_rows<T>(ctx, ly, L, cache, x, pl, seqs_dev, w, write_meta, pos_shift, s);
  attend_rows<T>(ctx, L, cache, pl, seqs_dev, w, n_splits, decode, pos_shift, 0, out, s);
}

template <typename T>
void layer_tail(alora_ctx *ctx, const alora_layer_desc *ly, const LayerDims &L, const T *x, const Workspace &w,
                int T_rows, T *out, hipStream_t s) {
  RowMeta none{};
  const bool mfma = w.mfma && std::is_same<T, bf16>::value;
  const int r = L.rank, n_ad = L.n_adapters;
  // Few rows with default options: gate/up, W_down and the adapters' down-projections in the kernel that streams weights past all rows
  auto streamed = [&](const GemmArgs &g, int epi) {
    return mfma && ctx->opt_gemm_splits == 0 && ctx->opt_gemm_tile == 0 && gemm_stream_supported(g, epi, ctx->n_cu);
  };
  auto linear = [&](const void *W, const void *W2, int N, int K) {
    GemmArgs g{};
    g.B = (const bf16 *)W; g.B2 = (const bf16 *)W2; g.ldb = K;
    g.M = T_rows; g.N = W2 ? 2 * N : N; g.K = K; g.rank = r;
    return g;
  };
  // Adapters of these linears (Eq.6 applied to them): on the MFMA path t = s_a A_a z is computed for all
  // adapters at once as a skinny GEMM against the stacked down-matrices [n_ad * parts * r, K] (exactly how
  // they are stored), each adapted row then picks its adapter's slice as a bf16 (hi, lo) pair, and the
  // up-projection runs as extra k-steps of the base GEMM; on the plain path the term is added afterwards.
  // Or, where the reduction is short enough for one workgroup (a step of 128 takes about 0.3 us), t of each row's adapter alone, in one
  // kernel: 139 rows, K = 4096, 11 us against 10 and 6. (K = 14336: 11 and 8.)
  auto lowrank_t = [&](const void *z, bool packed, int K, const void *A_all, int parts) {
    PrepArgs pa{};
    pa.T = T_rows; pa.d = K; pa.A = (const bf16 *)A_all; pa.rank = r; pa.parts = parts;
    pa.xh = (bf16 *)const_cast<void *>(z); pa.packed = packed ? 1 : 0; pa.tlow16 = (bf16 *)w.tlow; pa.rm = w.rm;
    if (K <= 8192 && prep_rows_mfma_supported(L.d, r) && t_rows_mfma_supported(pa)) {
      pa.n_used = w.pl->n_used; pa.adapted_tiles = w.pl->adapted_tiles;
      memcpy(pa.used, w.pl->used, sizeof pa.used);
      memcpy(pa.used_scale, w.pl->used_scale, sizeof pa.used_scale);
      launch_t_rows_mfma(pa, s);
      return;
    }
    GemmArgs g{};
    g.A = (const bf16 *)z; g.lda = K; g.packed = packed ? 1 : 0;
    g.B = (const bf16 *)A_all; g.ldb = K;
    g.M = T_rows; g.N = n_ad * parts * r; g.K = K;
    g.Cpart = w.Y;
    int splits;
    if (streamed(g, GEMM_EPI_PARTIAL)) {
      splits = g.k_splits = gemm_stream_segments(g, ctx->n_cu, (int)std::min<size_t>(32, w.y_floats / ((size_t)T_rows * g.N)));
      launch_gemm_stream(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
    } else {
      splits = gemm_mfma_pick_splits(T_rows, g.N, K, ctx->n_cu);
      while (splits > 1 && (size_t)splits * T_rows * g.N > w.y_floats) splits /= 2;
      g.k_splits = splits;
      g.k_segments = splits;
      launch_gemm_mfma(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
    }
    launch_tlow_select(w.Y, splits, T_rows, n_ad, parts, r, w.rm.adapter, w.scale_dev, (bf16 *)w.tlow, s);
  };
  auto set_lowrank = [&](GemmArgs &g, const void *B0, const void *B1, int parts, int width) {
    g.tlow = (const bf16 *)w.tlow; g.rank = r; g.lr_parts = parts;
    g.Bq = (const bf16 *)B0; g.Bk = (const bf16 *)B1; g.Bv = nullptr;
    g.n_q = width; g.n_kv = parts == 1 ? 0 : width;
    g.row_adapter = w.rm.adapter;
    g.present16 = prep_rows_mfma_supported(L.d, r) ? w.rm.present16 : nullptr;      // (the row preparation that wrote it)
  };
  // reduction segments of a linear [N, K] where neither the large tiles nor the streaming kernel takes the call: fixed by the weight shape (or by
  // the gemm_splits option), so that a row's result does not depend on the number of rows among such calls
  auto segments_of = [&](int N, int K) {
    if (ctx->opt_gemm_splits > 0) return K % (64 * ctx->opt_gemm_splits) == 0 ? ctx->opt_gemm_splits : 1;
    return gemm_mfma_fixed_segments(N, K, ctx->n_cu);
  };
  // More than 32 rows with default splits: the large-tile kernels, whose partial sums (when it takes several workgroups per output tile)
  // land in Y.  Returns their number, 0: not this way, 1: C is written.
  auto large = [&](GemmArgs &g) -> int {
    if (T_rows <= 32 || (T_rows <= 256 && g.tile_hint != 0) || ctx->opt_gemm_splits != 0 || g.tile_hint == 1 || g.tile_hint >= 4) return 0;
    int most = 8;
    while (most > 1 && ((size_t)most * T_rows * g.N > w.y_floats || T_rows > gemm_large_slice_rows(g.lda))) most /= 2;
    const GemmLargePlan pn = T_rows <= 256 ? gemm_few_plan(g, ctx->n_cu) : gemm_large_plan(g.tile_hint, g, ctx->n_cu, std::min(most, 4));
    if (pn.splits == 0 || pn.splits > most) return 0;
    g.k_splits = pn.splits;
    const int epi = pn.splits > 1 ? GEMM_EPI_PARTIAL : GEMM_EPI_BF16;
    if (!gemm_large_supported(g, epi, T_rows <= 256 ? pn.rows : 256)) return 0;
    g.Cpart = w.Y;
    launch_gemm_large(g, epi, pn, s);
    return pn.splits;
  };
  // C = A W^T (+ R), with the gated low-rank term of (Al, Bl) when given
  auto dense = [&](const void *A, const void *W, const void *R, void *C, int N, int K, const void *Al, const void *Bl,
                   int parts = 1, int part = 0, bool packed = false) {
    const bool lr = Al != nullptr && w.any_adapter;
    if (mfma) {
      if (lr) lowrank_t(A, packed, K, Al, 1);
      GemmArgs g{};
      g.A = (const bf16 *)A; g.lda = K;
      g.B = (const bf16 *)W; g.ldb = K;
      g.M = T_rows; g.N = N; g.K = K;
      g.tile_hint = ctx->opt_gemm_tile;
      if (lr) set_lowrank(g, Bl, nullptr, 1, N);
      g.C = (bf16 *)C; g.ldc = N; g.R = (const bf16 *)R;
      g.packed = packed ? 1 : 0;
      if (streamed(g, GEMM_EPI_BF16)) {
        launch_gemm_stream(g, GEMM_EPI_BF16, ctx->n_cu, s);
        return;
      }
      if (const int n = large(g)) {
        if (n > 1) launch_splitk_reduce(w.Y, n, (int64_t)T_rows * N, (const bf16 *)R, (bf16 *)C, s);
        return;
      }
      // few row tiles: every segment gets workgroups of its own to fill the chip, the segment sums go through
      // the Y buffer; otherwise one workgroup adds them itself, in the same order
      const int segs = segments_of(N, K);
      g.k_segments = segs;
      if (segs > 1 && gemm_mfma_split_segments(T_rows, N, ctx->n_cu) && (size_t)segs * T_rows * N <= w.y_floats &&
          ((int64_t)T_rows * N) % 4 == 0) {
        g.k_splits = segs;
        g.Cpart = w.Y;
        launch_gemm_mfma(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
        launch_splitk_reduce(w.Y, segs, (int64_t)T_rows * N, (const bf16 *)R, (bf16 *)C, s);
      } else {
        g.k_splits = 1;
        launch_gemm_mfma(g, GEMM_EPI_BF16, ctx->n_cu, s);
      }
    } else if (w.f0 != nullptr) {
      // bf16 on the plain kernels: base product, low-rank term and residual are added in fp32 and rounded once
      launch_gemm_plain_f32<T>((const T *)A, (const T *)W, w.f0, T_rows, N, K, s);
      if (lr)
        launch_lowrank_add_plain<T, float>((const T *)A, K, (const T *)Al, parts, part, (const T *)Bl, N, r, w.rm.adapter,
                                           w.scale_dev, w.f0, T_rows, s);
      launch_residual_store<T>(w.f0, (const T *)R, (T *)C, (int64_t)T_rows * N, s);
    } else {
      launch_gemm_plain<T>((const T *)A, (const T *)W, (const T *)R, (T *)C, T_rows, N, K, s);
      if (lr)
        launch_lowrank_add_plain<T, T>((const T *)A, K, (const T *)Al, parts, part, (const T *)Bl, N, r, w.rm.adapter,
                                       w.scale_dev, (T *)C, T_rows, s);
    }
  };
  // h1 = x + attn W_o^T, hn = RMSNorm(h1).  When the projection is split over the reduction axis anyway, the
  // kernel that adds the partial sums also normalises the row (from its fp32 value) -- one launch less.
  // Between streamed products rows travel in the order of the matrix operand (a request of 64 lanes is 1 KB in a row, not 32 bytes of
  // 32 rows): 128 rows of gate/up 66 -> 48 us.  (The adapters' down-projections read them too.)
  const bool gu_stream = streamed(linear(ly->W_gate, ly->W_up, ly->intermediate, L.d), GEMM_EPI_SWIGLU);
  const bool hn_packed = gu_stream && (!(ly->A_gu && w.any_adapter) || streamed(linear(ly->A_gu, nullptr, n_ad * 2 * r, L.d), GEMM_EPI_PARTIAL));
  const bool act_packed = gu_stream && streamed(linear(ly->W_down, nullptr, L.d, ly->intermediate), GEMM_EPI_BF16) &&
                          (!(ly->A_down && w.any_adapter) || streamed(linear(ly->A_down, nullptr, n_ad * r, ly->intermediate), GEMM_EPI_PARTIAL));
  bool normed = false;
  {
    ProfScope p(ctx, K_OPROJ, s);
    const int splits = mfma ? segments_of(L.d, L.n_q) : 1;
    const bool few = splits > 1 && gemm_mfma_split_segments(T_rows, L.d, ctx->n_cu) && (size_t)splits * T_rows * L.d <= w.y_floats;
    if (mfma && splitk_reduce_norm_supported(L.d) && (few || T_rows > 256)) {
      GemmArgs g{};
      g.A = (const bf16 *)w.attn; g.lda = L.n_q;
      g.B = (const bf16 *)ly->W_o; g.ldb = L.n_q;
      g.M = T_rows; g.N = L.d; g.K = L.n_q;
      g.tile_hint = ctx->opt_gemm_tile;
      if (ly->A_o && w.any_adapter) {
        lowrank_t(w.attn, false, L.n_q, ly->A_o, 1);
        set_lowrank(g, ly->B_o, nullptr, 1, L.d);
      }
      g.C = (bf16 *)w.h1; g.ldc = L.d; g.R = (const bf16 *)x;
      int parts = large(g);
      if (parts == 0 && few) {
        g.k_splits = parts = splits;
        g.k_segments = splits;
        g.Cpart = w.Y;
        launch_gemm_mfma(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
      }
      if (parts > 1) {
        launch_splitk_reduce_norm(w.Y, parts, T_rows, L.d, (const bf16 *)x, (const bf16 *)ly->rms2_gain, ly->rms_eps,
                                  (bf16 *)w.h1, (bf16 *)w.hn, hn_packed, s);
        normed = true;
      } else if (parts == 0) {
        g.k_splits = 1;
        g.k_segments = splits;
        launch_gemm_mfma(g, GEMM_EPI_BF16, ctx->n_cu, s);
      }
    } else {
      dense(w.attn, ly->W_o, x, w.h1, L.d, L.n_q, ly->A_o, ly->B_o);
    }
  }
  if (!normed) {
    ProfScope p(ctx, K_MLPNORM, s);
    if (mfma && prep_rows_mfma_supported(L.d, 0)) {
      PrepArgs pa{};
      pa.x = (const bf16 *)w.h1; pa.gain = (const bf16 *)ly->rms2_gain; pa.eps = ly->rms_eps;
      pa.T = T_rows; pa.d = L.d; pa.xh = (bf16 *)w.hn; pa.packed = hn_packed ? 1 : 0; pa.rm = none;
      launch_prep_rows_mfma(pa, s);
    } else {
      launch_prep_rows<T>((const T *)w.h1, (const T *)ly->rms2_gain, ly->rms_eps, T_rows, L.d, nullptr, 0, 0,
                          (const T *)nullptr, 0, false, (T *)w.hn, nullptr, nullptr, none, StagedCall{}, hn_packed, s);
    }
  }
  if (mfma) {   // act = silu(hn W_gate^T) * (hn W_up^T) in one pass
    ProfScope p(ctx, K_GATEUP, s);
    GemmArgs g{};
    g.A = (const bf16 *)w.hn; g.lda = L.d;
    g.B = (const bf16 *)ly->W_gate; g.B2 = (const bf16 *)ly->W_up; g.ldb = L.d;
    g.M = T_rows; g.N = 2 * ly->intermediate; g.K = L.d; g.k_splits = 1; g.k_segments = 1;
    g.tile_hint = ctx->opt_gemm_tile;
    if (ly->A_gu && w.any_adapter) {
      lowrank_t(w.hn, hn_packed, L.d, ly->A_gu, 2);
      set_lowrank(g, ly->B_gate, ly->B_up, 2, ly->intermediate);
    }
    g.C = (bf16 *)w.gate; g.ldc = ly->intermediate;
    g.packed = (hn_packed ? 1 : 0) | (act_packed ? 2 : 0);
    if (streamed(g, GEMM_EPI_SWIGLU)) launch_gemm_stream(g, GEMM_EPI_SWIGLU, ctx->n_cu, s);
    else launch_gemm_mfma(g, GEMM_EPI_SWIGLU, ctx->n_cu, s);
  } else if (w.f0 != nullptr) {
    // bf16 on the plain kernels: gate and up stay in fp32 until silu(gate) * up is rounded, once
    const bool lr = ly->A_gu != nullptr && w.any_adapter;
    {
      ProfScope p(ctx, K_GATEUP, s);
      launch_gemm_plain_f32<T>((const T *)w.hn, (const T *)ly->W_gate, w.f0, T_rows, ly->intermediate, L.d, s);
      launch_gemm_plain_f32<T>((const T *)w.hn, (const T *)ly->W_up, w.f1, T_rows, ly->intermediate, L.d, s);
      if (lr) {
        launch_lowrank_add_plain<T, float>((const T *)w.hn, L.d, (const T *)ly->A_gu, 2, 0, (const T *)ly->B_gate,
                                           ly->intermediate, r, w.rm.adapter, w.scale_dev, w.f0, T_rows, s);
        launch_lowrank_add_plain<T, float>((const T *)w.hn, L.d, (const T *)ly->A_gu, 2, 1, (const T *)ly->B_up,
                                           ly->intermediate, r, w.rm.adapter, w.scale_dev, w.f1, T_rows, s);
      }
    }
    {
      ProfScope p(ctx, K_SILU, s);
      launch_silu_mul_f32<T>(w.f0, w.f1, (T *)w.gate, (int64_t)T_rows * ly->intermediate, s);
    }
  } else {
    {
      ProfScope p(ctx, K_GATEUP, s);
      dense(w.hn, ly->W_gate, nullptr, w.gate, ly->intermediate, L.d, ly->A_gu, ly->B_gate, 2, 0);
      dense(w.hn, ly->W_up, nullptr, w.up, ly->intermediate, L.d, ly->A_gu, ly->B_up, 2, 1);
    }
    {
      ProfScope p(ctx, K_SILU, s);
      launch_silu_mul<T>((const T *)w.gate, (const T *)w.up, (T *)w.gate, (int64_t)T_rows * ly->intermediate, s);
    }
  }
  {
    ProfScope p(ctx, K_DOWN, s);
    dense(w.gate, ly->W_down, w.h1, out, L.d, ly->intermediate, ly->A_down, ly->B_down, 1, 0, act_packed);
  }
}

// Work list of the MFMA decode kernel: per (row, group of kv heads) items over ranges of the row's own cache rows, and -- when
// sequences name shared prefixes -- per (group of up to 32 / G rows with the same prefix, group of kv heads) items over
// ranges of that prefix.  A workgroup's eight waves are hw kv heads x kr sub-ranges of the item's keys.
struct DecodePlan {
  std::vector<DecItem> items;      // empty when the list is built on the device (the static entry point)
  std::vector<int32_t> rows;       // rows of the shared items
  std::vector<int32_t> counts;     // records per row: own, shared
  int n_own = 1, n_shared = 0;     // most own and shared records of a row
  int range = 0;                   // keys per own range, before it is evened out (dec_cut)
  int n_device_items = 0;          // size of the device-built list: rows x head groups x n_own
  int hw = 1, kr = 1, groups = 1, cols_max = 1;
  double us = 0;                   // what a step's attention would take (decode_cut_us)
};

// What one way of cutting the keys would take, in us: `n_of` [s] workgroups run s steps of 32 keys per wave, `records` partial records, at
// most `most` per (row, head), are merged.  Longest first on n_cu units, one workgroup each: either the longest chain of
// steps counts (3.76 us a step) or memory, which delivers 24 bytes per ns and unit once 5/8 of the units ask, and waits with the tail
// where fewer do.  4.8 us a round, 0.5 to join sub-ranges in LDS, 3 % for rows of which a workgroup reads but two heads; 2.8 where
// more than 16 records of more than 512 (row, head) pairs are merged by a wave each.  Fitted to
// 5600 measured plans (1 to 500 rows of 64 to 40000 keys, 1 to 16 kv heads, shared prefixes; 6 % mean error).  Picked by it, attention
// with its merge takes 1.8 % longer than with the best of those plans on average; the rule it replaces (at least 512 keys each in two
// rounds, or sub-ranges in one) 5.7 %, and up to 1.8 x: 256 rows of 64 keys 40 -> 28 us, 64 rows of 4000 214 -> 188, 33 of 4000 150 -> 105.
double decode_cut_us(const std::vector<int> &n_of, int n_cu, double bytes, bool join, bool two_heads, double records, int64_t pairs, int most) {
  int64_t steps = 0, n = 0;
  int first = 0, last = 0;                           // most and fewest steps
  for (int s = (int)n_of.size() - 1; s > 0; --s)
    if (n_of[s]) { steps += (int64_t)s * n_of[s]; n += n_of[s]; first = std::max(first, s); last = s; }
  const int ks = n_cu * 5 / 8;                       // units that keep memory busy
  const int rounds = (int)((n + n_cu - 1) / n_cu);
  double longest = first, busy = 0;                  // steps of the unit that ends last, and of the ks that do
  if (n <= n_cu) {
    for (int s = first, left = ks; s > 0 && left > 0; --s) { const int k = std::min(left, n_of[s]); busy += (double)k * s; left -= k; }
  } else if (n <= 2 * n_cu) {
    std::vector<int> d;
    d.reserve((size_t)n);
    for (int s = first; s > 0; --s) d.insert(d.end(), (size_t)n_of[s], s);
    for (int64_t i = n_cu; i < n; ++i) d[2 * n_cu - 1 - i] += d[i];
    d.resize(n_cu);
    std::nth_element(d.begin(), d.begin() + ks, d.end(), [](int x, int y) { return x > y; });
    for (int i = 0; i < ks; ++i) { busy += d[i]; longest = std::max(longest, (double)d[i]); }
  } else {
    const double mean = (double)steps / n_cu;
    longest = std::max(longest, mean + 0.5 * last);
    busy = ks * mean;
  }
  // (a round that fills the chip to the last unit: a hundredth more, 64 rows of 4000 keys 181 us in 192 workgroups and 196 in 256)
  const double full = !two_heads && n > n_cu * 15 / 16 && n <= n_cu ? 1.01 : 1.0;
  const double memory = bytes / (24e3 * n_cu) * (1.0 + (ks * longest - busy) / (double)steps) * full / (two_heads ? 0.97 : 1.0);
  return std::max(3.76 * longest, memory) + 4.8 * rounds + (join ? 0.5 : 0.0) + 200e-6 * records + (most > 1 ? 0.7 : 0.0) +
         (most > 16 && pairs > 512 ? 2.8 : 0.0) + 0.017 * most;
}

// the sequences of a call, those that name one prefix next to each other
std::vector<int32_t> by_prefix(const Plan &pl) {
  std::vector<int32_t> order(pl.B);
  for (int b = 0; b < pl.B; ++b) order[b] = b;
  auto before = [&](int x, int y) {
    if (pl.seqs[x].prefix_off != pl.seqs[y].prefix_off) return pl.seqs[x].prefix_off < pl.seqs[y].prefix_off;
    return pl.seqs[x].prefix_len < pl.seqs[y].prefix_len;
  };
  if (!std::is_sorted(order.begin(), order.end(), before)) std::stable_sort(order.begin(), order.end(), before);
  return order;
}

// `cap`: most records of either kind a row may have (every row's place in memory is that large).
DecodePlan plan_decode_items(const alora_ctx *ctx, const Plan &pl, const LayerDims &L, int cap, int n_steps, bool on_device) {
  DecodePlan dp;
  const int G = L.n_q_heads / L.n_kv_heads;
  const int pack = std::max(1, 32 / G);
  // rows that share one prefix, at most `pack` each
  struct Chunk { int64_t off; int len; int first, n; };
  std::vector<Chunk> chunks;
  dp.cols_max = G;
  if (pl.any_prefix) {
    const std::vector<int32_t> order = by_prefix(pl);
    for (int i = 0; i < pl.B; ++i) {
      const SeqMeta &m = pl.seqs[order[i]];
      if (m.n_new <= 0 || m.prefix_len <= 0) continue;
      if (chunks.empty() || chunks.back().n >= pack || chunks.back().off != m.prefix_off || chunks.back().len != m.prefix_len)
        chunks.push_back(Chunk{m.prefix_off, m.prefix_len, (int)dp.rows.size(), 0});
      dp.rows.push_back(m.row_start);
      dp.cols_max = std::max(dp.cols_max, ++chunks.back().n * G);
    }
  }
  auto own_keys = [&](const SeqMeta &m) { return m.P + n_steps - m.prefix_len; };      // of the last step, the new key included
  int64_t keys = 0;
  int longest = 1;
  // the rows' own keys, then the prefixes; equal neighbours are one entry
  struct Run { int len, n, rows; bool own; };      // (rows: that get a record of every range)
  std::vector<Run> runs;
  runs.reserve((size_t)pl.B + chunks.size());
  int n_lens = 0;
  auto put_len = [&](int len, int rows, bool own) {
    if (!runs.empty() && runs.back().len == len && runs.back().own == own) { ++runs.back().n; runs.back().rows += rows; }
    else runs.push_back(Run{len, 1, rows, own});
    ++n_lens;
    keys += len;
    longest = std::max(longest, len);
  };
  for (const SeqMeta &m : pl.seqs)
    if (m.n_new > 0) put_len(own_keys(m), 1, true);
  for (const Chunk &c : chunks) put_len(c.len, c.n, false);
  // A workgroup is eight kv heads side by side, each over the whole range, or (a long row among few, heads that are no multiple of
  // eight) two kv heads x four sub-ranges that join in LDS; the ranges are as long as gives nearly one round of workgroups, one,
  // two, or one workgroup per row and group of heads.  Whichever takes the least time (decode_cut_us).
  decode_mfma_shape(L.n_kv_heads, false, &dp.hw, &dp.kr);
  dp.groups = (L.n_kv_heads + dp.hw - 1) / dp.hw;
  const int least = (longest + cap - 1) / cap;
  int range = longest;
  if (ctx->opt_splits == 0) {
    const int n_cu = ctx->n_cu;
    double best = 1e30;
    const int wide = dp.hw;
    std::vector<int> n_of;
    auto consider = [&](int hw, int kr, int r) {
      const int groups = (L.n_kv_heads + hw - 1) / hw;
      auto steps_of = [&](int len) { return (((len + kr - 1) / kr) + 31) >> 5; };
      n_of.assign((size_t)steps_of(((r + 31) & ~31)) + 1, 0);      // (dec_cut's ranges are whole steps of r or less)
      double records = 0;
      int own = 0, shared = 0;
      for (const Run &q : runs) {
        const DecCut c = dec_cut(q.len, r);
        n_of[steps_of(c.len)] += (c.parts - 1) * groups * q.n;
        n_of[steps_of(q.len - (c.parts - 1) * c.len)] += groups * q.n;
        (q.own ? own : shared) = std::max(q.own ? own : shared, c.parts);
        records += (double)c.parts * q.rows;
      }
      const double us = decode_cut_us(n_of, n_cu, 512.0 * keys * L.n_kv_heads, kr > 1, hw < wide, records * L.n_q_heads, (int64_t)pl.T * L.n_q_heads, own + shared);
      if (us < best) { best = dp.us = us; dp.hw = hw; dp.kr = kr; range = r; }
    };
    for (int form = cap > 1 && wide > 2 ? 0 : 1; form < 2; ++form) {
      int hw, kr, last = 0;
      decode_mfma_shape(L.n_kv_heads, form == 0, &hw, &kr);
      const int64_t groups = (L.n_kv_heads + hw - 1) / hw;
      const int64_t n1 = groups * (int64_t)n_lens;      // workgroups, one range each
      // (the last one: where rows alone are more than that, a long row among them still wants to be cut)
      for (int64_t most : {(int64_t)(form == 0 ? 0 : n_cu * 15 / 16), (int64_t)n_cu, (int64_t)2 * n_cu, n1 > n_cu ? n1 + n1 / 8 : 0}) {
        if (most < n1 || (form == 0 && n1 > (L.n_kv_heads % 8 ? 4 : 2) * n_cu)) continue;
        // the shortest ranges that `most` workgroups take, to within a tenth
        int r = (int)std::max<int64_t>({(int64_t)32 * kr, keys * groups / most & ~31, (int64_t)least});
        for (int i = 0; i < 24 && r < longest; ++i) {
          int64_t n = 0;
          if (runs.size() > 16) {      // (a number of workgroups that is a little too large now and then)
            const float inv = 1.0f / (float)r;
            int k = 0;
            for (const Run &q : runs) k += ((int)((float)(q.len - 1) * inv) + 1) * q.n;
            n = k * groups;
          } else {
            for (const Run &q : runs) n += dec_cut(q.len, r).parts * q.n;
            n *= groups;
          }
          if (n <= most) break;
          r += std::max(32, (int)(r * (n - most) / most) & ~31);
        }
        if (r != last) consider(hw, kr, r);
        last = r;
      }
      if (form == 1 && n1 > n_cu * 15 / 16) consider(hw, kr, longest);
    }
    dp.groups = (L.n_kv_heads + dp.hw - 1) / dp.hw;
  }
  auto cut_of = [&](int n) {
    if (ctx->opt_splits > 0) return dec_cut(n, std::max(1, (n + ctx->opt_splits - 1) / ctx->opt_splits));
    return dec_cut(n, range);
  };
  dp.range = range;
  for (const SeqMeta &m : pl.seqs)
    if (m.n_new > 0) dp.n_own = std::max(dp.n_own, cut_of(own_keys(m)).parts);
  for (const Chunk &c : chunks) dp.n_shared = std::max(dp.n_shared, cut_of(c.len).parts);
  dp.n_device_items = pl.T * dp.groups * dp.n_own;
  if (on_device) return dp;
  dp.counts.assign((size_t)2 * pl.T, 0);
  for (const Chunk &c : chunks) {
    const DecCut cut = cut_of(c.len);
    for (int i = 0; i < c.n; ++i) dp.counts[2 * dp.rows[c.first + i] + 1] = cut.parts;
    for (int sp = 0; sp < cut.parts; ++sp)
      for (int gb = 0; gb < dp.groups; ++gb) {
        DecItem it{};
        it.key_row0 = c.off; it.row = c.first; it.kbeg = sp * cut.len; it.kend = std::min(c.len, it.kbeg + cut.len);
        it.n_rows = (int16_t)c.n; it.g = (int16_t)(gb * dp.hw); it.part = (int16_t)(dp.n_own + sp); it.shared = 1;
        dp.items.push_back(it);
      }
  }
  for (const SeqMeta &m : pl.seqs) {
    if (m.n_new <= 0) continue;
    const DecCut cut = cut_of(own_keys(m));
    dp.counts[2 * m.row_start] = cut.parts;
    for (int gb = 0; gb < dp.groups; ++gb)
      for (int sp = 0; sp < cut.parts; ++sp) {
        DecItem it{};
        it.key_row0 = m.pool_off + m.prefix_len; it.row = m.row_start; it.kbeg = sp * cut.len; it.kend = std::min(own_keys(m), it.kbeg + cut.len);
        it.n_rows = 1; it.g = (int16_t)(gb * dp.hw); it.part = (int16_t)sp; it.n_keys = m.P + 1 - m.prefix_len;
        dp.items.push_back(it);
      }
  }
  // longest first, so that the short ones even out the end
  auto longer = [](const DecItem &x, const DecItem &y) { return x.kend - x.kbeg > y.kend - y.kbeg; };
  if (!std::is_sorted(dp.items.begin(), dp.items.end(), longer)) std::stable_sort(dp.items.begin(), dp.items.end(), longer);
  return dp;
}

// Work list of the MFMA prefill attention kernel, part 1: how the keys of a (row, head) are cut up.  Sequences that
// name no shared prefix cut their visible keys into n_own ranges.  Sequences that do cut their own keys (positions
// from prefix_len on) into n_own ranges, and the prefix into n_sh ranges that are walked once for ALL rows of a run
// of consecutive sequences naming that same prefix (Section 2, "Cache reuse patterns": several adapters invoked on
// one context): the rows of such a run are neighbours in the packed batch, so up to 256 / G of them share a
// workgroup and the prefix keys and values are fetched once per run instead of once per sequence.
struct PrefixRun { int64_t prefix_off; int prefix_len, row0, n_rows; };
struct PrefillPlan {
  std::vector<PrefixRun> runs;
  int n_own = 1, n_sh = 0;
  double tiles = 0;      // what the cut would take (prefill_cut_tiles), where anything is compared with it
};
// keys of a sequence behind its prefix that prefill attention walks
int prefill_own_keys(const Plan &pl, const SeqMeta &m) { return m.P - m.prefix_len + (pl.cached_only ? 0 : m.n_new); }

// What cutting the keys in n_own / n_sh ranges would take, in 64-key tiles of one workgroup: an eighth of the items on an XCD, one at a
// time on a compute unit, longest first, each PREFILL_ITEM_TILES long besides its keys (first tiles, queries, result), and the records
// that the merge then reads.  (Lengths in 64 classes: a few microseconds of host time for all the cuts of a call.)  Against the best of nine fixed cuts
// of 40 uniform calls of 8 and 32 kv heads it is 1 % slower on average, 15 % at most.  Row tiles taken as if the last key were theirs, and the merge
// at 4 TB/s, were 7.5 %, 54 % at most: 2500 rows on 64 cached keys in two ranges 81 us and a merge of 33, in one 77.
constexpr int PREFILL_ITEM_TILES = 5;
double prefill_cut_tiles(const alora_ctx *ctx, const Plan &pl, const LayerDims &L, int tq, const PrefillPlan &pp, int longest, int n_own, int n_sh) {
  int len[64] = {}, count[64] = {};
  int64_t work = 0, rows = 0;
  auto add = [&](int l, int n) {
    if (n <= 0) return;
    const int c = (int)((int64_t)l * 63 / longest);
    len[c] = std::max(len[c], l);
    count[c] += n;
    work += (int64_t)n * (l + PREFILL_ITEM_TILES);
  };
  auto cut = [&](int keys, int parts, int q_tiles) {      // q_tiles row tiles against the ranges of so many keys
    if (parts == 0) return;
    const int chunk = std::max(1, ((keys + parts - 1) / parts + 63) / 64), t = (keys + 63) / 64, whole = t / chunk;
    add(chunk, whole * q_tiles);
    if (t > whole * chunk) add(t - whole * chunk, q_tiles);
    add(0, (parts - whole - (t > whole * chunk ? 1 : 0)) * q_tiles);
  };
  for (const SeqMeta &m : pl.seqs) {
    if (m.n_new <= 0) continue;
    rows += m.n_new;
    const int parts = m.prefix_len > 0 ? n_own : n_own + n_sh, before = m.P - m.prefix_len;
    if (pl.cached_only) cut(before, parts, (m.n_new + tq - 1) / tq);
    else for (int q0 = 0; q0 < m.n_new; q0 += tq) cut(before + std::min(m.n_new, q0 + tq), parts, 1);      // (its keys end with a tile's rows)
  }
  for (const PrefixRun &r : pp.runs) cut(r.prefix_len, n_sh, (r.n_rows + tq - 1) / tq);
  // no schedule ends before its rounds of the longest items do, or before the work is done
  const double cus = ctx->n_cu / 8.0, per = L.n_kv_heads / 8.0;
  double worst = (double)work * per / cus, items = 0;
  for (int c = 63; c >= 0; --c) {
    if (count[c] == 0) continue;
    items += count[c] * per;
    worst = std::max(worst, std::ceil(items / cus) * (len[c] + PREFILL_ITEM_TILES));
  }
  // Records written, and the merge, a tile being about 1.7 us: a wave per (row, head), as long with eight records as with two (128 rows of 32 heads
  // 6 us, 1024 17, 2500 33), or their bytes.  (The records of a run of decode steps, one more each, are in fp32 and go to another kernel.)
  const double pairs = 1e-3 * (double)rows * L.n_q_heads;
  const int n = n_own + n_sh;
  if (pl.cached_only) worst += 2.0 + pairs * n * (2 * 520) / 4e3 / 1.7 + (n >= 16 && pairs > 0.512 ? 1.6 : 0.0);
  else if (n > 1) worst += (5.0 + std::max(0.34 * pairs, pairs * n * 272 / 3.6e3) + pairs * n * 0.068) / 1.7;
  return worst;
}

PrefillPlan plan_prefill_ranges(const alora_ctx *ctx, const Plan &pl, const LayerDims &L, int B, int attn_waves) {
  PrefillPlan pp;
  const int tq = attn_prefill_mfma_tokens_per_tile(L, attn_waves);
  int64_t tiles = 0;
  int max_own = 0, max_pfx = 0;      // (0: nothing cached behind the prefixes, and cached_only)
  for (int b = 0; b < B; ++b) {
    const SeqMeta &m = pl.seqs[b];
    if (m.n_new <= 0) continue;
    tiles += (m.n_new + tq - 1) / tq;
    max_own = std::max(max_own, prefill_own_keys(pl, m));
    max_pfx = std::max(max_pfx, m.prefix_len);
    if (m.prefix_len <= 0) continue;
    if (!pp.runs.empty() && pp.runs.back().prefix_off == m.prefix_off && pp.runs.back().prefix_len == m.prefix_len &&
        pp.runs.back().row0 + pp.runs.back().n_rows == m.row_start)
      pp.runs.back().n_rows += m.n_new;
    else
      pp.runs.push_back(PrefixRun{m.prefix_off, m.prefix_len, m.row_start, m.n_new});
  }
  if (ctx->opt_splits > 0) {
    pp.n_own = max_own > 0 ? ctx->opt_splits : 0;
    pp.n_sh = pp.runs.empty() ? 0 : ctx->opt_splits;
    return pp;
  }
  pp.n_own = max_own > 0 ? 1 : 0;
  if (max_own + max_pfx == 0) return pp;
  // Ranges of at least four tiles, at most 16, the cut that takes the least.  Before, ranges were as long as two items per compute unit (shared
  // prefixes) or one (no prefix) would have them: 32 x 16 rows on four contexts of 16384 keys 249 -> 224 us with one range per unit instead
  // of two, eight sequences of 128 rows on 32768 keys 4285 -> 4228 (four layers).
  // (and at most 2^20 records of a kind: half a gigabyte)
  // (a run of decode steps has few rows to a context, and as many ranges as a step of it: one row on 131072 keys of one kv head, two steps 175 us
  // in 16 ranges, 62 in as many as are worth it; 67 a step at a time)
  const int limit = pl.cached_only ? 256 : 16;
  const int longest = std::max(max_own, max_pfx);
  int most = (int)std::max<int64_t>(1, std::min<int64_t>(std::min(limit, longest / 256), (1 << 20) / ((int64_t)pl.T * L.n_q_heads)));
  if (pp.runs.empty() && tiles * L.n_kv_heads >= 4 * (int64_t)ctx->n_cu) most = 1;      // more items than could be evened out by cutting them
  if (most == 1 && !pl.cached_only && pp.runs.empty()) return pp;      // (nothing to compare)
  double least = 0;
  int was_own = 0, was_sh = 0;
  for (int n = 1; n <= most; n += n < 16 ? 1 : n / 4) {
    const int len = std::max(4, ((longest + 63) / 64 + n - 1) / n);      // tiles of a range
    auto ranges = [&](int keys) { return std::max(1, std::min(limit, ((keys + 63) / 64 + len - 1) / len)); };
    const int own = max_own > 0 ? ranges(max_own) : 0, sh = pp.runs.empty() ? 0 : ranges(max_pfx);
    if (own == was_own && sh == was_sh) continue;
    was_own = own; was_sh = sh;
    const double t = prefill_cut_tiles(ctx, pl, L, tq, pp, (longest + 63) / 64, own, sh);
    if (n == 1 || t < least) { least = pp.tiles = t; pp.n_own = own; pp.n_sh = sh; }
  }
  return pp;
}

// Part 2: the items, one per workgroup, in launch order.  Workgroups are dealt round-robin to the 8 XCDs, each with
// its own L2, and an XCD starts them in list order as compute units become free.  All q-tiles of one (sequence or
// prefix run, kv head, key range) read the same keys and values, so such a group goes to one XCD: groups are
// handed out heaviest first to the XCD with the least work so far, and inside an XCD the items run longest first
// (which keeps the q-tiles of a group next to each other: their lengths differ least).
std::vector<AttnItem> build_prefill_items(const Plan &pl, const LayerDims &L, int B, int attn_waves, const PrefillPlan &pp) {
  const int tq = attn_prefill_mfma_tokens_per_tile(L, attn_waves);
  const int n_own = pp.n_own, n_sh = pp.n_sh;
  struct Group { int64_t cost; std::vector<AttnItem> items; };      // the items of a group stream the same keys
  std::vector<Group> groups;
  // range `sp` of `parts` over the key positions [lo, hi), in whole tiles of 64 keys
  auto cut = [](int lo, int hi, int parts, int sp, AttnItem *it) {
    int chunk = (std::max(hi - lo, 0) + parts - 1) / parts;
    chunk = (chunk + 63) & ~63;
    it->kbeg = (int)std::min<int64_t>(hi, lo + (int64_t)sp * chunk);
    it->kend = (int)std::min<int64_t>(hi, (int64_t)it->kbeg + chunk);
  };
  auto key_tiles = [](const AttnItem &it) { return (int64_t)(it.kend - it.kbeg + 63) / 64 + 1; };
  for (int b = 0; b < B; ++b) {
    const SeqMeta &m = pl.seqs[b];
    if (m.n_new <= 0) continue;
    // (a sequence without prefix still writes n_own + n_sh records per (row, head): all of them over its own keys)
    const int parts = m.prefix_len > 0 ? n_own : n_own + n_sh;
    const int last = ((m.n_new - 1) / tq) * tq;
    for (int g = 0; g < L.n_kv_heads; ++g)
      for (int sp = 0; sp < parts; ++sp) {
        Group gr{0, {}};
        for (int q0 = last; q0 >= 0; q0 -= tq) {
          AttnItem it{};
          it.ntok = std::min(tq, m.n_new - q0);
          it.row0 = m.row_start + q0;
          // key positions count from the sequence's first own row (position prefix_len)
          it.pos0 = pl.cached_only ? 1 << 30 : m.P + q0 - m.prefix_len;
          it.key_row0 = m.pool_off + m.prefix_len;
          it.n_addr = pl.cached_only ? prefill_own_keys(pl, m) : it.pos0 + it.ntok;      // keys visible to the item's last token
          cut(0, it.n_addr, parts, sp, &it);
          it.g = g;
          it.part = sp;
          gr.cost += key_tiles(it);
          gr.items.push_back(it);
        }
        groups.push_back(std::move(gr));
      }
  }
  for (const PrefixRun &r : pp.runs)
    for (int g = 0; g < L.n_kv_heads; ++g)
      for (int sp = 0; sp < n_sh; ++sp) {
        Group gr{0, {}};
        for (int r0 = 0; r0 < r.n_rows; r0 += tq) {
          AttnItem it{};
          it.ntok = std::min(tq, r.n_rows - r0);
          it.row0 = r.row0 + r0;
          it.pos0 = 1 << 30;                              // every prefix key is visible to every row of the run
          it.key_row0 = r.prefix_off;
          it.n_addr = r.prefix_len;
          cut(0, r.prefix_len, n_sh, sp, &it);
          it.g = g;
          it.part = n_own + sp;
          gr.cost += key_tiles(it);
          gr.items.push_back(it);
        }
        groups.push_back(std::move(gr));
      }
  std::stable_sort(groups.begin(), groups.end(), [](const Group &x, const Group &y) { return x.cost > y.cost; });
  std::vector<AttnItem> per_xcd[8];
  int64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (const Group &gr : groups) {
    int x = 0;
    for (int i = 1; i < 8; ++i)
      if (load[i] < load[x]) x = i;
    load[x] += gr.cost;
    per_xcd[x].insert(per_xcd[x].end(), gr.items.begin(), gr.items.end());
  }
  size_t longest = 0;
  for (int x = 0; x < 8; ++x) {
    std::stable_sort(per_xcd[x].begin(), per_xcd[x].end(),
                     [&](const AttnItem &p, const AttnItem &q) { return key_tiles(p) > key_tiles(q); });
    longest = std::max(longest, per_xcd[x].size());
  }
  std::vector<AttnItem> qtiles;
  qtiles.reserve(longest * 8);
  for (size_t i = 0; i < longest; ++i)
    for (int x = 0; x < 8; ++x)
      qtiles.push_back(i < per_xcd[x].size() ? per_xcd[x][i] : AttnItem{});        // ntok = 0: padding
  return qtiles;
}

// Work list of a run of decode steps whose cached keys prefill attention walks: the run's own new keys, an item per row and group of kv
// heads that ends at the row's position (row t * B + b: the t-th new token of sequence b), the longest first.
std::vector<DecItem> build_run_items(const Plan &pl, const LayerDims &L, int n_steps, int hw, int part) {
  std::vector<DecItem> items;
  items.reserve((size_t)n_steps * pl.T * ((L.n_kv_heads + hw - 1) / hw));
  for (int t = n_steps - 1; t >= 0; --t)
    for (const SeqMeta &m : pl.seqs)
      for (int g = 0; g < L.n_kv_heads; g += hw) {
        DecItem it{};
        it.key_row0 = m.pool_off + m.P; it.row = t * pl.T + m.row_start; it.kend = it.n_keys = t + 1;
        it.n_rows = 1; it.g = (int16_t)g; it.part = (int16_t)part;
        items.push_back(it);
      }
  return items;
}

// What the attention of a run of decode steps would take in one pass over what was cached before it, in us: the prefill items (a workgroup has its
// start to pay for, many of them more than the few tiles of a short cache), the decode items of the run's own keys, the records.  Against
// n_steps * (decode_cut_us + 2.5).  Fitted to 2254 measured runs (2 to 16 steps of 1 to 500 rows on 0 to 131072 keys, 1 to 32 kv heads, private
// and shared contexts): the way it picks takes 0.3 % longer than the better one on average and 24 % at most, the pass throughout 2.6 % and 4.7 x
// (two steps: 64 rows of 32 kv heads on 16 keys 180 us, 55 a step at a time; 500 rows of 8 on 300 keys 354 and 301).
double run_pass_us(const alora_ctx *ctx, const Plan &pl, const LayerDims &L, const PrefillPlan &pp, int n_steps) {
  const int tq = attn_prefill_mfma_tokens_per_tile(L, 8);
  int64_t items = 0;
  for (const SeqMeta &m : pl.seqs) items += (int64_t)((n_steps + tq - 1) / tq) * (m.prefix_len > 0 ? pp.n_own : pp.n_own + pp.n_sh);
  for (const PrefixRun &r : pp.runs) items += (int64_t)((r.n_rows + tq - 1) / tq) * pp.n_sh;
  items *= L.n_kv_heads;
  const int64_t own = (int64_t)pl.T * ((L.n_kv_heads + 7) / 8);
  const double start = items > 0 ? 7.0 + 11.0 * (double)items / ctx->n_cu : 0.0;
  return 1.6 * std::max(pp.tiles, start) + 4.0 * (double)((own + ctx->n_cu - 1) / ctx->n_cu) +
         1.7 * (double)pl.T * L.n_q_heads * (pp.n_own + pp.n_sh + 1) * (2 * 520) / 4e6;
}

alora_status run(alora_ctx *ctx, const alora_layer_desc *layers, int n_layers, alora_kv_cache *caches,
                 const void *x, const int32_t *cu, const int32_t *kps, const int32_t *aps, int B, void *out,
                 void *stream, bool stack, bool decode = false, int n_steps = 1, bool use_static = false) {
  if (!ctx) return ALORA_EINVAL;
  ctx->err.clear();
  if (n_layers < 1) return fail(ctx, ALORA_EINVAL, "n_layers = %d must be at least 1", n_layers);
  if (!layers || !caches) return fail(ctx, ALORA_EINVAL, "layers / caches is NULL");
  LayerDims L{};
  alora_status st = check_layer(ctx, &layers[0], stack, &L);
  if (st != ALORA_OK) return st;
  for (int l = 1; l < n_layers; ++l) {
    LayerDims Ll{};
    st = check_layer(ctx, &layers[l], stack, &Ll);
    if (st != ALORA_OK) return st;
    if (memcmp(&Ll, &L, sizeof L) != 0 || layers[l].dtype != layers[0].dtype ||
        layers[l].intermediate != layers[0].intermediate)
      return fail(ctx, ALORA_ESHAPE, "layer %d differs in shape or dtype from layer 0", l);
    if (layers[l].rope_theta != layers[0].rope_theta || layers[l].rms_eps != layers[0].rms_eps)
      return fail(ctx, ALORA_ESHAPE, "layer %d differs in rope_theta or rms_eps from layer 0 (one rotary table per call)", l);
    if (!caches[l].k || !caches[l].v) return fail(ctx, ALORA_EINVAL, "caches[%d] k / v is NULL", l);
    if (caches[l].pool_tokens != caches[0].pool_tokens)
      return fail(ctx, ALORA_ECAPACITY, "caches[%d] pool size differs from caches[0]", l);
  }
  Plan pl;
  pl.L = L;
  if (n_steps < 1) return fail(ctx, ALORA_EINVAL, "n_steps = %d must be at least 1", n_steps);
  st = check_batch(ctx, &layers[0], &caches[0], cu, kps, aps, B, n_steps, &pl);
  if (st != ALORA_OK) return st;
  if (pl.T > 0 && (!x || !out)) return fail(ctx, ALORA_EINVAL, "x / out is NULL");
  if (pl.T == 0) return ALORA_OK;
  if (use_static && pl.any_prefix)
    return fail(ctx, ALORA_EINVAL, "alora_decode_static does not take shared prefixes (prefix_len must be NULL or all zero)");
  // (the size question of the static entry point is answered on a validation-only context too, by the same plan)
  const auto validation_only = [&] { return fail(ctx, ALORA_EHIP, "arguments are valid, but this is a validation-only context (device -1)"); };
  if (ctx->device < 0 && !use_static) return validation_only();
  if (ctx->device >= 0) HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t s = (hipStream_t)stream;
  const size_t esz = layers[0].dtype == ALORA_BF16 ? 2 : 4;
  constexpr int RUN_ROWS = 1024;
  int run_steps = 1;
  // A run of decode steps has the inputs of all of them: their rows are prepared, projected and appended together, RUN_ROWS at most (their
  // workspace is bounded; one sum over K whatever the number of rows: base rows come out with the same bits as a step at a time).  A record
  // per row and step stands for a sequence of one new row.  Not where an output lies where a later input does.  16 steps of 64 rows:
  // 16 x 35 -> 115 us.  A longer run is several of about equal length, one after the other, each done like a short one: 17 steps of 64 rows
  // on 16 contexts of 16384 keys 3560 -> 666 us, 64 steps 13370 -> 1491, 1025 of one row on 8192 keys 13140 -> 335.
  Plan run_pl;
  if (n_steps > 1) {
    const size_t xb = (size_t)n_steps * pl.T * L.d * esz, ob = (size_t)n_steps * pl.T * L.n_q * esz;
    const bool apart = (const char *)x + xb <= (const char *)out || (const char *)out + ob <= (const char *)x;
    const int most = apart ? std::max(1, RUN_ROWS / pl.T) : 1;
    run_steps = std::min(n_steps, most);
    if (most > 1 && n_steps > most) {
      st = ensure_rope(ctx, pl.max_len, L.head_dim / 2, layers[0].rope_theta, s);      // (once, not for every part)
      if (st != ALORA_OK) return st;
      for (int t = 0, left = (n_steps + most - 1) / most; left > 0; --left) {
        const int n = (n_steps - t + left - 1) / left;
        st = run(ctx, layers, 1, caches, (const char *)x + (size_t)t * pl.T * L.d * esz, cu, kps, aps, B,
                 (char *)out + (size_t)t * pl.T * L.n_q * esz, stream, false, true, n);
        if (st != ALORA_OK) {      // (no memory: the run's rows do not count)
          for (int b = 0; b < B; ++b) caches[0].seq_len[b] -= (cu[b + 1] - cu[b]) * t;
          return st;
        }
        t += n;
      }
      return ALORA_OK;
    }
  }
  if (run_steps > 1) {
    run_pl = pl;
    run_pl.T = run_pl.B = run_steps * pl.T;
    run_pl.seqs.clear();
    run_pl.seqs.reserve(run_pl.T);
    for (int t = 0; t < run_steps; ++t)
      for (const SeqMeta &m : pl.seqs) {
        SeqMeta q = m;
        q.row_start += t * pl.T;
        q.P += t;
        run_pl.seqs.push_back(q);
      }
    count_adapted_tiles(&run_pl, 0);
  }
  const Plan &ppl = run_steps > 1 ? run_pl : pl;      // the rows that are projected together
  // kernel family: MFMA for bf16 shapes it covers, plain otherwise
  const bool mfma = layers[0].dtype == ALORA_BF16 && ctx->opt_kernels == 0 && L.d % 64 == 0 &&
                    (L.n_adapters == 0 || (L.rank % 8 == 0 && L.n_adapters <= 64)) && L.n_q % 32 == 0 &&
                    L.n_kv % 32 == 0 && (!stack || (layers[0].intermediate % 64 == 0 && L.n_q % 64 == 0));
  // The reduction axis of the QKV projection is one running sum where the kernel that streams the weights can take few rows, and
  // segments fixed by the weight shape where it cannot (unaligned weights, reductions that are no multiple of 128): 16 rows of the
  // 8B-class shape with unaligned weights are 43 us as one sum, 21 in segments.  Weights decide, never the number of rows, so that a
  // row's sums don't depend on it.  (Whether segments run in workgroups of their own or one after the other inside one does not
  // change a bit of the result.)
  int k_segments = 1;
  if (mfma && ctx->opt_gemm_splits > 0) {
    k_segments = L.d % (64 * ctx->opt_gemm_splits) == 0 ? ctx->opt_gemm_splits : 1;
  } else if (mfma) {
    bool streamed = true;
    for (int l = 0; l < n_layers; ++l) streamed = streamed && qkv_stream_supported(layers[l].W_qkv, L.n_qkv, L.d, L.head_dim);
    if (!streamed) k_segments = gemm_mfma_fixed_segments(L.n_qkv, L.d, ctx->n_cu);
  }
  int k_splits = (k_segments > 1 && gemm_mfma_split_segments(ppl.T, L.n_qkv, ctx->n_cu)) ? k_segments : 1;
  // What the static entry point needs with `n` partial records per (row, head) and `groups` work items per row and record
  auto static_bytes = [&](int n, int groups) {
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    return up(layout_workspace(nullptr, L, pl.T, esz, n, k_splits, 0, false).bytes) + up((size_t)B * sizeof(SeqMeta)) +
           up((size_t)pl.T * groups * n * sizeof(DecItem)) + up((size_t)2 * pl.T * sizeof(int32_t)) +
           (size_t)pl.T * (L.head_dim / 2) * sizeof(float2);
  };
  // A decode step whose segment sums alone keep it out of the static scratch array adds them inside the workgroups (both entry points
  // alike: they give the same bits).  Not where the option asked for the segments: such a call is refused.
  if (decode && ctx->opt_gemm_splits == 0 && k_splits > 1 && static_bytes(1, (L.n_kv_heads + 7) / 8) > SCRATCH_BYTES) k_splits = 1;
  // work lists of the MFMA attention kernels (the number of partial records per (row, head) comes out of them)
  const int attn_waves = ctx->opt_attn_waves == 4 ? 4 : 8;
  int n_splits = pick_splits(ctx, pl.T, L.n_kv_heads, pl.max_len);
  bool attn_mfma = layers[0].dtype == ALORA_BF16 && ctx->opt_kernels == 0 && !decode && attn_prefill_mfma_supported(L);
  bool decode_mfma = layers[0].dtype == ALORA_BF16 && ctx->opt_kernels == 0 && decode && attn_decode_mfma_supported(L);
  DecodePlan dp;
  PrefillPlan pp;
  auto plan_decode = [&](bool items) {
    // One long sequence among many short ones asks for many records in every row's place: bounded to about 130 MB at 32 heads,
    // and to what the static scratch array holds where one record per row fits there (both entry points cut the keys alike).
    int cap = pl.T <= 16 ? 256 : std::max(1, std::min(64, 8192 / pl.T));
    if (!pl.any_prefix && static_bytes(1, (L.n_kv_heads + 7) / 8) <= SCRATCH_BYTES)
      while (cap > 1 && static_bytes(cap, (L.n_kv_heads + 1) / 2) > SCRATCH_BYTES) --cap;
    return plan_decode_items(ctx, pl, L, cap, n_steps, !items);
  };
  // Rows of several steps that are projected together can attend in one pass: prefill attention walks the keys that were cached before them for
  // the rows of all steps, the cache read once instead of once a step.  The run's own keys are for items of the decode kernel that end at each
  // row's position: in a pass that masked them their values would still be multiplied, by probability 0, and a step whose row is Inf or NaN
  // would reach the steps before it.  16 steps of 64 rows on 16 contexts of 16384 keys 3412 -> 442 us, 22 of them the new keys.  Not for the
  // variants of the prefill kernel that the options choose.
  Plan run_att;
  // sequences by prefix, so that those of one context share its items wherever they stand in the batch: two steps of 64 rows on 16 contexts of 16384
  // keys, in turn, 977 us in the order of the batch (a step at a time 490), 368 like this
  std::vector<int32_t> run_order;
  bool run_prefill = decode_mfma && run_steps > 1 && attn_waves == 8 && ctx->opt_attn_fold && attn_prefill_mfma_supported(L);
  if (run_prefill) {
    run_att = pl;
    run_att.T = pl.T * n_steps;
    run_att.cached_only = true;
    if (pl.any_prefix) {
      run_order = by_prefix(pl);
      for (int b = 0; b < B; ++b) run_att.seqs[b] = pl.seqs[run_order[b]];
    }
    for (int b = 0; b < B; ++b) { run_att.seqs[b].n_new = n_steps; run_att.seqs[b].row_start = b * n_steps; }
    pp = plan_prefill_ranges(ctx, run_att, L, B, attn_waves);
    // (kv_splits leaves nothing to compare, and no decode step is done in less than its round and one step of keys)
    const double pass = run_pass_us(ctx, run_att, L, pp, n_steps);
    run_prefill = ctx->opt_splits > 0 || pass <= n_steps * (3.76 + 4.8 + 2.5) || pass <= n_steps * (plan_decode(false).us + 2.5);
  }
  if (run_prefill) {
    attn_mfma = true;
    decode_mfma = false;
    n_splits = pp.n_own + pp.n_sh + 1;      // (one more record per row: the run's own keys)
    decode_mfma_shape(L.n_kv_heads, false, &dp.hw, &dp.kr);
    dp.cols_max = L.n_q_heads / L.n_kv_heads;
    dp.items = build_run_items(pl, L, n_steps, dp.hw, n_splits - 1);
  } else if (decode_mfma) {
    run_order.clear();
    dp = plan_decode(!use_static);
    n_splits = dp.n_own + dp.n_shared;
  } else if (attn_mfma) {
    pp = plan_prefill_ranges(ctx, pl, L, B, attn_waves);
    n_splits = pp.n_own + pp.n_sh;
  }
  const Plan &att_pl = run_prefill ? run_att : pl;      // the rows that attend together: sequence after sequence (the kernel finds where they lie)
  const std::vector<DecItem> &ditems = dp.items;
  const int n_static_items = dp.n_device_items;
  const int dec_hw = dp.hw, dec_kr = dp.kr, dec_groups = dp.groups, dec_cols_max = dp.cols_max;
  const bool f32_tail = stack && !mfma && layers[0].dtype == ALORA_BF16;
  Workspace probe = layout_workspace(nullptr, L, ppl.T, esz, n_splits, k_splits, layers[0].intermediate, stack, f32_tail, att_pl.T);
  if (use_static) {
    // Everything the call needs beyond its inputs and outputs lives in the static scratch array of this GPU:
    //   [ workspace | per-sequence records | decode work list | rotary lines, one per row ]
    // No allocation, no staging copy: the records travel as kernel arguments, the work list and the rotary lines
    // are computed on the device.  Nothing in there has to start at zero (every byte a kernel reads was written
    // by a kernel of this call), so nothing is cleared.
    const size_t ws_bytes = (probe.bytes + 255) & ~(size_t)255;
    const size_t seq_b = ((size_t)B * sizeof(SeqMeta) + 255) & ~(size_t)255;
    const size_t item_b = ((size_t)n_static_items * sizeof(DecItem) + 255) & ~(size_t)255;
    const size_t rope_b = (size_t)pl.T * (L.head_dim / 2) * sizeof(float2);
    const size_t count_b = ((size_t)2 * pl.T * sizeof(int32_t) + 255) & ~(size_t)255;
    const size_t need = ws_bytes + seq_b + item_b + count_b + rope_b;
    if (need > SCRATCH_BYTES)
      return fail(ctx, ALORA_ECAPACITY, "alora_decode_static: this call needs %zu bytes of scratch, the static buffer holds %zu",
                  need, SCRATCH_BYTES);
    if (ctx->device < 0) return validation_only();
    if (!ctx->scratch_dev) return fail(ctx, ALORA_EHIP, "the static scratch array has no device address on this context");
    char *base = (char *)ctx->scratch_dev;
    SeqMeta *seqs_dev = (SeqMeta *)(base + ws_bytes);
    DecItem *items_dev = (DecItem *)(base + ws_bytes + seq_b);
    int32_t *counts_dev = (int32_t *)(base + ws_bytes + seq_b + item_b);
    for (int b0 = 0; b0 < B; b0 += STAGE_SEQS) {
      SeqChunk c;
      const int n = std::min(STAGE_SEQS, B - b0);
      memcpy(c.m, pl.seqs.data() + b0, (size_t)n * sizeof(SeqMeta));
      hipLaunchKernelGGL(stage_seqs_kernel, dim3(1), dim3(64), 0, s, c, n, seqs_dev + b0);
    }
    if (decode_mfma && n_static_items > 0)
      hipLaunchKernelGGL(make_decode_items_kernel, dim3((n_static_items + 255) / 256), dim3(256), 0, s, seqs_dev, B, items_dev,
                         counts_dev, dec_groups, dec_hw, dp.n_own, dp.range, ctx->opt_splits);
    Workspace w = layout_workspace(base, L, pl.T, esz, n_splits, k_splits, 0, false);
    w.mfma = mfma;
    w.k_splits = k_splits;
    w.k_segments = k_segments;
    w.lora_split = (k_splits > 1 && ctx->opt_lora_split != 2) || ctx->opt_lora_split == 1 ? 1 : 0;
    w.attn_mfma = false;
    w.decode_mfma = decode_mfma;
    w.attn_waves = attn_waves;
    w.ditems = items_dev;
    w.n_ditems = decode_mfma ? n_static_items : 0;
    w.dec_hw = dec_hw; w.dec_kr = dec_kr; w.dec_cols_max = dec_cols_max;
    w.any_adapter = pl.any_adapter;
    w.rope_by_row = true;
    if (decode_mfma) w.merge = MergeCounts{counts_dev, dp.n_own};
    w.rope_rows = (float2 *)(base + ws_bytes + seq_b + item_b + count_b);
    w.rope = w.rope_rows;
    const int saved_profile = ctx->opt_profile;
    ctx->opt_profile = 0;             // the event brackets of the profiling option create events: not here
    if (layers[0].dtype == ALORA_BF16)
      attention_block<bf16>(ctx, &layers[0], L, &caches[0], (const bf16 *)x, pl, seqs_dev, w, true, n_splits, true, 0, (bf16 *)out, s);
    else
      attention_block<float>(ctx, &layers[0], L, &caches[0], (const float *)x, pl, seqs_dev, w, true, n_splits, true, 0, (float *)out, s);
    ctx->opt_profile = saved_profile;
    HIP_TRY(ctx, hipGetLastError());
    for (int b = 0; b < B; ++b) caches[0].seq_len[b] += 1;
    return ALORA_OK;
  }
  st = ensure_workspace(ctx, probe.bytes);
  if (st != ALORA_OK) return st;
  st = ensure_rope(ctx, pl.max_len, L.head_dim / 2, layers[0].rope_theta, s);
  if (st != ALORA_OK) return st;
  // staged metadata: per-sequence records, then the work list of the MFMA attention kernel
  std::vector<AttnItem> qtiles;
  if (attn_mfma) qtiles = build_prefill_items(att_pl, L, B, attn_waves, pp);
  const size_t seq_bytes = (ppl.seqs.size() * sizeof(SeqMeta) + 15) & ~(size_t)15;
  const size_t list_bytes = (qtiles.size() * sizeof(AttnItem) + ditems.size() * sizeof(DecItem) + 15) & ~(size_t)15;   // (both: a run of decode steps)
  const size_t row_bytes = ((dp.rows.size() + dp.counts.size() + run_order.size()) * sizeof(int32_t) + 15) & ~(size_t)15;      // decode: shared items' rows, records per row; runs
  const size_t work_bytes = list_bytes + row_bytes;
  const size_t scale_bytes = stack ? (((size_t)L.n_adapters * sizeof(float) + 15) & ~(size_t)15) : 0;
  const size_t meta_bytes = seq_bytes + work_bytes + scale_bytes;
  MetaSlot *slot = nullptr;
  st = acquire_slot(ctx, meta_bytes, &slot);
  if (st != ALORA_OK) return st;
  memcpy(slot->host, ppl.seqs.data(), ppl.seqs.size() * sizeof(SeqMeta));
  if (!qtiles.empty()) memcpy(slot->host + seq_bytes, qtiles.data(), qtiles.size() * sizeof(AttnItem));
  const size_t dec_at = seq_bytes + qtiles.size() * sizeof(AttnItem);
  if (!ditems.empty()) memcpy(slot->host + dec_at, ditems.data(), ditems.size() * sizeof(DecItem));
  if (!dp.counts.empty()) memcpy(slot->host + seq_bytes + list_bytes, dp.counts.data(), dp.counts.size() * sizeof(int32_t));
  if (!dp.rows.empty()) memcpy(slot->host + seq_bytes + list_bytes + dp.counts.size() * sizeof(int32_t), dp.rows.data(), dp.rows.size() * sizeof(int32_t));
  const size_t order_at = seq_bytes + list_bytes + (dp.counts.size() + dp.rows.size()) * sizeof(int32_t);
  if (!run_order.empty()) memcpy(slot->host + order_at, run_order.data(), run_order.size() * sizeof(int32_t));
  if (scale_bytes) memcpy(slot->host + seq_bytes + work_bytes, layers[0].scale, (size_t)L.n_adapters * sizeof(float));
  const int n16 = (int)((meta_bytes + 15) / 16);
  const bool carried = ppl.B <= FEW_SEQS && n16 <= STAGE_N16 && !ctx->opt_stage_copy;      // by the call's first kernel
  if (carried) {
  } else if (ctx->opt_stage_copy) {
    HIP_TRY(ctx, hipMemcpyAsync(slot->dev, slot->host, meta_bytes, hipMemcpyHostToDevice, s));
  } else {
    hipLaunchKernelGGL(stage_meta_kernel, dim3((n16 + 255) / 256), dim3(256), 0, s, (const uint4 *)slot->host,
                       (uint4 *)slot->dev, n16);
  }
  const SeqMeta *seqs_dev = (const SeqMeta *)slot->dev;
  Workspace w = layout_workspace(ctx->ws, L, ppl.T, esz, n_splits, k_splits, layers[0].intermediate, stack, f32_tail, att_pl.T);
  w.mfma = mfma;
  w.k_splits = k_splits;
  w.k_segments = k_segments;
  // few row tiles and a split reduction: the workgroups are short and the prologue of split 0 would stick out
  w.lora_split = (k_splits > 1 && ctx->opt_lora_split != 2) || ctx->opt_lora_split == 1 ? 1 : 0;
  w.attn_mfma = attn_mfma;
  if (run_prefill) { w.run_steps = n_steps; w.run_seqs = B; w.run_order = run_order.empty() ? nullptr : (const int32_t *)(slot->dev + order_at); }
  w.decode_mfma = decode_mfma;
  w.attn_waves = attn_waves;
  w.qtiles = (const AttnItem *)(slot->dev + seq_bytes);
  w.n_qtiles = (int)qtiles.size();
  w.ditems = (const DecItem *)(slot->dev + dec_at);
  w.n_ditems = (int)ditems.size();
  if (!dp.counts.empty()) {
    w.merge = MergeCounts{(const int32_t *)(slot->dev + seq_bytes + list_bytes), dp.n_own};
    w.drows = w.merge.counts + dp.counts.size();
  }
  w.dec_hw = dec_hw; w.dec_kr = dec_kr; w.dec_cols_max = dec_cols_max;
  w.pl = &pl;
  w.scale_dev = scale_bytes ? (const float *)(slot->dev + seq_bytes + work_bytes) : nullptr;
  w.any_adapter = pl.any_adapter;
  w.rope = ctx->rope;
  if (carried) {
    w.stage_src = (const uint4 *)slot->host;
    w.stage_dst = (uint4 *)slot->dev;
    w.stage_n16 = n16;
  }

  const bool bf = layers[0].dtype == ALORA_BF16;
  if (!stack) {
    // n_steps > 1: a run of decode steps on the metadata staged once, projected together (run_steps = n_steps) or one at a time
    auto steps = [&](auto one) {
      using T = decltype(one);
      for (int t0 = 0; t0 < n_steps; t0 += run_steps) {
        project_rows<T>(ctx, &layers[0], L, &caches[0], (const T *)x + (size_t)t0 * pl.T * L.d, ppl, seqs_dev, w, true, t0, s);
        if (run_prefill) attend_rows<T>(ctx, L, &caches[0], att_pl, seqs_dev, w, n_splits, false, 0, 0, (T *)out, s);
        else for (int t = 0; t < run_steps; ++t)
          attend_rows<T>(ctx, L, &caches[0], pl, seqs_dev, w, n_splits, decode, t0 + t, t * pl.T, (T *)out + (size_t)(t0 + t) * pl.T * L.n_q, s);
      }
    };
    if (bf) steps(bf16{});
    else steps(float{});
  } else {
    const void *cur = x;
    for (int l = 0; l < n_layers; ++l) {
      void *nxt = (l == n_layers - 1) ? out : ((l & 1) ? w.xb : w.xa);
      if (bf) {
        attention_block<bf16>(ctx, &layers[l], L, &caches[l], (const bf16 *)cur, pl, seqs_dev, w, l == 0, n_splits, decode, 0, (bf16 *)w.attn, s);
        layer_tail<bf16>(ctx, &layers[l], L, (const bf16 *)cur, w, pl.T, (bf16 *)nxt, s);
      } else {
        attention_block<float>(ctx, &layers[l], L, &caches[l], (const float *)cur, pl, seqs_dev, w, l == 0, n_splits, decode, 0, (float *)w.attn, s);
        layer_tail<float>(ctx, &layers[l], L, (const float *)cur, w, pl.T, (float *)nxt, s);
      }
      cur = nxt;
    }
  }
  HIP_TRY(ctx, hipGetLastError());
  HIP_TRY(ctx, hipEventRecord(slot->ev, s));
  slot->in_flight = true;
  for (int b = 0; b < B; ++b) caches[0].seq_len[b] += (cu[b + 1] - cu[b]) * n_steps;
  return ALORA_OK;
}

}  // namespace

alora_status drain_profile(alora_ctx *ctx) {
  for (ProfEvent &e : ctx->prof_pending) {
    HIP_TRY(ctx, hipEventSynchronize(e.stop));
    float ms = 0.f;
    HIP_TRY(ctx, hipEventElapsedTime(&ms, e.start, e.stop));
    ctx->prof_ms[e.kernel] += ms;
    ctx->prof_n[e.kernel] += 1;
    ctx->prof_free.push_back(e.start);
    ctx->prof_free.push_back(e.stop);
  }
  ctx->prof_pending.clear();
  return ALORA_OK;
}

extern "C" {

alora_status alora_create(alora_ctx **out, int device) {
  if (!out) return ALORA_EINVAL;
  *out = nullptr;
  if (device == -1) {              // validation-only context: checks arguments, never launches
    alora_ctx *ctx = new alora_ctx();
    ctx->device = -1;
    *out = ctx;
    return ALORA_OK;
  }
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return ALORA_EHIP;
  if (hipSetDevice(device) != hipSuccess) return ALORA_EHIP;
  alora_ctx *ctx = new alora_ctx();
  ctx->device = device;
  // the device address of this GPU's copy of the static scratch array (the array's name is not one)
  void *sp = nullptr;
  if (hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) != hipSuccess || sp == nullptr) {
    delete ctx;
    return ALORA_EHIP;
  }
  ctx->scratch_dev = (unsigned char *)sp;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) == hipSuccess) ctx->n_cu = prop.multiProcessorCount;
  *out = ctx;
  return ALORA_OK;
}

void alora_destroy(alora_ctx *ctx) {
  if (!ctx) return;
  if (ctx->device < 0) { delete ctx; return; }
  (void)hipSetDevice(ctx->device);
  (void)hipDeviceSynchronize();
  if (ctx->ws) (void)hipFree(ctx->ws);
  if (ctx->rope) (void)hipFree(ctx->rope);
  (void)drain_profile(ctx);
  for (hipEvent_t e : ctx->prof_free) (void)hipEventDestroy(e);
  for (MetaSlot &sl : ctx->slots) {
    if (sl.host) (void)hipHostFree(sl.host);
    if (sl.dev) (void)hipFree(sl.dev);
    if (sl.ev) (void)hipEventDestroy(sl.ev);
  }
  delete ctx;
}

const char *alora_last_error(const alora_ctx *ctx) { return ctx ? ctx->err.c_str() : "context is NULL"; }

const char *alora_status_string(alora_status s) {
  switch (s) {
    case ALORA_OK: return "ALORA_OK";
    case ALORA_EINVAL: return "ALORA_EINVAL";
    case ALORA_ESHAPE: return "ALORA_ESHAPE";
    case ALORA_ECAPACITY: return "ALORA_ECAPACITY";
    case ALORA_EADAPTER: return "ALORA_EADAPTER";
    case ALORA_EDTYPE: return "ALORA_EDTYPE";
    case ALORA_EHIP: return "ALORA_EHIP";
  }
  return "unknown status";
}

alora_status alora_set_option(alora_ctx *ctx, const char *key, int value) {
  if (!ctx) return ALORA_EINVAL;
  ctx->err.clear();
  if (!key) return fail(ctx, ALORA_EINVAL, "option key is NULL");
  if (!strcmp(key, "kernels")) {
    if (value != 0 && value != 1) return fail(ctx, ALORA_EINVAL, "kernels must be 0 or 1");
    ctx->opt_kernels = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "kv_splits")) {
    if (value < 0 || value > 256) return fail(ctx, ALORA_EINVAL, "kv_splits must be in [0, 256]");
    ctx->opt_splits = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "gemm_splits")) {
    if (value < 0 || value > 64) return fail(ctx, ALORA_EINVAL, "gemm_splits must be in [0, 64]");
    ctx->opt_gemm_splits = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "lora_split")) {
    if (value < 0 || value > 2) return fail(ctx, ALORA_EINVAL, "lora_split must be 0, 1 or 2");
    ctx->opt_lora_split = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "stage_copy")) {
    if (value < 0 || value > 1) return fail(ctx, ALORA_EINVAL, "stage_copy must be 0 or 1");
    ctx->opt_stage_copy = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "attn_lazy")) {
    if (value < 0 || value > 16) return fail(ctx, ALORA_EINVAL, "attn_lazy must be in [0, 16]");
    ctx->opt_attn_lazy = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "attn_partials16")) {
    if (value != 0 && value != 1) return fail(ctx, ALORA_EINVAL, "attn_partials16 must be 0 or 1");
    ctx->opt_attn_partials16 = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "rope_fuse")) {
    if (value != 0 && value != 1) return fail(ctx, ALORA_EINVAL, "rope_fuse must be 0 or 1");
    ctx->opt_rope_fuse = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "attn_fold")) {
    if (value != 0 && value != 1) return fail(ctx, ALORA_EINVAL, "attn_fold must be 0 or 1");
    ctx->opt_attn_fold = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "attn_waves")) {
    if (value != 0 && value != 4 && value != 8) return fail(ctx, ALORA_EINVAL, "attn_waves must be 0, 4 or 8");
    ctx->opt_attn_waves = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "prep_split")) {
    if (value < 0 || value > 2) return fail(ctx, ALORA_EINVAL, "prep_split must be 0, 1 or 2");
    ctx->opt_prep_split = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "gemm_tile")) {
    if (value < 0 || value > 6) return fail(ctx, ALORA_EINVAL, "gemm_tile must be in [0, 6]");
    ctx->opt_gemm_tile = value;
    return ALORA_OK;
  }
  if (!strcmp(key, "profile")) {
    if (value != 0 && value != 1) return fail(ctx, ALORA_EINVAL, "profile must be 0 or 1");
    ctx->opt_profile = value;
    return ALORA_OK;
  }
  return fail(ctx, ALORA_EINVAL, "unknown option '%s'", key);
}

alora_status alora_profile_read(alora_ctx *ctx, const char *kernel, double *total_ms, int64_t *launches) {
  if (!ctx) return ALORA_EINVAL;
  ctx->err.clear();
  if (!kernel || !total_ms || !launches) return fail(ctx, ALORA_EINVAL, "NULL argument");
  alora_status st = drain_profile(ctx);
  if (st != ALORA_OK) return st;
  for (int i = 0; i < K_COUNT; ++i)
    if (!strcmp(kernel, KERNEL_NAMES[i])) {
      *total_ms = ctx->prof_ms[i];
      *launches = ctx->prof_n[i];
      return ALORA_OK;
    }
  return fail(ctx, ALORA_EINVAL, "unknown kernel name '%s'", kernel);
}

alora_status alora_lm_head(alora_ctx *ctx, alora_dtype dtype, int32_t d, int32_t vocab, const void *x_last,
                           const void *final_gain, float rms_eps, const void *W_vocab, int32_t B, float *logits,
                           int32_t *token, void *stream) {
  if (!ctx) return ALORA_EINVAL;
  ctx->err.clear();
  if (dtype != ALORA_F32 && dtype != ALORA_BF16)
    return fail(ctx, ALORA_EDTYPE, "dtype %d is neither ALORA_F32 nor ALORA_BF16", (int)dtype);
  if (d < 1 || d > 16000) return fail(ctx, ALORA_ESHAPE, "d = %d outside [1, 16000]", d);
  if (vocab < 1) return fail(ctx, ALORA_ESHAPE, "vocab = %d must be positive", vocab);
  if (B < 1 || B > 4096) return fail(ctx, ALORA_EINVAL, "B = %d outside [1, 4096]", B);
  if (!x_last || !W_vocab) return fail(ctx, ALORA_EINVAL, "x_last / W_vocab is NULL");
  if (!logits && !token) return fail(ctx, ALORA_EINVAL, "logits and token are both NULL: nothing to compute");
  if (ctx->device < 0) return fail(ctx, ALORA_EHIP, "validation-only context (device -1)");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t s = (hipStream_t)stream;
  const bool bf = dtype == ALORA_BF16;
  const size_t esz = bf ? 2 : 4;
  const int n_slabs = argmax_slabs(vocab);
  // workspace: normalised rows | logits (unless the caller keeps them) | per-slab maxima
  Bump probe(nullptr);
  probe.take<char>((size_t)B * d * esz);
  if (!logits) probe.take<float>((size_t)B * vocab);
  probe.take<float>((size_t)B * n_slabs);
  probe.take<int>((size_t)B * n_slabs);
  alora_status st = ensure_workspace(ctx, probe.off);
  if (st != ALORA_OK) return st;
  Bump b(ctx->ws);
  char *xh = b.take<char>((size_t)B * d * esz);
  float *lg = logits ? logits : b.take<float>((size_t)B * vocab);
  float *pv = b.take<float>((size_t)B * n_slabs);
  int *pi = b.take<int>((size_t)B * n_slabs);
  const bool mfma = bf && ctx->opt_kernels == 0 && gemm_mfma_supported(B, vocab, d);
  RowMeta none{};
  const void *rows = x_last;
  if (final_gain) {
    ProfScope p(ctx, K_MLPNORM, s);
    if (mfma && prep_rows_mfma_supported(d, 0)) {
      PrepArgs pa{};
      pa.x = (const bf16 *)x_last; pa.gain = (const bf16 *)final_gain; pa.eps = rms_eps;
      pa.T = B; pa.d = d; pa.xh = (bf16 *)xh; pa.rm = none;
      launch_prep_rows_mfma(pa, s);
    } else if (bf) {
      launch_prep_rows<bf16>((const bf16 *)x_last, (const bf16 *)final_gain, rms_eps, B, d, nullptr, 0, 0, nullptr, 0,
                             false, (bf16 *)xh, nullptr, nullptr, none, StagedCall{}, false, s);
    } else {
      launch_prep_rows<float>((const float *)x_last, (const float *)final_gain, rms_eps, B, d, nullptr, 0, 0, nullptr,
                              0, false, (float *)xh, nullptr, nullptr, none, StagedCall{}, false, s);
    }
    rows = xh;
  }
  {
    ProfScope p(ctx, K_LMHEAD, s);
    if (mfma) {
      GemmArgs g{};
      g.A = (const bf16 *)rows; g.lda = d;
      g.B = (const bf16 *)W_vocab; g.ldb = d;
      g.M = B; g.N = vocab; g.K = d;
      g.k_splits = 1;
      g.k_segments = 1;
      g.Cpart = lg;
      if (ctx->opt_gemm_splits == 0 && ctx->opt_gemm_tile == 0 && gemm_stream_supported(g, GEMM_EPI_PARTIAL, ctx->n_cu))
        launch_gemm_stream(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
      else
        launch_gemm_mfma(g, GEMM_EPI_PARTIAL, ctx->n_cu, s);
    } else if (bf) {
      launch_lm_logits_plain<bf16>((const bf16 *)rows, (const bf16 *)W_vocab, B, vocab, d, lg, s);
    } else {
      launch_lm_logits_plain<float>((const float *)rows, (const float *)W_vocab, B, vocab, d, lg, s);
    }
  }
  if (token) {
    ProfScope p(ctx, K_ARGMAX, s);
    launch_argmax(lg, B, vocab, pv, pi, token, s);
  }
  HIP_TRY(ctx, hipGetLastError());
  return ALORA_OK;
}

alora_status alora_profile_reset(alora_ctx *ctx) {
  if (!ctx) return ALORA_EINVAL;
  ctx->err.clear();
  alora_status st = drain_profile(ctx);
  if (st != ALORA_OK) return st;
  for (int i = 0; i < K_COUNT; ++i) { ctx->prof_ms[i] = 0.0; ctx->prof_n[i] = 0; }
  return ALORA_OK;
}

alora_status alora_prefill(alora_ctx *ctx, const alora_layer_desc *layer, alora_kv_cache *cache,
                           const void *x_suffix, const int32_t *cu_seqlens, const int32_t *k_per_seq,
                           const int32_t *adapter_per_seq, int32_t B, void *attn_out, void *stream) {
  return run(ctx, layer, 1, cache, x_suffix, cu_seqlens, k_per_seq, adapter_per_seq, B, attn_out, stream, false);
}

alora_status alora_decode(alora_ctx *ctx, const alora_layer_desc *layer, alora_kv_cache *cache, const void *x_tok,
                          const int32_t *k_per_seq, const int32_t *adapter_per_seq, int32_t B, void *attn_out,
                          void *stream) {
  if (!ctx) return ALORA_EINVAL;
  if (B < 1) return fail(ctx, ALORA_EINVAL, "B = %d must be at least 1", B);
  std::vector<int32_t> cu(B + 1);
  for (int b = 0; b <= B; ++b) cu[b] = b;
  return run(ctx, layer, 1, cache, x_tok, cu.data(), k_per_seq, adapter_per_seq, B, attn_out, stream, false, true);
}

alora_status alora_decode_static(alora_ctx *ctx, const alora_layer_desc *layer, alora_kv_cache *cache, const void *x_tok,
                                 const int32_t *k_per_seq, const int32_t *adapter_per_seq, int32_t B, void *attn_out,
                                 void *stream) {
  if (!ctx) return ALORA_EINVAL;
  if (B < 1) return fail(ctx, ALORA_EINVAL, "B = %d must be at least 1", B);
  if (B > 4096) return fail(ctx, ALORA_ECAPACITY, "alora_decode_static takes at most 4096 sequences per call (B = %d)", B);
  int32_t cu[4097];
  for (int b = 0; b <= B; ++b) cu[b] = b;
  return run(ctx, layer, 1, cache, x_tok, cu, k_per_seq, adapter_per_seq, B, attn_out, stream, false, true, 1, true);
}

alora_status alora_decode_steps(alora_ctx *ctx, const alora_layer_desc *layer, alora_kv_cache *cache,
                                const void *x_steps, const int32_t *k_per_seq, const int32_t *adapter_per_seq,
                                int32_t B, int32_t n_steps, void *attn_out, void *stream) {
  if (!ctx) return ALORA_EINVAL;
  if (B < 1) return fail(ctx, ALORA_EINVAL, "B = %d must be at least 1", B);
  std::vector<int32_t> cu(B + 1);
  for (int b = 0; b <= B; ++b) cu[b] = b;
  return run(ctx, layer, 1, cache, x_steps, cu.data(), k_per_seq, adapter_per_seq, B, attn_out, stream, false, true,
             n_steps);
}

alora_status alora_stack_prefill(alora_ctx *ctx, const alora_layer_desc *layers, int32_t n_layers,
                                 alora_kv_cache *caches, const void *x, const int32_t *cu_seqlens,
                                 const int32_t *k_per_seq, const int32_t *adapter_per_seq, int32_t B, void *out,
                                 void *stream) {
  return run(ctx, layers, n_layers, caches, x, cu_seqlens, k_per_seq, adapter_per_seq, B, out, stream, true);
}

alora_status alora_stack_decode(alora_ctx *ctx, const alora_layer_desc *layers, int32_t n_layers, alora_kv_cache *caches,
                                const void *x_tok, const int32_t *k_per_seq, const int32_t *adapter_per_seq, int32_t B,
                                void *out, void *stream) {
  if (!ctx) return ALORA_EINVAL;
  if (B < 1) return fail(ctx, ALORA_EINVAL, "B = %d must be at least 1", B);
  std::vector<int32_t> cu(B + 1);
  for (int b = 0; b <= B; ++b) cu[b] = b;
  return run(ctx, layers, n_layers, caches, x_tok, cu.data(), k_per_seq, adapter_per_seq, B, out, stream, true, true);
}

}  // extern "C"
