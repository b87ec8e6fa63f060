// C ABI of the library: host-side argument checks, then one launcher per entry point.
// The checks need no GPU, so every error path can be exercised on a CPU-only machine.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "common.h"
#include "launch.h"
#include "select_body.h"

namespace actqkv {

static thread_local char g_error[512] = "";

int set_error(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof(g_error), fmt, ap);
  va_end(ap);
  return code;
}

int hip_status(const char* what) {
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) return ACTQKV_OK;
  return set_error(ACTQKV_EHIP, "%s: %s", what, hipGetErrorString(e));
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static int check_shape(const actqkv_shape* sh) {
  if (sh == nullptr) return set_error(ACTQKV_EINVAL, "shape is NULL");
  if (sh->n_q_heads < 1 || sh->n_kv_heads < 1 || sh->head_dim < 1 || sh->n_rep < 1 ||
      sh->n_init < 0 || sh->n_local < 0)
    return set_error(ACTQKV_EINVAL, "shape has a non-positive field");
  if (sh->dtype != ACTQKV_F32 && sh->dtype != ACTQKV_BF16)
    return set_error(ACTQKV_EINVAL, "dtype %d is neither ACTQKV_F32 nor ACTQKV_BF16", sh->dtype);
  if (!(sh->softmax_scale >= 0.f) || !(sh->var_eps >= 0.f))
    return set_error(ACTQKV_EINVAL, "softmax_scale and var_eps must be >= 0");
  if (sh->head_dim != 64 && sh->head_dim != 128)
    return set_error(ACTQKV_ESHAPE, "head_dim %d not supported (64 or 128)", sh->head_dim);
  if (sh->n_q_heads % sh->n_kv_heads != 0)
    return set_error(ACTQKV_ESHAPE, "n_q_heads %d is not a multiple of n_kv_heads %d", sh->n_q_heads,
                     sh->n_kv_heads);
  const int g = sh->n_q_heads / sh->n_kv_heads;
  if (g < 1 || g > 8) return set_error(ACTQKV_ESHAPE, "group size %d not supported (1..8)", g);
  if (sh->block_size != 128)
    return set_error(ACTQKV_ESHAPE, "block_size %d not supported (128)", sh->block_size);
  if (sh->n_rep > 16) return set_error(ACTQKV_ESHAPE, "n_rep %d not supported (1..16)", sh->n_rep);
  if (sh->n_init % sh->block_size != 0 || sh->n_local % sh->block_size != 0)
    return set_error(ACTQKV_ESHAPE, "n_init and n_local must be multiples of block_size");
  if (sh->n_q_heads * sh->head_dim > 16384)
    return set_error(ACTQKV_ESHAPE, "H*D = %d not supported (at most 16384)",
                     sh->n_q_heads * sh->head_dim);
  return ACTQKV_OK;
}

static int check_batch(int batch) {
  if (batch < 1) return set_error(ACTQKV_EINVAL, "batch %d < 1", batch);
  if (batch > kMaxBatch) return set_error(ACTQKV_ESHAPE, "batch %d > %d", batch, kMaxBatch);
  return ACTQKV_OK;
}

static int check_blocks(int nb_capacity, int nb_begin, int k_cap, bool use_k) {
  if (nb_capacity < 0 || nb_begin < 0)
    return set_error(ACTQKV_EINVAL, "nb_capacity %d or nb_begin %d negative", nb_capacity, nb_begin);
  if (use_k && (k_cap < 1 || k_cap > 64))
    return set_error(ACTQKV_ESHAPE, "k_cap %d not supported (1..64)", k_cap);
  if (nb_capacity - nb_begin > 8192)
    return set_error(ACTQKV_ESHAPE, "%d blocks in one selection (at most 8192)",
                     nb_capacity - nb_begin);
  return ACTQKV_OK;
}

#define ACTQKV_REQUIRE_PTR(p)                                                       \
  do {                                                                              \
    if ((p) == nullptr) return set_error(ACTQKV_EINVAL, #p " is NULL");             \
    if (!aligned16(p)) return set_error(ACTQKV_EALIGN, #p " is not 16-byte aligned"); \
  } while (0)
#define ACTQKV_REQUIRE_SMALL(p, a)                                                          \
  do {                                                                                      \
    if ((p) == nullptr) return set_error(ACTQKV_EINVAL, #p " is NULL");                     \
    if ((reinterpret_cast<uintptr_t>(p) & ((a)-1)) != 0)                                    \
      return set_error(ACTQKV_EALIGN, #p " is not %d-byte aligned", int(a));                \
  } while (0)
#define ACTQKV_OPTIONAL_SMALL(p, a)                                                         \
  do {                                                                                      \
    if ((p) != nullptr && (reinterpret_cast<uintptr_t>(p) & ((a)-1)) != 0)                  \
      return set_error(ACTQKV_EALIGN, #p " is not %d-byte aligned", int(a));                \
  } while (0)
#define ACTQKV_OPTIONAL_PTR(p)                                                                   \
  do {                                                                                           \
    if ((p) != nullptr && !aligned16(p)) return set_error(ACTQKV_EALIGN, #p " is not 16-byte aligned"); \
  } while (0)
#define ACTQKV_TRY(expr)      \
  do {                        \
    int rc_ = (expr);         \
    if (rc_ != ACTQKV_OK) return rc_; \
  } while (0)

bool prefill_mfma_supported(const actqkv_shape& sh, int m);
bool prefill_merge_after(const actqkv_shape& sh, int s_lo);
int launch_attention_prefill_mfma(const actqkv_shape& sh, int batch, int m, const void* q,
                                  const void* k_cache, const void* v_cache, int64_t seq_stride,
                                  int nb_capacity, const int32_t* n_ctx, const int32_t* idx,
                                  const int32_t* n_sel, int k_cap, void* out, float* lse,
                                  const PfSplits& splits, float* scratch, unsigned int* counters,
                                  float scale, int sel_per_head, int first_cus, int late_cus,
                                  hipStream_t stream, hipStream_t stream_late, const SelectInside* inside);

bool prefill_f32_supported(const actqkv_shape& sh, int m);
size_t prefill_f32_scratch_bytes(const actqkv_shape& sh, int batch, int m);
size_t prefill_f32_scratch_most(const actqkv_shape& sh, int batch, int m);
int launch_attention_prefill_f32(const actqkv_shape& sh, int batch, int m, const void* q, const void* k_cache,
                                 const void* v_cache, int64_t seq_stride, int nb_capacity, const int32_t* n_ctx,
                                 const int32_t* idx, const int32_t* n_sel, int k_cap, void* out, float* lse,
                                 float* scratch, float scale, int sel_per_head,
                                 hipStream_t stream, const SelectInside* inside);
bool decode_fused_supported(const actqkv_shape& sh);
size_t decode_mfma_scratch_floats(const actqkv_shape& sh, int batch, int k_cap);
int launch_attention_decode_mfma(const actqkv_shape& sh, int batch, const void* q, const void* k_cache,
                                 const void* v_cache, int64_t seq_stride, int nb_capacity,
                                 const int32_t* n_ctx, const int32_t* idx, const int32_t* n_sel,
                                 int k_cap, void* out, float* lse, float* scratch,
                                 unsigned int* counters, float scale, int sel_per_head, hipStream_t stream);

int launch_attention_decode_select(const actqkv_shape& sh, int batch, const void* q, const void* k_cache,
                                   const void* v_cache, int64_t seq_stride, int nb_capacity,
                                   const int32_t* n_ctx, const float* scores, int64_t score_stride, int nb_begin,
                                   int nb_scored, const int32_t* nb_end, int k_cap, int flags, const float* budget_in,
                                   const float* theta_rest_sum, float* budget_after, int32_t* idx,
                                   int32_t* n_sel, float* theta, float* budget, void* out, float* lse,
                                   float* scratch, unsigned int* counters, float scale, hipStream_t stream);

// scratch of the attention alone: the ticket and queue counters, then the partial results
size_t attention_scratch_bytes(const actqkv_shape& sh, int batch, int m, int k_cap, int cus) {
  size_t attn = 0;
  if (m == 1) attn = decode_mfma_scratch_floats(sh, batch, k_cap) * sizeof(float);
  if (prefill_mfma_supported(sh, m)) {
    // partial results exist only where a query tile's key tiles are cut into pieces
    const PfSplits splits = prefill_splits(sh, batch, m, k_cap, cus);
    if (splits.slots > splits.n_qtiles)
      attn = size_t(batch) * sh.n_kv_heads * splits.slots * kPfPartialFloats * sizeof(float);
  }
  if (prefill_f32_supported(sh, m)) attn = prefill_f32_scratch_bytes(sh, batch, m);
  return kCounterBytes + align_up(attn, 256);
}

// what exactly this (batch, m) needs; the pieces a query tile is cut into, and with them the
// partial results, only grow with the compute units the attention may fill
size_t workspace_bytes(const actqkv_shape& sh, int batch, int m, int nb_capacity, int k_cap, int cus) {
  (void)nb_capacity;
  const size_t probe = kCounterBytes + align_up(probe_call_floats(sh, batch, m) * sizeof(float), 256);
  return std::max(probe, attention_scratch_bytes(sh, batch, m, k_cap, cus));
}

// What a caller should allocate: enough for every call with 1 .. batch entries and windows of
// 1 .. m tokens.  The need is not monotone: few short windows are cut into many pieces with
// partial results, many long ones into none; so a workspace sized for a layer's nominal window must also serve
// its ragged last window and a decode step.
static size_t workspace_bytes_upto(const actqkv_shape& sh, int batch, int m, int nb_capacity, int k_cap) {
  size_t need = 0;
  if (prefill_f32_supported(sh, m)) need = kCounterBytes + align_up(prefill_f32_scratch_most(sh, batch, m), 256);
  if (prefill_mfma_supported(sh, m)) need = kCounterBytes + prefill_partials_most(sh, batch, m);
  for (int b = 1; b <= batch; ++b) need = std::max(need, workspace_bytes(sh, b, 1, nb_capacity, k_cap));
  need = std::max(need, kCounterBytes + align_up(probe_call_floats(sh, batch, m) * sizeof(float), 256));
  return need + Workspace::spare_bytes(batch);
}

int launch_attention(const actqkv_shape& sh, int batch, int m, const void* q, const void* k_cache,
                     const void* v_cache, int64_t seq_stride, int nb_capacity, const int32_t* n_ctx,
                     const int32_t* idx, const int32_t* n_sel, int k_cap, void* out, float* lse,
                     const Workspace& ws, int sel_per_head, hipStream_t stream, int first_cus, int late_cus,
                     hipStream_t stream_late, bool pieces_of_one, const SelectInside* inside) {
  const float scale = sh.softmax_scale > 0.f ? sh.softmax_scale : 1.f / std::sqrt(float(sh.head_dim));
  if (m == 1)   // (no queue: one launch does all the work)
    return launch_attention_decode_mfma(sh, batch, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx,
                                        idx, n_sel, k_cap, out, lse, ws.scratch_f32(), ws.counters(), scale,
                                        sel_per_head, stream);
  if (prefill_mfma_supported(sh, m))
    return launch_attention_prefill_mfma(sh, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity,
                                         n_ctx, idx, n_sel, k_cap, out, lse,
                                         pieces_of_one ? prefill_splits(sh, 1, m, k_cap, kChipCus)
                                                       : prefill_splits(sh, batch, m, k_cap, first_cus), ws.scratch_f32(),
                                         ws.counters(), scale, sel_per_head, first_cus, late_cus, stream,
                                         stream_late, inside);
  return launch_attention_prefill_f32(sh, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx, n_sel,
                                      k_cap, out, lse, ws.scratch_f32(), scale, sel_per_head, stream, inside);
}

// Host-side checks of an attention call; `need` receives the scratch bytes the call uses.
int attention_validate(const actqkv_shape* shape, int batch, int m, const void* q, const void* k_cache,
                              const void* v_cache, int64_t seq_stride, int nb_capacity, const int32_t* n_ctx,
                              const int32_t* idx, const int32_t* n_sel, int k_cap, void* out, float* lse,
                              int first_cus, size_t* need) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (m < 1) return set_error(ACTQKV_EINVAL, "m %d < 1", m);
  if (m > kMaxWindow) return set_error(ACTQKV_ESHAPE, "m %d > %d", m, kMaxWindow);
  // (the attention selects nothing: the 8192-block limit of a selection does not apply to its cache)
  if (k_cap < 1 || k_cap > 64) return set_error(ACTQKV_ESHAPE, "k_cap %d not supported (1..64)", k_cap);
  if (nb_capacity < 1) return set_error(ACTQKV_EINVAL, "nb_capacity %d < 1", nb_capacity);
  if (int64_t(nb_capacity) * shape->block_size < m)
    return set_error(ACTQKV_EINVAL, "cache of %d blocks cannot hold a window of %d tokens", nb_capacity, m);
  if (int64_t(nb_capacity) * shape->block_size > (int64_t(1) << 30))
    return set_error(ACTQKV_ESHAPE, "cache of %d blocks exceeds 2^30 tokens", nb_capacity);
  ACTQKV_REQUIRE_PTR(q);
  ACTQKV_REQUIRE_PTR(k_cache);
  ACTQKV_REQUIRE_PTR(v_cache);
  ACTQKV_REQUIRE_SMALL(n_ctx, 4);
  ACTQKV_REQUIRE_SMALL(idx, 4);
  ACTQKV_REQUIRE_SMALL(n_sel, 4);
  ACTQKV_REQUIRE_PTR(out);
  ACTQKV_OPTIONAL_SMALL(lse, 4);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_kv_heads * shape->block_size * shape->head_dim;
  // seq_stride 0: all batch entries read one cache (several windows of one sequence)
  if (batch > 1 && seq_stride != 0 && seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "seq_stride %lld < one sequence's cache %lld", (long long)seq_stride,
                     (long long)per_seq);
  if (seq_stride % 8 != 0) return set_error(ACTQKV_EALIGN, "seq_stride must be a multiple of 8 elements");
  *need = attention_scratch_bytes(*shape, batch, m, k_cap, first_cus);
  return ACTQKV_OK;
}

}  // namespace actqkv

using namespace actqkv;

namespace actqkv {
// Grid-stride copy of n 16-byte words (traffic-counter calibration).
__global__ __launch_bounds__(256) void copy_bytes_kernel(u32x4* __restrict__ dst,
                                                         const u32x4* __restrict__ src, size_t n) {
  for (size_t i = size_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += size_t(gridDim.x) * 256)
    dst[i] = src[i];
}

// The same over the host link: few workgroups with many words in flight each.  The link takes about
// 57 GB/s whatever asks; a workgroup per 4 KB filled the memory system's queues with host accesses,
// and a 2 us kernel beside an 8 MB copy took 87 us.
// Stores into host memory go past the L2 (system scope: sc0 and sc1).  Ordinary ones stay there as dirty lines of
// memory behind the link, and every kernel on the chip waits for their evictions: the attention of four windows takes
// 171 us, 457 beside such a copy and 175 beside this one, which is also the faster copy (55 GB/s instead of 48).
// With fewer workgroups and ordinary stores it is one or the other: 2 of them 187 us and 45 GB/s, 4 281 us.
constexpr int kLinkWgs = 8, kLinkBatch = 8;
template <bool kToHost>
__global__ __launch_bounds__(256) void copy_bytes_link_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                              size_t n) {
  constexpr int kPiece = 256 * kLinkBatch;
  for (size_t i0 = size_t(blockIdx.x) * kPiece; i0 < n; i0 += size_t(gridDim.x) * kPiece) {
    u32x4 x[kLinkBatch];
#pragma unroll
    for (int b = 0; b < kLinkBatch; ++b) {
      const size_t i = i0 + b * 256 + threadIdx.x;
      x[b] = src[i < n ? i : n - 1];
    }
    if constexpr (kToHost) {
      constexpr int kSystemScope = 1 | 16;             // sc0, sc1
      const size_t left = n - i0;                      // (what lies behind the piece or the copy is not written)
      const __amdgpu_buffer_rsrc_t to =
          __builtin_amdgcn_make_buffer_rsrc(dst + i0, 0, int(left < kPiece ? left : kPiece) * 16, 0x00020000);
#pragma unroll
      for (int b = 0; b < kLinkBatch; ++b)
        __builtin_amdgcn_raw_buffer_store_b128(x[b], to, (b * 256 + int(threadIdx.x)) * 16, 0, kSystemScope);
    } else {
#pragma unroll
      for (int b = 0; b < kLinkBatch; ++b) {
        const size_t i = i0 + b * 256 + threadIdx.x;
        if (i < n) dst[i] = x[b];
      }
    }
  }
}
static bool in_host_memory(const void* p) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return a.type == hipMemoryTypeHost;
}
}  // namespace actqkv

extern "C" {

size_t actqkv_stats_floats(const actqkv_shape* shape) {
  if (check_shape(shape) != ACTQKV_OK) return 0;
  return stats_floats(*shape);
}

size_t actqkv_workspace_bytes(const actqkv_shape* shape, int batch, int m, int nb_capacity, int k_cap) {
  if (check_shape(shape) != ACTQKV_OK) return 0;
  if (batch < 1 || batch > kMaxBatch || m < 1 || nb_capacity < 0 || k_cap < 1 || k_cap > 64) {
    set_error(ACTQKV_EINVAL, "workspace_bytes: bad batch/m/nb_capacity/k_cap");
    return 0;
  }
  return workspace_bytes_upto(*shape, batch, m, nb_capacity, k_cap);
}

static int decode_retrieve_check(const actqkv_shape* shape, int batch, const void* q_tok, const void* k_new,
                                 const void* v_new, const int32_t* pos0, const void* k_cache, const void* v_cache,
                                 int64_t cache_seq_stride, const void* rep_keys, int64_t rep_seq_stride,
                                 int nb_capacity, int nb_begin, const int32_t* nb_end, const float* probe,
                                 const float* probe_kv, const float* probe_norm, const float* scores, int64_t score_stride,
                                 int k_cap, int flags, const float* budget_remaining, const float* theta_rest_sum,
                                 const int32_t* idx, const int32_t* n_sel, const float* theta, const float* budget) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (flags & ~(ACTQKV_SELECT_ENTROPY_TOPK | ACTQKV_DECODE_SCORES_ONLY))
    return set_error(ACTQKV_EINVAL, "decode_retrieve: unknown flag bits: %d", flags);
  const bool select_too = !(flags & ACTQKV_DECODE_SCORES_ONLY);
  if (nb_capacity < 1) return set_error(ACTQKV_EINVAL, "nb_capacity %d < 1", nb_capacity);
  if (int64_t(nb_capacity) * shape->block_size > (int64_t(1) << 30))
    return set_error(ACTQKV_ESHAPE, "cache of %d blocks exceeds 2^30 tokens", nb_capacity);
  ACTQKV_TRY(check_blocks(nb_capacity, nb_begin, k_cap, true));
  ACTQKV_REQUIRE_PTR(q_tok);
  const bool update = k_new != nullptr || v_new != nullptr || pos0 != nullptr;
  if (update) {
    ACTQKV_REQUIRE_PTR(k_new);
    ACTQKV_REQUIRE_PTR(v_new);
    ACTQKV_REQUIRE_SMALL(pos0, 4);
    ACTQKV_REQUIRE_PTR(k_cache);
    ACTQKV_REQUIRE_PTR(v_cache);
  }
  ACTQKV_REQUIRE_PTR(rep_keys);
  ACTQKV_REQUIRE_SMALL(nb_end, 4);
  ACTQKV_OPTIONAL_PTR(probe);
  ACTQKV_OPTIONAL_PTR(probe_kv);
  ACTQKV_OPTIONAL_SMALL(probe_norm, 4);
  ACTQKV_REQUIRE_SMALL(scores, 4);
  if (select_too) {
    ACTQKV_REQUIRE_SMALL(idx, 4);
    ACTQKV_REQUIRE_SMALL(n_sel, 4);
  }
  if ((budget_remaining == nullptr) != (theta_rest_sum == nullptr))
    return set_error(ACTQKV_EINVAL, "budget_remaining and theta_rest_sum must be given together");
  ACTQKV_OPTIONAL_SMALL(budget_remaining, 4);
  ACTQKV_OPTIONAL_SMALL(theta_rest_sum, 4);
  ACTQKV_OPTIONAL_SMALL(theta, 4);
  ACTQKV_OPTIONAL_SMALL(budget, 4);
  if (score_stride < nb_capacity)
    return set_error(ACTQKV_EINVAL, "score_stride %lld < nb_capacity %d", (long long)score_stride,
                     nb_capacity);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_kv_heads * shape->block_size * shape->head_dim;
  const int64_t rep_per_seq = int64_t(nb_capacity) * shape->n_rep * shape->n_kv_heads * shape->head_dim;
  if (batch > 1 && update && cache_seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "cache_seq_stride %lld < one sequence's cache %lld",
                     (long long)cache_seq_stride, (long long)per_seq);
  if (batch > 1 && rep_seq_stride < rep_per_seq)
    return set_error(ACTQKV_EINVAL, "rep_seq_stride %lld < one sequence's representative keys %lld",
                     (long long)rep_seq_stride, (long long)rep_per_seq);
  if (cache_seq_stride % 8 != 0 || rep_seq_stride % 8 != 0)
    return set_error(ACTQKV_EALIGN, "sequence strides must be multiples of 8 elements");
  return ACTQKV_OK;
}

static int build_probe_check(const actqkv_shape* shape, int batch, int m, const void* q_win, const float* stats,
                             int update_stats, const float* probe, const float* probe_kv, const float* probe_norm,
                             const float* weights, const void* workspace, size_t ws_bytes) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (m < 1) return set_error(ACTQKV_EINVAL, "m %d < 1", m);
  if (m > kMaxWindow) return set_error(ACTQKV_ESHAPE, "m %d > %d", m, kMaxWindow);
  ACTQKV_REQUIRE_PTR(q_win);
  ACTQKV_REQUIRE_PTR(probe);
  ACTQKV_REQUIRE_PTR(probe_kv);
  ACTQKV_REQUIRE_SMALL(probe_norm, 4);
  ACTQKV_OPTIONAL_SMALL(weights, 4);
  if (m > 1 || update_stats) ACTQKV_REQUIRE_PTR(stats);
  if (update_stats & ~(ACTQKV_STATS_UPDATE | ACTQKV_PROBE_MEAN_POOLING | ACTQKV_PROBE_WINDOW_CHAIN))
    return set_error(ACTQKV_EINVAL, "update_stats has unknown bits: %d", update_stats);
  if ((update_stats & ACTQKV_PROBE_WINDOW_CHAIN) && (!(update_stats & ACTQKV_STATS_UPDATE) || m < 2))
    return set_error(ACTQKV_EINVAL, "consecutive windows need ACTQKV_STATS_UPDATE and m >= 2");
  if (workspace == nullptr || !aligned16(workspace))
    return set_error(ACTQKV_EWORKSPACE, "workspace is NULL or not 16-byte aligned");
  size_t need = kCounterBytes + probe_call_floats(*shape, batch, m) * sizeof(float);
  if (ws_bytes < need)
    return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, build_probe needs %zu", ws_bytes, need);
  return ACTQKV_OK;
}

static int score_blocks_check(const actqkv_shape* shape, int batch, const float* probe_kv, const float* probe_norm,
                              const void* rep_keys, int64_t seq_stride, int nb_capacity, int nb_begin, const int32_t* nb_end,
                              const float* scores, int64_t score_stride) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  ACTQKV_TRY(check_blocks(nb_capacity, nb_begin, 1, false));
  ACTQKV_REQUIRE_PTR(probe_kv);
  ACTQKV_REQUIRE_SMALL(probe_norm, 4);
  ACTQKV_REQUIRE_PTR(rep_keys);
  ACTQKV_REQUIRE_SMALL(nb_end, 4);
  ACTQKV_REQUIRE_SMALL(scores, 4);
  if (score_stride < nb_capacity)
    return set_error(ACTQKV_EINVAL, "score_stride %lld < nb_capacity %d", (long long)score_stride,
                     nb_capacity);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_rep * shape->n_kv_heads * shape->head_dim;
  if (batch > 1 && seq_stride != 0 && seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "seq_stride %lld < one sequence's representative keys %lld",
                     (long long)seq_stride, (long long)per_seq);
  if (seq_stride % 8 != 0) return set_error(ACTQKV_EALIGN, "seq_stride must be a multiple of 8 elements");
  return ACTQKV_OK;
}

static int select_check(int batch, const float* scores, int64_t score_stride, int nb_capacity, int nb_begin,
                        const int32_t* nb_end, int k_cap, int flags, const float* budget_remaining,
                        const float* theta_rest_sum, const int32_t* idx, const int32_t* n_sel, const float* theta,
                        const float* budget) {
  if (flags & ~(ACTQKV_SELECT_ENTROPY_TOPK | ACTQKV_SELECT_DENSITY_ONLY | ACTQKV_SELECT_GIVEN_COUNT))
    return set_error(ACTQKV_EINVAL, "select: unknown flag bits: %d", flags);
  if ((flags & ACTQKV_SELECT_DENSITY_ONLY) && (flags & ACTQKV_SELECT_GIVEN_COUNT))
    return set_error(ACTQKV_EINVAL, "select: density only and a given count exclude each other");
  if ((flags & ACTQKV_SELECT_DENSITY_ONLY) && theta == nullptr)
    return set_error(ACTQKV_EINVAL, "select: density only needs theta");
  if ((flags & (ACTQKV_SELECT_DENSITY_ONLY | ACTQKV_SELECT_GIVEN_COUNT)) && budget_remaining != nullptr)
    return set_error(ACTQKV_EINVAL, "select: the cut-off state is not used with density only or a given count");
  ACTQKV_TRY(check_batch(batch));
  ACTQKV_TRY(check_blocks(nb_capacity, nb_begin, k_cap, true));
  ACTQKV_REQUIRE_SMALL(scores, 4);
  ACTQKV_REQUIRE_SMALL(nb_end, 4);
  ACTQKV_REQUIRE_SMALL(idx, 4);
  ACTQKV_REQUIRE_SMALL(n_sel, 4);
  if ((budget_remaining == nullptr) != (theta_rest_sum == nullptr))
    return set_error(ACTQKV_EINVAL, "budget_remaining and theta_rest_sum must be given together");
  ACTQKV_OPTIONAL_SMALL(budget_remaining, 4);
  ACTQKV_OPTIONAL_SMALL(theta_rest_sum, 4);
  ACTQKV_OPTIONAL_SMALL(theta, 4);
  ACTQKV_OPTIONAL_SMALL(budget, 4);
  if (score_stride < nb_capacity)
    return set_error(ACTQKV_EINVAL, "score_stride %lld < nb_capacity %d", (long long)score_stride,
                     nb_capacity);
  return ACTQKV_OK;
}

int actqkv_build_probe(const actqkv_shape* shape, int batch, int m, const void* q_win, float* stats,
                       int update_stats, float* probe, float* probe_kv, float* probe_norm,
                       float* weights, void* workspace, size_t ws_bytes, void* stream) {
  ACTQKV_TRY(build_probe_check(shape, batch, m, q_win, stats, update_stats, probe, probe_kv, probe_norm, weights, workspace,
                               ws_bytes));
  Workspace ws{workspace, ws_bytes};
  return launch_probe(*shape, batch, m, q_win, stats, update_stats, probe, probe_kv, probe_norm,
                      weights, ws, static_cast<hipStream_t>(stream));
}

int actqkv_score_blocks(const actqkv_shape* shape, int batch, const float* probe_kv,
                        const float* probe_norm, const void* rep_keys, int64_t seq_stride,
                        int nb_capacity, int nb_begin, const int32_t* nb_end, float* scores,
                        int64_t score_stride, void* stream) {
  ACTQKV_TRY(score_blocks_check(shape, batch, probe_kv, probe_norm, rep_keys, seq_stride, nb_capacity, nb_begin, nb_end, scores,
                                score_stride));
  return launch_score(*shape, batch, probe_kv, probe_norm, rep_keys, seq_stride, nb_capacity, nb_begin,
                      nb_end, scores, score_stride, static_cast<hipStream_t>(stream));
}

int actqkv_select(int batch, const float* scores, int64_t score_stride, int nb_capacity, int nb_begin,
                  const int32_t* nb_end, int k_cap, int flags, float* budget_remaining,
                  const float* theta_rest_sum, int32_t* idx, int32_t* n_sel, float* theta,
                  float* budget, void* stream) {
  ACTQKV_TRY(select_check(batch, scores, score_stride, nb_capacity, nb_begin, nb_end, k_cap, flags, budget_remaining,
                          theta_rest_sum, idx, n_sel, theta, budget));
  return launch_select(batch, scores, score_stride, nb_capacity, nb_begin, nb_end, k_cap, flags,
                       budget_remaining, theta_rest_sum, idx, n_sel, theta, budget,
                       static_cast<hipStream_t>(stream));
}

static int attention_checked(const actqkv_shape* shape, int batch, int m, const void* q, const void* k_cache,
                             const void* v_cache, int64_t seq_stride, int nb_capacity, const int32_t* n_ctx,
                             const int32_t* idx, const int32_t* n_sel, int k_cap, void* out, float* lse,
                             void* workspace, size_t ws_bytes, int sel_per_head, void* stream,
                             int first_cus = kChipCus, int late_cus = 0, void* stream_late = nullptr) {
  size_t need = 0;
  ACTQKV_TRY(attention_validate(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx, n_sel,
                                k_cap, out, lse, first_cus, &need));
  if (workspace == nullptr || !aligned16(workspace))
    return set_error(ACTQKV_EWORKSPACE, "workspace is NULL or not 16-byte aligned");
  if (ws_bytes < need)
    return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, retrieval_attention needs %zu", ws_bytes,
                     need);
  Workspace ws{workspace, ws_bytes};
  return launch_attention(*shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx,
                          n_sel, k_cap, out, lse, ws, sel_per_head, static_cast<hipStream_t>(stream), first_cus,
                          late_cus, static_cast<hipStream_t>(stream_late));
}

int actqkv_window_step(const actqkv_shape* shape, int batch, int m, const void* q_win, float* stats, int update_stats,
                       float* probe, float* probe_kv, float* probe_norm, float* weights, const void* rep_keys,
                       int64_t rep_seq_stride, int nb_scored, int nb_begin, const int32_t* nb_end, float* scores,
                       int64_t score_stride, int k_cap, int flags, float* budget_remaining, const float* theta_rest_sum,
                       int32_t* idx, int32_t* n_sel, float* theta, float* budget, const void* k_cache, const void* v_cache,
                       int64_t cache_seq_stride, int nb_capacity, const int32_t* n_ctx, void* out, float* lse,
                       void* workspace, size_t ws_bytes, void* stream) {
  // everything is checked before anything is launched
  ACTQKV_TRY(build_probe_check(shape, batch, m, q_win, stats, update_stats, probe, probe_kv, probe_norm, weights, workspace,
                               ws_bytes));
  ACTQKV_TRY(score_blocks_check(shape, batch, probe_kv, probe_norm, rep_keys, rep_seq_stride, nb_scored, nb_begin, nb_end,
                                scores, score_stride));
  ACTQKV_TRY(select_check(batch, scores, score_stride, nb_scored, nb_begin, nb_end, k_cap, flags, budget_remaining,
                          theta_rest_sum, idx, n_sel, theta, budget));
  size_t need = 0;
  ACTQKV_TRY(attention_validate(shape, batch, m, q_win, k_cache, v_cache, cache_seq_stride, nb_capacity, n_ctx, idx, n_sel,
                                k_cap, out, lse, kChipCus, &need));
  if (ws_bytes < need)
    return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, window_step needs %zu", ws_bytes, need);
  Workspace ws{workspace, ws_bytes};
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool apart = nb_scored > nb_begin && probe_finish_apart(*shape, batch, m, update_stats);
  ACTQKV_TRY(launch_probe(*shape, batch, m, q_win, stats, update_stats, probe, probe_kv, probe_norm, weights, ws, st, !apart));
  // The selection inside the attention launch (a workspace without room for the copy: a launch of its own).  A workgroup
  // writes the results while others still read, and they may be written where the cut-off state was read (budget_remaining
  // always is, theta may be theta_rest_sum): the scoring launch keeps a copy of it behind what the call needs of the workspace.
  // Four windows of 512 tokens at 64K with the selection as a launch of its own 244 us, inside 236; of 256 tokens with 64
  // channels 133, 128.
  float* copy = ws.spare(need, batch);
  if (apart && copy != nullptr && select_inside_supported(nb_scored - nb_begin, k_cap, flags)) {
    ACTQKV_TRY(launch_score_probe(*shape, probe, probe_kv, probe_norm, rep_keys, nb_scored, nb_begin, nb_end, scores,
                                  budget_remaining, theta_rest_sum, copy, st));
    SelectInside inside;
    inside.scores = scores;
    inside.nb_begin = nb_begin;
    inside.nb_capacity = nb_scored;
    inside.nb_end = nb_end;
    inside.entropy_topk = (flags & ACTQKV_SELECT_ENTROPY_TOPK) != 0;
    inside.io = SelectIo{budget_remaining != nullptr ? copy : nullptr, copy + 1, budget_remaining, idx, n_sel, theta, budget, false};
    if (flags & ACTQKV_SELECT_GIVEN_COUNT) inside.io.count_in = n_sel;   // (clamped twice it is the same)
    return launch_attention(*shape, batch, m, q_win, k_cache, v_cache, cache_seq_stride, nb_capacity, n_ctx, idx, n_sel, k_cap,
                            out, lse, ws, 0, st, kChipCus, 0, nullptr, false, &inside);
  }
  ACTQKV_TRY(apart ? launch_score_probe(*shape, probe, probe_kv, probe_norm, rep_keys, nb_scored, nb_begin, nb_end, scores,
                                        nullptr, nullptr, nullptr, st)
                   : launch_score(*shape, batch, probe_kv, probe_norm, rep_keys, rep_seq_stride, nb_scored, nb_begin, nb_end,
                                  scores, score_stride, st));
  ACTQKV_TRY(launch_select(batch, scores, score_stride, nb_scored, nb_begin, nb_end, k_cap, flags, budget_remaining,
                           theta_rest_sum, idx, n_sel, theta, budget, st));
  return launch_attention(*shape, batch, m, q_win, k_cache, v_cache, cache_seq_stride, nb_capacity, n_ctx, idx, n_sel, k_cap,
                          out, lse, ws, 0, st);
}

int actqkv_retrieval_attention(const actqkv_shape* shape, int batch, int m, const void* q,
                               const void* k_cache, const void* v_cache, int64_t seq_stride,
                               int nb_capacity, const int32_t* n_ctx, const int32_t* idx,
                               const int32_t* n_sel, int k_cap, void* out, float* lse, void* workspace,
                               size_t ws_bytes, void* stream) {
  return attention_checked(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx, n_sel,
                           k_cap, out, lse, workspace, ws_bytes, 0, stream);
}

int actqkv_retrieval_attention_teams(const actqkv_shape* shape, int batch, int m, const void* q,
                                     const void* k_cache, const void* v_cache, int64_t seq_stride,
                                     int nb_capacity, const int32_t* n_ctx, const int32_t* idx,
                                     const int32_t* n_sel, int k_cap, void* out, float* lse,
                                     void* workspace, size_t ws_bytes, int first_cus, int late_cus,
                                     void* stream, void* stream_late) {
  if (first_cus < 1 || first_cus > kChipCus)
    return set_error(ACTQKV_EINVAL, "first_cus %d outside 1..%d", first_cus, kChipCus);
  if (late_cus != 0 && shape != nullptr && (late_cus < shape->n_kv_heads || late_cus > kChipCus))
    return set_error(ACTQKV_EINVAL, "late_cus %d neither 0 nor in n_kv_heads..%d", late_cus, kChipCus);
  return attention_checked(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx, n_sel,
                           k_cap, out, lse, workspace, ws_bytes, 0, stream, first_cus, late_cus, stream_late);
}

int actqkv_retrieval_attention_windows(const actqkv_shape* shape, int n_windows, int m, const void* q,
                                       const void* k_cache, const void* v_cache, int nb_capacity,
                                       const int32_t* n_ctx, const int32_t* idx, const int32_t* n_sel, int k_cap,
                                       void* out, float* lse, void* workspace, size_t ws_bytes, int cus,
                                       void* stream) {
  if (cus < 1 || cus > kChipCus) return set_error(ACTQKV_EINVAL, "cus %d outside 1..%d", cus, kChipCus);
  size_t need = 0;
  ACTQKV_TRY(check_batch(n_windows));
  ACTQKV_TRY(attention_validate(shape, 1, m, q, k_cache, v_cache, 0, nb_capacity, n_ctx, idx, n_sel, k_cap, out, lse,
                                kChipCus, &need));
  if (!prefill_mfma_supported(*shape, m))
    return set_error(ACTQKV_ESHAPE, "retrieval_attention_windows: bf16 and windows of at least 2 tokens");
  need = kCounterBytes + (need - kCounterBytes) * n_windows;
  if (workspace == nullptr || !aligned16(workspace))
    return set_error(ACTQKV_EWORKSPACE, "workspace is NULL or not 16-byte aligned");
  if (ws_bytes < need)
    return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, retrieval_attention_windows needs %zu", ws_bytes, need);
  Workspace ws{workspace, ws_bytes};
  // a query tile in pieces has a ticket counter: as many windows in a launch as there are counters for (the pieces
  // of a window alone fill the chip, so more in a launch would gain nothing)
  const PfSplits splits = prefill_splits(*shape, 1, m, k_cap, kChipCus);
  const int per = splits.slots > splits.n_qtiles ? int(kTicketCounters) / (splits.n_qtiles * shape->n_kv_heads) : n_windows;
  const size_t row = size_t(m) * shape->n_q_heads, elem = shape->head_dim * sizeof(uint16_t);
  for (int w = 0; w < n_windows; w += per)
    ACTQKV_TRY(launch_attention(*shape, std::min(per, n_windows - w), m, static_cast<const char*>(q) + w * row * elem,
                                k_cache, v_cache, 0, nb_capacity, n_ctx + w, idx + size_t(w) * k_cap, n_sel + w, k_cap,
                                static_cast<char*>(out) + w * row * elem, lse == nullptr ? nullptr : lse + w * row, ws, 0,
                                static_cast<hipStream_t>(stream), cus, 0, nullptr, true));
  return ACTQKV_OK;
}

int actqkv_retrieval_attention_per_head(const actqkv_shape* shape, int batch, int m, const void* q,
                                        const void* k_cache, const void* v_cache, int64_t seq_stride,
                                        int nb_capacity, const int32_t* n_ctx, const int32_t* idx,
                                        const int32_t* n_sel, int k_cap, void* out, float* lse,
                                        void* workspace, size_t ws_bytes, void* stream) {
  return attention_checked(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx, n_sel,
                           k_cap, out, lse, workspace, ws_bytes, 1, stream);
}

int actqkv_decode_select_attention(const actqkv_shape* shape, int batch, const void* q,
                                   const void* k_cache, const void* v_cache, int64_t seq_stride,
                                   int nb_capacity, const int32_t* n_ctx, const float* scores,
                                   int64_t score_stride, int nb_begin, const int32_t* nb_end,
                                   int k_cap, int flags, const float* budget_in,
                                   const float* theta_rest_sum, float* budget_after, int32_t* idx,
                                   int32_t* n_sel, float* theta, float* budget, void* out,
                                   float* lse, void* workspace, size_t ws_bytes, void* stream) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (!decode_fused_supported(*shape))
    return set_error(ACTQKV_ESHAPE, "decode_select_attention: bf16, head_dim 128 and at most 8 query heads per KV head");
  if (flags & ~ACTQKV_SELECT_ENTROPY_TOPK)
    return set_error(ACTQKV_EINVAL, "decode_select_attention: unknown flag bits: %d", flags);
  if (nb_capacity < 1) return set_error(ACTQKV_EINVAL, "nb_capacity %d < 1", nb_capacity);
  if (int64_t(nb_capacity) * shape->block_size > (int64_t(1) << 30))
    return set_error(ACTQKV_ESHAPE, "cache of %d blocks exceeds 2^30 tokens", nb_capacity);
  ACTQKV_TRY(check_blocks(nb_capacity, nb_begin, k_cap, true));
  ACTQKV_REQUIRE_PTR(q);
  ACTQKV_REQUIRE_PTR(k_cache);
  ACTQKV_REQUIRE_PTR(v_cache);
  ACTQKV_REQUIRE_SMALL(n_ctx, 4);
  ACTQKV_REQUIRE_SMALL(scores, 4);
  ACTQKV_REQUIRE_SMALL(nb_end, 4);
  ACTQKV_REQUIRE_SMALL(idx, 4);
  ACTQKV_REQUIRE_SMALL(n_sel, 4);
  ACTQKV_REQUIRE_PTR(out);
  ACTQKV_OPTIONAL_SMALL(lse, 4);
  if ((budget_in == nullptr) != (theta_rest_sum == nullptr))
    return set_error(ACTQKV_EINVAL, "budget_in and theta_rest_sum must be given together");
  ACTQKV_OPTIONAL_SMALL(budget_in, 4);
  ACTQKV_OPTIONAL_SMALL(theta_rest_sum, 4);
  ACTQKV_OPTIONAL_SMALL(budget_after, 4);
  ACTQKV_OPTIONAL_SMALL(theta, 4);
  ACTQKV_OPTIONAL_SMALL(budget, 4);
  if (budget_after != nullptr && budget_after == budget_in)
    return set_error(ACTQKV_EINVAL, "budget_after must not be the array budget_in points to");
  if (score_stride < nb_capacity)
    return set_error(ACTQKV_EINVAL, "score_stride %lld < nb_capacity %d", (long long)score_stride,
                     nb_capacity);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_kv_heads * shape->block_size * shape->head_dim;
  if (batch > 1 && seq_stride != 0 && seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "seq_stride %lld < one sequence's cache %lld", (long long)seq_stride,
                     (long long)per_seq);
  if (seq_stride % 8 != 0) return set_error(ACTQKV_EALIGN, "seq_stride must be a multiple of 8 elements");
  if (workspace == nullptr || !aligned16(workspace))
    return set_error(ACTQKV_EWORKSPACE, "workspace is NULL or not 16-byte aligned");
  const size_t need = workspace_bytes(*shape, batch, 1, nb_capacity, k_cap);
  if (ws_bytes < need)
    return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, decode_select_attention needs %zu", ws_bytes,
                     need);
  Workspace ws{workspace, ws_bytes};
  const float scale = shape->softmax_scale > 0.f ? shape->softmax_scale : 1.f / std::sqrt(float(shape->head_dim));
  return launch_attention_decode_select(*shape, batch, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx,
                                        scores, score_stride, nb_begin, nb_capacity, nb_end, k_cap, flags, budget_in,
                                        theta_rest_sum, budget_after, idx, n_sel, theta, budget, out, lse,
                                        ws.scratch_f32(), ws.counters(), scale,
                                        static_cast<hipStream_t>(stream));
}

int actqkv_decode_layer(const actqkv_shape* shape, int batch, const void* q, const void* k_new,
                        const void* v_new, void* k_cache, void* v_cache, int64_t cache_seq_stride,
                        void* rep_keys, int64_t rep_seq_stride, int nb_capacity, const int32_t* n_ctx,
                        int nb_begin, const int32_t* nb_end, float* scores, int64_t score_stride, int k_cap,
                        int flags, const float* budget_in, const float* theta_rest_sum, float* budget_after,
                        int32_t* idx, int32_t* n_sel, float* theta, float* budget, void* out, float* lse,
                        void* workspace, size_t ws_bytes, void* stream) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (!decode_fused_supported(*shape))
    return set_error(ACTQKV_ESHAPE, "decode_layer: bf16, head_dim 128 and at most 8 query heads per KV head");
  if (flags & ~(ACTQKV_SELECT_ENTROPY_TOPK | ACTQKV_DECODE_NO_WAIT))
    return set_error(ACTQKV_EINVAL, "decode_layer: unknown flag bits: %d", flags);
  if (nb_capacity < 1) return set_error(ACTQKV_EINVAL, "nb_capacity %d < 1", nb_capacity);
  if (int64_t(nb_capacity) * shape->block_size > (int64_t(1) << 30))
    return set_error(ACTQKV_ESHAPE, "cache of %d blocks exceeds 2^30 tokens", nb_capacity);
  ACTQKV_TRY(check_blocks(nb_capacity, nb_begin, k_cap, true));
  if (batch > int(kSeqCounters / 2))
    return set_error(ACTQKV_ESHAPE, "decode_layer: batch %d > %d", batch, int(kSeqCounters / 2));
  ACTQKV_REQUIRE_PTR(q);
  if ((k_new == nullptr) != (v_new == nullptr))
    return set_error(ACTQKV_EINVAL, "k_new and v_new must be given together");
  ACTQKV_OPTIONAL_PTR(k_new);
  ACTQKV_OPTIONAL_PTR(v_new);
  ACTQKV_REQUIRE_PTR(k_cache);
  ACTQKV_REQUIRE_PTR(v_cache);
  ACTQKV_REQUIRE_PTR(rep_keys);
  ACTQKV_REQUIRE_SMALL(n_ctx, 4);
  ACTQKV_REQUIRE_SMALL(nb_end, 4);
  ACTQKV_REQUIRE_SMALL(scores, 4);
  ACTQKV_REQUIRE_SMALL(idx, 4);
  ACTQKV_REQUIRE_SMALL(n_sel, 4);
  ACTQKV_REQUIRE_PTR(out);
  ACTQKV_OPTIONAL_SMALL(lse, 4);
  if ((budget_in == nullptr) != (theta_rest_sum == nullptr))
    return set_error(ACTQKV_EINVAL, "budget_in and theta_rest_sum must be given together");
  ACTQKV_OPTIONAL_SMALL(budget_in, 4);
  ACTQKV_OPTIONAL_SMALL(theta_rest_sum, 4);
  ACTQKV_OPTIONAL_SMALL(budget_after, 4);
  ACTQKV_OPTIONAL_SMALL(theta, 4);
  ACTQKV_OPTIONAL_SMALL(budget, 4);
  if (budget_after != nullptr && budget_after == budget_in)
    return set_error(ACTQKV_EINVAL, "budget_after must not be the array budget_in points to");
  if (score_stride < nb_capacity)
    return set_error(ACTQKV_EINVAL, "score_stride %lld < nb_capacity %d", (long long)score_stride,
                     nb_capacity);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_kv_heads * shape->block_size * shape->head_dim;
  const int64_t rep_per_seq = int64_t(nb_capacity) * shape->n_rep * shape->n_kv_heads * shape->head_dim;
  if (batch > 1 && cache_seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "cache_seq_stride %lld < one sequence's cache %lld",
                     (long long)cache_seq_stride, (long long)per_seq);
  if (batch > 1 && rep_seq_stride < rep_per_seq)
    return set_error(ACTQKV_EINVAL, "rep_seq_stride %lld < one sequence's representative keys %lld",
                     (long long)rep_seq_stride, (long long)rep_per_seq);
  if (cache_seq_stride % 8 != 0 || rep_seq_stride % 8 != 0)
    return set_error(ACTQKV_EALIGN, "sequence strides must be multiples of 8 elements");
  if (workspace == nullptr || !aligned16(workspace))
    return set_error(ACTQKV_EWORKSPACE, "workspace is NULL or not 16-byte aligned");
  const size_t need = workspace_bytes(*shape, batch, 1, nb_capacity, k_cap);
  if (ws_bytes < need)
    return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, decode_layer needs %zu", ws_bytes, need);
  Workspace ws{workspace, ws_bytes};
  const float scale = shape->softmax_scale > 0.f ? shape->softmax_scale : 1.f / std::sqrt(float(shape->head_dim));
  // the wait for the other workgroups' scores is bounded: 2 ms is a hundred times a whole launch
  const int wait_us = (flags & ACTQKV_DECODE_NO_WAIT) ? 0 : 2000;
  return launch_decode_layer(*shape, batch, q, k_new, v_new, k_cache, v_cache, cache_seq_stride, rep_keys,
                             rep_seq_stride, nb_capacity, n_ctx, nb_begin, nb_end, scores, score_stride, k_cap,
                             flags & ACTQKV_SELECT_ENTROPY_TOPK, budget_in, theta_rest_sum, budget_after, idx,
                             n_sel, theta, budget, out, lse, ws.scratch_f32(), ws.counters(), scale, wait_us,
                             static_cast<hipStream_t>(stream));
}

int actqkv_score_blocks_per_head(const actqkv_shape* shape, int batch, const float* probe, const void* rep_keys,
                                 int64_t seq_stride, int nb_capacity, int nb_begin, const int32_t* nb_end,
                                 float* scores, int64_t score_stride, void* stream) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  ACTQKV_TRY(check_blocks(nb_capacity, nb_begin, 1, false));
  ACTQKV_REQUIRE_PTR(probe);
  ACTQKV_REQUIRE_PTR(rep_keys);
  ACTQKV_REQUIRE_SMALL(nb_end, 4);
  ACTQKV_REQUIRE_SMALL(scores, 4);
  if (score_stride < nb_capacity)
    return set_error(ACTQKV_EINVAL, "score_stride %lld < nb_capacity %d", (long long)score_stride,
                     nb_capacity);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_rep * shape->n_kv_heads * shape->head_dim;
  if (batch > 1 && seq_stride != 0 && seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "seq_stride %lld < one sequence's representative keys %lld",
                     (long long)seq_stride, (long long)per_seq);
  if (seq_stride % 8 != 0) return set_error(ACTQKV_EALIGN, "seq_stride must be a multiple of 8 elements");
  return launch_score_per_head(*shape, batch, probe, rep_keys, seq_stride, nb_capacity, nb_begin, nb_end,
                               scores, score_stride, static_cast<hipStream_t>(stream));
}

int actqkv_copy_bytes(void* dst, const void* src, size_t bytes, void* stream) {
  if (dst == nullptr || src == nullptr) return set_error(ACTQKV_EINVAL, "copy_bytes: null pointer");
  if (bytes % 16 != 0) return set_error(ACTQKV_EINVAL, "copy_bytes: %zu bytes is not a multiple of 16", bytes);
  if (reinterpret_cast<uintptr_t>(dst) % 16 != 0 || reinterpret_cast<uintptr_t>(src) % 16 != 0)
    return set_error(ACTQKV_EALIGN, "copy_bytes: pointers must be 16-byte aligned");
  if (bytes == 0) return ACTQKV_OK;
  const size_t n = bytes / 16;
  const bool to_host = in_host_memory(dst);
  if (to_host || in_host_memory(src)) {
    hipLaunchKernelGGL(to_host ? copy_bytes_link_kernel<true> : copy_bytes_link_kernel<false>, dim3(kLinkWgs), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<u32x4*>(dst), static_cast<const u32x4*>(src), n);
    return hip_status("copy_bytes");
  }
  const unsigned blocks = unsigned(std::min<size_t>((n + 255) / 256, 256 * 16));
  hipLaunchKernelGGL(copy_bytes_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<u32x4*>(dst), static_cast<const u32x4*>(src), n);
  return hip_status("copy_bytes");
}

int actqkv_gather_blocks(const actqkv_shape* shape, int batch, const void* k_store, const void* v_store,
                         int64_t store_seq_stride, int nb_store, const int32_t* idx, const int32_t* n_sel,
                         int k_cap, void* k_cache, void* v_cache, int64_t cache_seq_stride,
                         int nb_capacity, int slot0, int32_t* idx_slots, void* stream) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (k_cap < 1 || k_cap > 64) return set_error(ACTQKV_ESHAPE, "k_cap %d outside 1..64", k_cap);
  if (nb_store < 1 || nb_capacity < 1) return set_error(ACTQKV_EINVAL, "gather_blocks: empty store or cache");
  if (slot0 < 0 || int64_t(slot0) + k_cap > nb_capacity)
    return set_error(ACTQKV_EINVAL, "gather_blocks: slots %d .. %d outside the cache of %d blocks", slot0,
                     slot0 + k_cap - 1, nb_capacity);
  ACTQKV_REQUIRE_PTR(k_store);
  ACTQKV_REQUIRE_PTR(v_store);
  ACTQKV_REQUIRE_PTR(k_cache);
  ACTQKV_REQUIRE_PTR(v_cache);
  ACTQKV_REQUIRE_SMALL(idx, 4);
  ACTQKV_REQUIRE_SMALL(n_sel, 4);
  ACTQKV_OPTIONAL_SMALL(idx_slots, 4);
  const int64_t block_elems = int64_t(shape->n_kv_heads) * shape->block_size * shape->head_dim;
  if (batch > 1 && (store_seq_stride < nb_store * block_elems || cache_seq_stride < nb_capacity * block_elems))
    return set_error(ACTQKV_EINVAL, "gather_blocks: a sequence stride is smaller than one sequence");
  if (store_seq_stride % 8 != 0 || cache_seq_stride % 8 != 0)
    return set_error(ACTQKV_EALIGN, "sequence strides must be multiples of 8 elements");
  return launch_gather(*shape, batch, k_store, v_store, store_seq_stride, nb_store, idx, n_sel, k_cap, k_cache,
                       v_cache, cache_seq_stride, slot0, idx_slots, static_cast<hipStream_t>(stream));
}

int actqkv_gather_blocks_cached(const actqkv_shape* shape, int n_windows, const void* k_store, const void* v_store,
                                int nb_store, const int32_t* idx, const int32_t* n_sel, int k_cap, void* k_cache,
                                void* v_cache, int nb_capacity, int slot0, int n_slots, int here0_lo, int here0_hi,
                                int here0_at, int here1_lo, int here1_hi, int here1_at, int group, int32_t* state,
                                int32_t* idx_slots, void* stream) {
  ACTQKV_TRY(check_shape(shape));
  if (k_cap < 1 || k_cap > 64) return set_error(ACTQKV_ESHAPE, "k_cap %d outside 1..64", k_cap);
  if (n_windows < 1 || n_windows > kSlotSelections / k_cap)
    return set_error(ACTQKV_ESHAPE, "gather_blocks_cached: %d windows of up to %d blocks (at most %d selections)", n_windows,
                     k_cap, kSlotSelections);
  if (nb_store < 1 || nb_capacity < 1) return set_error(ACTQKV_EINVAL, "gather_blocks_cached: empty store or cache");
  if (n_slots < 2 * n_windows * k_cap || n_slots > 2 * kSlotSelections)
    return set_error(ACTQKV_EINVAL, "gather_blocks_cached: %d slots outside %d..%d", n_slots, 2 * n_windows * k_cap,
                     2 * kSlotSelections);
  if (slot0 < 0 || int64_t(slot0) + n_slots > nb_capacity)
    return set_error(ACTQKV_EINVAL, "gather_blocks_cached: slots %d .. %d outside the cache of %d blocks", slot0,
                     slot0 + n_slots - 1, nb_capacity);
  if (group < 0) return set_error(ACTQKV_EINVAL, "gather_blocks_cached: group %d", group);
  const HereRange ranges[2] = {{here0_lo, here0_hi, here0_at}, {here1_lo, here1_hi, here1_at}};
  for (const HereRange& h : ranges) {
    if (h.hi <= h.lo) continue;
    const int64_t end = int64_t(h.at) + (int64_t(h.hi) - h.lo);
    if (h.lo < 0 || h.at < 0 || end > nb_capacity || (end > slot0 && h.at < slot0 + n_slots))
      return set_error(ACTQKV_EINVAL, "gather_blocks_cached: blocks %d .. %d at %d overlap the slots or leave the cache",
                       h.lo, h.hi - 1, h.at);
  }
  ACTQKV_REQUIRE_PTR(k_store);
  ACTQKV_REQUIRE_PTR(v_store);
  ACTQKV_REQUIRE_PTR(k_cache);
  ACTQKV_REQUIRE_PTR(v_cache);
  ACTQKV_REQUIRE_SMALL(idx, 4);
  ACTQKV_REQUIRE_SMALL(n_sel, 4);
  ACTQKV_REQUIRE_SMALL(state, 4);
  ACTQKV_REQUIRE_SMALL(idx_slots, 4);
  return launch_gather_cached(*shape, n_windows, k_store, v_store, nb_store, idx, n_sel, k_cap, k_cache, v_cache, slot0,
                              n_slots, ranges[0], ranges[1], group, state, idx_slots,
                              static_cast<hipStream_t>(stream));
}

static int append_checked(const actqkv_shape* shape, int batch, int m, const void* k_new, const void* v_new,
                          const int32_t* pos0, void* k_cache, void* v_cache, int64_t cache_seq_stride,
                          void* rep_keys, int64_t rep_seq_stride, int nb_capacity, const void* q_tok,
                          float* probe, float* probe_kv, float* probe_norm, void* stream) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (m < 1) return set_error(ACTQKV_EINVAL, "m %d < 1", m);
  if (m > kMaxWindow) return set_error(ACTQKV_ESHAPE, "m %d > %d", m, kMaxWindow);
  if (nb_capacity < 1) return set_error(ACTQKV_EINVAL, "nb_capacity %d < 1", nb_capacity);
  if (int64_t(nb_capacity) * shape->block_size > (int64_t(1) << 30))
    return set_error(ACTQKV_ESHAPE, "cache of %d blocks exceeds 2^30 tokens", nb_capacity);
  ACTQKV_REQUIRE_PTR(k_new);
  ACTQKV_REQUIRE_PTR(v_new);
  ACTQKV_REQUIRE_SMALL(pos0, 4);
  ACTQKV_REQUIRE_PTR(k_cache);
  ACTQKV_REQUIRE_PTR(v_cache);
  ACTQKV_OPTIONAL_PTR(rep_keys);
  const int64_t per_seq = int64_t(nb_capacity) * shape->n_kv_heads * shape->block_size * shape->head_dim;
  const int64_t rep_per_seq = int64_t(nb_capacity) * shape->n_rep * shape->n_kv_heads * shape->head_dim;
  if (batch > 1 && cache_seq_stride < per_seq)
    return set_error(ACTQKV_EINVAL, "cache_seq_stride %lld < one sequence's cache %lld",
                     (long long)cache_seq_stride, (long long)per_seq);
  if (batch > 1 && rep_keys != nullptr && rep_seq_stride < rep_per_seq)
    return set_error(ACTQKV_EINVAL, "rep_seq_stride %lld < one sequence's representative keys %lld",
                     (long long)rep_seq_stride, (long long)rep_per_seq);
  if (cache_seq_stride % 8 != 0 || rep_seq_stride % 8 != 0)
    return set_error(ACTQKV_EALIGN, "sequence strides must be multiples of 8 elements");
  return launch_append(*shape, batch, m, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                       rep_seq_stride, nb_capacity, q_tok, probe, probe_kv, probe_norm,
                       static_cast<hipStream_t>(stream));
}

int actqkv_append_kv(const actqkv_shape* shape, int batch, int m, const void* k_new, const void* v_new,
                     const int32_t* pos0, void* k_cache, void* v_cache, int64_t cache_seq_stride,
                     void* rep_keys, int64_t rep_seq_stride, int nb_capacity, void* stream) {
  return append_checked(shape, batch, m, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                        rep_seq_stride, nb_capacity, nullptr, nullptr, nullptr, nullptr, stream);
}

int actqkv_append_kv_probe(const actqkv_shape* shape, int batch, const void* q_tok, const void* k_new,
                           const void* v_new, const int32_t* pos0, void* k_cache, void* v_cache,
                           int64_t cache_seq_stride, void* rep_keys, int64_t rep_seq_stride,
                           int nb_capacity, float* probe, float* probe_kv, float* probe_norm,
                           void* stream) {
  ACTQKV_REQUIRE_PTR(q_tok);
  ACTQKV_REQUIRE_PTR(probe);
  ACTQKV_REQUIRE_PTR(probe_kv);
  ACTQKV_REQUIRE_SMALL(probe_norm, 4);
  return append_checked(shape, batch, 1, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                        rep_seq_stride, nb_capacity, q_tok, probe, probe_kv, probe_norm, stream);
}

int actqkv_decode_retrieve(const actqkv_shape* shape, int batch, const void* q_tok, const void* k_new,
                           const void* v_new, const int32_t* pos0, void* k_cache, void* v_cache,
                           int64_t cache_seq_stride, void* rep_keys, int64_t rep_seq_stride,
                           int nb_capacity, int nb_begin, const int32_t* nb_end, float* probe,
                           float* probe_kv, float* probe_norm, float* scores, int64_t score_stride,
                           int k_cap, int flags, float* budget_remaining,
                           const float* theta_rest_sum, int32_t* idx, int32_t* n_sel, float* theta,
                           float* budget, void* stream) {
  ACTQKV_TRY(decode_retrieve_check(shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                                   rep_seq_stride, nb_capacity, nb_begin, nb_end, probe, probe_kv, probe_norm, scores,
                                   score_stride, k_cap, flags, budget_remaining, theta_rest_sum, idx, n_sel, theta, budget));
  return launch_decode_retrieve(*shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride,
                                rep_keys, rep_seq_stride, nb_capacity, nb_begin, nb_end, probe, probe_kv,
                                probe_norm, scores, score_stride, k_cap, flags, budget_remaining,
                                theta_rest_sum, idx, n_sel, theta, budget, static_cast<hipStream_t>(stream));
}

int actqkv_decode_step(const actqkv_shape* shape, int batch, const void* q_tok, const void* k_new, const void* v_new,
                       const int32_t* pos0, void* k_cache, void* v_cache, int64_t cache_seq_stride, void* rep_keys,
                       int64_t rep_seq_stride, int nb_scored, int nb_begin, const int32_t* nb_end, float* probe,
                       float* probe_kv, float* probe_norm, float* scores, int64_t score_stride, int k_cap, int flags,
                       float* budget_remaining, const float* theta_rest_sum, int32_t* idx, int32_t* n_sel, float* theta,
                       float* budget, int nb_capacity, const int32_t* n_ctx, void* out, float* lse, void* workspace,
                       size_t ws_bytes, void* stream) {
  // everything is checked before anything is launched
  if (flags & ACTQKV_DECODE_SCORES_ONLY) return set_error(ACTQKV_EINVAL, "decode_step: unknown flag bits: %d", flags);
  ACTQKV_TRY(decode_retrieve_check(shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                                   rep_seq_stride, nb_scored, nb_begin, nb_end, probe, probe_kv, probe_norm, scores,
                                   score_stride, k_cap, flags, budget_remaining, theta_rest_sum, idx, n_sel, theta, budget));
  size_t need = 0;
  ACTQKV_TRY(attention_validate(shape, batch, 1, q_tok, k_cache, v_cache, cache_seq_stride, nb_capacity, n_ctx, idx, n_sel,
                                k_cap, out, lse, kChipCus, &need));
  if (workspace == nullptr || !aligned16(workspace))
    return set_error(ACTQKV_EWORKSPACE, "workspace is NULL or not 16-byte aligned");
  if (ws_bytes < need) return set_error(ACTQKV_EWORKSPACE, "workspace has %zu bytes, decode_step needs %zu", ws_bytes, need);
  Workspace ws{workspace, ws_bytes};
  hipStream_t st = static_cast<hipStream_t>(stream);
  // The selection inside the attention launch, on a copy of the cut-off state that the scoring launch makes, where one wavefront
  // selects (a workspace without room for the copy, and rows that a launch gives to 1024 threads: a launch of its own, in which a
  // row is selected once and not by every workgroup).  The attention walks the local span before the selected blocks then, so its
  // sums have another order; bf16 with 128 channels has actqkv_decode_select_attention for that, and keeps the bits of the two calls here.
  // (The other attention in that order too: 8 sequences of 32K tokens, a selection per KV head, 29.2 -> 30.2 us, because full
  // blocks and no longer a part of the last one are left for the last round.)
  const bool inside = !decode_fused_supported(*shape) && select_inside_supported(nb_scored - nb_begin, k_cap, flags);
  float* copy = inside ? ws.spare(need, batch) : nullptr;
  ACTQKV_TRY(launch_decode_retrieve(*shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                                    rep_seq_stride, nb_scored, nb_begin, nb_end, probe, probe_kv, probe_norm, scores,
                                    score_stride, k_cap, copy != nullptr ? flags | ACTQKV_DECODE_SCORES_ONLY : flags,
                                    budget_remaining, theta_rest_sum, idx, n_sel, theta, budget, st, copy));
  if (copy == nullptr)
    return launch_attention(*shape, batch, 1, q_tok, k_cache, v_cache, cache_seq_stride, nb_capacity, n_ctx, idx, n_sel, k_cap,
                            out, lse, ws, 0, st);
  const float scale = shape->softmax_scale > 0.f ? shape->softmax_scale : 1.f / std::sqrt(float(shape->head_dim));
  return launch_attention_decode_select(*shape, batch, q_tok, k_cache, v_cache, cache_seq_stride, nb_capacity, n_ctx, scores,
                                        score_stride, nb_begin, nb_scored, nb_end, k_cap, flags,
                                        budget_remaining != nullptr ? copy : nullptr, copy + batch, budget_remaining, idx,
                                        n_sel, theta, budget, out, lse, ws.scratch_f32(), ws.counters(), scale, st);
}

int actqkv_cutoff_budgets(int batch, int n_layers, float k_mean, int k_cap, const float* theta, float* budget,
                          int32_t* count, float* budget_left, void* stream) {
  ACTQKV_TRY(check_batch(batch));
  if (n_layers < 1 || n_layers > 1024)
    return set_error(ACTQKV_ESHAPE, "n_layers %d not supported (1..1024)", n_layers);
  if (!(k_mean > 0.f)) return set_error(ACTQKV_EINVAL, "k_mean must be positive");
  if (k_cap < 1 || k_cap > 64) return set_error(ACTQKV_ESHAPE, "k_cap %d not supported (1..64)", k_cap);
  ACTQKV_REQUIRE_SMALL(theta, 4);
  ACTQKV_REQUIRE_SMALL(budget, 4);
  ACTQKV_REQUIRE_SMALL(count, 4);
  ACTQKV_OPTIONAL_SMALL(budget_left, 4);
  return launch_cutoff_budgets(batch, n_layers, k_mean, k_cap, theta, budget, count, budget_left,
                               static_cast<hipStream_t>(stream));
}

int actqkv_cutoff_next_step(int batch, int n_layers, float k_mean, float theta_prior,
                            const float* theta_prev, float* theta_sum, float* n_steps,
                            float* budget_remaining, float* theta_rest_sum, void* stream) {
  ACTQKV_TRY(check_batch(batch));
  if (n_layers < 1 || n_layers > 1024)
    return set_error(ACTQKV_ESHAPE, "n_layers %d not supported (1..1024)", n_layers);
  if (!(k_mean > 0.f)) return set_error(ACTQKV_EINVAL, "k_mean must be positive");
  if (!(theta_prior >= 0.f)) return set_error(ACTQKV_EINVAL, "theta_prior must not be negative");
  ACTQKV_OPTIONAL_SMALL(theta_prev, 4);
  ACTQKV_REQUIRE_SMALL(theta_sum, 4);
  ACTQKV_REQUIRE_SMALL(n_steps, 4);
  ACTQKV_REQUIRE_SMALL(budget_remaining, 4);
  ACTQKV_REQUIRE_SMALL(theta_rest_sum, 4);
  return launch_cutoff_next_step(batch, n_layers, k_mean, theta_prior, theta_prev, theta_sum, n_steps,
                                 budget_remaining, theta_rest_sum, static_cast<hipStream_t>(stream));
}

const char* actqkv_last_error(void) { return g_error; }

int actqkv_prefill_cut(const actqkv_shape* shape, int batch, int m, int k_cap, int cus, int32_t* cut) {
  ACTQKV_TRY(check_shape(shape));
  ACTQKV_TRY(check_batch(batch));
  if (m > kMaxWindow || !prefill_mfma_supported(*shape, m))
    return set_error(ACTQKV_ESHAPE, "prefill_cut: bf16 and windows of 2 to %d tokens", kMaxWindow);
  if (k_cap < 1 || k_cap > 64) return set_error(ACTQKV_ESHAPE, "k_cap %d not supported (1..64)", k_cap);
  if (cus < 1 || cus > kChipCus) return set_error(ACTQKV_EINVAL, "cus %d outside 1..%d", cus, kChipCus);
  if (cut == nullptr) return set_error(ACTQKV_EINVAL, "cut is NULL");
  const PfSplits c = prefill_splits(*shape, batch, m, k_cap, cus);
  cut[0] = 256 / c.ks;
  cut[1] = c.n_qtiles;
  cut[2] = c.slots;
  cut[3] = batch == 1 && prefill_merge_after(*shape, c.s_lo);
  return ACTQKV_OK;
}

int actqkv_version(void) { return ACTQKV_VERSION; }

}  // extern "C"
