// Retrieval attention of a prefill window in fp32 (Sec. 3.1, Eq. (2)): fp32 storage, and fp32
// products and sums throughout (v_mfma_f32_32x32x2_f32), so nothing is rounded below fp32.
//
// What bounds it: the matrix pipe, 256 fp32 operations per clock and compute unit, a sixteenth of
// its bf16 rate.  Everything else (LDS reads, softmax, loads) is small beside a 64-cycle MFMA, so
// the kernel is the bf16 one with fewer precautions: a workgroup of 4 wavefronts owns 128 query
// rows that share a KV head (numbered position by position, the G heads side by side), a
// wavefront 32 of them; half a block of keys at a time (16 KB of keys, 16 KB of values) goes from
// memory straight into LDS, double buffered; two workgroups share a compute unit, so each SIMD
// has a second wavefront for the matrix pipe while the first one is in its softmax.
//
// S^T = K Q^T leaves a lane with scores of ONE query (column lane % 32), and register r of lane
// half h holds key 8 (r / 4) + 4 h + r % 4 of a 32-key group.  An MFMA of O^T += V^T P^T takes one
// key from either half, so register r of both halves IS its B operand, without a conversion or a
// lane exchange; its A operand is the same key pair of the V^T row, four keys per 16-byte LDS read.
// The channels of the first product are dealt to the halves four at a time for the same reason.
//
// A single window has few query tiles; then the key tiles are cut into pieces, one workgroup
// each, and the workgroup that finishes last among the pieces of a query tile merges them.
// A pass over 8192 tokens, windows of 256, 8 query and 2 KV heads of 64 channels: the attention
// takes 244 us (96 TFLOP/s of the 153 a large fp32 product reaches), against 1645 us as one thread
// per query row; what is left of the gap is that all its workgroups are resident at once and the
// first windows see fewer keys.
#include <algorithm>
#include <mutex>

#include "common.h"
#include "launch.h"

namespace actqkv {

constexpr int kFfThreads = 256;
constexpr int kFfWaves = 4;
constexpr int kFfRows = 32 * kFfWaves;            // query rows of a workgroup
constexpr int kFfTileBytes = 16384;               // K or V^T of a tile
constexpr int kFfLdsBytes = 2 * 2 * kFfTileBytes; // 2 stages x (K, V^T)
// Workgroups of a full launch: two per compute unit; with 128 channels a little less, so that their
// partial results fit the library's own scratch array.
template <int D> constexpr int kFfSlots = D == 64 ? 512 : 480;
template <int D> constexpr size_t kFfPieceBytes = size_t(kFfWaves) * (D / 4 + 1) * 64 * 8;
static_assert(kFfSlots<128> * kFfPieceBytes<128> + kCounterBytes <= ACTQKV_STATIC_SCRATCH_BYTES, "partial results");
constexpr int kFfMaxSplits = 8;

struct FfParams {
  const float* q;
  const float* k_cache;
  const float* v_cache;
  int64_t seq_stride;
  int nb_capacity;
  const int32_t* n_ctx;
  const int32_t* idx;
  const int32_t* n_sel;
  int k_cap;
  float* out;
  float* lse;
  uint64_t* part;          // [workgroup][wavefront][D / 4 pairs of O | (max, sum)][64 lanes]
  unsigned int* counters;  // one ticket counter per (sequence, query tile, KV head), zero between launches
  int m, n_q_heads, n_kv_heads, n_init, n_local, n_qtiles, splits;
  int sel_per_head;
  float scale_log2e;
};

// Final normalisation and store of one lane's share of a query row.
template <int D>
__device__ __forceinline__ void ff_store_row(const FfParams& p, const f32x16 (&acc_o)[D / 32], float m_run, float l_tot,
                                             int s, int row, int head, int half) {
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  float* op = p.out + ((size_t(s) * p.m + row) * p.n_q_heads + head) * D + 4 * half;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4*>(op + db * 32 + 8 * j) =
          f32x4{acc_o[db][4 * j] * inv, acc_o[db][4 * j + 1] * inv, acc_o[db][4 * j + 2] * inv, acc_o[db][4 * j + 3] * inv};
  if (p.lse != nullptr && half == 0)
    p.lse[(size_t(s) * p.n_q_heads + head) * p.m + row] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
}

template <int D>
__global__ __launch_bounds__(kFfThreads, 2) void attn_prefill_f32_kernel(FfParams p) {
  constexpr int kKeys = kFfTileBytes / (4 * D);     // keys of a tile: 64 or 32
  constexpr int kPerBlock = kBlock / kKeys;
  constexpr int kG = kKeys / 32, kDb = D / 32, kQ = D / 8;
  constexpr uint32_t kKRow = D * 4, kVRow = kKeys * 4;   // bytes of a K / V^T row in LDS
  extern __shared__ __attribute__((aligned(16))) char ff_lds[];
  __shared__ int32_t idx_lds[64];
  __shared__ int last_flag;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, half = lane >> 5;
  const int group = p.n_q_heads / p.n_kv_heads;
  // consecutive workgroups differ in the KV head (they go round the XCDs: a head's tiles stay in few L2s)
  const int hk = blockIdx.x % p.n_kv_heads, rest = blockIdx.x / p.n_kv_heads;
  const int split = rest % p.splits, qt = rest / p.splits;
  const int qtile = qt % p.n_qtiles, s = qt / p.n_qtiles;

  const size_t sel_row = p.sel_per_head ? size_t(s) * p.n_kv_heads + hk : size_t(s);
  const int32_t my_idx = tid < p.k_cap ? p.idx[sel_row * p.k_cap + tid] : -1;
  const int n_ctx_raw = p.n_ctx[s], n_sel_raw = p.n_sel[sel_row];
  if (tid < 64) idx_lds[tid] = my_idx;
  __syncthreads();
  const int n_ctx = min(max(n_ctx_raw, p.m), p.nb_capacity * kBlock);
  const WindowGeom g = window_geom(n_ctx, p.m, p.n_init, p.n_local);
  const int row_end = p.m * group;
  const int row_hi = (min((qtile + 1) * kFfRows, row_end) - 1) / group;
  const TileList tl = make_tile_list(g, g.w0 + row_hi, idx_lds, n_sel_raw, p.k_cap, p.nb_capacity);
  const int n_tiles = tl.count() * kPerBlock;
  const int per = (n_tiles + p.splits - 1) / p.splits;
  const int t_begin = split * per, t_end = min(n_tiles, t_begin + per);

  const int frow0 = qtile * kFfRows + wave * 32;             // first query row of this wavefront
  const bool wave_ok = frow0 < row_end;
  const int wpos_lo = g.w0 + min(frow0, row_end - 1) / group;
  const int wpos_hi = g.w0 + min(frow0 + 31, row_end - 1) / group;
  const bool row_ok = frow0 + n < row_end;
  const int frow = min(frow0 + n, row_end - 1);
  const int my_row = frow / group, head = hk * group + (frow - my_row * group);
  const int my_pos = g.w0 + my_row;

  f32x4 qreg[kQ];                                            // channels 8 j + 4 half .. + 3 of this lane's query
  {
    const float* qp = p.q + ((size_t(s) * p.m + my_row) * p.n_q_heads + head) * D + 4 * half;
#pragma unroll
    for (int j = 0; j < kQ; ++j) qreg[j] = *reinterpret_cast<const f32x4*>(qp + 8 * j);
  }
  f32x16 acc_o[kDb];
#pragma unroll
  for (int i = 0; i < kDb; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc_o[i][j] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;                      // running max (log2 units), this lane's share of the sum

  // LDS rows are split into 16-byte chunks, XOR-swizzled with a key made of the row so that 16
  // consecutive rows hit all banks: row % 16, or (row / 2) % 8 where two rows span the banks.
  auto k_key = [](int r) { return uint32_t(r & 15); };
  auto v_key = [](int r) { return uint32_t(kVRow == 256 ? r & 15 : (r >> 1) & 7); };
  constexpr int kKPer = 1024 / kKRow, kVPer = 1024 / kVRow;  // rows of a 1 KB piece (a wavefront's load)
  uint32_t gk[4], gv[4];                                     // byte offsets of this lane's loads inside a block's tile
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int kr = (4 * wave + i) * kKPer + lane / (64 / kKPer), kc = lane % (64 / kKPer);
    gk[i] = uint32_t(kr) * kKRow + ((uint32_t(kc) ^ k_key(kr)) << 4);
    const int vr = (4 * wave + i) * kVPer + lane / (64 / kVPer), vc = lane % (64 / kVPer);
    gv[i] = uint32_t(vr) * (kBlock * 4) + ((uint32_t(vc) ^ v_key(vr)) << 4);
  }
  const char* kbase = reinterpret_cast<const char*>(p.k_cache + size_t(s) * p.seq_stride);
  const char* vbase = reinterpret_cast<const char*>(p.v_cache + size_t(s) * p.seq_stride);
  auto tile_at = [&](int t, int& key0, int& lo, int& hi) {   // first key, and the visible span within the tile
    int block;
    tl.get(t / kPerBlock, block, lo, hi);
    key0 = block * kBlock + (t % kPerBlock) * kKeys;
    lo = max(lo, key0);
    hi = min(hi, key0 + kKeys);
    key0 = __builtin_amdgcn_readfirstlane(key0);
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
  };
  auto fetch_tile = [&](int key0, int stage) {
    constexpr uint32_t kBlockBytes = uint32_t(kBlock) * D * 4;
    const int block = key0 / kBlock, k0 = key0 % kBlock;
    const size_t off = (size_t(block) * p.n_kv_heads + hk) * kBlockBytes;
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(kbase + off), 0, kBlockBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vbase + off), 0, kBlockBytes, 0x00020000);
    char* dst = ff_lds + stage * 2 * kFfTileBytes + wave * 4096;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, gk[i], k0 * kKRow, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (__attribute__((address_space(3))) void*)(dst + kFfTileBytes + i * 1024), 16, gv[i], k0 * 4, 0, 0);
    }
  };

  int key0 = 0, lo = 0, hi = 0;
  if (t_begin < t_end) {
    tile_at(t_begin, key0, lo, hi);
    fetch_tile(key0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  for (int t = t_begin; t < t_end; ++t) {
    const int stage = (t - t_begin) & 1;
    int key_next = 0, lo_next = 0, hi_next = 0;
    if (t + 1 < t_end) tile_at(t + 1, key_next, lo_next, hi_next);
    // the wavefront skips tiles none of its rows can see; it masks tiles that are clipped or reach
    // past its first row's position
    const bool visible = wave_ok && hi > lo && lo <= wpos_hi;
    const bool masked = lo > key0 || hi < key0 + kKeys || hi - 1 > wpos_lo;
    const char* ks_ = ff_lds + stage * 2 * kFfTileBytes;
    const char* vs_ = ks_ + kFfTileBytes;
    f32x16 acc_s[kG];
    if (visible) {
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_s[gg][i] = 0.f;
#pragma unroll
      for (int j = 0; j < kQ; ++j) {
        f32x4 ka[kG];
#pragma unroll
        for (int gg = 0; gg < kG; ++gg)
          ka[gg] = *reinterpret_cast<const f32x4*>(ks_ + uint32_t(gg * 32 + n) * kKRow + ((uint32_t(2 * j + half) ^ k_key(n)) << 4));
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int gg = 0; gg < kG; ++gg)
            acc_s[gg] = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[gg][i], qreg[j][i], acc_s[gg], 0, 0, 0);
      }
    }
    // (the next tile is requested behind the score reads: see attn_prefill_mfma.hip)
    if (t + 1 < t_end) fetch_tile(key_next, stage ^ 1);
    if (visible) {
      if (masked) {
#pragma unroll
        for (int gg = 0; gg < kG; ++gg)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int kp = key0 + gg * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
            const bool ok = kp >= lo && kp < hi && kp <= my_pos;
            acc_s[gg][i] = ok ? acc_s[gg][i] : -INFINITY;
          }
      }
      float mx = acc_s[0][0];
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc_s[gg][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run, mx * p.scale_log2e);
      const float m_safe = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
      m_run = m_new;
      if (!__all(alpha == 1.f)) {
#pragma unroll
        for (int db = 0; db < kDb; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc_o[db][i] *= alpha;
        l_run *= alpha;
      }
      float psum = 0.f;
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          acc_s[gg][i] = __builtin_amdgcn_exp2f(fmaf(acc_s[gg][i], p.scale_log2e, -m_safe));
          psum += acc_s[gg][i];
        }
      l_run += psum;
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 va[kDb];
#pragma unroll
          for (int db = 0; db < kDb; ++db)
            va[db] = *reinterpret_cast<const f32x4*>(vs_ + uint32_t(db * 32 + n) * kVRow + ((uint32_t(gg * 8 + 2 * j + half) ^ v_key(n)) << 4));
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int db = 0; db < kDb; ++db)
              acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[db][i], acc_s[gg][4 * j + i], acc_o[db], 0, 0, 0);
        }
    }
    key0 = key_next;
    lo = lo_next;
    hi = hi_next;
    __builtin_amdgcn_s_waitcnt(0);   // this wavefront's pieces of the next tile have landed in LDS
    __syncthreads();
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (p.splits == 1) {
    if (row_ok) ff_store_row<D>(p, acc_o, m_run, l_tot, s, my_row, head, half);
    return;
  }
  // ---- a piece stores its unnormalised output in the order the registers hold it, plus its max and sum
  constexpr int kWords = D / 4 + 1;                          // 64-bit words per lane
  const size_t pieces0 = (size_t(qt) * p.n_kv_heads + hk) * p.splits;
  uint64_t* mine = p.part + ((pieces0 + split) * kFfWaves + wave) * (kWords * 64) + lane;
  auto pack = [](float a, float b) { return uint64_t(__float_as_uint(a)) | (uint64_t(__float_as_uint(b)) << 32); };
#pragma unroll
  for (int db = 0; db < kDb; ++db)
#pragma unroll
    for (int i = 0; i < 8; ++i) st_agent(mine + (db * 8 + i) * 64, pack(acc_o[db][2 * i], acc_o[db][2 * i + 1]));
  st_agent(mine + (kWords - 1) * 64, pack(m_run, l_tot));
  if (!last_of_group(p.counters + size_t(qt) * p.n_kv_heads + hk, unsigned(p.splits), &last_flag)) return;
  // ---- the last piece to finish merges them, in piece order:
  //   out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s
  const uint64_t* piece0 = p.part + (pieces0 * kFfWaves + wave) * (kWords * 64) + lane;
  constexpr size_t kPieceStride = size_t(kFfWaves) * kWords * 64;
  uint64_t ml[kFfMaxSplits];
#pragma unroll
  for (int i = 0; i < kFfMaxSplits; ++i)
    ml[i] = i < p.splits ? ld_agent(piece0 + i * kPieceStride + (kWords - 1) * 64) : pack(-INFINITY, 0.f);
  float m_all = -INFINITY;
#pragma unroll
  for (int i = 0; i < kFfMaxSplits; ++i) m_all = fmaxf(m_all, __uint_as_float(uint32_t(ml[i])));
  const float m_safe = m_all == -INFINITY ? 0.f : m_all;
  float l_all = 0.f;
#pragma unroll
  for (int db = 0; db < kDb; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc_o[db][i] = 0.f;
#pragma unroll
  for (int i = 0; i < kFfMaxSplits; ++i) {
    if (i < p.splits) {
      uint64_t raw[kWords - 1];
#pragma unroll
      for (int k = 0; k < kWords - 1; ++k) raw[k] = ld_agent(piece0 + i * kPieceStride + k * 64);
      const float w = __builtin_amdgcn_exp2f(__uint_as_float(uint32_t(ml[i])) - m_safe);
      l_all += w * __uint_as_float(uint32_t(ml[i] >> 32));
#pragma unroll
      for (int db = 0; db < kDb; ++db)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          acc_o[db][2 * k] += w * __uint_as_float(uint32_t(raw[db * 8 + k]));
          acc_o[db][2 * k + 1] += w * __uint_as_float(uint32_t(raw[db * 8 + k] >> 32));
        }
    }
  }
  if (row_ok) ff_store_row<D>(p, acc_o, m_all, l_all, s, my_row, head, half);
}

bool prefill_f32_supported(const actqkv_shape& sh, int m) { return sh.dtype == ACTQKV_F32 && m > 1; }

static int prefill_f32_qtiles(const actqkv_shape& sh, int m) {
  return (m * (sh.n_q_heads / sh.n_kv_heads) + kFfRows - 1) / kFfRows;
}

static int prefill_f32_slots(const actqkv_shape& sh) { return sh.head_dim == 64 ? kFfSlots<64> : kFfSlots<128>; }

// Pieces per query tile: as many as fill the chip, at most 8 (every piece is written and read once
// more by the merge).
static int prefill_f32_splits(const actqkv_shape& sh, int batch, int m) {
  const int items = batch * sh.n_kv_heads * prefill_f32_qtiles(sh, m);
  return std::min(std::max(prefill_f32_slots(sh) / items, 1), kFfMaxSplits);
}

// Partial results of this call, and the most any call with up to `batch` windows of up to `m` tokens needs.
static size_t prefill_f32_piece_bytes(const actqkv_shape& sh) { return sh.head_dim == 64 ? kFfPieceBytes<64> : kFfPieceBytes<128>; }
size_t prefill_f32_scratch_bytes(const actqkv_shape& sh, int batch, int m) {
  const int splits = prefill_f32_splits(sh, batch, m);
  return splits == 1 ? 0 : size_t(batch) * sh.n_kv_heads * prefill_f32_qtiles(sh, m) * splits * prefill_f32_piece_bytes(sh);
}
size_t prefill_f32_scratch_most(const actqkv_shape& sh, int batch, int m) {
  const size_t items = size_t(batch) * sh.n_kv_heads * prefill_f32_qtiles(sh, m);
  return std::min(size_t(prefill_f32_slots(sh)), items * kFfMaxSplits) * prefill_f32_piece_bytes(sh);
}

template <int D>
static int launch_ff(const FfParams& p, int grid, hipStream_t stream) {
  static std::mutex mu;
  static bool attr_set = false;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!attr_set) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_prefill_f32_kernel<D>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, kFfLdsBytes);
      if (e != hipSuccess) return set_error(ACTQKV_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
      attr_set = true;
    }
  }
  hipLaunchKernelGGL(attn_prefill_f32_kernel<D>, dim3(grid), dim3(kFfThreads), kFfLdsBytes, stream, p);
  return hip_status("attention (prefill, fp32)");
}

int launch_attention_prefill_f32(const actqkv_shape& sh, int batch, int m, const void* q, const void* k_cache,
                                 const void* v_cache, int64_t seq_stride, int nb_capacity, const int32_t* n_ctx,
                                 const int32_t* idx, const int32_t* n_sel, int k_cap, void* out, float* lse,
                                 float* scratch, unsigned int* counters, float scale, int sel_per_head,
                                 hipStream_t stream) {
  FfParams p;
  p.q = static_cast<const float*>(q);
  p.k_cache = static_cast<const float*>(k_cache);
  p.v_cache = static_cast<const float*>(v_cache);
  p.seq_stride = seq_stride;
  p.nb_capacity = nb_capacity;
  p.n_ctx = n_ctx;
  p.idx = idx;
  p.n_sel = n_sel;
  p.k_cap = k_cap;
  p.out = static_cast<float*>(out);
  p.lse = lse;
  p.part = reinterpret_cast<uint64_t*>(scratch);
  p.counters = counters;
  p.m = m;
  p.n_q_heads = sh.n_q_heads;
  p.n_kv_heads = sh.n_kv_heads;
  p.n_init = sh.n_init;
  p.n_local = sh.n_local;
  p.n_qtiles = prefill_f32_qtiles(sh, m);
  p.splits = prefill_f32_splits(sh, batch, m);
  p.sel_per_head = sel_per_head;
  p.scale_log2e = scale * 1.4426950408889634f;
  const int64_t items = int64_t(batch) * sh.n_kv_heads * p.n_qtiles;
  if (p.splits > 1 && items > int64_t(kTicketCounters))
    return set_error(ACTQKV_EINVAL, "prefill attention: more split query tiles than ticket counters");
  if (items * p.splits > int64_t(INT32_MAX))
    return set_error(ACTQKV_ESHAPE, "prefill attention: %lld query tiles in a call", (long long)items);
  const int grid = int(items * p.splits);
  return sh.head_dim == 64 ? launch_ff<64>(p, grid, stream) : launch_ff<128>(p, grid, stream);
}

}  // namespace actqkv
