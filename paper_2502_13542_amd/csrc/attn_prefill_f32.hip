// Retrieval attention of a prefill window in fp32 (Sec. 3.1, Eq. (2)): fp32 storage, and results as close to the exact
// ones as fp32 products and sums give them, or closer.
//
// The fp32 matrix instruction does 256 operations per clock and compute unit, a sixteenth of the 16-bit one.  So a value
// enters as three bf16 parts, each what rounding to bf16 left of the one before: 8 + 8 + 8 bits are all of its 24, and
// bf16 has the exponents of fp32, so the parts together ARE the value, whatever lies beside it (from 2^-109 on, smaller
// ones to 2^-134; a query row enters times the softmax scale, to 2^-26).  A product is six of the nine products of parts,
// exact each, summed in fp32, small ones first; the three left out are below 2^-24 of it together, half a unit of its last
// place.  Two f16 halves and three products are faster (32 windows of 256 tokens 102 us, 146 so), but hold 23 bits, and
// those only of values near the largest that shares their factor: not taken.  Values above the largest bf16, infinite ones
// among them, have no parts: where a tile has one its scores are taken again, or its large values added, in fp32 products.
// Relative error against 64 bits, normal inputs, 64 channels: 32 windows of 256 tokens 6.4e-7 (fp32 products 7.6e-7), one
// such window 3.3e-7 (4.2e-7), one of 4096 tokens 8.4e-7 (9.8e-7); 128 channels 6.8e-7 (8.1e-7), 4.0e-7 (4.9e-7), 1.18e-6 (1.37e-6).
//
// A workgroup of 4 wavefronts owns 128 query rows that share a KV head (numbered position by position, the G heads side
// by side), a wavefront 32 of them.  A tile is 4096 / D keys, 16 KB of keys and 16 KB of values: every wavefront brings a
// quarter of each into registers while the tile before is worked on, and cuts it into parts in LDS (48 KB, one tile) between
// two barriers.  Two workgroups share a compute unit, so a SIMD has a second wavefront while the first is in its softmax
// or at a barrier.  What bounds it: 96 matrix instructions per tile and wavefront and six vector ones beside each, which a
// wavefront hardly overlaps with its own matrix ones; the matrix pipe is busy in 63 % of the cycles (32 windows of 256 tokens).
//
// S^T = K Q^T leaves a lane with scores of ONE query (column lane % 32).  Bits 2 and 3 of a key's number within 16 change
// places on the way into the first product, so that register i of lane half h holds key 16 (i / 8) + 8 h + i % 8 of a
// 32-key group: 8 registers are the B operand of a 16-key step of O^T += V^T P^T, without a lane exchange.
//
// A single window has few query tiles; then the key tiles are cut into pieces, one workgroup each, which a second launch
// merges.  64 channels, 8 query and 2 KV heads, 8 blocks retrieved, against fp32 products with the merge in the last
// workgroup: 32 windows of 256 tokens 218 -> 146 us, one of them 57 -> 22, of 4096 tokens 301 -> 179; 128 channels, 32
// windows 427 -> 296.
#include <algorithm>
#include <mutex>

#include "common.h"
#include "launch.h"
#include "select_body.h"

namespace actqkv {

constexpr int kFfThreads = 256;
constexpr int kFfWaves = 4;
constexpr int kFfRows = 32 * kFfWaves;            // query rows of a workgroup
constexpr int kFfPart = 8192;                     // one of the three parts of K or V^T of a tile
constexpr int kFfLdsBytes = 6 * kFfPart;
constexpr float kFfMax = 3.3895314e38f;           // the largest bf16: what is larger has no parts
// Workgroups of a full launch: two per compute unit; with 128 channels a little less, so that their
// partial results fit the library's own scratch array.
template <int D> constexpr int kFfSlots = D == 64 ? 512 : 480;
template <int D> constexpr size_t kFfPieceBytes = size_t(kFfWaves) * (D / 2 + 2) * 64 * 4;
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
  float* part;             // [query tile and KV head][piece][wavefront][D / 8 x 4 of O | (max, sum)][64 lanes]
  int m, n_q_heads, n_kv_heads, n_init, n_local, n_qtiles, splits;
  int per_chip;            // query tiles whose workgroups make one for every compute unit
  int sel_per_head;
  float scale_log2e;
  SelectInside sel;        // one sequence: its selection is made here
};

// Two fp32 values -> their three parts, packed.  What is left of a value after a part is exact.
__device__ __forceinline__ void ff_split(float x0, float x1, uint32_t (&part)[3]) {
  part[0] = pack_bf16x2(x0, x1);
  x0 -= bf16_lo(part[0]), x1 -= bf16_hi(part[0]);
  part[1] = pack_bf16x2(x0, x1);
  x0 -= bf16_lo(part[1]), x1 -= bf16_hi(part[1]);
  part[2] = pack_bf16x2(x0, x1);
}
// The same of the values times scale, to 2^-26 of them.
__device__ __forceinline__ void ff_split_scaled(float x0, float x1, float scale, uint32_t (&part)[3]) {
  part[0] = pack_bf16x2(x0 * scale, x1 * scale);
  x0 = fmaf(x0, scale, -bf16_lo(part[0])), x1 = fmaf(x1, scale, -bf16_hi(part[0]));
  part[1] = pack_bf16x2(x0, x1);
  x0 -= bf16_lo(part[1]), x1 -= bf16_hi(part[1]);
  part[2] = pack_bf16x2(x0, x1);
}
__device__ __forceinline__ bf16x8 ff_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ f32x16 ff_mfma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// The six products of a step, small ones first: part kFfOf[i][0] of one factor, kFfOf[i][1] of the other.
constexpr int kFfProducts = 6;
constexpr int kFfOf[kFfProducts][2] = {{2, 0}, {1, 1}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};

// What wavefront `wave` of piece `split` of a (query tile, KV head) leaves: D / 2 floats of output per lane, then (max, sum).
template <int D>
__device__ __forceinline__ float* ff_piece(const FfParams& p, int item, int split, int wave) {
  return p.part + ((size_t(item) * p.splits + split) * kFfWaves + wave) * ((D / 2 + 2) * 64);
}

// Final normalisation and store of one lane's share of a query row.
template <int D>
__device__ __forceinline__ void ff_store_row(const FfParams& p, const f32x16 (&acc_o)[D / 32], float m_run,
                                             float l_tot, int s, int row, int head, int half) {
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
  constexpr int kKeys = 4096 / D;                   // keys of a tile: 64 or 32
  constexpr int kPerBlock = kBlock / kKeys;
  constexpr int kG = kKeys / 32, kDb = D / 32, kQ = D / 16;
  constexpr uint32_t kKRow = D * 2, kVRow = kKeys * 2;   // bytes of a K / V^T row in one of its parts in LDS
  extern __shared__ __attribute__((aligned(16))) char ff_lds[];   // three parts of K, three of V^T
  // whether a wavefront brought values above kFfMax: [K, V^T][wavefront]
  __shared__ __attribute__((aligned(16))) uint32_t no_parts[2][kFfWaves];
  __shared__ int32_t idx_lds[64];
  __shared__ SelectWaveLds sel_lds;
  __shared__ int sel_count;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, half = lane >> 5;
  const int group = p.n_q_heads / p.n_kv_heads;
  // consecutive workgroups differ in the KV head (they go round the XCDs: a head's tiles stay in few L2s)
  const int hk = blockIdx.x % p.n_kv_heads, rest = blockIdx.x / p.n_kv_heads;
  const int split = rest % p.splits, qt = rest / p.splits;
  const int s = qt / p.n_qtiles;
  int qtile = qt % p.n_qtiles;
  // The last rows of a window see up to a window more keys than the first: the two workgroups that share a compute unit
  // (per_chip query tiles apart) take them in opposite orders.  A window of 4096 tokens 198 -> 180 us, four of 1024 110 -> 103.
  if (p.per_chip >= p.n_qtiles) {
    if ((s * p.n_qtiles / p.per_chip) & 1) qtile = p.n_qtiles - 1 - qtile;
  } else {
    const int turn = qtile / p.per_chip;
    if ((turn & 1) && (turn + 1) * p.per_chip <= p.n_qtiles) qtile = (2 * turn + 1) * p.per_chip - 1 - qtile;
  }

  // (the last wavefront selects before it asks for anything else; the others have the first tile and their queries on the way)
  const bool inside = p.sel.scores != nullptr;
  const size_t sel_row = p.sel_per_head ? size_t(s) * p.n_kv_heads + hk : size_t(s);
  const int32_t my_idx = !inside && tid < p.k_cap ? p.idx[sel_row * p.k_cap + tid] : -1;
  const int n_ctx_raw = p.n_ctx[s];
  int n_sel_raw = inside ? 0 : p.n_sel[sel_row];
  if (inside && wave == kFfWaves - 1) p.sel.run(p.k_cap, blockIdx.x == 0, sel_lds, idx_lds, &sel_count);
  const int n_ctx = min(max(n_ctx_raw, p.m), p.nb_capacity * kBlock);
  const WindowGeom g = window_geom(n_ctx, p.m, p.n_init, p.n_local);
  const int row_end = p.m * group;
  const int row_hi = (min((qtile + 1) * kFfRows, row_end) - 1) / group;
  const int frow0 = qtile * kFfRows + wave * 32;             // first query row of this wavefront
  const bool wave_ok = frow0 < row_end;
  const int wpos_lo = g.w0 + min(frow0, row_end - 1) / group;
  const int wpos_hi = g.w0 + min(frow0 + 31, row_end - 1) / group;
  const bool row_ok = frow0 + n < row_end;
  const int frow = min(frow0 + n, row_end - 1);
  const int my_row = frow / group, head = hk * group + (frow - my_row * group);
  const int my_pos = g.w0 + my_row;

  // ---- tiles: a wavefront brings a quarter of the rows of K and of V^T into registers, 4 x 1 KB each
  constexpr int kKPer = 1024 / (4 * D), kVPer = 1024 / (4 * kKeys);   // rows of 1 KB in memory
  const int kc = lane % (64 / kKPer), vc = lane % (64 / kVPer);       // 16-byte piece of a row
  const int kr0 = wave * (kKeys / 4) + lane / (64 / kKPer), vr0 = wave * (D / 4) + lane / (64 / kVPer);
  const uint32_t gk = uint32_t(kr0) * (4 * D) + kc * 16, gv = uint32_t(vr0) * (4 * kBlock) + vc * 16;
  // LDS rows are split into 16-byte chunks, XOR-swizzled with a key made of the row so that 16 rows that
  // are read together hit all banks.
  auto k_key = [](int r) { return uint32_t(D == 64 ? (r >> 1) & 7 : r & 15); };
  auto v_key = [](int r) { return uint32_t(D == 64 ? (r >> 1) & 7 : (r >> 2) & 3); };
  uint32_t wk[4], wv[4];                                     // where this lane's pieces go in a part
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int kr = kr0 + i * kKPer, vr = vr0 + i * kVPer;
    wk[i] = uint32_t(kr) * kKRow + ((uint32_t(kc >> 1) ^ k_key(kr)) << 4) + 8 * (kc & 1);
    wv[i] = uint32_t(vr) * kVRow + ((uint32_t(vc >> 1) ^ v_key(vr)) << 4) + 8 * (vc & 1);
  }
  const char* kbase = reinterpret_cast<const char*>(p.k_cache + size_t(s) * p.seq_stride);
  const char* vbase = reinterpret_cast<const char*>(p.v_cache + size_t(s) * p.seq_stride);
  constexpr uint32_t kBlockBytes = uint32_t(kBlock) * D * 4;
  struct Tile { int key0, lo, hi; };                         // first key, and the visible span within the tile
  auto block_offset = [&](int key0) { return (size_t(key0 / kBlock) * p.n_kv_heads + hk) * kBlockBytes; };
  f32x4 xk[4], xv[4];                                        // a tile on its way
  auto fetch_tile = [&](const Tile& t) {
    const size_t off = block_offset(t.key0);
    const int k0 = t.key0 % kBlock;
    const char* kp = kbase + off + size_t(k0) * (4 * D) + gk;
    const char* vp = vbase + off + size_t(k0) * 4 + gv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      xk[i] = *reinterpret_cast<const f32x4*>(kp + i * 1024);
      xv[i] = *reinterpret_cast<const f32x4*>(vp + i * kVPer * (4 * kBlock));
    }
  };
  auto too_large = [&](const f32x4 (&x)[4]) {                // whether any of the wavefront's values is (NaN is not)
    float mx = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; j += 2) mx = fmaxf(fmaxf(fabsf(x[i][j]), fabsf(x[i][j + 1])), mx);
    return __any(mx > kFfMax) != 0;
  };
  // the tile in registers -> LDS, in parts; keys that no row of the workgroup sees count as zeros
  auto store_tile = [&](const Tile& t) {
    if (t.lo > t.key0 || t.hi < t.key0 + kKeys) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kp = t.key0 + kr0 + i * kKPer, vp = t.key0 + 4 * vc;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          xk[i][j] = kp >= t.lo && kp < t.hi ? xk[i][j] : 0.f;
          xv[i][j] = vp + j >= t.lo && vp + j < t.hi ? xv[i][j] : 0.f;
        }
      }
    }
    const bool k_large = too_large(xk), v_large = too_large(xv);
    if (__builtin_expect(v_large, 0)) {                      // the others; these are added by the reader
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) xv[i][j] = fabsf(xv[i][j]) > kFfMax ? 0.f : xv[i][j];
    }
    if (lane == 0) {
      no_parts[0][wave] = k_large;
      no_parts[1][wave] = v_large;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t a[3], b[3];
      ff_split(xk[i][0], xk[i][1], a);
      ff_split(xk[i][2], xk[i][3], b);
#pragma unroll
      for (int c = 0; c < 3; ++c) *reinterpret_cast<u32x2*>(ff_lds + c * kFfPart + wk[i]) = u32x2{a[c], b[c]};
      ff_split(xv[i][0], xv[i][1], a);
      ff_split(xv[i][2], xv[i][3], b);
#pragma unroll
      for (int c = 0; c < 3; ++c) *reinterpret_cast<u32x2*>(ff_lds + (3 + c) * kFfPart + wv[i]) = u32x2{a[c], b[c]};
    }
  };

  // the first piece begins with the initial tokens, whatever is selected
  Tile now{0, 0, 0};
  const bool early = split == 0 && g.i0 > 0;
  if (early) fetch_tile(now);
  // ---- the queries: channels 16 j + 8 half .. + 7 of this lane's row times scale_log2e, in parts: scores come in units of log2
  // then, and that of the key with the maximum less the maximum is 0 (fmaf(score, scale_log2e, -maximum) is not)
  const float* qrow = p.q + ((size_t(s) * p.m + my_row) * p.n_q_heads + head) * D;
  u32x4 qp[3][kQ];
  bool q_large;
  {
    f32x4 x[2 * kQ];
    float mx = 0.f;
#pragma unroll
    for (int j = 0; j < kQ; ++j) {
      x[2 * j] = *reinterpret_cast<const f32x4*>(qrow + 16 * j + 8 * half);
      x[2 * j + 1] = *reinterpret_cast<const f32x4*>(qrow + 16 * j + 8 * half + 4);
    }
#pragma unroll
    for (int j = 0; j < 2 * kQ; ++j)
#pragma unroll
      for (int i = 0; i < 4; i += 2) mx = fmaxf(fmaxf(fabsf(x[j][i]), fabsf(x[j][i + 1])), mx);
    q_large = __any(mx > kFfMax || mx * p.scale_log2e > kFfMax);
#pragma unroll
    for (int j = 0; j < kQ; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t part[3];
        ff_split_scaled(x[2 * j + (i >> 1)][2 * (i & 1)], x[2 * j + (i >> 1)][2 * (i & 1) + 1], p.scale_log2e, part);
#pragma unroll
        for (int c = 0; c < 3; ++c) qp[c][j][i] = part[c];
      }
  }
  if (!inside && tid < 64) idx_lds[tid] = my_idx;
  __syncthreads();
  if (inside) n_sel_raw = sel_count;
  const TileList tl = make_tile_list(g, g.w0 + row_hi, idx_lds, n_sel_raw, p.k_cap, p.nb_capacity);
  const int n_tiles = tl.count() * kPerBlock;
  const int per = (n_tiles + p.splits - 1) / p.splits;
  const int t_begin = split * per, t_end = min(n_tiles, t_begin + per);
  auto tile_at = [&](int t) {
    int block, lo, hi;
    tl.get(t / kPerBlock, block, lo, hi);
    const int key0 = block * kBlock + (t % kPerBlock) * kKeys;
    return Tile{__builtin_amdgcn_readfirstlane(key0), __builtin_amdgcn_readfirstlane(max(lo, key0)),
                __builtin_amdgcn_readfirstlane(min(hi, key0 + kKeys))};
  };
  if (t_begin < t_end) {
    now = tile_at(t_begin);
    if (!early) fetch_tile(now);
  }
  f32x16 acc_o[kDb];
#pragma unroll
  for (int i = 0; i < kDb; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc_o[i][j] = 0.f;
  // the row's maximum (log2 units), this lane's share of the sum
  float m_run = -INFINITY, l_run = 0.f;

  const int kn = (n & 0x13) | ((n & 4) << 1) | ((n & 8) >> 1);   // the key of this lane's row in the first product
  for (int t = t_begin; t < t_end; ++t) {
    const int key0 = now.key0, lo = now.lo, hi = now.hi;
    if (t > t_begin) __syncthreads();                        // everybody is done with the tile before
    store_tile(now);
    __syncthreads();
    if (t + 1 < t_end) {
      now = tile_at(t + 1);
      fetch_tile(now);
    }
    // the wavefront skips tiles none of its rows can see; it masks tiles that are clipped or reach
    // past its first row's position
    const bool visible = wave_ok && hi > lo && lo <= wpos_hi;
    const bool masked = lo > key0 || hi < key0 + kKeys || hi - 1 > wpos_lo;
    if (!visible) continue;
    bool k_large = q_large, v_large = false;
    {
      const u32x4 of_k = *reinterpret_cast<const u32x4*>(no_parts[0]), of_v = *reinterpret_cast<const u32x4*>(no_parts[1]);
      k_large |= __any((of_k.x | of_k.y | of_k.z | of_k.w) != 0u);
      v_large = __any((of_v.x | of_v.y | of_v.z | of_v.w) != 0u);
    }
    f32x16 acc_s[kG];
#pragma unroll
    for (int gg = 0; gg < kG; ++gg)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc_s[gg][i] = 0.f;
    bf16x8 kp[2][3][kG];                                     // a step's operands are requested a step ahead
    auto read_k = [&](int j) {
#pragma unroll
      for (int gg = 0; gg < kG; ++gg) {
        const char* at = ff_lds + uint32_t(gg * 32 + kn) * kKRow + ((uint32_t(2 * j + half) ^ k_key(kn)) << 4);
#pragma unroll
        for (int c = 0; c < 3; ++c) kp[j & 1][c][gg] = ff_bf16x8(*reinterpret_cast<const u32x4*>(at + c * kFfPart));
      }
    };
    read_k(0);
#pragma unroll
    for (int j = 0; j < kQ; ++j) {
      if (j + 1 < kQ) read_k(j + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kFfProducts; ++i)
#pragma unroll
        for (int gg = 0; gg < kG; ++gg)
          acc_s[gg] = ff_mfma(kp[j & 1][kFfOf[i][0]][gg], ff_bf16x8(qp[kFfOf[i][1]][j]), acc_s[gg]);
    }
    if (__builtin_expect(k_large, 0)) {
      // a key or query without parts: the scores anew in fp32 products, from memory
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_s[gg][i] = 0.f;
      const float* kt = reinterpret_cast<const float*>(kbase + block_offset(key0)) + size_t(key0 % kBlock + kn) * D + half;
#pragma unroll 1
      for (int c = 0; c < D; c += 2)
#pragma unroll
        for (int gg = 0; gg < kG; ++gg)
          acc_s[gg] = __builtin_amdgcn_mfma_f32_32x32x2f32(kt[gg * 32 * D + c], qrow[c + half], acc_s[gg], 0, 0, 0);
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_s[gg][i] *= p.scale_log2e;
    }
    if (masked) {
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int kpos = key0 + gg * 32 + 16 * (i >> 3) + 8 * half + (i & 7);
          const bool ok = kpos >= lo && kpos < hi && kpos <= my_pos;
          acc_s[gg][i] = ok ? acc_s[gg][i] : -INFINITY;
        }
    }
    float mx = acc_s[0][0];
#pragma unroll
    for (int gg = 0; gg < kG; ++gg)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc_s[gg][i]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // (every lane takes the same branch.  A reference that lags behind by up to 2^8 is 1 to 3 % faster, but probabilities
    // above 1 overflow sums over values near the largest fp32)
    if (!__all(mx <= m_run)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
      m_run = m_new;
#pragma unroll
      for (int db = 0; db < kDb; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_o[db][i] *= alpha;
      l_run *= alpha;
    }
    const float m_safe = m_run == -INFINITY ? 0.f : m_run;
    float psum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int gg = 0; gg < kG; ++gg)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc_s[gg][i] = __builtin_amdgcn_exp2f(acc_s[gg][i] - m_safe);
        psum[i & 3] += acc_s[gg][i];
      }
    l_run += (psum[0] + psum[1]) + (psum[2] + psum[3]);
#pragma unroll
    for (int st = 0; st < 2 * kG; ++st) {
      u32x4 pp[3];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t part[3];
        ff_split(acc_s[st >> 1][8 * (st & 1) + 2 * i], acc_s[st >> 1][8 * (st & 1) + 2 * i + 1], part);
#pragma unroll
        for (int c = 0; c < 3; ++c) pp[c][i] = part[c];
      }
#pragma unroll
      for (int d0 = 0; d0 < kDb; d0 += 2) {
        bf16x8 vp[3][2];
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          const char* at = ff_lds + 3 * kFfPart + uint32_t((d0 + db) * 32 + n) * kVRow + ((uint32_t(2 * st + half) ^ v_key(n)) << 4);
#pragma unroll
          for (int c = 0; c < 3; ++c) vp[c][db] = ff_bf16x8(*reinterpret_cast<const u32x4*>(at + c * kFfPart));
        }
#pragma unroll
        for (int i = 0; i < kFfProducts; ++i)
#pragma unroll
          for (int db = 0; db < 2; ++db)
            acc_o[d0 + db] = ff_mfma(vp[kFfOf[i][0]][db], ff_bf16x8(pp[kFfOf[i][1]]), acc_o[d0 + db]);
      }
    }
    if (__builtin_expect(v_large, 0)) {
      // values without parts went in as zeros; their products in fp32, from memory
      const float* vt = reinterpret_cast<const float*>(vbase + block_offset(key0)) + size_t(n) * kBlock + key0 % kBlock;
#pragma unroll
      for (int gg = 0; gg < kG; ++gg)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int k = gg * 32 + 16 * (i >> 3) + 8 * half + (i & 7);
          const bool seen = key0 + k >= lo && key0 + k < hi;
#pragma unroll
          for (int db = 0; db < kDb; ++db) {
            const float x = vt[db * 32 * kBlock + k];
            acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(seen && fabsf(x) > kFfMax ? x : 0.f, acc_s[gg][i], acc_o[db], 0, 0, 0);
          }
        }
    }
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (p.splits == 1) {
    if (row_ok) ff_store_row<D>(p, acc_o, m_run, l_tot, s, my_row, head, half);
    return;
  }
  // ---- a piece stores its unnormalised output in the order the registers hold it, plus its max and sum
  float* mine = ff_piece<D>(p, (s * p.n_qtiles + qtile) * p.n_kv_heads + hk, split, wave);
#pragma unroll
  for (int db = 0; db < kDb; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4*>(mine + ((db * 4 + j) * 64 + lane) * 4) =
          f32x4{acc_o[db][4 * j], acc_o[db][4 * j + 1], acc_o[db][4 * j + 2], acc_o[db][4 * j + 3]};
  *reinterpret_cast<f32x2*>(mine + (D / 2) * 64 + lane * 2) = f32x2{m_run, l_tot};
}

// The pieces of a query tile, in their order:  out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s.
// grid (4 wavefronts' rows of every query tile and KV head); a wavefront here takes a quarter of the channels of the
// 32 rows.  A launch of its own: the last of 8 pieces to finish needed 31 us to read the others' 256 KB back (one
// compute unit gets 8 GB/s of coherent 8-byte loads), with fp32 products a window of 256 tokens 57 us, so 33 of them.
template <int D>
__global__ __launch_bounds__(256) void attn_prefill_f32_merge_kernel(FfParams p) {
  constexpr int kSlots = D / 32;                             // 16-byte groups of a lane here
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int n = lane & 31, half = lane >> 5, group = p.n_q_heads / p.n_kv_heads;
  const int wave = blockIdx.x % kFfWaves, item = blockIdx.x / kFfWaves;
  const int hk = item % p.n_kv_heads, qt = item / p.n_kv_heads, qtile = qt % p.n_qtiles, s = qt / p.n_qtiles;
  const int frow = qtile * kFfRows + wave * 32 + n;
  f32x2 ml[kFfMaxSplits];
  f32x4 o[kFfMaxSplits][kSlots];
#pragma unroll
  for (int i = 0; i < kFfMaxSplits; ++i) {                   // all loads first: they overlap
    const float* piece = ff_piece<D>(p, item, min(i, p.splits - 1), wave);
    ml[i] = *reinterpret_cast<const f32x2*>(piece + (D / 2) * 64 + lane * 2);
#pragma unroll
    for (int k = 0; k < kSlots; ++k) o[i][k] = *reinterpret_cast<const f32x4*>(piece + ((part * kSlots + k) * 64 + lane) * 4);
  }
  float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int i = 0; i < kFfMaxSplits; ++i) m_all = fmaxf(m_all, i < p.splits ? ml[i].x : -INFINITY);
  const float m_safe = m_all == -INFINITY ? 0.f : m_all;
  f32x4 sum[kSlots];
#pragma unroll
  for (int k = 0; k < kSlots; ++k) sum[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < kFfMaxSplits; ++i) {
    if (i < p.splits) {
      const float w = __builtin_amdgcn_exp2f(ml[i].x - m_safe);
      l_all += w * ml[i].y;
#pragma unroll
      for (int k = 0; k < kSlots; ++k) sum[k] += w * o[i][k];
    }
  }
  if (frow >= p.m * group) return;
  const int row = frow / group, head = hk * group + (frow - row * group);
  const float inv = l_all > 0.f ? 1.f / l_all : 0.f;
  float* op = p.out + ((size_t(s) * p.m + row) * p.n_q_heads + head) * D + 4 * half;
#pragma unroll
  for (int k = 0; k < kSlots; ++k) *reinterpret_cast<f32x4*>(op + 8 * (part * kSlots + k)) = sum[k] * inv;
  if (p.lse != nullptr && half == 0 && part == 0)
    p.lse[(size_t(s) * p.n_q_heads + head) * p.m + row] = (m_all + log2f(l_all)) * 0.6931471805599453f;
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
  if (p.splits > 1)
    hipLaunchKernelGGL(attn_prefill_f32_merge_kernel<D>, dim3(grid / p.splits * kFfWaves), dim3(256), 0, stream, p);
  return hip_status("attention (prefill, fp32)");
}

int launch_attention_prefill_f32(const actqkv_shape& sh, int batch, int m, const void* q, const void* k_cache,
                                 const void* v_cache, int64_t seq_stride, int nb_capacity, const int32_t* n_ctx,
                                 const int32_t* idx, const int32_t* n_sel, int k_cap, void* out, float* lse,
                                 float* scratch, float scale, int sel_per_head,
                                 hipStream_t stream, const SelectInside* inside) {
  FfParams p;
  if (inside != nullptr) p.sel = *inside;
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
  p.part = scratch;
  p.m = m;
  p.n_q_heads = sh.n_q_heads;
  p.n_kv_heads = sh.n_kv_heads;
  p.n_init = sh.n_init;
  p.n_local = sh.n_local;
  p.n_qtiles = prefill_f32_qtiles(sh, m);
  p.splits = prefill_f32_splits(sh, batch, m);
  p.per_chip = std::max(kChipCus / (sh.n_kv_heads * p.splits), 1);
  p.sel_per_head = sel_per_head;
  p.scale_log2e = scale * 1.4426950408889634f;
  const int64_t items = int64_t(batch) * sh.n_kv_heads * p.n_qtiles;
  if (items * p.splits > int64_t(INT32_MAX))
    return set_error(ACTQKV_ESHAPE, "prefill attention: %lld query tiles in a call", (long long)items);
  const int grid = int(items * p.splits);
  return sh.head_dim == 64 ? launch_ff<64>(p, grid, stream) : launch_ff<128>(p, grid, stream);
}

}  // namespace actqkv
