// Retrieval attention of a prefill window on the matrix cores
// (Sec. 3.1, Eq. (2): O^t = Attention(Q^t, [K^t, K*], [V^t, V*]); bf16 storage, fp32 accumulation).
//
// Work split.  A workgroup of 8 wavefronts owns 256 / KS query rows that share one KV
// head, 32 of them for KS wavefronts (KS = 1, 2 or 4), which share the keys of every tile and merge
// in LDS at the end; prefill_splits says when.  The rows are numbered position by position with
// the G heads of the KV head side by side, so every group size fills the wavefronts (with a
// wavefront per head, seven heads left one of eight idle: 1.92 instead of 1.87 ms for a pass over
// 50001 tokens).  The key tiles of the window - initial tokens, the blocks chosen by
// actqkv_select (read from device memory), the local span and the causal part of the window -
// form one list of 128-key blocks; it is cut into `splits` contiguous pieces, one workgroup
// each, so that a 512-token window still fills all 256 compute units; the workgroup that
// finishes last among the pieces of a query tile merges them, or, of many pieces, a second launch.  Workgroups of one
// KV head sit on one XCD (blockIdx % Hk picks the head), so that head's gathered
// tiles stay in that XCD's L2.
//
// Data flow per tile.  K [128 keys][D] and V^T [D][128 keys] (D = 64 or 128 channels) go from HBM
// straight into LDS (buffer_load_dwordx4 ... lds, double buffered, 16-byte chunks XOR-swizzled with
// the row index so that operand reads of 16 consecutive rows hit all 64 banks).  A 16x16x32 tiling
// with one wavefront per SIMD and no key splits was measured and rejected: one wavefront
// can only issue a 1 KB LDS operand read every ~35 cycles, which caps a 16-cycle MFMA per
// read at ~40 % and left that variant at 0.4 PFLOP/s.  Each wavefront computes S^T = K Q^T with
// v_mfma_f32_32x32x16_bf16 (A = K rows from LDS, B = Q^T kept in registers), so a
// lane ends up holding scores of ONE query: the softmax needs no cross-lane work
// except one exchange between the two half-waves, and the probabilities are
// already in the register layout the next product wants as its B operand:
// O^T += V^T P^T (A = V^T rows from LDS).  To make that work the K rows are fed in
// a permuted order (bits 2 and 3 of the row index swapped); the permutation is
// undone for free because a lane's 8 consecutive accumulator registers then hold
// 8 consecutive keys.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "common.h"
#include "launch.h"
#include "select_body.h"

namespace actqkv {

constexpr int kPfThreads = 512;
constexpr int kPfWaves = 8;
// Whether key tiles may be cut into pieces: fp32 partial results of a whole query tile with 128 channels would be
// twice kPfPartialFloats (and 256 of them more than the library's own scratch array holds).
template <int D, int KS, bool kTwoTermP> constexpr bool kPfPieces = D == 64 || KS > 1 || !kTwoTermP;
template <int KS> constexpr int kPfRows = 32 * kPfWaves / KS;   // query rows of a workgroup
template <int D> constexpr int kPfTileBytes = kBlock * D * 2;           // one K or V^T tile of a (block, KV head)
template <int D> constexpr int kPfLdsBytes = 2 * 2 * kPfTileBytes<D>;   // 2 stages x (K, V^T)
constexpr int kMaxPfSplits = 8;
constexpr int kMergeWaves = 2;                       // wavefronts of a workgroup of the merge launch
constexpr float kLazyMaxLog2 = 8.f;                  // how far a tile's maximum may exceed the reference one
constexpr int kPfOrderMax = 64;                      // batch entries the queue hands out longest first
// Index of the "left" counter behind the per-head queue counters: 16384 channels in heads of 64 are 256 KV heads.
// It is the first of the decode layer's counters; every launch leaves both at zero, and calls that share a workspace
// are ordered.
constexpr int kPfQueueDone = 256;
static_assert(kPfQueueDone + 1 <= kSeqCounterOffset - kTicketCounters + kSeqCounters, "queue counters");

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// sum += the eight bf16 values of a packed operand (as fp32): four dot products of a pair with
// (1, 1).  (Written as assembly: the compiler's builtin for this instruction takes the first
// pair of a packed vector whatever element is asked for.)
__device__ __forceinline__ void add_bf16x8(float& sum, bf16x8 v, uint32_t ones) {
  const u32x4 w = __builtin_bit_cast(u32x4, v);
  asm("v_dot2c_f32_bf16 %0, %1, %2" : "+v"(sum) : "v"(w.x), "v"(ones));
  asm("v_dot2c_f32_bf16 %0, %1, %2" : "+v"(sum) : "v"(w.y), "v"(ones));
  asm("v_dot2c_f32_bf16 %0, %1, %2" : "+v"(sum) : "v"(w.z), "v"(ones));
  asm("v_dot2c_f32_bf16 %0, %1, %2" : "+v"(sum) : "v"(w.w), "v"(ones));
}

// 8 fp32 -> 8 bf16 (round to nearest even), packed as an MFMA operand
__device__ __forceinline__ bf16x8 pack8(float a0, float a1, float a2, float a3, float a4, float a5,
                                        float a6, float a7) {
  typedef __attribute__((ext_vector_type(8))) float f32x8;
  f32x8 v = {a0, a1, a2, a3, a4, a5, a6, a7};
  return __builtin_convertvector(v, bf16x8);
}

// A pointer that is the same in all lanes, pinned to scalar registers (so that adding a
// 32-bit lane offset to it becomes the scalar-base addressing mode of the load).
__device__ __forceinline__ const char* uniform_ptr(const char* ptr) {
  const uint64_t v = reinterpret_cast<uint64_t>(ptr);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
  return reinterpret_cast<const char*>((uint64_t(hi) << 32) | lo);
}

// MFMA row -> key row inside a 32-key group: swap bits 2 and 3.
__device__ __forceinline__ int perm_row(int i) {
  return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1);
}

struct PfParams {
  const uint16_t* q;
  const uint16_t* k_cache;
  const uint16_t* v_cache;
  int64_t seq_stride;
  int nb_capacity;
  const int32_t* n_ctx;
  const int32_t* idx;
  const int32_t* n_sel;
  int k_cap;
  uint16_t* out;
  float* lse;
  uint64_t* part;          // [workgroup][split][wave][its 32-channel groups x 4 x 4 bf16 | (max, sum)][64 lanes]; or PfPiece
  int merge_after;         // 1: a second launch merges the pieces, 0: the workgroup that finishes last (prefill_merge_after)
  unsigned int* counters;  // one ticket counter per (sequence, query tile, KV head), zero between launches
  int m, n_q_heads, n_kv_heads, n_init, n_local;
  int s_lo, rem, slots, n_qtiles;   // pieces per query tile (PfSplits)
  int items_per_head, wgs_per_head; // work items and (first-team) workgroups of one KV head
  int team_total;                   // workgroups of both teams together (the last one to leave resets the queue)
  int late;                         // 1: this launch is the second team, which only draws from the queue
  int sel_per_head;                 // 1: idx and n_sel have a row per (sequence, KV head), 0: per sequence
  unsigned int* queue;              // per KV head: items handed out beyond the first round; [kPfQueueDone]: workgroups that left
  float scale_log2e;
  SelectInside sel;                 // one sequence: its selection is made here
};

// The selection of a work item in LDS.
struct PfChosen {
  int32_t idx[64];
  int count;                        // (with PfParams::sel)
  SelectWaveLds work;
};

// The partial result of one wavefront of a piece for the merge launch: kSlots times 16 bytes per lane, then (maximum, sum).
template <int D, int KS, bool kTwoTermP>
struct PfPiece {
  static constexpr int kDb = D / 32;
  static constexpr int kMine = kDb > KS ? kDb / KS : 1;      // 32-channel groups of a wavefront after its merge in LDS
  static constexpr bool kHalf = KS == 1 && !kTwoTermP;       // normalised and bf16
  static constexpr int kSlots = (kHalf ? 2 : 4) * kMine;
  static constexpr int kWords = kSlots * 64 + 32;            // 16-byte words
  static constexpr int kTake = 2;                            // slots of a wavefront of the merge
  static constexpr int kUnits = kPfWaves / KS * (kDb < KS ? kDb : KS) * (kSlots / kTake);   // its wavefronts per query tile
  static_assert(kPfPieces<D, KS, kTwoTermP> ? kPfWaves * kWords * 4 <= kPfPartialFloats && kUnits % kMergeWaves == 0 : true, "pieces");
  static __device__ __forceinline__ u32x4* at(const PfParams& p, int s, int hk, int slot, int wave) {
    return reinterpret_cast<u32x4*>(p.part) + (((size_t(s) * p.n_kv_heads + hk) * p.slots + slot) * kPfWaves + wave) * kWords;
  }
};

// Final normalisation and store of one lane's share of a query row:
// acc_o[j][4i + r] is channel (db0 + j)*32 + 8i + 4*half + r.
template <int D, int N>
__device__ __forceinline__ void store_rows(const PfParams& p, const f32x16 (&acc_o)[N], int db0, float m_run,
                                           float l_tot, int s, int my_row, int head, int half) {
  const size_t grow = (size_t(s) * p.m + my_row) * p.n_q_heads + head;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  uint16_t* op = p.out + grow * D + db0 * 32;
#pragma unroll
  for (int db = 0; db < N; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u32x2 v;
      v.x = pack_bf16x2(acc_o[db][4 * j + 0] * inv, acc_o[db][4 * j + 1] * inv);
      v.y = pack_bf16x2(acc_o[db][4 * j + 2] * inv, acc_o[db][4 * j + 3] * inv);
      *reinterpret_cast<u32x2*>(op + db * 32 + 8 * j + 4 * half) = v;
    }
  if (p.lse != nullptr && half == 0 && db0 == 0)
    p.lse[(size_t(s) * p.n_q_heads + head) * p.m + my_row] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
}

// One work item: piece `slot` of the query tiles of (sequence s, KV head hk).  kTwoTermP: see prefill_two_terms.
template <int D, int KS, bool kTwoTermP, bool kInLoop>
__device__ __forceinline__ void attn_prefill_item(const PfParams& p, uint16_t* lds, PfChosen& chosen, int hk, int slot, int s) {
  constexpr int kDb = D / 32, kKs = D / 16;      // 32-channel groups of the output, 16-channel steps of a score
  constexpr int kRows = kPfRows<KS>, kRowGroups = kPfWaves / KS;   // query rows, groups of 32 of them
  constexpr int kNg = 4 / KS;                    // 32-key groups of a tile that are this wavefront's
  // (inside an item loop the thread index is made opaque, so that nothing derived from it is
  // hoisted out of the loop and kept in registers across the whole item)
  int tid = threadIdx.x;
  if (kInLoop) asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, half = lane >> 5;
  const int rg = wave % kRowGroups, quarter = wave / kRowGroups;   // its rows, its share of the keys of every tile
  const int kb0 = quarter * kNg;
  const int group = p.n_q_heads / p.n_kv_heads;

  // The slots of a (sequence, KV head) are the pieces of its query tiles, in order.
  const int n_lo = p.n_qtiles - p.rem;
  int qtile, split, splits;
  if (slot < n_lo * p.s_lo) {
    qtile = slot / p.s_lo;
    split = slot - qtile * p.s_lo;
    splits = p.s_lo;
  } else {
    const int r = slot - n_lo * p.s_lo;
    splits = p.s_lo + 1;
    qtile = n_lo + r / splits;
    split = r - (qtile - n_lo) * splits;
  }

  // the selected block indices are requested together with the two scalars they are used
  // with, not after them (one memory round trip less before the first tile can be fetched); or the last wavefront
  // selects, before it asks for anything else
  const bool inside = p.sel.scores != nullptr;
  const size_t sel_row = p.sel_per_head ? size_t(s) * p.n_kv_heads + hk : size_t(s);
  const int32_t my_idx = !inside && tid < p.k_cap ? p.idx[sel_row * p.k_cap + tid] : -1;
  const int n_ctx_raw = p.n_ctx[s];
  int n_sel_raw = inside ? 0 : p.n_sel[sel_row];
  if (!kInLoop && inside && wave == kPfWaves - 1)
    p.sel.run(p.k_cap, blockIdx.x == 0, chosen.work, chosen.idx, &chosen.count);
  const int n_ctx = min(max(n_ctx_raw, p.m), p.nb_capacity * kBlock);
  const WindowGeom g = window_geom(n_ctx, p.m, p.n_init, p.n_local);
  // The query rows of a (sequence, KV head) are numbered position by position, the G heads of a
  // position next to each other; a workgroup takes kRows consecutive ones, a wavefront 32.
  const int row_end = p.m * group;
  const int row_hi = (min((qtile + 1) * kRows, row_end) - 1) / group;
  const int frow0 = qtile * kRows + rg * 32;                 // first query row of this wavefront
  const bool wave_ok = frow0 < row_end;
  const int wpos_lo = g.w0 + min(frow0, row_end - 1) / group;         // positions of its first and last row
  const int wpos_hi = g.w0 + min(frow0 + 31, row_end - 1) / group;
  const bool row_ok = frow0 + n < row_end;
  const int frow = min(frow0 + n, row_end - 1);
  const int my_row = frow / group;                           // window row (position) and head of this lane
  const int head = hk * group + (frow - my_row * group);
  const int my_pos = g.w0 + my_row;                          // this lane's query position

  // Q^T as B operand: lane (n, half) holds d = ks*16 + 8*half .. +7 of query row n.  (Folding
  // scale * log2(e) into these operands, rounded to bf16 again, and starting the score
  // accumulators at minus the reference maximum would spare the multiply-add per score, but the
  // second rounding of the queries moves large logits by 2^-9 of their size: 2 % output error on
  // heavy-tailed inputs.)
  bf16x8 qreg[kKs];
  {
    const uint16_t* qp = p.q + ((size_t(s) * p.m + my_row) * p.n_q_heads + head) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks)
      qreg[ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(qp + ks * 16));
  }

  f32x16 acc_o[kDb];
#pragma unroll
  for (int i = 0; i < kDb; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc_o[i][j] = 0.f;
  float m_run = -INFINITY;                // running max (log2 units)
  const uint32_t bf16_ones = 0x3f803f80u;

  const char* kc = reinterpret_cast<const char*>(p.k_cache + size_t(s) * p.seq_stride);
  const char* vc = reinterpret_cast<const char*>(p.v_cache + size_t(s) * p.seq_stride);
  constexpr uint32_t kTileBytes = kPfTileBytes<D>;
  // LDS: stage s holds K at 2s * kTileBytes and V^T at (2s + 1) * kTileBytes
  char* lds_b = reinterpret_cast<char*>(lds);

  // Tiles go from HBM straight into LDS (buffer_load_dwordx4 ... lds: lane i of a wavefront
  // fills the i-th 16-byte chunk of a contiguous 1 KB piece of LDS; no staging registers, no
  // ds_write).  Each wavefront fills an eighth of a K and of a V^T tile.  The 16-byte chunks of
  // an LDS row are XOR-swizzled with a key made of the row, so that the 16 rows an MFMA operand
  // load touches hit all 64 banks: rows of 256 bytes (V^T, and K with 128 channels) take
  // row % 16, rows of 128 bytes (K with 64 channels: two of them span the banks) take
  // (row / 2) % 8.  The swizzle is applied on the global side: the lane that fills chunk c' of
  // row r fetches chunk c' ^ key(r) of that row.
  constexpr int kLoads = D / 32;                       // 1 KB pieces of a tile per wavefront
  constexpr uint32_t kKRow = D * 2;                    // bytes of a K row
  constexpr int kKPerPiece = 1024 / kKRow;             // K rows of a piece
  // per-lane byte offsets inside a tile, one per load; the tile's base and the LDS
  // destination are the same for all lanes and stay in scalar registers
  uint32_t gk[kLoads], gv[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    const int kr = (kLoads * wave + i) * kKPerPiece + lane / (64 / kKPerPiece);
    const int kc16 = lane % (64 / kKPerPiece);
    gk[i] = uint32_t(kr) * kKRow + (uint32_t(kc16 ^ (D == 128 ? kr & 15 : (kr >> 1) & 7)) << 4);
    const int vr = (kLoads * wave + i) * 4 + (lane >> 4);
    gv[i] = uint32_t(vr) * 256 + (uint32_t((lane & 15) ^ (vr & 15)) << 4);
  }
  auto fetch_tile = [&](int block, int stage) {
    const size_t off = (size_t(block) * p.n_kv_heads + hk) * kTileBytes;
    const char* kt = uniform_ptr(kc + off);
    const char* vt = uniform_ptr(vc + off);
    char* dst = lds_b + stage * 2 * kTileBytes + wave * (kTileBytes / 8);
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(kt), 0, kTileBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vt), 0, kTileBytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, gk[i], 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (__attribute__((address_space(3))) void*)(dst + kTileBytes + i * 1024), 16, gv[i], 0, 0, 0);
    }
  };
  // the first piece begins with the initial tokens, whatever is selected
  const bool early = split == 0 && g.i0 > 0;
  if (early) fetch_tile(0, 0);
  if (!inside && tid < 64) chosen.idx[tid] = my_idx;
  __syncthreads();
  if (inside) n_sel_raw = chosen.count;
  const TileList tl = make_tile_list(g, g.w0 + row_hi, chosen.idx, n_sel_raw, p.k_cap, p.nb_capacity);
  const int n_tiles = tl.count();
  const int per = (n_tiles + splits - 1) / splits;
  const int t_begin = split * per, t_end = min(n_tiles, t_begin + per);

  // tile t of the list -> its block and visible span, in scalar registers
  auto tile_at = [&](int t, int& block, int& lo, int& hi) {
    tl.get(t, block, lo, hi);
    block = __builtin_amdgcn_readfirstlane(block);
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
  };

  int block = 0, lo = 0, hi = 0;
  if (t_begin < t_end) {
    tile_at(t_begin, block, lo, hi);
    if (!early) fetch_tile(block, 0);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const int a_row = perm_row(n);
  // Byte offsets of this lane's MFMA A operands inside a K / V^T tile.  K: row perm(n), chunk
  // 2*ks + half; V^T: row n, chunk c = 4*kb + 2*s2 + half; both XOR-ed with the row's swizzle
  // key.  The offset of chunk pair c is that of pair 0 with c << 5 XOR-ed in: one register per
  // operand kind and one XOR per read, instead of eight registers each.  The 32-row blocks
  // (kb, db) add a compile-time constant.
  uint32_t a_off0 = uint32_t(a_row) * kKRow + (uint32_t(half ^ (D == 128 ? a_row & 15 : (a_row >> 1) & 7)) << 4);
  uint32_t v_off0 = uint32_t(n) * 256 + (uint32_t(half ^ (n & 15)) << 4);
  float l_run = 0.f;                           // this lane's share of the running sum of its query row
  for (int t = t_begin; t < t_end; ++t) {
    const int stage = (t - t_begin) & 1;
    // (opaque per iteration: the XOR-ed offsets are recomputed, not kept across the loop)
    asm volatile("" : "+v"(a_off0), "+v"(v_off0));

    int block_next = 0, lo_next = 0, hi_next = 0;
    if (t + 1 < t_end) tile_at(t + 1, block_next, lo_next, hi_next);
    const int kpos0 = block * kBlock;
    // the wavefront skips tiles none of its rows can see; it masks tiles that are
    // clipped or that reach past its first row's position
    const int sub0 = kpos0 + kb0 * 32;             // first key of this wavefront's share
    const bool visible = wave_ok && hi > max(lo, sub0) && max(lo, sub0) <= wpos_hi;
    const bool masked = lo > kpos0 || hi < kpos0 + kBlock || hi - 1 > wpos_lo;
    const char* ks_ = lds_b + stage * 2 * kTileBytes;
    const char* vs_ = ks_ + kTileBytes;
    f32x16 acc_s[kNg];
    if (visible) {
      // ---- S^T = K Q^T : kNg groups of 32 keys
      const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      // the key groups take turns (a single one is summed in two halves), so that an MFMA does not
      // wait for the one just before it (a dependent 32x32x16 MFMA issues only about 90 cycles
      // after its producer, an independent one after 32)
      // (written in the order it should issue: a ring of 8 operands, each read 8 MFMAs ahead)
      constexpr int kChains = kNg == 1 ? 2 : kNg;
      auto k_read = [&](int i) {
        return *reinterpret_cast<const u32x4*>(ks_ + (a_off0 ^ (uint32_t(i / kNg) << 5)) + (kb0 + i % kNg) * 32 * kKRow);
      };
      constexpr int kScore = kNg * kKs, kRing = kScore < 8 ? kScore : 8;      // MFMAs of the scores
      u32x4 ring[kRing];
      f32x16 acc[kChains];
#pragma unroll
      for (int i = 0; i < kRing; ++i) ring[i] = k_read(i);
#pragma unroll
      for (int i = 0; i < kScore; ++i) {
        const int c = i % kChains;
        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ring[i % kRing]), qreg[i / kNg], i < kChains ? zero16 : acc[c], 0, 0, 0);
        if (i + kRing < kScore) ring[i % kRing] = k_read(i + kRing);
      }
      // issue order: 8 operand reads ahead of the first MFMA, then one read per MFMA, so that an
      // operand is requested about 8 MFMAs before it is needed (0x100 = LDS read, 0x008 = MFMA)
      __builtin_amdgcn_sched_group_barrier(0x100, kRing, 0);
#pragma unroll
      for (int i = 0; i < kScore - kRing; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, kRing, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kb = 0; kb < kNg; ++kb) acc_s[kb] = acc[kb];
      if constexpr (kNg == 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_s[0][i] += acc[1][i];
      }
    }
    // The next tile is requested here, after the score MFMAs and not at the top of the
    // iteration: while an LDS-direct load (a FLAT-encoded instruction) is in flight the
    // compiler must treat LDS operations as completing out of order and waits for ALL
    // outstanding operand reads before each use, which stalled the score phase every 8 MFMAs.
    // It still has the softmax and the value phase of this tile to land.
    if (t + 1 < t_end) fetch_tile(block_next, stage ^ 1);
    if (visible) {
      // register i of group kb holds key kpos0 + (kb0 + kb)*32 + 16*(i/8) + 8*half + (i%8)
      if (masked) {
#pragma unroll
        for (int kb = 0; kb < kNg; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int kp = kpos0 + (kb0 + kb) * 32 + 16 * (i >> 3) + 8 * half + (i & 7);
            const bool ok = kp >= lo && kp < hi && kp <= my_pos;
            acc_s[kb][i] = ok ? acc_s[kb][i] : -INFINITY;
          }
      }
      // ---- online softmax, one query per lane (two lanes share a query: n and n+32)
      // the first V^T operands are requested now and land during the max reduction;
      // operand j = kDb * (2*kb + s2) + db belongs to keys (kb0 + kb)*32 + s2*16 .. +15, rows db*32 .. +31
      auto v_read = [&](int j) {
        return *reinterpret_cast<const u32x4*>(vs_ + (v_off0 ^ (uint32_t(2 * kb0 + j / kDb) << 5)) + (j % kDb) * 32 * 256);
      };
      constexpr int kValue = 2 * kNg * kDb, kVRing = kValue < 8 ? kValue : 8;
      u32x4 vring[kVRing];
#pragma unroll
      for (int i = 0; i < kVRing; ++i) vring[i] = v_read(i);
      float mx = acc_s[0][0];
#pragma unroll
      for (int kb = 0; kb < kNg; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc_s[kb][i]);
      mx = lane_pair<32>(mx, [](float x, float y) { return fmaxf(x, y); });
      // the reference maximum follows the true one lazily: it moves only when a tile exceeds
      // it by more than 2^8, so the rescaling of the accumulators below is rare after the first
      // tiles; probabilities up to 2^8 are as exact in bf16 and fp32 as those up to 1
      const float m_tile = mx * p.scale_log2e;
      const float m_new = m_tile - m_run > kLazyMaxLog2 ? m_tile : m_run;
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
#pragma unroll
      for (int i = 0; i < 16; ++i) acc_s[0][i] = __builtin_amdgcn_exp2f(acc_s[0][i] * p.scale_log2e - m_safe);
      __builtin_amdgcn_sched_barrier(0);
      // ---- O^T += V^T P^T.  Written in issue order: the exponentials of the next 32 keys sit
      // between the MFMAs of these 32 (the vector ALU works while the matrix pipe does), and every
      // V^T operand is read 8 MFMAs ahead.  The row sums add the bf16 probabilities the product
      // itself uses, a pair per instruction, each lane summing its own 64 keys of the tile (with two
      // terms the fp32 ones).
#pragma unroll
      for (int g8 = 0; g8 < 2 * kNg; ++g8) {
        const int kb = g8 >> 1, s2 = g8 & 1;
        const bf16x8 pb = pack8(acc_s[kb][8 * s2 + 0], acc_s[kb][8 * s2 + 1], acc_s[kb][8 * s2 + 2],
                                acc_s[kb][8 * s2 + 3], acc_s[kb][8 * s2 + 4], acc_s[kb][8 * s2 + 5],
                                acc_s[kb][8 * s2 + 6], acc_s[kb][8 * s2 + 7]);
        bf16x8 pl;                         // with two terms: what the rounding to bf16 left of the probabilities
        if constexpr (kTwoTermP) {
          typedef __attribute__((ext_vector_type(8))) float f32x8;
          const f32x8 wide = __builtin_convertvector(pb, f32x8);
          float left[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) left[i] = acc_s[kb][8 * s2 + i] - wide[i];
#pragma unroll
          for (int i = 0; i < 8; i += 2) l_run += acc_s[kb][8 * s2 + i] + acc_s[kb][8 * s2 + i + 1];
          pl = pack8(left[0], left[1], left[2], left[3], left[4], left[5], left[6], left[7]);
        } else {
          add_bf16x8(l_run, pb, bf16_ones);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < kDb; ++db) {
          if (kb < kNg - 1) {
            constexpr int kExp = 8 / kDb;
#pragma unroll
            for (int i = 8 * s2 + kExp * db; i < 8 * s2 + kExp * (db + 1); ++i)
              acc_s[kb + 1][i] = __builtin_amdgcn_exp2f(acc_s[kb + 1][i] * p.scale_log2e - m_safe);
          }
          __builtin_amdgcn_sched_barrier(0);
          const int j = kDb * g8 + db;
          acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vring[j % kVRing]), pb, acc_o[db], 0, 0, 0);
          if constexpr (kTwoTermP)
            acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vring[j % kVRing]), pl, acc_o[db], 0, 0, 0);
          if (j + kVRing < kValue) vring[j % kVRing] = v_read(j + kVRing);
        }
      }
    }
    block = block_next;
    lo = lo_next;
    hi = hi_next;
    __builtin_amdgcn_s_waitcnt(0);   // this wavefront's pieces of the next tile have landed in LDS
    __syncthreads();
  }

  // ---- epilogue
  float l_tot = lane_pair<32>(l_run, [](float x, float y) { return x + y; });
  // The wavefronts that share query rows merge in LDS (the tiles are no longer needed): each puts down
  // its output, its maximum and its sum and takes over kMine of the 32-channel groups:
  //   out = sum_w 2^(m_w - M) o_w / sum_w 2^(m_w - M) l_w
  constexpr int kMine = kDb > KS ? kDb / KS : 1;     // channel groups of a wavefront from here on
  f32x16 acc_f[kMine];
  const int db0 = quarter * kMine;
  const bool has_mine = db0 < kDb;
  if constexpr (KS == 1) {
#pragma unroll
    for (int db = 0; db < kDb; ++db) acc_f[db] = acc_o[db];
  } else {
    __shared__ float ml_lds[kPfWaves][2][32];
    f32x4* o_lds = reinterpret_cast<f32x4*>(lds);    // [wavefront][channel group][register / 4][lane]
#pragma unroll
    for (int db = 0; db < kDb; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o_lds[((wave * kDb + db) * 4 + i) * 64 + lane] =
            f32x4{acc_o[db][4 * i], acc_o[db][4 * i + 1], acc_o[db][4 * i + 2], acc_o[db][4 * i + 3]};
    if (half == 0) {
      ml_lds[wave][0][n] = m_run;
      ml_lds[wave][1][n] = l_tot;
    }
    __syncthreads();
    float m_of[KS], l_of[KS], m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      m_of[w] = ml_lds[w * kRowGroups + rg][0][n];
      l_of[w] = ml_lds[w * kRowGroups + rg][1][n];
      m_all = fmaxf(m_all, m_of[w]);
    }
    const float m_ref = m_all == -INFINITY ? 0.f : m_all;
    l_tot = 0.f;
#pragma unroll
    for (int db = 0; db < kMine; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc_f[db][i] = 0.f;
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      const float weight = __builtin_amdgcn_exp2f(m_of[w] - m_ref);
      l_tot += weight * l_of[w];
      if (has_mine) {
#pragma unroll
        for (int db = 0; db < kMine; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const f32x4 o = o_lds[(((w * kRowGroups + rg) * kDb + db0 + db) * 4 + i) * 64 + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) acc_f[db][4 * i + r] += weight * o[r];
          }
      }
    }
    m_run = m_all;
  }
  if (splits == 1 || !kPfPieces<D, KS, kTwoTermP>) {
    if (row_ok && has_mine) store_rows<D, kMine>(p, acc_f, db0, m_run, l_tot, s, my_row, head, half);
    return;
  }
  // A piece for the merge launch: in the order the registers hold it, 1 KB in a row per store instruction, normalised and as
  // bf16 where PfPiece says so.
  if (p.merge_after) {
    using Piece = PfPiece<D, KS, kTwoTermP>;
    if (!has_mine) return;
    u32x4* mine = Piece::at(p, s, hk, slot, wave) + lane;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
#pragma unroll
    for (int k = 0; k < Piece::kSlots; ++k) {
      u32x4 v;
      if constexpr (Piece::kHalf) {
        const f32x16& o = acc_f[k / 2];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = pack_bf16x2(o[8 * (k % 2) + 2 * i] * inv, o[8 * (k % 2) + 2 * i + 1] * inv);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(acc_f[k / 4][4 * (k % 4) + i]);
      }
      mine[k * 64] = v;
    }
    reinterpret_cast<f32x2*>(mine - lane + Piece::kSlots * 64)[lane] = f32x2{m_run, l_tot};
    return;
  }
  // Otherwise the piece stores its output in the order the registers hold it (register-major, lane-minor: every
  // store instruction writes one contiguous 512-byte row), plus its running max and sum: of a whole
  // query tile of one-term probabilities normalised and as bf16 (64 KB), otherwise as it is.
  constexpr bool kHalf = KS == 1 && !kTwoTermP;
  constexpr int kPerGroup = kHalf ? 4 : 8;         // 64-bit words of a channel group
  constexpr int kWords = kPerGroup * kMine + 1;    // 64-bit words per lane: the output, then (max, sum)
  __shared__ int last_flag;
  const size_t group_id = (size_t(s) * p.n_qtiles + qtile) * p.n_kv_heads + hk;
  uint64_t* group_part = p.part + ((size_t(s) * p.n_kv_heads + hk) * p.slots + (slot - split)) *
                                      (kPfWaves * (kWords * 64));
  if (has_mine) {
    uint64_t* mine = group_part + (size_t(split) * kPfWaves + wave) * (kWords * 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
#pragma unroll
    for (int db = 0; db < kMine; ++db)
#pragma unroll
      for (int i = 0; i < kPerGroup; ++i) {
        uint32_t lo, hi;
        if constexpr (kHalf) {
          lo = pack_bf16x2(acc_f[db][4 * i] * inv, acc_f[db][4 * i + 1] * inv);
          hi = pack_bf16x2(acc_f[db][4 * i + 2] * inv, acc_f[db][4 * i + 3] * inv);
        } else {
          lo = __float_as_uint(acc_f[db][2 * i]);
          hi = __float_as_uint(acc_f[db][2 * i + 1]);
        }
        st_agent(mine + (db * kPerGroup + i) * 64 + lane, uint64_t(lo) | (uint64_t(hi) << 32));
      }
    st_agent(mine + (kWords - 1) * 64 + lane, uint64_t(__float_as_uint(m_run)) | (uint64_t(__float_as_uint(l_tot)) << 32));
  }
  if (!last_of_group(p.counters + group_id, unsigned(splits), &last_flag) || !has_mine) return;

  // ---- the last piece of the query tile merges all of them, in order:
  //   out = sum_s w_s o_s / sum_s w_s with w_s = l_s 2^(m_s - M), M = max_s m_s, o_s normalised
  //   (not normalised: sum_s v_s O_s / sum_s v_s l_s with v_s = 2^(m_s - M))
  // (its own piece is read back like the others, so the result does not depend on who is last)
  const uint64_t* piece0 = group_part + size_t(wave) * (kWords * 64) + lane;
  const size_t piece_stride = size_t(kPfWaves) * (kWords * 64);
  // the loads of the first pieces go out together with the (max, sum) words of all pieces
  constexpr int kMergeBatch = kWords <= 9 ? 4 : 3;
  uint64_t ml[kMaxPfSplits], raw[kMergeBatch][kWords - 1];
#pragma unroll
  for (int s2 = 0; s2 < kMaxPfSplits; ++s2)
    ml[s2] = s2 < splits ? ld_agent(piece0 + s2 * piece_stride + (kWords - 1) * 64) : 0;
#pragma unroll
  for (int j = 0; j < kMergeBatch; ++j)
#pragma unroll
    for (int k = 0; k < kWords - 1; ++k) raw[j][k] = j < splits ? ld_agent(piece0 + j * piece_stride + k * 64) : 0;
  __builtin_amdgcn_sched_barrier(0);
  float w_s[kMaxPfSplits + kMergeBatch];
  float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int s2 = 0; s2 < kMaxPfSplits; ++s2)
    if (s2 < splits) m_all = fmaxf(m_all, __uint_as_float(uint32_t(ml[s2])));
  const float m_safe = m_all == -INFINITY ? 0.f : m_all;
#pragma unroll
  for (int s2 = 0; s2 < kMaxPfSplits + kMergeBatch; ++s2) {
    const uint64_t of = ml[s2 < kMaxPfSplits ? s2 : 0];
    const float v = s2 < splits ? __builtin_amdgcn_exp2f(__uint_as_float(uint32_t(of)) - m_safe) : 0.f;
    const float vl = s2 < splits ? v * __uint_as_float(uint32_t(of >> 32)) : 0.f;
    l_all = fmaf(v, s2 < splits ? __uint_as_float(uint32_t(of >> 32)) : 0.f, l_all);
    w_s[s2] = kHalf ? vl : v;
  }
#pragma unroll
  for (int db = 0; db < kMine; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc_f[db][i] = 0.f;
#pragma unroll
  for (int b0 = 0; b0 < kMaxPfSplits; b0 += kMergeBatch) {
    if (b0 < splits) {
      if (b0 > 0) {
#pragma unroll
        for (int j = 0; j < kMergeBatch; ++j)
#pragma unroll
          for (int k = 0; k < kWords - 1; ++k)
            raw[j][k] = b0 + j < splits ? ld_agent(piece0 + (b0 + j) * piece_stride + k * 64) : 0;
      }
#pragma unroll
      for (int j = 0; j < kMergeBatch; ++j) {
        const float w = w_s[b0 + j];
#pragma unroll
        for (int db = 0; db < kMine; ++db)
#pragma unroll
          for (int i = 0; i < kPerGroup; ++i) {
            const uint32_t lo = uint32_t(raw[j][db * kPerGroup + i]), hi = uint32_t(raw[j][db * kPerGroup + i] >> 32);
            if constexpr (kHalf) {
              acc_f[db][4 * i + 0] = fmaf(w, bf16_lo(lo), acc_f[db][4 * i + 0]);
              acc_f[db][4 * i + 1] = fmaf(w, bf16_hi(lo), acc_f[db][4 * i + 1]);
              acc_f[db][4 * i + 2] = fmaf(w, bf16_lo(hi), acc_f[db][4 * i + 2]);
              acc_f[db][4 * i + 3] = fmaf(w, bf16_hi(hi), acc_f[db][4 * i + 3]);
            } else {
              acc_f[db][2 * i] = fmaf(w, __uint_as_float(lo), acc_f[db][2 * i]);
              acc_f[db][2 * i + 1] = fmaf(w, __uint_as_float(hi), acc_f[db][2 * i + 1]);
            }
          }
      }
    }
  }
  if (row_ok) store_rows<D, kMine>(p, acc_f, db0, m_all, l_all, s, my_row, head, half);
}

// The pieces of a query tile of one window (prefill_merge_after), in their order:
//   out = sum_s w_s o_s / sum_s w_s  with w_s = l_s 2^(m_s - M), M = max_s m_s, o_s normalised
//   (not normalised: sum_s v_s O_s / sum_s v_s l_s  with v_s = 2^(m_s - M)).
// A wavefront merges kTake 16-byte slots of the 32 rows of a wavefront of the attention, all its loads in flight at once; blocks
// deal the KV heads like the attention's, so that a head's pieces are read on the XCD that wrote them.  Bound by its launch and one
// round trip: 4 to 5 us for 256 pieces (prefill_merge_after has both sides).
template <int D, int KS, bool kTwoTermP>
__global__ __launch_bounds__(64 * kMergeWaves) void attn_prefill_merge_kernel(PfParams p) {
  using Piece = PfPiece<D, KS, kTwoTermP>;
  constexpr int kTake = Piece::kTake, kParts = Piece::kSlots / kTake;
  constexpr int kRowGroups = kPfWaves / KS, kRows = kPfRows<KS>;
  const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  const int hk = blockIdx.x % p.n_kv_heads;
  const int unit = __builtin_amdgcn_readfirstlane((blockIdx.x / p.n_kv_heads) * kMergeWaves + (threadIdx.x >> 6));
  const int qtile = unit / Piece::kUnits, wave = unit % Piece::kUnits / kParts, part = unit % kParts;
  const int n_lo = p.n_qtiles - p.rem;
  const int splits = qtile < n_lo ? p.s_lo : p.s_lo + 1;
  const int slot0 = qtile < n_lo ? qtile * p.s_lo : n_lo * p.s_lo + (qtile - n_lo) * splits;
  const u32x4* piece = Piece::at(p, 0, hk, slot0, wave);
  f32x2 ml[kMaxPfSplits];
  u32x4 raw[kMaxPfSplits][kTake];
#pragma unroll
  for (int i = 0; i < kMaxPfSplits; ++i) {
    ml[i] = f32x2{-INFINITY, 0.f};
#pragma unroll
    for (int k = 0; k < kTake; ++k) raw[i][k] = u32x4{0, 0, 0, 0};
    if (i < splits) {
      const u32x4* from = piece + size_t(i) * (kPfWaves * Piece::kWords);
      ml[i] = reinterpret_cast<const f32x2*>(from + Piece::kSlots * 64)[lane];
#pragma unroll
      for (int k = 0; k < kTake; ++k) raw[i][k] = from[(part * kTake + k) * 64 + lane];
    }
  }
  float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int i = 0; i < kMaxPfSplits; ++i)
    if (i < splits) m_all = fmaxf(m_all, ml[i].x);
  const float m_safe = m_all == -INFINITY ? 0.f : m_all;
  float sum[kTake][Piece::kHalf ? 8 : 4];
#pragma unroll
  for (int k = 0; k < kTake; ++k)
#pragma unroll
    for (int j = 0; j < (Piece::kHalf ? 8 : 4); ++j) sum[k][j] = 0.f;
#pragma unroll
  for (int i = 0; i < kMaxPfSplits; ++i) {
    if (i < splits) {
      const float v = __builtin_amdgcn_exp2f(ml[i].x - m_safe), vl = v * ml[i].y;
      l_all = fmaf(v, ml[i].y, l_all);
#pragma unroll
      for (int k = 0; k < kTake; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (Piece::kHalf) {
            sum[k][2 * j] = fmaf(vl, bf16_lo(raw[i][k][j]), sum[k][2 * j]);
            sum[k][2 * j + 1] = fmaf(vl, bf16_hi(raw[i][k][j]), sum[k][2 * j + 1]);
          } else {
            sum[k][j] = fmaf(v, __uint_as_float(raw[i][k][j]), sum[k][j]);
          }
        }
    }
  }
  const int group = p.n_q_heads / p.n_kv_heads;
  const int frow = qtile * kRows + (wave % kRowGroups) * 32 + n;
  if (frow >= p.m * group) return;
  const int row = frow / group, head = hk * group + (frow - row * group);
  const int db0 = (wave / kRowGroups) * Piece::kMine;
  const float inv = l_all > 0.f ? 1.f / l_all : 0.f;
  uint16_t* op = p.out + (size_t(row) * p.n_q_heads + head) * D + db0 * 32 + 4 * half;
#pragma unroll
  for (int k = 0; k < kTake; ++k)
#pragma unroll
    for (int j = 0; j < (Piece::kHalf ? 2 : 1); ++j) {
      const int at = (part * kTake + k) * (Piece::kHalf ? 2 : 1) + j;    // group of 8 channels
      u32x2 v;
      v.x = pack_bf16x2(sum[k][4 * j] * inv, sum[k][4 * j + 1] * inv);
      v.y = pack_bf16x2(sum[k][4 * j + 2] * inv, sum[k][4 * j + 3] * inv);
      *reinterpret_cast<u32x2*>(op + 8 * at) = v;
    }
  if (p.lse != nullptr && half == 0 && db0 == 0 && part == 0)
    p.lse[size_t(head) * p.m + row] = (m_all + log2f(l_all)) * 0.6931471805599453f;
}

// blockIdx.x = w * Hk + hk: consecutive ids differ in hk, and ids are dealt round-robin to the
// XCDs, so each XCD serves few KV heads and that head's tiles stay in its L2.  The items of a
// KV head are its (sequence, slot) pairs.  If there are no more of them than workgroups, each
// workgroup takes one.  Otherwise (several windows in one call, fewer compute units than
// items) the workgroups of a head draw the remaining items from a counter: windows differ in
// how many blocks they retrieve, and a fixed assignment would wait for the unluckiest
// workgroup.  Nobody waits for anybody: a workgroup leaves when the counter runs out, and the
// last one to leave puts the counters back to zero for the next launch.
template <int D, int KS, bool kTwoTermP>
__global__ __launch_bounds__(kPfThreads) void attn_prefill_mfma_kernel(PfParams p) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  __shared__ PfChosen chosen;
  const int item = blockIdx.x / p.n_kv_heads, s = item / p.slots;
  attn_prefill_item<D, KS, kTwoTermP, false>(p, lds, chosen, blockIdx.x % p.n_kv_heads, item - s * p.slots, s);
}

template <int D, int KS, bool kTwoTermP>
__global__ __launch_bounds__(kPfThreads) void attn_prefill_mfma_queued_kernel(PfParams p) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  __shared__ int next_item;
  __shared__ PfChosen chosen;
  const int hk = blockIdx.x % p.n_kv_heads;
  // (one window: the same selection for all of its items; the barrier of the first item is behind it)
  if (p.sel.scores != nullptr && threadIdx.x >= kPfThreads - 64)
    p.sel.run(p.k_cap, blockIdx.x == 0, chosen.work, chosen.idx, &chosen.count);
  auto draw = [&]() {
    if (threadIdx.x == 0)
      next_item = p.wgs_per_head + int(__hip_atomic_fetch_add(p.queue + hk, 1u, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT));
    __syncthreads();
    return next_item;
  };
  // Longest items first, so that the launch does not end with a few workgroups on long items
  // while the others have left: the batch entries in descending order of the number of blocks
  // they retrieve (ties: ascending index), and within an entry the later query tiles, which see
  // more of the window, before the earlier ones.
  __shared__ int order[kPfOrderMax];
  const int batch = p.items_per_head / p.slots;
  const bool sorted = batch <= kPfOrderMax;
  if (sorted) {
    const int t = threadIdx.x;
    if (t < batch) {
      const size_t stride = p.sel_per_head ? p.n_kv_heads : 1, off = p.sel_per_head ? hk : 0;
      const int mine = p.n_sel[size_t(t) * stride + off];
      int rank = 0;
      for (int j = 0; j < batch; ++j) {
        const int other = p.n_sel[size_t(j) * stride + off];
        rank += (other > mine) || (other == mine && j < t);
      }
      order[rank] = t;
    }
    __syncthreads();
  }
  // A second team of workgroups (a launch of its own, on compute units that were busy with
  // something else when the first team started) has no first-round items: it only draws.
  int item = p.late ? draw() : int(blockIdx.x) / p.n_kv_heads;
  while (item < p.items_per_head) {
    int s = item / p.slots, slot = item - s * p.slots;
    if (sorted) {
      s = order[s];
      slot = p.slots - 1 - slot;
    }
    attn_prefill_item<D, KS, kTwoTermP, true>(p, lds, chosen, hk, __builtin_amdgcn_readfirstlane(slot), __builtin_amdgcn_readfirstlane(s));
    __syncthreads();                         // everybody is done with the LDS tiles of this item
    item = draw();
  }
  if (threadIdx.x == 0) {
    unsigned int* done = p.queue + kPfQueueDone;
    const unsigned int t = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == unsigned(p.team_total) - 1u) {
      for (int h = 0; h < p.n_kv_heads; ++h)
        __hip_atomic_store(p.queue + h, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

bool prefill_mfma_supported(const actqkv_shape& sh, int m) {
  return sh.dtype == ACTQKV_BF16 && m > 1;
}

// Two-term probabilities: they enter the second product as the value rounded to bf16 plus what the rounding left,
// again as bf16, which keeps 16 of their bits; their sums and the partial results are fp32.  Always with 64
// channels, and with 128 where the longest possible tile list (64 selected blocks) passes 96 tiles: these calls
// had fp32 probabilities before they came to the matrix cores, the others have always had bf16 ones.
// Relative error against 64 bits, a window of 4096 tokens, 32 query and 8 KV heads of 64 channels: 2.2954e-3 with
// one term, 1.6583e-3 with two and as fp32, which is what the rounding of the output alone gives; 128 channels:
// 2.3107e-3, 1.6582e-3, 1.6582e-3.  It costs half as many MFMAs again: 158 -> 210 us, 235 -> 317 us; a window of 256 tokens of
// 8 query and 2 KV heads of 64 channels 13.5 -> 14.0 us.  (As one thread per query row: 10.7 ms, 27.8 ms, 1.4 ms.)
static bool prefill_two_terms(const actqkv_shape& sh, int m) {
  return sh.head_dim == 64 || sh.n_init / kBlock + 64 + sh.n_local / kBlock + (m + kBlock - 1) / kBlock + 2 > 96;
}

static int prefill_mfma_qtiles(const actqkv_shape& sh, int m, int ks) {
  const int rows = kPfRows<1> / ks;
  return (m * (sh.n_q_heads / sh.n_kv_heads) + rows - 1) / rows;
}

// Whether a second launch merges the pieces of a query tile: in a single window, from four pieces on (five with fewer than four
// KV heads); otherwise the workgroup that finishes last does.  That one reads the others' results back at 8 bytes a lane past
// the L2s, 32 KB a piece (64 KB of 128 rows) and 8 KB per us, which nothing overlaps in a single window; the launch costs 4 us
// whatever their number.  Of several windows in a call the last workgroup merges beside other items (a host-cache pass of 32K
// tokens in groups of four windows of 512: 3520 us so, 3696 with the launch).  Both do the same operations in the same order,
// written as fmaf, so windows in one call have the bits of single ones.
// Single windows, last workgroup | launch, us:
//   32 query and 8 KV heads of 128: 384 tokens, 5 pieces of 256 rows 30.2 | 24.8; 1024, 2 of 256 49.2 | 50.0; 256, 4 of 128 23.2 | 21.3;
//   512, 2 of 128 29.1 | 29.6; 64, 8 of 64 17.7 | 13.9; 128, 4 of 64 17.4 | 16.0; 200, 2 of 64 19.7 | 20.1
//   28 and 4 heads: 768 tokens, 3 pieces of 256 rows 36.9 | 37.1
//   8 and 2 heads (a query tile's pieces are on more XCDs, which the launch reads from more slowly): 256 tokens, 8 pieces of 64
//   rows 19.4 | 16.0; 768, 5 of 128 25.5 | 23.7; 1024, 4 of 128 27.0 | 27.4; of 64 channels 256, 8 13.9 | 12.3; 512, 4 14.6 | 15.0
bool prefill_merge_after(const actqkv_shape& sh, int s_lo) {
  return s_lo >= (sh.n_kv_heads >= 4 ? 4 : 5);
}

// How a call is cut up: the query rows of a workgroup (kPfRows of ks), the pieces of the key tiles.
//
// Whole query tiles of 256 rows use the matrix cores and the L2 best, but a single window has few of them, and pieces of
// their key tiles cost partial results, out and back.  With fewer rows per workgroup (its wavefronts share the keys of a tile and
// merge in LDS) there are fewer pieces and less to merge, but a tile costs more per row.
static PfSplits prefill_cut(const actqkv_shape& sh, int batch, int m, int cus, int ks, bool pieces) {
  const int pairs = batch * sh.n_kv_heads;
  PfSplits c;
  c.ks = ks;
  c.n_qtiles = prefill_mfma_qtiles(sh, m, ks);
  // pieces where the query tiles leave compute units idle, never more than 8 per query tile; of whole
  // query tiles, what does not divide evenly goes to the last ones of the window
  const int per_pair = std::max(cus / pairs, c.n_qtiles);    // workgroups one pair may have
  c.s_lo = pieces ? std::min(per_pair / c.n_qtiles, kMaxPfSplits) : 1;
  c.rem = c.s_lo == kMaxPfSplits || ks > 1 || !pieces ? 0 : per_pair - c.s_lo * c.n_qtiles;
  c.slots = c.s_lo * c.n_qtiles + c.rem;
  return c;
}

// Several windows or sequences in a call, whose items differ in length with what each retrieves: the least of what the busiest
// compute unit needs by these figures, in us, with half of k_cap retrieved; 32 windows of 512 tokens, 32 query and 8 KV heads of
// 128 channels: 597 as 256 rows, 692 as 128, 1009 as 64.  With 64 channels a tile is half the work and with two-term
// probabilities half as much again, in the same proportions: over windows of 32 to 4096 tokens and groups of 1, 4 and 7 heads, up
// to 32 in a call, the choice took at most 8 % longer than the best of the three, as a rule 0 to 3 %.
static double prefill_many_us(const actqkv_shape& sh, int batch, int m, int k_cap, int cus, const PfSplits& c) {
  constexpr double kTileUs[] = {3.7, 2.1, 1.5}, kMergeUs[] = {6., 3.5, 2.}, kMergePieceUs[] = {1.1, 0.7, 0.5};
  constexpr double kItemUs = 8.;
  const int i = c.ks >> 1;
  const double longest = (sh.n_init + sh.n_local + m) / double(kBlock) + k_cap / 2.0, average = longest - m / double(2 * kBlock);
  const double rounds = double(batch) * sh.n_kv_heads * c.slots / cus;
  double us = std::max(std::ceil(longest / c.s_lo), rounds * average / c.s_lo) * kTileUs[i] + kItemUs * std::max(rounds, 1.);
  if (c.slots > c.n_qtiles) us += kMergeUs[i] + kMergePieceUs[i] * c.s_lo;
  return us;
}
static PfSplits prefill_splits_many(const actqkv_shape& sh, int batch, int m, int k_cap, int cus) {
  const bool two = prefill_two_terms(sh, m);
  PfSplits r{};
  double best = 0.;
  for (int i = 0; i < 3; ++i) {
    const PfSplits c = prefill_cut(sh, batch, m, cus, 1 << i, sh.head_dim == 64 || i > 0 || !two);    // kPfPieces
    const double us = prefill_many_us(sh, batch, m, k_cap, cus, c);
    if (i == 0 || us < best) {
      best = us;
      r = c;
    }
  }
  return r;
}

// A single window with two-term probabilities: another cut than that where these figures, in us, make less of its launch: a
// tile (64 channels 0.75 of it, 128 1.28 times), an item's start and end, and merging.  Against 490 launches measured they are
// 9 % off in the root mean square.
// One-term probabilities keep the cut above: they are rounded to bf16 against the running maximum of the wavefronts that share a
// tile, so another cut rounds them elsewhere and gives outputs that differ by 1e-3 of themselves (two terms have 16 bits: 1e-4 of
// the output at most, where a value lies close to the middle between two).  It costs time: 28 query and 4 KV heads, 640
// tokens, as 70 items of 64 rows for each of the 4, a few more than compute units, 37.8 us, as 35 of 128 rows 29.8.
// Windows that come as groups in one call take the cut of a single one (actqkv_retrieval_attention_windows), so it must not
// cost four of them time by the figures above.  64 channels, 32 query and 8 KV heads, 16 blocks, alone | four, the cut above
// against the other one: 640 tokens 45.5 -> 29.8 | 122 -> 100 us (taken), 768 37.1 -> 34.2 | 106 -> 120 (not), 1200 63 -> 55 | 192 -> 204
// (not); 8 query and 2 KV heads, 3000 tokens 55.6 -> 47.3 | 197 -> 145 (taken).
PfSplits prefill_splits(const actqkv_shape& sh, int batch, int m, int k_cap, int cus) {
  PfSplits r{1, 0, 1, 1, 1};
  if (!prefill_mfma_supported(sh, m)) return r;
  const PfSplits many = prefill_splits_many(sh, batch, m, k_cap, cus);
  if (batch > 1 || !prefill_two_terms(sh, m)) return many;
  constexpr double kTileUs[] = {3.4, 2.23, 1.73};
  constexpr double kItemUs = 2.2;
  const double tile_scale = sh.head_dim == 64 ? 0.75 : 1.28;
  // the window's own key tiles, which the first query tile does not see; those that 256 query rows span
  const double own = m / double(kBlock), span = kPfRows<1> / double(sh.n_q_heads / sh.n_kv_heads) / kBlock;
  auto needs = [&](const PfSplits& c, double retrieved) {
    // key tiles of the last query tile and of an average one
    const double longest = (sh.n_init + sh.n_local) / double(kBlock) + own + retrieved, average = longest - own / 2;
    const double tile = kTileUs[c.ks >> 1] * tile_scale;
    const double rounds = double(sh.n_kv_heads) * c.slots / cus, share = double(c.n_qtiles) / c.slots;
    // the longest item (of the last query tile, or of the last one with a piece less), all of them over the compute units,
    // and the two that share a compute unit where there are some more items than those
    double most = std::ceil(longest / (c.s_lo + (c.rem > 0)));
    if (c.rem > 0) most = std::max(most, std::ceil((longest - c.rem * span) / c.s_lo));
    double us = std::max(most * tile + kItemUs, rounds * (average * share * tile + kItemUs));
    if (rounds > 1.) us = std::max(us, 2 * ((longest - own / rounds) * share * tile + kItemUs));
    if (c.slots > c.n_qtiles) {
      const double kb = kPfRows<1> / c.ks * sh.head_dim * 4 / 1024.;    // of a piece
      us += prefill_merge_after(sh, c.s_lo) ? 5.2 + 0.54 / 1024 * kb * sh.n_kv_heads * c.slots : 1.3 + 2.7 / 64 * kb * c.s_lo;
    }
    return us;
  };
  r = many;
  constexpr int kGroup = 4;
  const double group_us = prefill_many_us(sh, kGroup, m, k_cap, cus, many);
  // (only with fewer wavefronts to a row: in a group a tile's cost per row counts)
  for (int i = 0; 1 << i < many.ks; ++i) {
    const PfSplits c = prefill_cut(sh, 1, m, cus, 1 << i, sh.head_dim == 64 || i > 0);
    // a cut-off leaves a third of k_cap or less, without one there are as many: it has to be better for both
    if (prefill_many_us(sh, kGroup, m, k_cap, cus, c) <= group_us && needs(c, 0.25 * k_cap) < needs(r, 0.25 * k_cap) &&
        needs(c, k_cap) < needs(r, k_cap))
      r = c;
  }
  return r;
}

// Partial results of any call of up to `batch` windows of up to m tokens: pieces exist only while they
// and the query tiles fit the compute units.
size_t prefill_partials_most(const actqkv_shape& sh, int batch, int m) {
  const size_t most = size_t(batch) * sh.n_kv_heads * prefill_mfma_qtiles(sh, m, 4) * kMaxPfSplits;
  return std::min(size_t(kChipCus), most) * kPfPartialFloats * sizeof(float);
}

// hipFuncSetAttribute once per process and variant, from whichever thread comes first
template <int D, int KS, bool kTwoTermP>
static int prefill_lds_attribute() {
  static std::mutex mu;
  static bool attr_set = false;
  std::lock_guard<std::mutex> lock(mu);
  if (attr_set) return ACTQKV_OK;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_prefill_mfma_kernel<D, KS, kTwoTermP>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kPfLdsBytes<D>);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_prefill_mfma_queued_kernel<D, KS, kTwoTermP>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kPfLdsBytes<D>);
  if (e != hipSuccess) return set_error(ACTQKV_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
  attr_set = true;
  return ACTQKV_OK;
}

template <int D, int KS, bool kTwoTermP>
static int launch_pf(PfParams p, int late_per_head, hipStream_t stream, hipStream_t stream_late) {
  if (int rc = prefill_lds_attribute<D, KS, kTwoTermP>()) return rc;
  dim3 grid(p.wgs_per_head * p.n_kv_heads);
  if (p.items_per_head > p.wgs_per_head)
    hipLaunchKernelGGL((attn_prefill_mfma_queued_kernel<D, KS, kTwoTermP>), grid, dim3(kPfThreads), kPfLdsBytes<D>, stream, p);
  else
    hipLaunchKernelGGL((attn_prefill_mfma_kernel<D, KS, kTwoTermP>), grid, dim3(kPfThreads), kPfLdsBytes<D>, stream, p);
  if (int rc = hip_status("attention (prefill, matrix cores)")) return rc;
  if constexpr (kPfPieces<D, KS, kTwoTermP>) if (p.merge_after) {
    const int units = p.n_qtiles * PfPiece<D, KS, kTwoTermP>::kUnits;     // per KV head
    hipLaunchKernelGGL((attn_prefill_merge_kernel<D, KS, kTwoTermP>), dim3(units / kMergeWaves * p.n_kv_heads),
                       dim3(64 * kMergeWaves), 0, stream, p);
    if (int rc = hip_status("attention (prefill, matrix cores, merge)")) return rc;
  }
  if (late_per_head > 0) {
    p.late = 1;
    hipLaunchKernelGGL((attn_prefill_mfma_queued_kernel<D, KS, kTwoTermP>), dim3(late_per_head * p.n_kv_heads), dim3(kPfThreads),
                       kPfLdsBytes<D>, stream_late, p);
    // (if this launch fails after the first one went out, the first team still does all the work, but
    // the queue is not put back to zero: the workspace must be zero-filled again before its next use)
    if (int rc = hip_status("attention (prefill, matrix cores, second team)")) return rc;
  }
  return ACTQKV_OK;
}
template <int D, bool kTwoTermP>
static int launch_pf_ks(int ks, const PfParams& p, int late_per_head, hipStream_t stream, hipStream_t stream_late) {
  return ks == 1   ? launch_pf<D, 1, kTwoTermP>(p, late_per_head, stream, stream_late)
         : ks == 2 ? launch_pf<D, 2, kTwoTermP>(p, late_per_head, stream, stream_late)
                   : launch_pf<D, 4, kTwoTermP>(p, late_per_head, stream, stream_late);
}

// first_cus: compute units the first team may fill (the pieces in `splits` were chosen for it);
// late_cus > 0: a second team of that many workgroups is launched on stream_late by the same
// call, so that the two launches can never disagree about the queue they share.
int launch_attention_prefill_mfma(const actqkv_shape& sh, int batch, int m, const void* q,
                                  const void* k_cache, const void* v_cache, int64_t seq_stride,
                                  int nb_capacity, const int32_t* n_ctx, const int32_t* idx,
                                  const int32_t* n_sel, int k_cap, void* out, float* lse,
                                  const PfSplits& splits, float* scratch, unsigned int* counters,
                                  float scale, int sel_per_head, int first_cus, int late_cus,
                                  hipStream_t stream, hipStream_t stream_late, const SelectInside* inside) {
  PfParams p;
  if (inside != nullptr) p.sel = *inside;
  p.q = static_cast<const uint16_t*>(q);
  p.k_cache = static_cast<const uint16_t*>(k_cache);
  p.v_cache = static_cast<const uint16_t*>(v_cache);
  p.seq_stride = seq_stride;
  p.nb_capacity = nb_capacity;
  p.n_ctx = n_ctx;
  p.idx = idx;
  p.n_sel = n_sel;
  p.sel_per_head = sel_per_head;
  p.k_cap = k_cap;
  p.out = static_cast<uint16_t*>(out);
  p.lse = lse;
  p.part = reinterpret_cast<uint64_t*>(scratch);
  p.counters = counters;
  p.m = m;
  p.n_q_heads = sh.n_q_heads;
  p.n_kv_heads = sh.n_kv_heads;
  p.n_init = sh.n_init;
  p.n_local = sh.n_local;
  p.s_lo = splits.s_lo;
  p.rem = splits.rem;
  p.slots = splits.slots;
  p.n_qtiles = splits.n_qtiles;
  p.scale_log2e = scale * 1.4426950408889634f;
  if (splits.slots < p.n_qtiles || splits.slots != splits.s_lo * p.n_qtiles + splits.rem)
    return set_error(ACTQKV_EINVAL, "prefill attention: inconsistent split of the key tiles");
  if (splits.slots > p.n_qtiles && size_t(batch) * p.n_qtiles * sh.n_kv_heads > kTicketCounters)
    return set_error(ACTQKV_EINVAL, "prefill attention: more split query tiles than ticket counters");
  p.items_per_head = splits.slots * batch;
  // On the first team's own stream a second team would come when all is done: its workgroups belong to the first one
  // then (the cut stays that for first_cus).
  int team_cus = first_cus;
  if (late_cus > 0 && stream_late == stream) {
    team_cus = std::min(first_cus + late_cus, kChipCus);
    late_cus = 0;
  }
  p.wgs_per_head = std::min(p.items_per_head, std::max(1, team_cus / sh.n_kv_heads));
  p.queue = counters + kTicketCounters;
  int late_per_head = late_cus / sh.n_kv_heads;
  if (p.items_per_head <= p.wgs_per_head) late_per_head = 0;   // a workgroup per item: no queue, no second team
  p.merge_after = batch == 1 && prefill_merge_after(sh, splits.s_lo);
  p.team_total = (p.wgs_per_head + late_per_head) * sh.n_kv_heads;
  p.late = 0;
  if (sh.head_dim == 64) return launch_pf_ks<64, true>(splits.ks, p, late_per_head, stream, stream_late);
  return prefill_two_terms(sh, m) ? launch_pf_ks<128, true>(splits.ks, p, late_per_head, stream, stream_late)
                                  : launch_pf_ks<128, false>(splits.ks, p, late_per_head, stream, stream_late);
}

}  // namespace actqkv
