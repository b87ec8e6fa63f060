// Selected blocks from a block store into the working cache (Sec. 3.1: the key-value cache
// may be kept in CPU memory and only what a step retrieves is brought to the GPU).
//
// The store holds the whole context in the blocked layouts of the cache; it is usually pinned
// host memory, which the kernel reads in place over the host link (no staging copy, no host
// synchronisation: the block indices come from actqkv_select on the device).  Block idx[s][j],
// j < n_sel[s], goes to block slot0 + j of the working cache, whose other blocks hold what is
// always resident: the initial tokens before the slots, the local span and the window behind
// them.  Attention then runs on the working cache with the slot numbers as its selection.
//
// grid (kGatherWgs, batch), 256 threads.  A few persistent workgroups walk over the (block, KV
// head) tiles of a sequence; a thread keeps 2 x kGatherBatch 16-byte loads in flight.  The host
// link needs about 100 KB of requests in flight to stay busy (60 GB/s times 2 us); a workgroup
// per tile had fifty times that outstanding, which fills the memory system's queues with slow
// host reads and slows every other kernel on the chip (a 9 us probe kernel beside such a
// gather took 200 us).
#include "common.h"
#include "launch.h"

namespace actqkv {

constexpr int kGatherThreads = 256;
constexpr int kGatherBatch = 4;   // 16-byte loads per tile kind a thread keeps in flight
constexpr int kGatherWgs = 8;
constexpr int kFetchWgs = 16;     // (part of what fetch_listed moves comes from HBM)

// One (block, KV head) tile of keys and of values, by all threads of a workgroup.
__device__ __forceinline__ void move_tile(const u32x4* k_src, const u32x4* v_src, u32x4* k_dst, u32x4* v_dst,
                                          int tile16) {
  for (int c0 = threadIdx.x; c0 < tile16; c0 += kGatherThreads * kGatherBatch) {
    u32x4 kk[kGatherBatch], vv[kGatherBatch];
#pragma unroll
    for (int i = 0; i < kGatherBatch; ++i) {
      const int c = c0 + i * kGatherThreads;
      kk[i] = k_src[c < tile16 ? c : c0];
      vv[i] = v_src[c < tile16 ? c : c0];
    }
#pragma unroll
    for (int i = 0; i < kGatherBatch; ++i) {
      const int c = c0 + i * kGatherThreads;
      if (c < tile16) {
        k_dst[c] = kk[i];
        v_dst[c] = vv[i];
      }
    }
  }
}

__global__ __launch_bounds__(kGatherThreads) void gather_blocks_kernel(
    const u32x4* __restrict__ k_store, const u32x4* __restrict__ v_store, int64_t store_stride16,
    int nb_store, const int32_t* __restrict__ idx, const int32_t* __restrict__ n_sel, int k_cap,
    u32x4* __restrict__ k_cache, u32x4* __restrict__ v_cache, int64_t cache_stride16, int slot0,
    int32_t* __restrict__ idx_slots, int n_kv_heads, int tile16) {
  const int s = blockIdx.y;
  const int e = min(max(n_sel[s], 0), k_cap);
  if (blockIdx.x == 0 && idx_slots != nullptr) {
    for (int j = threadIdx.x; j < k_cap; j += kGatherThreads) {
      const int b = idx[size_t(s) * k_cap + j];
      idx_slots[size_t(s) * k_cap + j] = (j < e && b >= 0 && b < nb_store) ? slot0 + j : -1;
    }
  }
  for (int tile = blockIdx.x; tile < e * n_kv_heads; tile += gridDim.x) {
    const int j = tile / n_kv_heads, hk = tile - j * n_kv_heads;
    const int b = idx[size_t(s) * k_cap + j];
    if (b < 0 || b >= nb_store) continue;
    const size_t src = size_t(s) * store_stride16 + (size_t(b) * n_kv_heads + hk) * tile16;
    const size_t dst = size_t(s) * cache_stride16 + (size_t(slot0 + j) * n_kv_heads + hk) * tile16;
    move_tile(k_store + src, v_store + src, k_cache + dst, v_cache + dst, tile16);
  }
}

// ---- the slots as a cache of the store -----------------------------------------------------
// Neighbouring windows of a pass select mostly the same blocks, and the host link is the narrowest
// way of the chip (57 GB/s; the 960 selections of a 32K pass are 0.5 GB, their distinct blocks a
// tenth of that).  So a block keeps its slot until the slot is needed.  assign_slots gives every
// block that one of a group of windows selects a slot, the one it already has or else the least
// recently used one, and lists the blocks to bring in; fetch_listed moves them, from the store or,
// where the working cache still holds them at their place in the sequence, from there.  Slots that
// the group before used are not given away (its attention may be reading them): with
// n_slots >= 2 n_windows k_cap there is always one to give.
//
// state, int32: slot of every block of the store, or negative [nb_store]; block of every slot, or
// negative [n_slots]; last group that used the slot [n_slots]; number of listed blocks; the list,
// (slot, block) pairs.
struct SlotState {
  int32_t *slot_of_block, *block_of_slot, *used, *count, *list;
  __device__ __forceinline__ SlotState(int32_t* s, int nb_store, int n_slots)
      : slot_of_block(s), block_of_slot(s + nb_store), used(block_of_slot + n_slots), count(used + n_slots), list(count + 1) {}
};

// One workgroup, a thread per selected block.
__global__ __launch_bounds__(kSlotSelections) void assign_slots_kernel(int n_windows, const int32_t* __restrict__ idx,
                                                                       const int32_t* __restrict__ n_sel, int k_cap,
                                                                       int nb_store, int n_slots, int slot0, int group,
                                                                       int32_t* state, int32_t* __restrict__ idx_slots) {
  __shared__ int block[kSlotSelections], slot[kSlotSelections], give[kSlotSelections];
  __shared__ int used[2 * kSlotSelections];
  __shared__ int wave_new[kSlotSelections / 64];
  const SlotState st(state, nb_store, n_slots);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int c = tid; c < n_slots; c += kSlotSelections) used[c] = st.used[c];
  int b = -1;
  if (tid < n_windows * k_cap && tid % k_cap < n_sel[tid / k_cap]) b = idx[tid];
  if (b >= nb_store) b = -1;
  block[tid] = b;
  give[tid] = -1;
  int mine = b >= 0 ? st.slot_of_block[b] : -1;
  if (mine >= n_slots) mine = -1;
  __syncthreads();
  if (mine >= 0) used[mine] = st.used[mine] = group;
  // of the threads that name one missing block, the first brings it in
  int first = tid;
  if (b >= 0 && mine < 0)
    for (first = 0; block[first] != b; ++first) {}
  const bool bring = b >= 0 && mine < 0 && first == tid;
  const unsigned long long votes = __ballot(bring);
  if (lane == 0) wave_new[wave] = __popcll(votes);
  __syncthreads();
  int before = __popcll(votes & ((1ull << lane) - 1ull)), total = 0;
  for (int w = 0; w < kSlotSelections / 64; ++w) {
    before += w < wave ? wave_new[w] : 0;
    total += wave_new[w];
  }
  if (total > 0) {
    // slots in the order they may be given away: longest unused first, then by number
    for (int c = tid; c < n_slots; c += kSlotSelections) {
      const int u = used[c];
      if (u >= group - 1) continue;
      int rank = 0;
      for (int o = 0; o < n_slots; ++o) rank += used[o] < u || (used[o] == u && o < c);
      if (rank < total) give[rank] = c;
    }
    __syncthreads();
    if (bring) {
      mine = give[before];
      if (mine >= 0) {
        const int old = st.block_of_slot[mine];
        if (old >= 0 && old < nb_store) st.slot_of_block[old] = -1;
        st.slot_of_block[b] = mine;
        st.block_of_slot[mine] = b;
        st.used[mine] = group;
      }
      st.list[2 * before] = mine;
      st.list[2 * before + 1] = b;
    }
  }
  slot[tid] = mine;
  __syncthreads();
  if (mine < 0 && b >= 0) mine = slot[first];
  if (tid < n_windows * k_cap) idx_slots[tid] = mine >= 0 ? slot0 + mine : -1;
  if (tid == 0) *st.count = total;
}

__global__ __launch_bounds__(kGatherThreads) void fetch_listed_kernel(
    const u32x4* k_store, const u32x4* v_store, int nb_store, int n_slots, int slot0, u32x4* k_cache, u32x4* v_cache,
    HereRange here0, HereRange here1, int32_t* state, int n_kv_heads, int tile16) {
  const SlotState st(state, nb_store, n_slots);
  const int n = min(*st.count, kSlotSelections);
  for (int tile = blockIdx.x; tile < n * n_kv_heads; tile += gridDim.x) {
    const int j = tile / n_kv_heads, hk = tile - j * n_kv_heads;
    const int to = st.list[2 * j], b = st.list[2 * j + 1];
    if (to < 0 || to >= n_slots || b < 0 || b >= nb_store) continue;
    int from = b;
    const bool in0 = b >= here0.lo && b < here0.hi, here = in0 || (b >= here1.lo && b < here1.hi);
    if (here) from = in0 ? here0.at + (b - here0.lo) : here1.at + (b - here1.lo);
    const size_t src = (size_t(from) * n_kv_heads + hk) * tile16;
    const size_t dst = (size_t(slot0 + to) * n_kv_heads + hk) * tile16;
    move_tile((here ? k_cache : k_store) + src, (here ? v_cache : v_store) + src, k_cache + dst, v_cache + dst, tile16);
  }
}

int launch_gather_cached(const actqkv_shape& sh, int n_windows, const void* k_store, const void* v_store, int nb_store,
                         const int32_t* idx, const int32_t* n_sel, int k_cap, void* k_cache, void* v_cache, int slot0,
                         int n_slots, HereRange here0, HereRange here1, int group, int32_t* state, int32_t* idx_slots,
                         hipStream_t stream) {
  const int tile16 = sh.block_size * sh.head_dim / (sh.dtype == ACTQKV_F32 ? 4 : 8);
  hipLaunchKernelGGL(assign_slots_kernel, dim3(1), dim3(kSlotSelections), 0, stream, n_windows, idx, n_sel, k_cap,
                     nb_store, n_slots, slot0, group, state, idx_slots);
  hipLaunchKernelGGL(fetch_listed_kernel, dim3(kFetchWgs), dim3(kGatherThreads), 0, stream,
                     static_cast<const u32x4*>(k_store), static_cast<const u32x4*>(v_store), nb_store, n_slots, slot0,
                     static_cast<u32x4*>(k_cache), static_cast<u32x4*>(v_cache), here0, here1, state,
                     sh.n_kv_heads, tile16);
  return hip_status("gather_blocks_cached");
}

int launch_gather(const actqkv_shape& sh, int batch, const void* k_store, const void* v_store,
                  int64_t store_stride, int nb_store, const int32_t* idx, const int32_t* n_sel, int k_cap,
                  void* k_cache, void* v_cache, int64_t cache_stride, int slot0, int32_t* idx_slots,
                  hipStream_t stream) {
  const int elem = sh.dtype == ACTQKV_F32 ? 4 : 2;
  const int per16 = 16 / elem;                                   // elements per 16 bytes
  const int tile16 = sh.block_size * sh.head_dim / per16;
  hipLaunchKernelGGL(gather_blocks_kernel, dim3(kGatherWgs, batch), dim3(kGatherThreads), 0, stream,
                     static_cast<const u32x4*>(k_store), static_cast<const u32x4*>(v_store),
                     store_stride / per16, nb_store, idx, n_sel, k_cap, static_cast<u32x4*>(k_cache),
                     static_cast<u32x4*>(v_cache), cache_stride / per16, slot0, idx_slots, sh.n_kv_heads,
                     tile16);
  return hip_status("gather_blocks");
}

}  // namespace actqkv
