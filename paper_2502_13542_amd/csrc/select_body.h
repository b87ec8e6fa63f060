// The selection step as a device function: information density, per-layer budget and the
// tournament for the best blocks (Sec. 4.2, Eq. (11), Eq. (12); Alg. 1, second and third loop).
// Shared by the selection kernels (one workgroup of 1024 threads per sequence, or one wavefront:
// select_wave) and by the decode attention that selects for itself (every workgroup of 512 threads, or
// a wavefront of it, repeats its sequence's selection while the first keys and values are on their way).
//
// The density is a two-pass softmax entropy over the eligible scores (or, as a variant, over the
// scores of the k_cap best blocks once the tournament has found them).  The E best blocks come
// from a tournament: every wavefront bitonic-sorts 64 (score, index) keys at a time across its
// lanes with shuffles and keeps a running sorted top-64; the lists are then merged pairwise
// through LDS, each merge keeping the better 64.  Keys are 64-bit: order-preserving score bits
// above the inverted block index, so equal scores rank by ascending index and the result does
// not depend on timing.
#pragma once

#include "common.h"

namespace actqkv {

__device__ __forceinline__ unsigned long long select_key(float s, int block) {
  s += 0.f;  // -0 -> +0, so the two zeros tie
  uint32_t u = __float_as_uint(s);
  u ^= (u >> 31) ? 0xffffffffu : 0x80000000u;
  return (static_cast<unsigned long long>(u) << 32) | (0xffffffffu - uint32_t(block));
}
// the score a tournament key was made from
__device__ __forceinline__ float key_score(unsigned long long key) {
  uint32_t u = uint32_t(key >> 32);
  u ^= (u >> 31) ? 0x80000000u : 0xffffffffu;
  return __uint_as_float(u);
}
__device__ __forceinline__ unsigned long long shfl64(unsigned long long v, int src) {
  uint32_t lo = __shfl(uint32_t(v), src, 64), hi = __shfl(uint32_t(v >> 32), src, 64);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}
template <int J>
__device__ __forceinline__ unsigned long long lane_xor64(unsigned long long v) {
  const uint32_t lo = lane_xor32<J>(uint32_t(v)), hi = lane_xor32<J>(uint32_t(v >> 32));
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}
__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) {
  return a > b ? a : b;
}
__device__ __forceinline__ unsigned long long umin64(unsigned long long a, unsigned long long b) {
  return a < b ? a : b;
}
// one compare-exchange step of a bitonic network at lane distance J; keep_max per lane
template <int J>
__device__ __forceinline__ unsigned long long bitonic_step(unsigned long long v, bool keep_max) {
  const unsigned long long o = lane_xor64<J>(v);
  return keep_max ? umax64(v, o) : umin64(v, o);
}
// A bitonic sequence across the 64 lanes -> sorted, lane 0 largest.
__device__ __forceinline__ unsigned long long bitonic_merge_desc(unsigned long long v, int lane) {
  v = bitonic_step<32>(v, (lane & 32) == 0);
  v = bitonic_step<16>(v, (lane & 16) == 0);
  v = bitonic_step<8>(v, (lane & 8) == 0);
  v = bitonic_step<4>(v, (lane & 4) == 0);
  v = bitonic_step<2>(v, (lane & 2) == 0);
  v = bitonic_step<1>(v, (lane & 1) == 0);
  return v;
}
// Any 64 keys across the lanes -> sorted, lane 0 largest.  Stage k sorts runs of k lanes,
// alternating in direction ((lane & k) == 0: descending), by steps at distances k/2 .. 1.
template <int K, int J>
__device__ __forceinline__ unsigned long long bitonic_stage(unsigned long long v, int lane) {
  v = bitonic_step<J>(v, ((lane & K) == 0) == ((lane & J) == 0));
  if constexpr (J > 1) v = bitonic_stage<K, J / 2>(v, lane);
  return v;
}
__device__ __forceinline__ unsigned long long bitonic_sort_desc(unsigned long long v, int lane) {
  v = bitonic_stage<2, 1>(v, lane);
  v = bitonic_stage<4, 2>(v, lane);
  v = bitonic_stage<8, 4>(v, lane);
  v = bitonic_stage<16, 8>(v, lane);
  v = bitonic_stage<32, 16>(v, lane);
  v = bitonic_stage<64, 32>(v, lane);      // (lane & 64) == 0 for every lane: descending
  return v;
}

// Cut-off state in, results out (global memory; the arrays have an entry per sequence).
struct SelectIo {
  const float* budget_in;        // B_kv before this layer, or NULL: no cut-off, the k_cap best
  const float* theta_rest_sum;   // R of this layer (with budget_in)
  float* budget_after;           // B_kv - B^l; may be the array budget_in points to
  int32_t* idx;                  // [k_cap] per sequence
  int32_t* n_sel;
  float* theta;                  // optional
  float* budget;                 // optional: B^l
  bool write;                    // false: nothing is stored (the caller reads the result from LDS)
  // The two halves of Alg. 1 as it is printed (every density first, then every budget, then the
  // selections): density_only stops after Eq. (11) and stores theta alone; count_in (per sequence,
  // device memory) is an E^l that was computed elsewhere and replaces Eq. (12) in this call.
  bool density_only = false;
  const int32_t* count_in = nullptr;
};

// What Eq. (12) needs of the cut-off state, requested before anything else.
struct CutoffIn {
  float b_kv, rest;
  int count;
  __device__ __forceinline__ CutoffIn(int s, const SelectIo& io)
      : b_kv(io.budget_in != nullptr ? io.budget_in[s] : 0.f), rest(io.budget_in != nullptr ? io.theta_rest_sum[s] : 0.f),
        count(io.count_in != nullptr ? io.count_in[s] : 0) {}
};
// Eq. (12), the budget update that follows it, and E^l (Alg. 1).
struct Cutoff {
  float theta, b_l, after;
  int e;
  __device__ __forceinline__ Cutoff(float theta_, int n, int k_cap, const CutoffIn& in, const SelectIo& io)
      : theta(theta_), b_l(0.f), after(0.f), e(0) {
    if (io.density_only) return;
    if (io.count_in != nullptr) {
      e = min(max(in.count, 0), min(k_cap, n));
      b_l = float(e);
    } else if (io.budget_in != nullptr) {
      const float den = theta + in.rest;
      b_l = den > 0.f ? theta / den * in.b_kv : in.b_kv;
      e = min(int(fminf(fmaxf(floorf(b_l + 0.5f), 1.f), float(k_cap))), n);
      after = in.b_kv - b_l;
    } else {
      e = min(k_cap, n);
      b_l = float(e);
    }
  }
  // called by one thread
  __device__ __forceinline__ void store(int s, const SelectIo& io) const {
    if (io.theta) io.theta[s] = theta;
    if (io.density_only) return;
    io.n_sel[s] = e;
    if (io.budget) io.budget[s] = b_l;
    if (io.count_in == nullptr && io.budget_in != nullptr && io.budget_after != nullptr) io.budget_after[s] = after;
  }
};
__device__ __forceinline__ int cutoff_count(float theta, int s, int n, int k_cap, const CutoffIn& in, const SelectIo& io) {
  const Cutoff c(theta, n, k_cap, in, io);
  if (io.write) c.store(s, io);
  return c.e;
}

// LDS of one selecting workgroup; after select_body, count and sel[0 .. k_cap) hold the result.
template <int kThreads>
struct SelectLds {
  float red[32];
  unsigned long long lists[kThreads / 64][64];
  int count;
  int sel[64];
};

// Called by all kThreads threads of a workgroup for sequence (row) s; n >= 0 eligible blocks
// starting at nb_begin; sc[i] is the score of block nb_begin + i and is only ever indexed with
// i = threadIdx.x + c * kThreads.  Ends with a barrier.
template <int kThreads, typename Scores>
__device__ __forceinline__ void select_body(const Scores& sc, int s, int n, int nb_begin, int k_cap,
                                            int entropy_topk, const SelectIo& io, SelectLds<kThreads>& lds) {
  constexpr int kWaves = kThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t* my_idx = io.idx + size_t(s) * k_cap;
  const CutoffIn state(s, io);
  if (n == 0) {
    if (io.density_only) {
      if (tid == 0 && io.write && io.theta) io.theta[s] = 0.f;
      __syncthreads();
      return;
    }
    if (tid < k_cap) {
      lds.sel[tid] = -1;
      if (io.write) my_idx[tid] = -1;
    }
    if (tid == 0) {
      lds.count = 0;
      if (io.write) {
        io.n_sel[s] = 0;
        if (io.theta) io.theta[s] = 0.f;
        if (io.budget) io.budget[s] = 0.f;
        if (io.budget_in != nullptr && io.budget_after != nullptr) io.budget_after[s] = io.budget_in[s];
      }
    }
    __syncthreads();
    return;
  }
  if (!entropy_topk) {
    // Eq. (11): theta = -sum P ln P with P = softmax(s) = ln Z + max - sum P s
    float mx = -INFINITY;
    for (int i = tid; i < n; i += kThreads) mx = fmaxf(mx, sc[i]);
    mx = block_max(mx, lds.red);
    float z = 0.f, t = 0.f;
    for (int i = tid; i < n; i += kThreads) {
      float v = sc[i], e = __expf(v - mx);
      z += e;
      t += e * v;
    }
    z = block_sum(z, lds.red);
    t = block_sum(t, lds.red);
    if (tid == 0) lds.count = cutoff_count(fmaxf(logf(z) + mx - t / z, 0.f), s, n, k_cap, state, io);
    if (io.density_only) {
      __syncthreads();
      return;
    }
  }
  // Alg. 1, third loop: the best blocks, best first
  unsigned long long run = 0ull;
  for (int c = 0; c * kThreads < n; ++c) {
    int i = c * kThreads + wave * 64 + lane;
    unsigned long long key = i < n ? select_key(sc[i], nb_begin + i) : 0ull;
    key = bitonic_sort_desc(key, lane);
    if (c == 0) {
      run = key;
    } else {
      run = umax64(run, shfl64(key, 63 - lane));
      run = bitonic_merge_desc(run, lane);
    }
  }
  lds.lists[wave][lane] = run;
  for (int stride = kWaves / 2; stride > 0; stride >>= 1) {
    __syncthreads();
    if (wave < stride) {
      run = umax64(run, lds.lists[wave + stride][63 - lane]);
      run = bitonic_merge_desc(run, lane);
      lds.lists[wave][lane] = run;
    }
  }
  if (entropy_topk && wave == 0) {
    // the same entropy over the scores of the min(k_cap, n) best blocks, which sit in lanes
    // 0 .. of wavefront 0, best first (lane 0 holds the maximum)
    const bool in = lane < min(k_cap, n);
    const float v = in ? key_score(run) : 0.f;
    const float mx = __shfl(v, 0, 64);
    const float e = in ? __expf(v - mx) : 0.f;
    float z = e, t = e * v;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      z += __shfl_xor(z, o, 64);
      t += __shfl_xor(t, o, 64);
    }
    if (lane == 0) lds.count = cutoff_count(fmaxf(logf(z) + mx - t / z, 0.f), s, n, k_cap, state, io);
  }
  __syncthreads();
  if (io.density_only) return;        // (density over the best blocks: the tournament had to run first)
  if (wave == 0 && lane < k_cap) {
    const int b = lane < lds.count ? int(0xffffffffu - uint32_t(run)) : -1;
    lds.sel[lane] = b;
    if (io.write) my_idx[lane] = b;
  }
  __syncthreads();
}

// ---- the same step by ONE wavefront, for rows of at most 64 * kSelWavePerLane scores ----------
// A selection spread over a workgroup couples its wavefronts at a dozen barriers; one wavefront needs
// none.  In the decode attention that selects for itself the others are stuck handing 32 KB of
// load requests each to a full memory pipeline meanwhile; as a launch of its own the step is nothing
// but latency: an instruction that waits for the one before it takes 8 cycles.  Lane l keeps the scores of blocks l, l + 64, ...
// in registers.  The density is two passes over them.  Then the candidates: of a row of more than 64 blocks those that are
// no smaller than the E-th largest of the lanes' maxima (E values at least are that large, so the E best are among them;
// of random scores a few more than E), put one to a lane through LDS in the order of their blocks.  A candidate's place is the
// number of larger ones, counted against every one of them: three instructions each and none that waits.  Up to 4 blocks
// (3 of 62: 3.4 us round by round, 4.0 so), and more than 64 candidates (many equal scores, or E beyond 32), come out
// round by round, 130 cycles each and more where lanes have to search again: every lane knows its three best scores and
// where they are, the best of all lanes is a 32-bit maximum by row shifts and broadcasts (an instruction per
// step), a ballot names its lane (several lanes with equal scores: the lowest block of them), and that lane goes on with
// its next; only a lane that has given all three looks through its registers again, for what comes behind them.
// As a launch of its own, round by round / by candidates: 10 of 60 blocks 3.9 / 3.4 us, 10 of 500 4.5 / 3.6, 32 of 500 8.5 / 4.2,
// 32 of 1000 in 32 rows 12.0 / 5.3 (an empty launch behind another takes 1.7).
// Same ties, same Eq. (11), Eq. (12) as select_body; the sums run in another order.
constexpr int kSelWavePerLane = 16;
constexpr int kSelFewRounds = 4;

struct SelectWaveLds {
  uint32_t key[64];
  int block[64];
};

// How many of the keys of lanes 0 .. count - 1 come before this lane's: larger ones, and equal ones of lower lanes.
// (count is wave-uniform; lanes from count on hold 0.)
__device__ __forceinline__ int wave_place(uint32_t key, int count, int lane) {
  int before = 0;
  for (int j0 = 0; j0 < count; j0 += 16) {
#pragma unroll
    for (int j = j0; j < j0 + 16; ++j) before += uint32_t(__builtin_amdgcn_readlane(int(key), j)) > key;
  }
  // equal keys share a place: then the places do not add up
  const float sum = wave_sum_scalar(lane < count ? float(before) : 0.f);     // (at most 2016: exact)
  if (sum != float(count * (count - 1) / 2)) {
    for (int j = 0; j < count; ++j) before += uint32_t(__builtin_amdgcn_readlane(int(key), j)) == key && j < lane;
  }
  return before;
}

// Called by all 64 lanes of one wavefront; sel[0 .. 64) and *count (LDS) receive the result (sel[i] = -1 from E on), then
// publish() is called, then the global outputs are written if io.write.
template <typename Publish>
__device__ __forceinline__ void select_wave(const float* __restrict__ sc_mem, int s, int n, int nb_begin, int k_cap,
                                            int entropy_topk, const SelectIo& io, SelectWaveLds& lds, int* sel, int* count,
                                            Publish&& publish) {
  constexpr int kPer = kSelWavePerLane, kPart = 4;               // registers are walked a part at a time, as far as n goes
  const int lane = threadIdx.x & 63;
  const int per = __builtin_amdgcn_readfirstlane((n + 63) >> 6);
  float v[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {                               // every load before the first use
    const int b = lane + 64 * i;
    v[i] = b < n ? sc_mem[b] : -INFINITY;
  }
  const CutoffIn in(s, io);
  float theta = 0.f;
  if (!entropy_topk && n > 0) {
    float mx = v[0];
#pragma unroll
    for (int c = 0; c < kPer; c += kPart)
      if (c < per) {
#pragma unroll
        for (int i = c; i < c + kPart; ++i) mx = fmaxf(mx, v[i]);
      }
    mx = wave_max(mx);
    float z = 0.f, t = 0.f;
#pragma unroll
    for (int c = 0; c < kPer; c += kPart)
      if (c < per) {
#pragma unroll
        for (int i = c; i < c + kPart; ++i) {
          const bool in = lane + 64 * i < n;
          const float e = in ? __expf(v[i] - mx) : 0.f;
          z += e;
          t += in ? e * v[i] : 0.f;
        }
      }
    z = wave_sum_scalar(z);
    t = wave_sum_scalar(t);
    theta = fmaxf(logf(z) + mx - t / z, 0.f);
  }
  Cutoff cut(theta, n, k_cap, in, io);
  if (n == 0) cut.b_l = 0.f, cut.after = in.b_kv;                // nothing to select, nothing spent
  int mine = -1;                                                 // lane r: the r-th best block
  uint32_t mine_key = 0u;
  const int rounds = __builtin_amdgcn_readfirstlane(io.density_only && !entropy_topk ? 0 : entropy_topk ? min(k_cap, n) : cut.e);
  sel[lane] = -1;
  if (rounds > 0) {
    uint32_t key[kPer];                                          // 0: no block
#pragma unroll
    for (int i = 0; i < kPer; ++i) key[i] = 0u;
#pragma unroll
    for (int c = 0; c < kPer; c += kPart)
      if (c < per) {
#pragma unroll
        for (int i = c; i < c + kPart; ++i)
          key[i] = lane + 64 * i < n ? max(uint32_t(select_key(v[i], 0) >> 32), 1u) : 0u;
      }
    uint32_t cand = key[0];
    int block = lane, n_cand = rounds > kSelFewRounds ? n : 65;
    if (per > 1 && rounds > kSelFewRounds) {
      uint32_t best = key[0];
#pragma unroll
      for (int c = 0; c < kPer; c += kPart)
        if (c < per) {
#pragma unroll
          for (int i = c; i < c + kPart; ++i) best = max(best, key[i]);
        }
      int before = 0;
#pragma unroll
      for (int j = 0; j < 64; ++j) before += uint32_t(__builtin_amdgcn_readlane(int(best), j)) > best;
      const uint32_t least = ~wave_max_u32(before < rounds ? ~best : 0u);   // (best > 0: every lane has a block)
      n_cand = 0;
#pragma unroll
      for (int c = 0; c < kPer; c += kPart)
        if (c < per) {
#pragma unroll
          for (int i = c; i < c + kPart; ++i) {
            const unsigned long long who = __ballot(key[i] >= least);
            const int at = n_cand + int(__builtin_amdgcn_mbcnt_hi(uint32_t(who >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(who), 0u)));
            if (key[i] >= least && at < 64) {
              lds.key[at] = key[i];
              lds.block[at] = lane + 64 * i;
            }
            n_cand += __builtin_popcountll(who);
          }
        }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      cand = lane < n_cand ? lds.key[lane] : 0u;
      block = lds.block[lane];
    }
    if (n_cand <= 64) {
      const int place = wave_place(cand, n_cand, lane);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (lane < n_cand && place < rounds) {
        sel[place] = nb_begin + block;
        lds.key[place] = cand;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      mine = sel[lane];
      mine_key = lds.key[lane];
    } else {
      // the lane's three best behind (than, at_than) in the order of descending keys and ascending registers, and the
      // registers they are in
      uint32_t best, next, third;
      int at, at2, at3;
      auto find_three = [&](uint32_t than, int at_than) {
        best = next = third = 0u;
        at = at2 = at3 = 0;
#pragma unroll
        for (int c = 0; c < kPer; c += kPart)
          if (c < per) {
#pragma unroll
            for (int i = c; i < c + kPart; ++i) {
              const uint32_t k = key[i] < than || (key[i] == than && i > at_than) ? key[i] : 0u;
              const bool c1 = k > best, c2 = k > next, c3 = k > third;
              at3 = c2 ? at2 : c3 ? i : at3;
              at2 = c1 ? at : c2 ? i : at2;
              at = c1 ? i : at;
              third = max(third, min(next, k));
              next = max(next, min(best, k));
              best = max(best, k);
            }
          }
      };
      find_three(0xffffffffu, -1);
      int left = n > lane ? (n - lane + 63) >> 6 : 0;              // the lane's blocks that have not come out
      for (int r = 0; r < rounds; ++r) {
        const uint32_t top = wave_max_u32(best);
        const unsigned long long who = __ballot(best == top);
        int w = __builtin_ctzll(who);
        if ((who & (who - 1ull)) != 0ull) {
          const uint32_t low = wave_max_u32(best == top ? ~uint32_t(lane + 64 * at) : 0u);
          w = int(~low) & 63;
        }
        const int i_top = __builtin_amdgcn_readlane(at, w), b = w + 64 * i_top;
        mine = lane == r ? nb_begin + b : mine;
        mine_key = lane == r ? top : mine_key;
        const bool won = lane == w;
        best = won ? next : best;
        at = won ? at2 : at;
        next = won ? third : next;
        at2 = won ? at3 : at2;
        third = won ? 0u : third;
        left -= won;
        if (per > 3 && __ballot(won && best == 0u && left > 0) != 0ull) {
          if (won) find_three(top, i_top);
        }
      }
    }
  }
  if (entropy_topk && n > 0) {
    const bool have = lane < rounds;
    const float sv = have ? key_score(static_cast<unsigned long long>(mine_key) << 32) : 0.f;
    const float mx = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sv)));
    const float e = have ? __expf(sv - mx) : 0.f;
    const float z = wave_sum(e), t = wave_sum(e * sv);
    cut = Cutoff(fmaxf(logf(z) + mx - t / z, 0.f), n, k_cap, in, io);
  }
  if (lane >= cut.e) mine = -1;
  sel[lane] = mine;
  if (lane == 0) *count = cut.e;
  publish();
  if (io.write) {
    if (lane < k_cap && !io.density_only) io.idx[size_t(s) * k_cap + lane] = mine;
    if (lane == 0) cut.store(s, io);
  }
}

// The selection of a window's one sequence inside its attention launch (scores NULL: idx and n_sel hold it already).  Every
// workgroup repeats it, by one wavefront, while the others ask for their queries and the initial tokens; the first one writes it
// out.  io.budget_in and io.theta_rest_sum are copies: budget_after and theta, which may be the arrays these were, are written
// while other workgroups still read.
struct SelectInside {
  const float* scores = nullptr;
  int nb_begin = 0, nb_capacity = 0;
  const int32_t* nb_end = nullptr;
  int entropy_topk = 0;
  SelectIo io = {};
  // called by one wavefront
  __device__ __forceinline__ void run(int k_cap, bool write, SelectWaveLds& lds, int* sel, int* count) const {
    const int end = min(max(nb_end[0], nb_begin), nb_capacity);
    SelectIo mine = io;
    mine.write = write;
    select_wave(scores + nb_begin, 0, max(end - nb_begin, 0), nb_begin, k_cap, entropy_topk, mine, lds, sel, count, [] {});
  }
};

// The scores of one sequence as select_body reads them: the first kThreads stay in a register
// per thread for all passes (their load does not wait for anything), the others come from memory.
template <int kThreads>
struct ScoreRow {
  const float* mem;
  float first;
  __device__ __forceinline__ float operator[](int i) const { return i < kThreads ? first : mem[i]; }
};

}  // namespace actqkv
