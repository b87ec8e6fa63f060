// Activation Bias and probe-Query (Sec. 4.1, Eq. (7)-(9)).
//
// The statistics of Eq. (8) reduce over the rows of the window and the weights of Eq. (9)
// over the channels, so the call is a chain of three short kernels over the window's
// queries Q^t [m][d] (a kernel boundary is the cheapest grid-wide dependency on this chip:
// device-scope fences inside a kernel write back and invalidate the whole L2):
//   stats_bias  a workgroup owns a slab of channels for ALL rows: merges the window into the
//               running (n, mean, M2) of Eq. (8), then sums phi of Eq. (7) over its channels,
//               one partial |phi_j|_1 per row and slab;
//   weigh       adds the slabs' partials to a_j = |phi_j|_1, w_j = a_j / sum a, and forms its
//               slab of probe = sum_j w_j q_j of Eq. (9);
//   finish      norm of the probe and its per-KV-head sum.
// All sums are fp32 and are taken in a fixed order, so results are reproducible.
//
// Consecutive windows of one sequence can be taken in one call: Eq. (8) merges the windows
// into the running statistics one after the other, but a merge is a function of each window's
// own (mean, M2) only, so everything else is done for all windows at once (kernels further
// down).  Four launches for n windows instead of 3 n.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "probe_identity.h"

namespace actqkv {

constexpr int kColLanes = 8;      // 16-byte column lanes of a slab

// Sums of values of eight row lanes: x[i] of the wavefront's lanes cl, cl + 8, ..., cl + 56 (column lane cl).  Halves of the
// lanes take halves of the values (an exchange and an addition for two of them): lane bit 5 says which half of the 2 V values,
// bit 4 which half of those; the V / 2 sums left are the same in both lanes of bit 3.
template <int V>
__device__ __forceinline__ void row_lane_sums(const float (&x)[2 * V], float (&out)[V / 2]) {
  float y[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[V + i]), false, false);
    y[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < V / 2; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(y[i]), __float_as_uint(y[V / 2 + i]), false, false);
    const float t = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    out[i] = t + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(t), 0x128, 0xF, 0xF, true));   // row_ror:8
  }
}

// apart[j] = sum over the slab's channels of (q_jc - mean_c)^2 / var_c for the rows of the
// window (Eq. (7) summed over a slab); x holds pass 0 of the rows when there is one pass only.
template <typename T, int RL, int R, typename LoadPass>
__device__ __forceinline__ void bias_partials(typename Vec<T>::raw (&x)[R], LoadPass&& load_pass,
                                              const float* mu_lds, const float* iv_lds,
                                              float* __restrict__ apart, int m, int m_pad, int n_pass,
                                              int cl, int rl) {
  constexpr int V = Vec<T>::N;
  float mu[V], iv[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    mu[v] = mu_lds[cl * V + v];
    iv[v] = iv_lds[cl * V + v];
  }
  for (int pass = 0; pass < n_pass; ++pass) {
    if (n_pass > 1) load_pass(pass);
    const int r0 = (pass * RL + rl) * R;
    float a[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      float f[V];
      Vec<T>::widen(x[i], f);
      float t = 0.f;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        float e = f[v] - mu[v];
        t += e * e * iv[v];
      }
      // the 8 column lanes of a row are neighbouring lanes of one wave
      t += lane_xor_f32<1>(t);
      t += lane_xor_f32<2>(t);
      t += lane_xor_f32<4>(t);
      a[i] = r0 + i < m ? t : 0.f;
    }
    if (cl == 0 && r0 < m_pad) {
#pragma unroll
      for (int i = 0; i < R; i += 4) {
        f32x4 o = {a[i], a[i + 1], a[i + 2], a[i + 3]};
        *reinterpret_cast<f32x4*>(apart + r0 + i) = o;
      }
    }
  }
}

// grid (column slabs of 8*V channels, batch); 8 column lanes x RL row lanes; row lane rl takes rows
// rl R .. rl R + R - 1 of every pass of R RL rows.
// Pass 1 (update != 0): sums of (q - shift), shift = the old mean (or the window's first
// query when there is no history), which keeps the squares free of cancellation; pairwise
// merge into the running mean and M2.  The count n is published by the next kernel of the
// chain (every workgroup here reads the old one).
// Pass 2 (m > 1): apart[slab][j] = sum over the slab's channels of (q_jc - mean_c)^2 / var_c.
// A window of at most R RL rows stays in registers between the passes.  RL and R follow the window's
// length (launch_probe_t): there is one workgroup per slab however long the window is, a pass costs a memory round trip,
// and what a thread does with its rows is instructions one after the other: as many row lanes as the window has use for,
// the fewest rows each.  The probe's three launches with 32 or 64 row lanes of 16 rows each, and what is written below at weigh,
// before / now: 256 tokens, 512 channels 11.9 / 10.1 us, 4096 channels 13.5 / 10.6; 600 tokens 13.9 / 12.6, 17.4 / 14.5; 2048 tokens
// 20.4 / 18.3, 28.2 / 22.6.
template <typename T, int RL, int R>
__global__ __launch_bounds__(kColLanes * RL) void probe_stats_bias_kernel(const T* __restrict__ q_win,
                                                               float* __restrict__ stats,
                                                               float* __restrict__ scratch, int update,
                                                               int m, int m_pad, int d, float eps,
                                                               size_t stats_stride,
                                                               size_t scratch_stride) {
  constexpr int V = Vec<T>::N;
  constexpr int SLAB = kColLanes * V;
  typedef typename Vec<T>::raw raw_t;
  __shared__ __attribute__((aligned(16))) float red[2][RL / 8][SLAB];
  __shared__ float mu_lds[SLAB], iv_lds[SLAB];
  const int s = blockIdx.y;
  const T* q = q_win + size_t(s) * m * d;
  float* st = stats + size_t(s) * stats_stride;
  float* apart = scratch + size_t(s) * scratch_stride + size_t(blockIdx.x) * m_pad;
  const int cl = threadIdx.x % kColLanes, rl = threadIdx.x / kColLanes;
  const int ch0 = blockIdx.x * SLAB + cl * V;
  const bool col_ok = ch0 < d;
  // the old statistics and the window's first query are requested before the queries: the counter of
  // outstanding loads is in order, and asked for later they would be a round trip of their own
  const float n_old = st[0];
  const int col = threadIdx.x, ch = blockIdx.x * SLAB + col;      // the first threads: the channel they merge
  float mean_a = 0.f, m2_a = 0.f, first = 0.f;
  if (col < SLAB && ch < d) {
    mean_a = st[4 + ch];
    m2_a = st[4 + d + ch];
    first = to_f32(q[ch]);
  }
  float c[V], c_first[V];
#pragma unroll
  for (int v = 0; v < V; ++v) c[v] = c_first[v] = 0.f;
  if (update && col_ok) {
#pragma unroll
    for (int v = 0; v < V; ++v) c[v] = st[4 + ch0 + v];
    Vec<T>::load(q + ch0, c_first);
  }
  const int n_pass = (m + RL * R - 1) / (RL * R);

  raw_t x[R];
  auto load_pass = [&](int pass) {
#pragma unroll
    for (int i = 0; i < R; ++i) {   // all loads first: they overlap
      const int r = (pass * RL + rl) * R + i;
      x[i] = Vec<T>::load_raw(q + size_t(r < m ? r : 0) * d + (col_ok ? ch0 : 0));
    }
  };
  load_pass(0);

  if (update) {
    float s1[V], s2[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      c[v] = n_old > 0.f ? c[v] : c_first[v];
      s1[v] = s2[v] = 0.f;
    }
    for (int pass = 0; pass < n_pass; ++pass) {
      if (pass > 0) load_pass(pass);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if ((pass * RL + rl) * R + i < m) {
          float f[V];
          Vec<T>::widen(x[i], f);
#pragma unroll
          for (int v = 0; v < V; ++v) {
            float t = f[v] - c[v];
            s1[v] += t;
            s2[v] += t * t;
          }
        }
      }
    }
    float both[2 * V], sum[V / 2];
#pragma unroll
    for (int v = 0; v < V; ++v) both[v] = s1[v], both[V + v] = s2[v];
    row_lane_sums<V>(both, sum);
    const int lane = threadIdx.x & 63;
    if ((lane & 8) == 0) {
      float* to = &red[lane >> 5][threadIdx.x >> 6][cl * V + ((lane >> 4) & 1) * (V / 2)];
#pragma unroll
      for (int i = 0; i < V / 2; ++i) to[i] = sum[i];
    }
    __syncthreads();
  }
  {
    if (col < SLAB && ch >= d) mu_lds[col] = iv_lds[col] = 0.f;
    if (col < SLAB && ch < d) {
      float mean, m2, n_new;
      if (update) {
        float t1 = 0.f, t2 = 0.f;
#pragma unroll
        for (int k = 0; k < RL / 8; ++k) {
          t1 += red[0][k][col];
          t2 += red[1][k][col];
        }
        const float nb = float(m);
        n_new = n_old + nb;
        const float shift = n_old > 0.f ? mean_a : first;
        const float mean_b = shift + t1 / nb;
        const float m2_b = fmaxf(t2 - t1 * t1 / nb, 0.f);
        const float delta = mean_b - mean_a;
        mean = n_old > 0.f ? mean_a + delta * (nb / n_new) : mean_b;
        m2 = n_old > 0.f ? m2_a + m2_b + delta * delta * (n_old * nb / n_new) : m2_b;
        st[4 + ch] = mean;
        st[4 + d + ch] = m2;
      } else {
        n_new = n_old;
        mean = mean_a;
        m2 = m2_a;
      }
      const float var = n_new > 1.f ? m2 / (n_new - 1.f) : 0.f;
      mu_lds[col] = mean;
      iv_lds[col] = 1.f / fmaxf(var, eps);
    }
  }
  if (m == 1) return;   // a single token is its own probe: no weights needed
  __syncthreads();

  bias_partials<T, RL, R>(x, load_pass, mu_lds, iv_lds, apart, m, m_pad, n_pass, cl, rl);
}

// ---- consecutive windows of one sequence in one call
// With many windows in a call there is enough work to read the queries the way they lie in
// memory: a workgroup takes 64 whole rows (rows x all channels, 16-byte loads of consecutive
// lanes are consecutive in memory), where the one-window kernels above take 128-byte column
// slabs of all rows.  Reductions over rows leave one partial per 64-row chunk, summed in chunk
// order by the next kernel; reductions over channels are whole-row sums inside a wavefront, so
// the bias weight a_j of a row is complete while the row is still in registers and Eq. (9)'s
// weighted sum is taken in the same pass: the queries are read twice, not three times.
//   rows_moments     (chunks x windows): sums of (q - c) and (q - c)^2 per channel over the
//                    chunk's rows, c = the window's first query, for a single window the old mean
//                    where there is one;
//   chain_stats      per channel: every window's own (mean, M2) from its chunks, then the merges
//                    of Eq. (8) window after window, which give the (mean, 1/var) each window
//                    sees; stores the final statistics;
//   rows_bias_weigh  (chunks x windows): a_j = |phi_j|_1 per row, sum of a_j q_j over the chunk's
//                    rows per channel, sum of a_j;
//   chain_finish     per window: probe = sum over chunks / sum of a_j, norm, per-KV-head sum,
//                    weights.
// Scratch per call, in floats: part [n][chunks][2][d], stat [n][3][d] (mean, 1/var, the window's
// own mean), pprobe [n][chunks][d], asum [n][chunks rounded up to 16], a [n][m rounded up to 16].
constexpr int kRmThreads = 256;

// The point a channel's sums are about.  (An old mean that is infinite or NaN would make the window's own mean NaN too, and that
// one is the probe where the bias weights are NaN.)
__device__ __forceinline__ float moments_about(float first, float n_run, float old_mean) {
  return n_run > 0.f && fabsf(old_mean) <= 3.4028235e38f ? old_mean : first;
}

// grid (chunks, windows, ceil(d / V / cols)): a workgroup takes `cols` 16-byte channel groups (64 .. 256) of the chunk's
// rows, row lane rl of 256 / cols the rows rl, rl + lanes, ..., and the lanes' sums are added in their order.  A compute
// unit does not get more than 35-50 GB/s, so the channels are cut finer where there are few chunks; 16 rows are
// requested together.
template <typename T>
__global__ __launch_bounds__(kRmThreads) void probe_rows_moments_kernel(const T* __restrict__ q_win,
                                                                        const float* __restrict__ stats,
                                                                        float* __restrict__ part, int m, int d,
                                                                        int n_chunks, int cols) {
  constexpr int V = Vec<T>::N;
  constexpr int R = 16;                              // rows requested together
  typedef typename Vec<T>::raw raw_t;
  __shared__ f32x4 sums[kRmThreads * 2 * V / 4];
  const int rc = blockIdx.x, w = blockIdx.y;
  const T* q = q_win + size_t(w) * m * d;
  const int rls = kRmThreads / cols, rl = int(threadIdx.x) / cols, col = int(threadIdx.x) - rl * cols;
  const int ch = (int(blockIdx.z) * cols + col) * V;
  const bool ok = ch < d && rl < rls;
  float c[V], s1[V], s2[V], mean[V];
  const bool single = gridDim.y == 1;
  const float n_run = single ? stats[0] : 0.f;
  Vec<T>::load(q + (ok ? ch : 0), c);
#pragma unroll
  for (int v = 0; v < V; ++v) mean[v] = single ? stats[4 + (ok ? ch : 0) + v] : 0.f;   // (asked for with the rest, used or not)
#pragma unroll
  for (int v = 0; v < V; ++v) s1[v] = s2[v] = 0.f;
  const int r0 = rc * kRowChunk, r1 = min(r0 + kRowChunk, m);
  raw_t x[R];
  auto load_rows = [&](int r) {
#pragma unroll
    for (int i = 0; i < R; ++i) x[i] = Vec<T>::load_raw(q + size_t(min(r + i * rls, r1 - 1)) * d + (ok ? ch : 0));
  };
  load_rows(r0 + rl);
  __builtin_amdgcn_sched_barrier(0);                 // (n sums of squares about a point lose n * its distance^2)
#pragma unroll
  for (int v = 0; v < V; ++v) c[v] = moments_about(c[v], n_run, mean[v]);
  for (int r = r0 + rl; r < r1; r += R * rls) {
    if (r != r0 + rl) load_rows(r);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (r + i * rls < r1) {
        float f[V];
        Vec<T>::widen(x[i], f);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float t = f[v] - c[v];
          s1[v] += t;
          s2[v] += t * t;
        }
      }
    }
  }
  if (rls > 1) {
    f32x4* mine = sums + threadIdx.x * (2 * V / 4);
#pragma unroll
    for (int v = 0; v < V; v += 4) {
      mine[v / 4] = f32x4{s1[v], s1[v + 1], s1[v + 2], s1[v + 3]};
      mine[(V + v) / 4] = f32x4{s2[v], s2[v + 1], s2[v + 2], s2[v + 3]};
    }
    __syncthreads();
    if (rl > 0) return;
    for (int o = 1; o < rls; ++o) {
      const f32x4* from = sums + (o * cols + col) * (2 * V / 4);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        s1[v] += from[v / 4][v % 4];
        s2[v] += from[(V + v) / 4][v % 4];
      }
    }
  }
  if (!ok) return;
  float* p1 = part + (size_t(w) * n_chunks + rc) * 2 * d;
#pragma unroll
  for (int v = 0; v < V; v += 4) {
    *reinterpret_cast<f32x4*>(p1 + ch + v) = f32x4{s1[v], s1[v + 1], s1[v + 2], s1[v + 3]};
    *reinterpret_cast<f32x4*>(p1 + d + ch + v) = f32x4{s2[v], s2[v + 1], s2[v + 2], s2[v + 3]};
  }
}

// grid (d / 32), 1024 threads = 32 channels x 32 lanes.  The chunk sums of every window become the window's own
// (mean, M2) in LDS: with fewer than 32 windows several lanes share one (32 / n, rounded down to a power of two), lane
// u of them the chunks u, u + share, ..., whose sums are added in lane order.  Then lane 0 merges the windows into the
// running statistics in window order (the merge of Eq. (8), as in probe_stats_bias_kernel): one window after the other, so
// its quotients of counts and the 1/var that follow from it are made by all lanes, before and after.  The count is published
// by the next kernel (every thread here reads the old one; `before` is what launches of this call have added to it).  At most
// kChainTile windows a launch: 132 KB of LDS, and 8 KB for the lanes' sums.
// With both in the loop 11.6 us for 32 windows of 256 tokens with 512 channels in fp32, 5.8 so; 18.5 for 32 of 512 with 4096
// beside the attention, 12.4 so.  The tiles in one launch, as a loop: a window of 4096 tokens with 512 channels 24.3 instead of 23.7.
constexpr int kChainTile = 512;
template <typename T>
__global__ __launch_bounds__(1024) void probe_chain_stats_kernel(const T* __restrict__ q_win,
                                                                 const float* __restrict__ part,
                                                                 float* __restrict__ stats,
                                                                 float* __restrict__ stat_out, int n, int m,
                                                                 int d, int n_chunks, float eps, float before, int single) {
  extern __shared__ float wm[];                      // [n][2][32]: the windows' own mean and M2, then the running ones | [n][2]
  __shared__ float lane_sum[2][32][32];
  constexpr int kBatch = 8;                          // chunks requested together
  const int cl = threadIdx.x & 31, wl = threadIdx.x >> 5;
  const int ch = blockIdx.x * 32 + cl;
  const float nb = float(m);
  int share = 1;
  while (share * 2 * n <= 32) share *= 2;
  const int u = wl % share;
  float mean = 0.f, m2 = 0.f;
  const float n_run = stats[0] + before;
  if (wl == 0 && ch < d) mean = stats[4 + ch], m2 = stats[4 + d + ch];   // (in flight meanwhile)
  float* count_of = wm + size_t(n) * 64;             // nb / n_new, n_old nb / n_new
  for (int w0 = 0; w0 < n; w0 += 32 / share) {
    const int w = w0 + wl / share;
    const bool live = w < n && ch < d;
    float t1 = 0.f, t2 = 0.f;
    const float first = live ? to_f32(q_win[size_t(w) * m * d + ch]) : 0.f;
    if (live) {
      const float* p1 = part + size_t(w) * n_chunks * 2 * d + ch;
      for (int rc = u; rc < n_chunks; rc += kBatch * share) {
        float a[kBatch], b[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {           // all loads first: they overlap
          const int c = rc + i * share < n_chunks ? rc + i * share : rc;
          a[i] = p1[size_t(c) * 2 * d];
          b[i] = p1[size_t(c) * 2 * d + d];
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          t1 += rc + i * share < n_chunks ? a[i] : 0.f;
          t2 += rc + i * share < n_chunks ? b[i] : 0.f;
        }
      }
    }
    if (share > 1) {                                 // (one round: all windows have their lanes)
      lane_sum[0][wl][cl] = t1;
      lane_sum[1][wl][cl] = t2;
      __syncthreads();
      if (u == 0)
        for (int o = 1; o < share; ++o) {
          t1 += lane_sum[0][wl + o][cl];
          t2 += lane_sum[1][wl + o][cl];
        }
    }
    if (live && u == 0) {
      const float mean_b = (single ? moments_about(first, n_run, mean) : first) + t1 / nb;   // (a single window: lane 0 alone comes here)
      wm[(w * 2 + 0) * 32 + cl] = mean_b;
      wm[(w * 2 + 1) * 32 + cl] = fmaxf(t2 - t1 * t1 / nb, 0.f);
      stat_out[size_t(w) * 3 * d + 2 * d + ch] = mean_b;
    }
  }
  for (int w = threadIdx.x; w < n; w += 1024) {
    const float n_old = n_run + float(w) * nb, n_new = n_old + nb;
    count_of[2 * w] = nb / n_new;
    count_of[2 * w + 1] = n_old * nb / n_new;
  }
  __syncthreads();
  if (wl == 0 && ch < d) {
    for (int w = 0; w < n; ++w) {
      const float mean_b = wm[(w * 2 + 0) * 32 + cl], m2_b = wm[(w * 2 + 1) * 32 + cl];
      if (w > 0 || n_run > 0.f) {
        const float delta = mean_b - mean;
        mean += delta * count_of[2 * w];
        m2 += m2_b + delta * delta * count_of[2 * w + 1];
      } else {
        mean = mean_b;
        m2 = m2_b;
      }
      wm[(w * 2 + 0) * 32 + cl] = mean;
      wm[(w * 2 + 1) * 32 + cl] = m2;
    }
    stats[4 + ch] = mean;
    stats[4 + d + ch] = m2;
  }
  __syncthreads();
  if (ch >= d) return;
  for (int w = wl; w < n; w += 32) {
    const float n_new = n_run + float(w) * nb + nb;
    const float var = n_new > 1.f ? wm[(w * 2 + 1) * 32 + cl] / (n_new - 1.f) : 0.f;
    float* o = stat_out + size_t(w) * 3 * d + ch;
    o[0] = wm[(w * 2 + 0) * 32 + cl];
    o[d] = 1.f / fmaxf(var, eps);
  }
}

// grid (chunks, windows), NW wavefronts; wavefront v takes rows v, v + NW, ... of the chunk, a lane
// the 16-byte groups lane, lane + 64, ... of a row (NI of them: d <= 64 * NI * V channels), R rows at a time and the
// next R in flight meanwhile (8 groups of each; with NI = 1 the chunk is R * NW rows and nothing follows).  For rows that are
// not there the chunk's last one is requested once more (branches around the loads: 4 windows of 512 tokens with 4096 channels
// 36.4 us instead of 35.3), and no weight is applied (0 times an infinite query is NaN).  NI is the least that holds a row:
// with room for 4096 channels whatever the row (and half of the lanes of rows_moments idle, 8 rows at once), the four launches
// of 32 windows of 256 tokens with 512 channels took 49 us, 26 so; of 4 windows of 512 tokens with 4096 channels 50, 36 (chunks of 32 rows).
// LDS: mean and 1/var of the window (2 kRowLen floats), reused for the sum over the wavefronts.
template <typename T, int NI, int NW, int R>
__global__ __launch_bounds__(64 * NW) void probe_rows_bias_weigh_kernel(
    const T* __restrict__ q_win, const float* __restrict__ stat_in, float* __restrict__ stats, float add_count,
    int mean_pooling, float* __restrict__ pprobe, float* __restrict__ asum, float* __restrict__ a_rows, int m,
    int m_pad, int d, int rows, int n_chunks, int asum_stride) {
  constexpr int V = Vec<T>::N;
  typedef typename Vec<T>::raw raw_t;
  constexpr int kRowLen = 64 * NI * V;                             // channels a wavefront covers
  extern __shared__ __attribute__((aligned(16))) float rw_lds[];   // [max(2 kRowLen, NW / 2 d)]
  __shared__ float red[NW];
  const int rc = blockIdx.x, w = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const T* q = q_win + size_t(w) * m * d;
  float* mu = rw_lds;
  float* iv = rw_lds + kRowLen;
  const int r0 = rc * rows, r1 = min(r0 + rows, m);
  auto load_rows = [&](int r, raw_t (&x)[R][NI]) {
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = (lane + 64 * i) * V;
        x[j][i] = Vec<T>::load_raw(q + size_t(min(r + j * NW, r1 - 1)) * d + (c < d ? c : 0));
      }
  };
  raw_t x[R][NI];
  load_rows(r0 + wave, x);
  // channels past d (rows shorter than a wavefront's 64 * NI * V) get mean 0 and weight 0
  for (int i = threadIdx.x * 4; i < kRowLen; i += 64 * NW * 4) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f32x4*>(mu + i) = i < d ? *reinterpret_cast<const f32x4*>(stat_in + size_t(w) * 3 * d + i) : zero;
    *reinterpret_cast<f32x4*>(iv + i) = i < d ? *reinterpret_cast<const f32x4*>(stat_in + size_t(w) * 3 * d + d + i) : zero;
  }
  if (add_count != 0.f && rc == 0 && w == 0 && threadIdx.x == 0) stats[0] += add_count;
  __syncthreads();
  float acc[NI][V];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[i][v] = 0.f;
  float a_sum = 0.f;
  for (int r = r0 + wave; r < r1; r += R * NW) {
    // the wavefront's next rows are requested before these are used
    raw_t xn[R][NI];
    if constexpr (NI > 1) load_rows(r + R * NW, xn);
    float t[R];
#pragma unroll
    for (int j = 0; j < R; ++j) t[j] = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = (lane + 64 * i) * V;
      f32x4 mu4[V / 4], iv4[V / 4];
#pragma unroll
      for (int u = 0; u < V / 4; ++u) {
        mu4[u] = *reinterpret_cast<const f32x4*>(mu + c + 4 * u);
        iv4[u] = *reinterpret_cast<const f32x4*>(iv + c + 4 * u);
      }
#pragma unroll
      for (int j = 0; j < R; ++j) {
        float f[V];
        Vec<T>::widen(x[j][i], f);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float e = f[v] - mu4[v >> 2][v & 3];
          t[j] += e * e * iv4[v >> 2][v & 3];
        }
      }
    }
    float a[R];                                      // |phi_j|_1 of Eq. (7), the row's weight before normalisation
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int row = r + j * NW;
      a[j] = wave_sum(t[j]);
      if (mean_pooling) a[j] = 1.f;
      if (row >= r1) a[j] = 0.f;
      if (lane == 0 && row < r1) a_rows[size_t(w) * m_pad + row] = a[j];
      a_sum += a[j];
    }
#pragma unroll
    for (int j = 0; j < R; ++j)
      if (r + j * NW < r1) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float f[V];
          Vec<T>::widen(x[j][i], f);
#pragma unroll
          for (int v = 0; v < V; ++v) acc[i][v] += a[j] * f[v];
        }
      }
    if constexpr (NI == 1) break;
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) x[j][i] = xn[j][i];
  }
  // sum over the wavefronts, in a fixed order: halves onto halves
  __syncthreads();                                   // mean and 1/var are no longer needed
  if (lane == 0) red[wave] = a_sum;
  auto put = [&](float* dst) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = (lane + 64 * i) * V;
      if (c < d) {
#pragma unroll
        for (int v = 0; v < V; v += 4)
          *reinterpret_cast<f32x4*>(dst + c + v) = f32x4{acc[i][v], acc[i][v + 1], acc[i][v + 2], acc[i][v + 3]};
      }
    }
  };
  auto add = [&](const float* src) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = (lane + 64 * i) * V;
      if (c < d) {
#pragma unroll
        for (int v = 0; v < V; ++v) acc[i][v] += src[c + v];
      }
    }
  };
#pragma unroll
  for (int h = NW / 2; h > 0; h /= 2) {
    if (wave >= h && wave < 2 * h) put(rw_lds + (wave - h) * d);
    __syncthreads();
    if (wave < h) add(rw_lds + wave * d);
    if (h > 1) __syncthreads();
  }
  if (wave == 0) {
    put(pprobe + (size_t(w) * n_chunks + rc) * d);
    if (lane == 0) {
#pragma unroll
      for (int h = NW / 2; h > 0; h /= 2)
#pragma unroll
        for (int v = 0; v < h; ++v) red[v] += red[v + h];
      asum[size_t(w) * asum_stride + rc] = red[0];
    }
  }
}

// Per window: the sums over its chunks, Eq. (9)'s normalisation (uniform weights, i.e. the window's mean, if every bias
// is zero) and the weights; with one workgroup per window also what probe_finish computes.  grid (windows, slabs): a
// workgroup takes d / slabs channels, four to a thread and the chunks shared among 4096 / d threads (the one of u takes u,
// u + share, ..., added in the order of u: whatever the slabs, the sums are the same).  All that bounds it is round trips: a thread
// per channel and the chunks eight at a time, the sum of a_j one scalar load after the other, took 15.0 us for one
// window of 4096 tokens with 1024 channels (64 chunks), now 4.8.
constexpr int kCfThreads = 1024;
__global__ __launch_bounds__(kCfThreads) void probe_chain_finish_kernel(
    const float* __restrict__ pprobe, const float* __restrict__ asum, const float* __restrict__ a_rows,
    const float* __restrict__ stat_in, float* __restrict__ probe_out, float* __restrict__ probe_kv_out,
    float* __restrict__ probe_norm_out, float* __restrict__ weights_out, int m, int m_pad, int d, int n_chunks,
    int asum_stride, int n_q_heads, int n_kv_heads, int head_dim) {
  __shared__ float red[32];
  __shared__ f32x4 part[kCfThreads];
  extern __shared__ __attribute__((aligned(16))) float probe_lds[];   // [d]
  const int w = blockIdx.x, per = d / int(gridDim.y), groups = per / 4, share = 4 * kCfThreads / d;
  const int u = int(threadIdx.x) / groups, ch = int(blockIdx.y) * per + (int(threadIdx.x) - u * groups) * 4;
  const float* mine = pprobe + size_t(w) * n_chunks * d + ch;
  f32x4 t = {0.f, 0.f, 0.f, 0.f};
  auto add_chunks = [&](auto batch) {
    constexpr int kBatch = decltype(batch)::value;
    for (int rc = u; rc < n_chunks; rc += kBatch * share) {
      f32x4 x[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i)               // all loads first: they overlap
        x[i] = *reinterpret_cast<const f32x4*>(mine + size_t(rc + i * share < n_chunks ? rc + i * share : rc) * d);
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (rc + i * share < n_chunks) t += x[i];
    }
  };
  if (u < share) {
    if (n_chunks <= share) add_chunks(std::integral_constant<int, 1>{});
    else if (n_chunks <= 8 * share) add_chunks(std::integral_constant<int, 8>{});
    else add_chunks(std::integral_constant<int, 16>{});
  }
  float total = 0.f;
  for (int rc = threadIdx.x & 63; rc < n_chunks; rc += 64) total += asum[size_t(w) * asum_stride + rc];
  total = wave_sum(total);
  const bool uniform = !(total > 0.f);
  const float inv = uniform ? 0.f : 1.f / total;
  if (weights_out != nullptr) {
    for (int j = int(blockIdx.y * blockDim.x + threadIdx.x); j < m; j += int(gridDim.y * blockDim.x))
      weights_out[size_t(w) * m + j] = uniform ? 1.f / float(m) : a_rows[size_t(w) * m_pad + j] * inv;
  }
  if (share > 1) {
    part[threadIdx.x] = t;
    __syncthreads();
    if (u == 0)
      for (int o = 1; o < min(share, n_chunks); ++o) t += part[o * groups + threadIdx.x];
  }
  float ss = 0.f;
  if (u == 0) {
    t = uniform ? *reinterpret_cast<const f32x4*>(stat_in + size_t(w) * 3 * d + 2 * d + ch) : t * inv;
    *reinterpret_cast<f32x4*>(probe_out + size_t(w) * d + ch) = t;
    *reinterpret_cast<f32x4*>(probe_lds + ch) = t;
    ss = (t.x * t.x + t.y * t.y) + (t.z * t.z + t.w * t.w);
  }
  if (gridDim.y > 1) return;                         // (the scoring launch forms the norm and the per-KV-head sum)
  ss = block_sum(ss, red);                           // also orders the LDS writes before the reads below
  if (threadIdx.x == 0) probe_norm_out[w] = sqrtf(ss);
  const int g = n_q_heads / n_kv_heads;
  float* probe_kv = probe_kv_out + size_t(w) * n_kv_heads * head_dim;
  for (int e = threadIdx.x; e < n_kv_heads * head_dim; e += kCfThreads) {
    const int hk = e / head_dim, dd = e - hk * head_dim;
    float kv = 0.f;
    for (int i = 0; i < g; ++i) kv += probe_lds[(hk * g + i) * head_dim + dd];
    probe_kv[e] = kv;
  }
}

constexpr int kWeighRows = 8;    // rows a thread takes per pass

// grid (column slabs of 8*V channels, batch); 8 column lanes x RL row lanes.
// Every workgroup adds the slabs' partials up to a_j (slab order), turns them into the
// weights of Eq. (9) and sums w_j q_j over all rows for its channels.  The queries of the
// first pass are requested before the partials, so both are in flight together.  The partials are read four rows to a
// thread, at most 16 slabs to a thread while there are threads for the rest (instead of a row to a thread and all slabs one
// after the other, four times as many loads; with one workgroup in four barriers more for 8 slabs: 0.6 us slower).
template <typename T, int RL>
__global__ __launch_bounds__(kColLanes * RL) void probe_weigh_kernel(const T* __restrict__ q_win,
                                                          const float* __restrict__ scratch,
                                                          float* __restrict__ stats, int add_count,
                                                          int mean_pooling,
                                                          float* __restrict__ probe_out,
                                                          float* __restrict__ weights_out, int m,
                                                          int m_pad, int n_slabs, int d,
                                                          size_t scratch_stride, size_t stats_stride) {
  constexpr int V = Vec<T>::N;
  constexpr int SLAB = kColLanes * V;
  constexpr int kThreads = kColLanes * RL, kRows = RL * kWeighRows;      // threads, rows of a pass
  typedef typename Vec<T>::raw raw_t;
  __shared__ float red[32];
  __shared__ __attribute__((aligned(16))) float w_lds[kMaxWindow];
  __shared__ f32x4 part[kThreads];
  __shared__ float buf[kThreads / 64][SLAB];
  const int s = blockIdx.y;
  const T* q = q_win + size_t(s) * m * d;
  const float* apart = scratch + size_t(s) * scratch_stride;
  const int cl = threadIdx.x % kColLanes, rl = threadIdx.x / kColLanes;
  const int ch0 = blockIdx.x * SLAB + cl * V;
  const bool col_ok = ch0 < d;
  if (add_count && blockIdx.x == 0 && threadIdx.x == 0) stats[size_t(s) * stats_stride] += float(m);

  raw_t x[kWeighRows];
  auto load_pass = [&](int pass) {
#pragma unroll
    for (int i = 0; i < kWeighRows; ++i) {
      const int r = pass * kRows + rl * kWeighRows + i;
      x[i] = Vec<T>::load_raw(q + size_t(r < m ? r : 0) * d + (col_ok ? ch0 : 0));
    }
  };
  load_pass(0);

  // thread (group of four rows, slab lane u): slabs u, u + share, ...  (m_pad is a multiple of 16; rows from m on hold 0)
  float tsum = 0.f;
  if (!mean_pooling) {
    constexpr int kBatch = 16;
    const int groups = m_pad / 4, u = int(threadIdx.x) / groups;
    const int share = max(min(kThreads / groups, (n_slabs + kBatch - 1) / kBatch), 1);
    for (int g = int(threadIdx.x) - u * groups; g < groups && u < share; g += kThreads) {
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
      for (int s0 = u; s0 < n_slabs; s0 += kBatch * share) {
        f32x4 p[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i)             // all loads first: they overlap
          p[i] = *reinterpret_cast<const f32x4*>(apart + size_t(s0 + i * share < n_slabs ? s0 + i * share : s0) * m_pad + 4 * g);
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
          if (s0 + i * share < n_slabs) t += p[i];
      }
      if (share == 1) {
        *reinterpret_cast<f32x4*>(w_lds + 4 * g) = t;
        tsum += (t.x + t.y) + (t.z + t.w);
      } else {
        part[threadIdx.x] = t;
      }
    }
    if (share > 1) {
      __syncthreads();
      if (int(threadIdx.x) < groups) {
        f32x4 t = part[threadIdx.x];
        for (int o = 1; o < min(share, n_slabs); ++o) t += part[o * groups + threadIdx.x];
        *reinterpret_cast<f32x4*>(w_lds + 4 * threadIdx.x) = t;
        tsum = (t.x + t.y) + (t.z + t.w);
      }
    }
  }
  const float total = block_sum(tsum, red);          // |Phi|_1; orders the LDS writes as well
  const float inv_total = total > 0.f ? 1.f / total : 0.f;
  const float uniform = 1.f / float(m);

  float acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0.f;
  const int n_pass = (m + kRows - 1) / kRows;
  for (int pass = 0; pass < n_pass; ++pass) {
    if (pass > 0) load_pass(pass);
#pragma unroll
    for (int i = 0; i < kWeighRows; ++i) {
      const int r = pass * kRows + rl * kWeighRows + i;
      const float w = r < m ? (total > 0.f ? w_lds[r] * inv_total : uniform) : 0.f;
      float f[V];
      Vec<T>::widen(x[i], f);
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += w * f[v];
    }
  }
  // the 8 row lanes of a wave first, then the waves through LDS
#pragma unroll
  for (int v = 0; v < V; ++v) {
    acc[v] += lane_xor_f32<8>(acc[v]);
    acc[v] += lane_xor_f32<16>(acc[v]);
    acc[v] += lane_xor_f32<32>(acc[v]);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane < kColLanes) {
#pragma unroll
    for (int v = 0; v < V; ++v) buf[wv][cl * V + v] = acc[v];
  }
  __syncthreads();
  if (threadIdx.x < SLAB) {
    const int ch = blockIdx.x * SLAB + threadIdx.x;
    if (ch < d) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < kThreads / 64; ++i) t += buf[i][threadIdx.x];
      probe_out[size_t(s) * d + ch] = t;
    }
  }
  if (blockIdx.x == 0 && weights_out != nullptr) {
    for (int j = threadIdx.x; j < m; j += kThreads)
      weights_out[size_t(s) * m + j] = total > 0.f ? w_lds[j] * inv_total : uniform;
  }
}

// One workgroup per sequence: the norm of the probe and its per-KV-head sum.  All latency (one
// workgroup, 16 KB), so every element is read once, 16 bytes a lane, and serves both.
constexpr int kFinishThreads = 512;
__global__ __launch_bounds__(kFinishThreads) void probe_finish_kernel(const float* __restrict__ probe,
                                                                      float* __restrict__ probe_kv_out,
                                                                      float* __restrict__ probe_norm_out,
                                                                      int n_q_heads, int n_kv_heads,
                                                                      int head_dim) {
  __shared__ float red[32];
  const int s = blockIdx.x, g = n_q_heads / n_kv_heads, dk = n_kv_heads * head_dim;
  const float* p = probe + size_t(s) * n_q_heads * head_dim;
  float ss = 0.f;
  for (int e = threadIdx.x * 4; e < dk; e += kFinishThreads * 4) {     // (head_dim is a multiple of 4)
    const int hk = e / head_dim, dd = e - hk * head_dim;
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int i = 0; i < g; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(p + (hk * g + i) * head_dim + dd);
      ss += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
      t += v;
    }
    *reinterpret_cast<f32x4*>(probe_kv_out + size_t(s) * dk + e) = t;
  }
  ss = block_sum(ss, red);
  if (threadIdx.x == 0) probe_norm_out[s] = sqrtf(ss);
}

// A window of one token (decode): the probe is the query (probe_identity.h).
template <typename T>
__global__ __launch_bounds__(1024) void probe_identity_kernel(
    const T* __restrict__ q_win, float* __restrict__ stats, int add_count, size_t stats_stride,
    float* __restrict__ probe_out, float* __restrict__ probe_kv_out, float* __restrict__ probe_norm_out,
    float* __restrict__ weights_out, int n_q_heads, int n_kv_heads, int head_dim) {
  __shared__ float red[32];
  extern __shared__ __attribute__((aligned(16))) float probe_lds[];   // [d]
  const int d = n_q_heads * head_dim;
  const int s = blockIdx.x;
  if (add_count && threadIdx.x == 0) stats[size_t(s) * stats_stride] += 1.f;
  probe_identity_body<T>(q_win + size_t(s) * d, probe_out + size_t(s) * d,
                         probe_kv_out + size_t(s) * n_kv_heads * head_dim, probe_norm_out + s,
                         weights_out != nullptr ? weights_out + s : nullptr, n_q_heads, n_kv_heads, head_dim,
                         probe_lds, red);
}

// A long window is a chain of one: a slab has one workgroup however long the window is, and holds 2048 rows in registers.
// A window's step without its attention, in slabs / row by row: 2048 tokens 24.2 / 25.1 us (512 channels), 25.2 / 27.1 (1024),
// 25.7 / 30.1 (2048); 2112 tokens 30.2 / 24.8, 31.8 / 26.8, 34.2 / 31.3; 4096 tokens 35.3 / 26.1, 37.3 / 28.3, 39.8 / 32.5.
// With 4096 channels the slabs are many: 2112 tokens 38.0 / 44.2, 3584 tokens 45.5 / 47.5, 4096 tokens 48.7 / 47.6.
static bool long_window(const actqkv_shape& sh, int batch, int m, int update_stats) {
  const int d = sh.n_q_heads * sh.head_dim;
  return batch == 1 && (update_stats & ACTQKV_STATS_UPDATE) && m > 2048 && (d <= 2048 || (d <= 64 * 64 && m >= 4096));
}

template <typename T>
static int launch_probe_t(const actqkv_shape& sh, int batch, int m, const T* q_win, float* stats,
                          int update_stats, float* probe, float* probe_kv, float* probe_norm,
                          float* weights, const Workspace& ws, hipStream_t stream, bool finish) {
  constexpr int V = Vec<T>::N;
  const int d = sh.n_q_heads * sh.head_dim;
  const float eps = sh.var_eps > 0.f ? sh.var_eps : 1e-12f;
  const size_t stats_stride = stats_floats(sh);
  const size_t scratch_stride = probe_scratch_floats(sh, m);
  const int m_pad = int(probe_a_floats(m));
  const int n_slabs = probe_slabs(sh);
  static_assert(kColLanes * 8 == kProbeSlabBytes / 2 && kColLanes * 4 == kProbeSlabBytes / 4, "slab width");
  float* scratch = ws.scratch_f32();
  const int mean_pooling = (update_stats & ACTQKV_PROBE_MEAN_POOLING) != 0;
  if ((update_stats & ACTQKV_PROBE_WINDOW_CHAIN) || long_window(sh, batch, m, update_stats)) {
    // the batch entries are consecutive windows of one sequence with one set of statistics
    if (d > 64 * 64) {          // (not a long window)
      // rows wider than a wavefront of the row-major kernels holds: window after window
      const int dk = sh.n_kv_heads * sh.head_dim;
      for (int w = 0; w < batch; ++w) {
        const int rc = launch_probe_t<T>(sh, 1, m, q_win + size_t(w) * m * d, stats,
                                         update_stats & ~ACTQKV_PROBE_WINDOW_CHAIN, probe + size_t(w) * d,
                                         probe_kv + size_t(w) * dk, probe_norm + w,
                                         weights != nullptr ? weights + size_t(w) * m : nullptr, ws, stream, true);
        if (rc != ACTQKV_OK) return rc;
      }
      return ACTQKV_OK;
    }
    const ChainScratch cl = chain_scratch(sh, batch, m);
    float* part = scratch;
    float* stat = part + cl.part;
    float* pprobe = stat + cl.stat;
    float* asum = pprobe + cl.pprobe;
    float* a_rows = asum + cl.asum;
    const int n_chunks = cl.n_chunks, groups = d / V;
    // channels of a workgroup: fewer where the chunks alone would leave compute units idle
    int cols = std::min(groups, kRmThreads);
    while (cols > 64 && batch * n_chunks * ((groups + cols - 1) / cols) < kChipCus) cols = std::max(cols / 2, 64);
    hipLaunchKernelGGL(probe_rows_moments_kernel<T>, dim3(n_chunks, batch, (groups + cols - 1) / cols), dim3(kRmThreads), 0,
                       stream, q_win, stats, part, m, d, n_chunks, cols);
    for (int w = 0; w < batch; w += kChainTile) {
      const int n = std::min(batch - w, kChainTile);
      hipLaunchKernelGGL(probe_chain_stats_kernel<T>, dim3((d + 31) / 32), dim3(1024), size_t(n) * 66 * sizeof(float), stream,
                         q_win + size_t(w) * m * d, part + size_t(w) * n_chunks * 2 * d, stats, stat + size_t(w) * 3 * d, n, m, d,
                         n_chunks, eps, float(w) * float(m), int(batch == 1));
    }
    // Few chunks: half as long in the second pass.  Twice as many partial probes take the place of the moments, which
    // chain_stats has used up, and their sums that of the partial probes.
    const bool halves = batch * n_chunks <= kChipCus / 2 && n_chunks <= 16;
    const int rows = halves ? kRowChunk / 2 : kRowChunk, n_parts = (m + rows - 1) / rows;
    const int asum_stride = halves ? (n_parts + 15) / 16 * 16 : cl.asum_stride;
    if (halves) {
      asum = pprobe;                                  // (2 chunks floats and less than 16 more of chunks * d)
      pprobe = part;
    }
    auto bias_weigh = [&](auto kernel, int ni, int waves) {
      const size_t lds = std::max(size_t(2) * 64 * ni * V, size_t(waves / 2) * d) * sizeof(float);
      hipLaunchKernelGGL(kernel, dim3(n_parts, batch), dim3(64 * waves), lds, stream, q_win, stat, stats,
                         float(batch) * float(m), mean_pooling, pprobe, asum, a_rows, m, m_pad, d, rows, n_parts, asum_stride);
    };
    if (groups <= 64 && halves) bias_weigh(probe_rows_bias_weigh_kernel<T, 1, 8, 4>, 1, 8);
    else if (groups <= 64) bias_weigh(probe_rows_bias_weigh_kernel<T, 1, 8, 8>, 1, 8);
    else if (groups <= 128) bias_weigh(probe_rows_bias_weigh_kernel<T, 2, 8, 4>, 2, 8);
    else if (groups <= 256) bias_weigh(probe_rows_bias_weigh_kernel<T, 4, 8, 2>, 4, 8);
    else if (groups <= 512) bias_weigh(probe_rows_bias_weigh_kernel<T, 8, 4, 1>, 8, 4);
    else if constexpr (V == 4) bias_weigh(probe_rows_bias_weigh_kernel<T, 16, 4, 1>, 16, 4);   // (4096 channels of 16 bits are 512)
    // One window, whose norm and per-KV-head sum the scoring launch forms, or, for wide rows, a launch of their own (4096
    // tokens with 4096 channels: 40.9 us, one workgroup for all of it 46.2).
    const bool spread = batch == 1 && d % 256 == 0 && (!finish || d > 2048);
    const int slabs = spread ? d / 256 : 1;
    hipLaunchKernelGGL(probe_chain_finish_kernel, dim3(batch, slabs), dim3(spread ? 64 * (4 * kCfThreads / d) : kCfThreads),
                       size_t(d) * sizeof(float), stream, pprobe,
                       asum, a_rows, stat, probe, probe_kv, probe_norm, weights, m, m_pad, d, n_parts, asum_stride,
                       sh.n_q_heads, sh.n_kv_heads, sh.head_dim);
    if (spread && finish)
      hipLaunchKernelGGL(probe_finish_kernel, dim3(1), dim3(kFinishThreads), 0, stream, probe, probe_kv, probe_norm,
                         sh.n_q_heads, sh.n_kv_heads, sh.head_dim);
    return hip_status("probe");
  }
  update_stats &= ACTQKV_STATS_UPDATE;
  if (update_stats || (m > 1 && !mean_pooling)) {
    auto launch = [&](auto kernel, int row_lanes) {
      hipLaunchKernelGGL(kernel, dim3(n_slabs, batch), dim3(kColLanes * row_lanes), 0, stream, q_win, stats, scratch,
                         update_stats, m, m_pad, d, eps, stats_stride, scratch_stride);
    };
    if (m <= 64 * 4) launch(probe_stats_bias_kernel<T, 64, 4>, 64);
    else if (m <= 64 * 8) launch(probe_stats_bias_kernel<T, 64, 8>, 64);
    else if (m <= 128 * 8) launch(probe_stats_bias_kernel<T, 128, 8>, 128);
    else launch(probe_stats_bias_kernel<T, 128, 16>, 128);
  }
  if (m == 1) {
    hipLaunchKernelGGL(probe_identity_kernel<T>, dim3(batch), dim3(1024), size_t(d) * sizeof(float),
                       stream, q_win, stats,
                       update_stats, stats_stride, probe, probe_kv, probe_norm, weights, sh.n_q_heads,
                       sh.n_kv_heads, sh.head_dim);
    return hip_status("probe");
  }
  auto weigh = [&](auto kernel, int row_lanes) {
    hipLaunchKernelGGL(kernel, dim3(n_slabs, batch), dim3(kColLanes * row_lanes), 0, stream, q_win, scratch, stats,
                       update_stats, mean_pooling, probe, weights, m, m_pad, n_slabs, d, scratch_stride, stats_stride);
  };
  if (m <= 64 * kWeighRows) weigh(probe_weigh_kernel<T, 64>, 64);
  else weigh(probe_weigh_kernel<T, 128>, 128);
  if (finish)
    hipLaunchKernelGGL(probe_finish_kernel, dim3(batch), dim3(kFinishThreads), 0, stream, probe, probe_kv,
                       probe_norm, sh.n_q_heads, sh.n_kv_heads, sh.head_dim);
  return hip_status("probe");
}

bool probe_finish_apart(const actqkv_shape& sh, int batch, int m, int update_stats) {
  return batch == 1 && m > 1;
}

int launch_probe(const actqkv_shape& sh, int batch, int m, const void* q_win, float* stats,
                 int update_stats, float* probe, float* probe_kv, float* probe_norm, float* weights,
                 const Workspace& ws, hipStream_t stream, bool finish) {
  if (sh.dtype == ACTQKV_F32)
    return launch_probe_t<float>(sh, batch, m, static_cast<const float*>(q_win), stats, update_stats,
                                 probe, probe_kv, probe_norm, weights, ws, stream, finish);
  return launch_probe_t<uint16_t>(sh, batch, m, static_cast<const uint16_t*>(q_win), stats,
                                  update_stats, probe, probe_kv, probe_norm, weights, ws, stream, finish);
}

}  // namespace actqkv
