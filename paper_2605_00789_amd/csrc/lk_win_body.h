// Device-side body of the window partition (lk_windows.hip, where the algorithm is described).  It takes the sequence and
// a block of LDS as arguments and is written for any number of waves, so that a launch can run it next to other work
// (lk_rows.hip) as well as on its own.
#pragma once
#include "lk_common.h"
#include "lk_launch.h"

namespace lk {

struct WinArgs {
  const int32_t *cu_vis, *pos;
  // "next stage" form: the tokens are those of the PREVIOUS stage (cu_vis, pos); a token takes part if
  // new_index[i] >= 0 and is listed under that index; cu_out holds the sequence offsets after compaction.
  // Both NULL: the plain form (every token takes part under its own index).
  const int32_t *new_index, *cu_out;
  int batch, tiles, grid_h, grid_w, w, win_per_seq;
  int32_t *win_offsets, *win_tokens;
  // optional: the per-window counts in the same launch -- the window sizes are in LDS here anyway.
  int count_mode;             // WIN_NO_COUNTS, or a mode of window_counts_kernel (0 ratio, 1 edges, 2 token budget)
  double rho;                 // modes 0 and 1
  const int32_t *cu_target;   // mode 2: [batch + 1] offsets of the sequences after the step the windows are built for
  int32_t *win_remove, *status;
  int dir;
};
constexpr int WIN_NO_COUNTS = -1;

// index under which token i is listed, or -1 if it does not take part
__device__ __forceinline__ int listed_as(const WinArgs &g, int i) { return g.new_index ? g.new_index[i] : i; }

__device__ __forceinline__ int window_of(const WinArgs &g, int p) {
  if (g.w == 0) return 0;
  const int cells = g.grid_h * g.grid_w;
  p = p < 0 ? 0 : p;
  int tile = p / cells;
  const int cell = p - tile * cells;
  tile = tile >= g.tiles ? g.tiles - 1 : tile;
  int row = cell / g.grid_w;
  const int col = cell - row * g.grid_w;
  row = row >= g.grid_h ? g.grid_h - 1 : row;
  return tile * g.w * g.w + (row * g.w / g.grid_h) * g.w + (col * g.w / g.grid_w);
}

// r_w (mode 0) or k_w (mode 1) of a window of v tokens from the ratio; a double, so that the floor is the one a host
// program would take
__device__ __forceinline__ int count_from_ratio(int mode, double rho, int v, int dir) {
  long long r, cap;
  if (mode == 0) { r = (long long)floor(rho * (double)v + 1e-9); cap = side_a(v, dir); }
  else           { r = (long long)floor(rho * (double)v / 2.0 + 1e-9); cap = (long long)((v + 1) / 2) * (v / 2); }
  return (int)(r < 0 ? 0 : (r > cap ? cap : r));
}
// the most a window of v tokens can give: its proposing side; a single token has nobody to merge into
__device__ __forceinline__ int window_cap(int v, int dir) {
  const int c = v >= 2 ? side_a(v, dir) : 0;
  return c < 65535 ? c : 65535;
}

// Bytes of LDS the partition of one sequence of n tokens over wps windows needs: the (run, window) counts, then the
// window bases.
__host__ __device__ __forceinline__ size_t win_table_bytes(int n, int wps) {
  const size_t entries = (size_t)((n + 63) / 64) * (size_t)wps;
  return (entries + 7) / 8 * 16 + ((size_t)wps + 1) * sizeof(int32_t);
}

// ---- the token budget of a sequence spread over its windows (Sec. 3.2.2: the ratios P given as target lengths), by ONE
// wave.  With cap_w the most a window can give and q the largest level for which sum_w min(cap_w, q) stays within the
// budget, window w gives min(cap_w, q), and the first windows (in order) that can give more than q give one more until
// the budget is met.  A budget that cannot be met (negative, or above sum_w cap_w): every window gives its cap (nothing
// for a negative budget) and the status word is set.
// The level is found by filling: from level q with `missing` tokens left and `open` windows that can still give, the
// level rises by missing / open, which can never overshoot; it is final once missing < open.  Equal windows take two
// rounds.  A round is two sums over the windows in one pass of shuffles, so the wave needs no barrier at all (the
// binary search this replaces took two workgroup barriers per probe, 5-8 probes).
__device__ __forceinline__ long long wave_sum_ll(long long v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <typename SizeFn>
__device__ __forceinline__ void counts_target_wave(int W, int budget, int dir, SizeFn size_of, int32_t *win_remove,
                                                   int32_t *status) {
  const int lane = threadIdx.x & 63;
  long long t = 0;
  for (int w = lane; w < W; w += 64) t += window_cap(size_of(w), dir);
  const long long total = wave_sum_ll(t);
  const bool infeasible = budget < 0 || budget > total;
  if (status && lane == 0) *status = infeasible ? 1 : 0;
  if (infeasible) {   // more than every set A holds: all of them go; a negative budget: nothing goes
    for (int w = lane; w < W; w += 64) win_remove[w] = budget < 0 ? 0 : window_cap(size_of(w), dir);
    return;
  }
  int q = 0, missing = budget;
  for (;;) {   // uniform; q rises by at least one per round and is bounded by the largest cap
    int open = 0, given = 0;
    for (int w = lane; w < W; w += 64) {
      const int c = window_cap(size_of(w), dir);
      open += c > q ? 1 : 0;
      given += c < q ? c : q;
    }
    const long long both = wave_sum_ll(((long long)open << 32) | (unsigned)given);   // given <= budget < 2^31
    open = (int)(both >> 32);
    missing = budget - (int)(both & 0xffffffffll);
    if (open == 0 || missing < open) break;
    q += missing / open;
  }
  int before = 0;   // windows with cap > q before this pass
  for (int w0 = 0; w0 < W; w0 += 64) {   // uniform
    const int w = w0 + lane;
    const int c = w < W ? window_cap(size_of(w), dir) : 0;
    const bool more = c > q;
    const unsigned long long m = __ballot(more);
    const int rank = before + __popcll(m & ((1ull << lane) - 1ull));
    if (w < W) win_remove[w] = (c < q ? c : q) + ((more && rank < missing) ? 1 : 0);
    before += __popcll(m);
  }
}

// Partition of sequence b by NT threads; `lds` holds win_table_bytes(tokens of the sequence, win_per_seq).
// KEEP: passes of NT tokens whose window and rank stay in registers between counting and placing (later ones are
// recomputed).
template <int NT, int KEEP>
__device__ __forceinline__ void build_windows_body(const WinArgs &g, int b, char *lds) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int base = g.cu_vis[b];
  const int n = g.cu_vis[b + 1] - base;
  const int out_base = g.cu_out ? g.cu_out[b] : base;                 // first listed index of the sequence
  const int out_n = g.cu_out ? g.cu_out[b + 1] - out_base : n;        // tokens that take part
  const int target_n = g.count_mode == 2 ? g.cu_target[b + 1] - g.cu_target[b] : 0;
  const int wps = g.win_per_seq;
  const int wbase = b * wps;
  const int runs = (n + 63) >> 6;
  uint16_t *table = reinterpret_cast<uint16_t *>(lds);   // [runs][wps] counts, then exclusive prefixes over the runs
  const int words = (runs * wps + 7) >> 3;               // 16-byte pieces
  int *winbase = reinterpret_cast<int *>(lds + (size_t)words * 16);   // [wps + 1]

  // phase 1: per-run counts.  All loads of the kept passes go out before anything is used.
  int k_id[KEEP], k_wr[KEEP];   // listed index; window << 6 | rank inside the run's group (a window is below 2^17)
#pragma unroll
  for (int p = 0; p < KEEP; ++p) {
    const int i = p * NT + tid;
    k_id[p] = -1; k_wr[p] = 0;
    if (p * NT < n) {   // uniform
      const int ic = i < n ? i : n - 1;
      const int id = listed_as(g, base + ic);
      k_wr[p] = g.pos[base + ic];
      k_id[p] = i < n ? id : -1;
    }
  }
  for (int e = tid; e < words; e += NT) reinterpret_cast<uint4 *>(table)[e] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  const int bits = 32 - __clz(wps > 1 ? wps - 1 : 1);
  // rank of this lane among the lanes of its wave with the same window: lanes agreeing on every bit of the window's
  // number (a ballot per bit, whatever the number of distinct windows in the run)
  auto rank_in_run = [&](int wid, bool valid, int i, int &rank) {
    unsigned long long same = __ballot(valid);
    for (int k = 0; k < bits; ++k) {   // uniform
      const bool one = (wid >> k) & 1;
      const unsigned long long m = __ballot(one);
      same &= one ? m : ~m;
    }
    rank = __popcll(same & ((1ull << lane) - 1ull));
    if (valid && rank == 0) table[(i >> 6) * wps + wid] = (uint16_t)__popcll(same);
  };
#pragma unroll
  for (int p = 0; p < KEEP; ++p) {
    if (p * NT < n) {   // uniform
      const bool valid = k_id[p] >= 0;
      const int wid = window_of(g, k_wr[p]);
      int rank;
      rank_in_run(wid, valid, p * NT + tid, rank);
      k_wr[p] = (wid << 6) | rank;
    }
  }
  for (int i0 = KEEP * NT; i0 < n; i0 += NT) {
    const int i = i0 + tid;
    const bool valid = i < n && listed_as(g, base + (i < n ? i : 0)) >= 0;
    const int wid = window_of(g, g.pos[base + (i < n ? i : 0)]);
    int rank;
    rank_in_run(wid, valid, i, rank);
  }
  __syncthreads();
  // phase 2: exclusive prefix over the runs for every window (a thread per window, eight counts in flight)
  for (int w = tid; w < wps; w += NT) {
    int total = 0;
    for (int r0 = 0; r0 < runs; r0 += 8) {
      int c[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] = table[(r0 + u < runs ? r0 + u : runs - 1) * wps + w];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (r0 + u < runs) { table[(r0 + u) * wps + w] = (uint16_t)total; total += c[u]; }
    }
    winbase[w] = total;
  }
  __syncthreads();
  // ... and over the windows, by the first wave: 64 at a time
  if (tid < 64) {
    int carry = 0;
    for (int w0 = 0; w0 < wps; w0 += 64) {   // uniform
      const int w = w0 + lane;
      const int total = w < wps ? winbase[w] : 0;
      int inc = total;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
      }
      if (w < wps) winbase[w] = carry + inc - total;
      carry += __shfl(inc, 63, 64);
    }
    if (lane == 0) winbase[wps] = out_n;
  }
  __syncthreads();
  for (int w = tid; w < wps; w += NT) g.win_offsets[wbase + w] = out_base + winbase[w];
  if (tid == 0 && b == g.batch - 1) g.win_offsets[wbase + wps] = out_base + out_n;
  // counts: the sizes of the windows are the differences of winbase[]
  auto size_of = [&](int w) { return winbase[w + 1] - winbase[w]; };
  if (g.count_mode == 2) {
    // the last wave, which has the fewest tokens to place (in a small sequence none at all)
    if (tid >= NT - 64)
      counts_target_wave(wps, out_n - target_n, g.dir, size_of, g.win_remove + wbase, g.status ? g.status + b : nullptr);
  } else if (g.count_mode >= 0) {
    for (int w = tid; w < wps; w += NT) g.win_remove[wbase + w] = count_from_ratio(g.count_mode, g.rho, size_of(w), g.dir);
    if (g.status && tid == 0) g.status[b] = 0;
  }
  // phase 3: slots
#pragma unroll
  for (int p = 0; p < KEEP; ++p) {
    const int i = p * NT + tid;
    if (k_id[p] >= 0) {
      const int wid = k_wr[p] >> 6, rank = k_wr[p] & 63;
      g.win_tokens[out_base + winbase[wid] + table[(i >> 6) * wps + wid] + rank] = k_id[p];
    }
  }
  for (int i0 = KEEP * NT; i0 < n; i0 += NT) {
    const int i = i0 + tid;
    const int id = i < n ? listed_as(g, base + (i < n ? i : 0)) : -1;
    const bool valid = id >= 0;
    const int wid = window_of(g, g.pos[base + (i < n ? i : 0)]);
    unsigned long long same = __ballot(valid);
    for (int k = 0; k < bits; ++k) {
      const bool one = (wid >> k) & 1;
      const unsigned long long m = __ballot(one);
      same &= one ? m : ~m;
    }
    if (valid)
      g.win_tokens[out_base + winbase[wid] + table[(i >> 6) * wps + wid] + __popcll(same & ((1ull << lane) - 1ull))] = id;
  }
}

}  // namespace lk
