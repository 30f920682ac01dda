// Device-side body of the window partition (lk_windows.hip, where the algorithm is described).  It takes the sequence and
// a block of LDS as arguments and is written for any number of waves, so that a launch can run it next to other work
// (lk_rows.hip) as well as on its own.
#pragma once
#include "lk_common.h"
#include "lk_launch.h"

namespace lk {

// Division of 0 <= n < 2^31 by a divisor known on the host (Granlund and Montgomery, "Division by invariant integers using
// multiplication"): with s = ceil(log2 d) and m = floor(2^32 (2^s - d) / d) + 1, n / d = (mulhi(m, n) + n) >> s.  The partition
// needs four per token, and the compiler's own sequence for an unknown divisor is some forty instructions: 16384 tokens in 16
// windows 38.5 -> 28 us.
struct FastDiv {
  uint32_t m, s;
  __device__ __forceinline__ int div(int n) const { return (int)((__umulhi(m, (uint32_t)n) + (uint32_t)n) >> s); }
};
inline FastDiv make_fast_div(uint32_t d) {
  uint32_t s = 0;
  while (((uint64_t)1 << s) < d) ++s;
  return FastDiv{(uint32_t)((((((uint64_t)1 << s) - d) << 32) / d) + 1), s};
}

struct WinArgs {
  const int32_t *cu_vis, *pos;
  // "next stage" form: the tokens are those of the PREVIOUS stage (cu_vis, pos); a token takes part if
  // new_index[i] >= 0 and is listed under that index; cu_out holds the sequence offsets after compaction.
  // Both NULL: the plain form (every token takes part under its own index).
  const int32_t *new_index, *cu_out;
  int batch, tiles, grid_h, grid_w, w, win_per_seq;
  FastDiv by_cells, by_grid_h, by_grid_w;
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
  p = p < 0 ? 0 : p;
  int tile = g.by_cells.div(p);
  const int cell = p - tile * (g.grid_h * g.grid_w);
  tile = tile >= g.tiles ? g.tiles - 1 : tile;
  const int row = g.by_grid_w.div(cell);   // below grid_h
  const int col = cell - row * g.grid_w;
  return tile * g.w * g.w + g.by_grid_h.div(row * g.w) * g.w + g.by_grid_w.div(col * g.w);
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
// window bases, then a word per wave.
constexpr size_t WIN_SCRATCH = 16 * sizeof(long long);
__host__ __device__ __forceinline__ size_t win_table_bytes(int n, int wps) {
  const size_t entries = (size_t)((n + 63) / 64) * (size_t)wps;
  return (entries + 7) / 8 * 16 + (((size_t)wps + 2) & ~(size_t)1) * sizeof(int32_t) + WIN_SCRATCH;
}

// Sum over the NW waves that work on a sequence's counts; `scratch` holds NW values (not used by a single wave).
template <int NW>
__device__ __forceinline__ long long group_sum_ll(long long v, long long *scratch) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  if constexpr (NW > 1) {
    __syncthreads();   // scratch may still be read from the call before
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) v += scratch[i];
  }
  return v;
}

// ---- the token budget of a sequence spread over its windows (Sec. 3.2.2: the ratios P given as target lengths), by ONE
// wave, or by the NW waves of a workgroup.  With cap_w the most a window can give and q the largest level for which
// sum_w min(cap_w, q) stays within the budget, window w gives min(cap_w, q), and the first windows (in order) that can give
// more than q give one more until the budget is met.  A budget that cannot be met (negative, or above sum_w cap_w): every
// window gives its cap (nothing for a negative budget) and the status word is set.
// The level is found by filling: from level q with `missing` tokens left and `open` windows that can still give, the
// level rises by missing / open, which can never overshoot; it is final once missing < open.  Equal windows take two
// rounds.  A round is two sums over the windows in one pass of shuffles, so a single wave needs no barrier at all (a
// binary search took two workgroup barriers per probe, 5-8 probes).  A wave takes 64 windows a step, though, and with many of
// them the whole workgroup is the faster form (lightkv_window_counts, one wave / four: 64 windows 3.4 / 4.1 us, 180 4.3 / 4.3,
// 512 5.9 / 4.6, 1024 9.5 / 6.1, 8192 47.5 / 23.0).  Inside the partition the single wave counts while the others place
// tokens, so it keeps more of them there.
constexpr int COUNTS_WAVE_MAX = 192, COUNTS_WAVE_MAX_BESIDE = 512;
template <int NW, typename SizeFn>
__device__ __forceinline__ void counts_target(int W, int budget, int dir, SizeFn size_of, int32_t *win_remove,
                                              int32_t *status, long long *scratch) {
  constexpr int NT = 64 * NW;
  const int lane = threadIdx.x & 63, wave = NW > 1 ? (int)threadIdx.x >> 6 : 0, t = wave * 64 + lane;
  long long sum = 0;
  for (int w = t; w < W; w += NT) sum += window_cap(size_of(w), dir);
  const long long total = group_sum_ll<NW>(sum, scratch);
  const bool infeasible = budget < 0 || budget > total;
  if (status && t == 0) *status = infeasible ? 1 : 0;
  if (infeasible) {   // more than every set A holds: all of them go; a negative budget: nothing goes
    for (int w = t; w < W; w += NT) win_remove[w] = budget < 0 ? 0 : window_cap(size_of(w), dir);
    return;
  }
  int q = 0, missing = budget;
  for (;;) {   // uniform; q rises by at least one per round and is bounded by the largest cap
    int open = 0, given = 0;
    for (int w = t; w < W; w += NT) {
      const int c = window_cap(size_of(w), dir);
      open += c > q ? 1 : 0;
      given += c < q ? c : q;
    }
    const long long both = group_sum_ll<NW>(((long long)open << 32) | (unsigned)given, scratch);   // given <= budget < 2^31
    open = (int)(both >> 32);
    missing = budget - (int)(both & 0xffffffffll);
    if (open == 0 || missing < open) break;
    q += missing / open;
  }
  int before = 0;   // windows with cap > q before this pass
  for (int w0 = 0; w0 < W; w0 += NT) {   // uniform
    const int w = w0 + t;
    const int c = w < W ? window_cap(size_of(w), dir) : 0;
    const bool more = c > q;
    const unsigned long long m = __ballot(more);
    int rank = before + __popcll(m & ((1ull << lane) - 1ull)), all = __popcll(m);
    if constexpr (NW > 1) {
      __syncthreads();
      if (lane == 0) scratch[wave] = all;
      __syncthreads();
      all = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        rank += i < wave ? (int)scratch[i] : 0;
        all += (int)scratch[i];
      }
    }
    if (w < W) win_remove[w] = (c < q ? c : q) + ((more && rank < missing) ? 1 : 0);
    before += all;
  }
}

// Partition of sequence b by NT threads; `lds` holds win_table_bytes(tokens of the sequence, win_per_seq).
// The tokens go by in passes of NT, KEEP passes at a time whose loads are in flight together: a pass on its own is a trip to
// memory, and 16384 tokens are 64 passes of 256 threads, twice.  The window and rank of the first KEEP passes stay in
// registers between counting and placing, those of the others are computed again.
template <int NT, int KEEP>
__device__ __forceinline__ void build_windows_body(const WinArgs &g, int b, char *lds) {
  static_assert(NT / 64 * sizeof(long long) <= WIN_SCRATCH, "a word per wave");
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
  long long *scratch = reinterpret_cast<long long *>(winbase + ((wps + 2) & ~1));

  int k_id[KEEP], k_wr[KEEP];   // listed index; cell, then window << 6 | rank inside the run's group (a window is below 2^17)
  auto load = [&](int i0) {
#pragma unroll
    for (int p = 0; p < KEEP; ++p) {
      const int i = i0 + p * NT + tid;
      k_id[p] = -1; k_wr[p] = 0;
      if (i0 + p * NT < n) {   // uniform
        const int ic = i < n ? i : n - 1;
        const int id = listed_as(g, base + ic);
        k_wr[p] = g.pos[base + ic];
        k_id[p] = i < n ? id : -1;
      }
    }
  };
  const int bits = 32 - __clz(wps > 1 ? wps - 1 : 1);
  // window of a token, and its rank among the lanes of its wave with the same window: lanes agreeing on every bit of the
  // window's number (a ballot per bit, whatever the number of distinct windows in the run)
  auto rank_all = [&](int i0, bool count) {
#pragma unroll
    for (int p = 0; p < KEEP; ++p) {
      if (i0 + p * NT < n) {   // uniform
        const bool valid = k_id[p] >= 0;
        const int wid = window_of(g, k_wr[p]);
        unsigned long long same = __ballot(valid);
        for (int k = 0; k < bits; ++k) {   // uniform
          const bool one = (wid >> k) & 1;
          const unsigned long long m = __ballot(one);
          same &= one ? m : ~m;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        if (count && valid && rank == 0) table[((i0 + p * NT + tid) >> 6) * wps + wid] = (uint16_t)__popcll(same);
        k_wr[p] = (wid << 6) | rank;
      }
    }
  };
  // phase 1: per-run counts (the first loads go out before anything else)
  load(0);
  for (int e = tid; e < words; e += NT) reinterpret_cast<uint4 *>(table)[e] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  // (backwards, so that the first passes are the ones left in registers)
  for (int i0 = (n - 1) / (KEEP * NT) * (KEEP * NT); i0 > 0; i0 -= KEEP * NT) { load(i0); rank_all(i0, true); }
  if (n > KEEP * NT) load(0);
  rank_all(0, true);
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
  // ... and over the windows: up to 64 by the first wave, more by all of them
  auto wave_scan = [&](int v) {   // inclusive
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(v, o, 64);
      if (lane >= o) v += t;
    }
    return v;
  };
  if (wps <= 64) {
    if (tid < 64) {
      const int total = lane < wps ? winbase[lane] : 0;
      const int inc = wave_scan(total);
      if (lane < wps) winbase[lane] = inc - total;
    }
  } else {
    int carry = 0;
    for (int w0 = 0; w0 < wps; w0 += NT) {   // uniform
      const int w = w0 + tid;
      const int total = w < wps ? winbase[w] : 0;
      const int inc = wave_scan(total);
      if (w0 > 0) __syncthreads();   // scratch may still be read from the step before
      if (lane == 63) scratch[tid >> 6] = inc;
      __syncthreads();
      int before = carry;
#pragma unroll
      for (int i = 0; i < NT / 64; ++i) {
        before += i < (tid >> 6) ? (int)scratch[i] : 0;
        carry += (int)scratch[i];
      }
      if (w < wps) winbase[w] = before + inc - total;
    }
  }
  if (tid == 0) winbase[wps] = out_n;
  __syncthreads();
  for (int w = tid; w < wps; w += NT) g.win_offsets[wbase + w] = out_base + winbase[w];
  if (tid == 0 && b == g.batch - 1) g.win_offsets[wbase + wps] = out_base + out_n;
  // counts: the sizes of the windows are the differences of winbase[]
  auto size_of = [&](int w) { return winbase[w + 1] - winbase[w]; };
  if (g.count_mode == 2) {
    int32_t *status = g.status ? g.status + b : nullptr;
    if (wps > COUNTS_WAVE_MAX_BESIDE) counts_target<NT / 64>(wps, out_n - target_n, g.dir, size_of, g.win_remove + wbase, status, scratch);
    // otherwise the last wave, which has the fewest tokens to place (in a small sequence none at all)
    else if (tid >= NT - 64) counts_target<1>(wps, out_n - target_n, g.dir, size_of, g.win_remove + wbase, status, nullptr);
  } else if (g.count_mode >= 0) {
    for (int w = tid; w < wps; w += NT) g.win_remove[wbase + w] = count_from_ratio(g.count_mode, g.rho, size_of(w), g.dir);
    if (g.status && tid == 0) g.status[b] = 0;
  }
  // phase 3: slots
  for (int i0 = 0; i0 < n; i0 += KEEP * NT) {
    if (i0 > 0) { load(i0); rank_all(i0, false); }
#pragma unroll
    for (int p = 0; p < KEEP; ++p) {
      const int i = i0 + p * NT + tid;
      if (k_id[p] >= 0) {
        const int wid = k_wr[p] >> 6, rank = k_wr[p] & 63;
        g.win_tokens[out_base + winbase[wid] + table[(i >> 6) * wps + wid] + rank] = k_id[p];
      }
    }
  }
}

}  // namespace lk
