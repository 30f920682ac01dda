// Selection under full pairwise matching (appendix, "Bipartite vs. full pairwise matching").  The appendix reports
// accuracy and cost of matching every token against every other token of its window but gives no merge rule; the
// reading implemented here (and in the test oracle): the tokens of a window are visited in ascending order of their
// nearest-neighbour FD (ties: earlier in the window first); a visited token is merged into its nearest neighbour
// unless a token merged earlier was merged INTO it (a token that has received others stays) or its nearest neighbour
// has itself been merged away already; the visit ends after r_w merges.  At most r_w tokens leave a window.
//
// One workgroup per window (at most 4096 tokens), everything in LDS:
//   1. rank of every token among the (FD bits, position) keys of the window, by counting smaller keys
//   2. the visit, which is sequential by definition, as a fixed point: a token can be decided as soon as every token
//      visited before it that could affect it is decided -- the earlier-ranked tokens that name it as their nearest
//      neighbour (any of them leaving makes it a destination) and its own nearest neighbour if that one ranks
//      earlier (it may be gone).  Every round decides at least the lowest-ranked undecided token, so the loop ends
//      after at most v rounds (in practice a handful: chains of nearest neighbours are short); it is bounded by v.
//   3. the first r_w of the tokens that may leave, in rank order (a scan over ranks)
//   4. dst, the number of sources of every destination, and the rank of every source among the sources of its
//      destination in ascending token order -- what select_scan_kernel turns into new_index and the inverse map.
// Bound: barriers and dependent LDS reads of one workgroup.  So the workgroup is no larger than the window needs (256
// threads up to 256 tokens), threads without a token of their own share the counting loops, and a round of the visit
// is three barriers: the minima of the next round are reset while this one's are read, and the count of undecided tokens
// travels with the last barrier.  Windows of 36 / 120 / 400 tokens: 13 / 18 / 36 us -> 6.1 / 8.0 / 14.5 us.
#include "lk_common.h"
#include "lk_launch.h"

namespace lk {

constexpr int PS_MAX = 4096;              // tokens of the largest window

struct PairSelArgs {
  int n_windows, sum_n, cap;              // cap: the caller's bound on the tokens of a window
  const int32_t *win_offsets, *win_tokens, *win_remove;
  const unsigned long long *keys;         // [sum_n] by list position
  float *best_fd;
  int32_t *best_dst, *dst, *cnt, *src_rank;
};

enum : unsigned char { PS_UNDECIDED = 0, PS_LEAVES = 1, PS_STAYS = 2 };

// NT threads, windows of at most CAP tokens (the launcher's bound).
template <int NT, int CAP>
__global__ __launch_bounds__(NT) void pair_select_kernel(PairSelArgs g) {
  fetch_args<PairSelArgs>();
  constexpr int ITEMS = CAP / NT;
  // order-preserving FD bits (step 1); then the neighbour of every token that leaves (step 4)
  __shared__ __attribute__((aligned(16))) uint32_t key[CAP + 4];
  __shared__ uint32_t minpend[2][CAP];      // per position, the lowest rank among the undecided tokens that name it
  __shared__ int count[CAP];                // ranks (step 1), then sources of every position (step 4)
  __shared__ uint16_t nbr[CAP];             // nearest neighbour (list position), 0xffff: none
  __shared__ uint16_t rnk[CAP];
  __shared__ uint16_t by_rank[CAP];         // token at every rank
  __shared__ unsigned char state[CAP];
  __shared__ unsigned char received[CAP];
  __shared__ int wave_tot[NT / 64];
  const int w = blockIdx.x;
  const int off = g.win_offsets[w];
  int v = g.win_offsets[w + 1] - off;
  const int v_all = v;
  v = v < g.cap ? v : g.cap;
  v = v < CAP ? v : CAP;
  int r = g.win_remove[w];
  r = r < 0 ? 0 : r;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // tokens of a window beyond the bound are neither scored nor merged
  for (int l = v + tid; l < v_all; l += NT) {
    const int t = g.win_tokens[off + l];
    if ((unsigned)t < (unsigned)g.sum_n) {
      g.dst[t] = -1; g.cnt[t] = 0; g.src_rank[t] = 0;
      g.best_fd[t] = __uint_as_float(0x7f800000u); g.best_dst[t] = -1;
    }
  }
  // ---- 0. keys -> LDS, best_fd / best_dst
  const int v4 = (v + 3) & ~3;
  int tok[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int l = k * NT + tid;
    tok[k] = -1;
    if (k * NT >= v4) continue;   // uniform
    if (l < v4) { key[l] = l < v ? 0xfffffffeu : 0xffffffffu; nbr[l] = 0xffffu; }   // (without a neighbour: behind +inf, in order)
    if (l < v) {
      state[l] = PS_STAYS; received[l] = 0; minpend[0][l] = 0xffffffffu; count[l] = 0;
      const int t = g.win_tokens[off + l];
      const unsigned long long kk = g.keys[off + l];
      const bool okt = (unsigned)t < (unsigned)g.sum_n;
      const unsigned nb = (unsigned)(kk & 0xffffffffu);
      const float fd = __uint_as_float((unsigned)(kk >> 32));
      const bool scored = okt && kk != ~0ull && nb < (unsigned)v && fd >= 0.f;   // NaN or negative never competes
      const int nt = g.win_tokens[off + (scored ? (int)nb : 0)];
      const bool has = scored && (unsigned)nt < (unsigned)g.sum_n;
      tok[k] = okt ? t : -1;
      if (has) { key[l] = f32_order_key(fd); nbr[l] = (uint16_t)nb; state[l] = PS_UNDECIDED; }
      if (okt) {
        g.best_fd[t] = scored ? fd : __uint_as_float(0x7f800000u);
        g.best_dst[t] = has ? nt : -1;
      }
    }
  }
  __syncthreads();
  // ---- 1. ranks by counting (keys beyond v are all-ones: never smaller).  In a window of at most half the workgroup's
  // threads, `segs` threads share a position and split the list.
  int span = 64;                       // positions the threads are laid over: a power of two of at least v
  while (span < v && span < NT) span <<= 1;
  const int segs = ITEMS == 1 ? NT / span : 1;
  const int seg_len = ((v4 / 4 + segs - 1) / segs) * 4;
  const int my_l = ITEMS == 1 ? (tid & (span - 1)) : tid, my_begin = ITEMS == 1 ? (tid / span) * seg_len : 0;
  const int my_end = min(v4, my_begin + seg_len);
  if (ITEMS == 1) {
    if (my_l < v && my_begin < my_end) {
      const int c = count_before(key, key[my_l], my_l, my_begin, my_end);
      if (c) atomicAdd(&count[my_l], c);
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int l = k * NT + tid;
    if (l < v) {
      const int c = ITEMS == 1 ? count[l] : count_before(key, key[l], l, 0, v4);
      rnk[l] = (uint16_t)c;
      by_rank[c] = (uint16_t)l;
      count[l] = 0;
    }
  }
  __syncthreads();
  // ---- 2. the visit as a fixed point
  for (int round = 0; round <= v; ++round) {   // bounded: every round decides at least one token
    uint32_t *pend = minpend[round & 1], *next = minpend[(round & 1) ^ 1];
    for (int l = tid; l < v; l += NT)
      if (state[l] == PS_UNDECIDED) atomicMin(&pend[nbr[l]], (uint32_t)rnk[l]);
    __syncthreads();
    unsigned char decided[ITEMS];
    int left = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int l = k * NT + tid;
      decided[k] = PS_UNDECIDED;
      if (l < v) {
        next[l] = 0xffffffffu;
        if (state[l] == PS_UNDECIDED) {
          const int b = nbr[l];
          const uint32_t my_rank = rnk[l];
          const unsigned char sb = state[b];
          const bool ready = pend[l] >= my_rank && (sb != PS_UNDECIDED || rnk[b] > my_rank);
          if (ready) decided[k] = (received[l] || sb == PS_LEAVES) ? PS_STAYS : PS_LEAVES;
          else left = 1;
        }
      }
    }
    __syncthreads();   // every thread has read the states of this round before any is changed
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int l = k * NT + tid;
      if (decided[k] != PS_UNDECIDED) {
        state[l] = decided[k];
        if (decided[k] == PS_LEAVES) received[nbr[l]] = 1;
      }
    }
    if (!__syncthreads_or(left)) break;   // uniform
  }
  // ---- 3. the first r leavers in rank order: by_rank[q] -> leavers before rank q (exclusive scan over ranks)
  {
    int carry = 0;
    for (int q0 = 0; q0 < v; q0 += NT) {   // uniform
      const int q = q0 + tid;
      const int flag = (q < v && state[by_rank[q]] == PS_LEAVES) ? 1 : 0;
      int inc = flag;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(inc, o, 64); if (lane >= o) inc += t; }
      if (q0 > 0) __syncthreads();   // wave_tot may still be read from the pass before
      if (lane == 63) wave_tot[wave] = inc;
      __syncthreads();
      int before = carry;
      for (int k = 0; k < wave; ++k) before += wave_tot[k];
      if (q < v && flag && before + inc - flag >= r) state[by_rank[q]] = PS_STAYS;   // beyond the r-th merge: stays after all
      int total = 0;
      for (int k = 0; k < NT / 64; ++k) total += wave_tot[k];
      carry += total;
    }
  }
  __syncthreads();
  // ---- 4. destinations, source counts, source ranks.  key[] now holds the neighbour of every token that leaves
  // (all-ones: stays), count[] the sources of every position.
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int l = k * NT + tid;
    if (l < v4) {
      const bool leaves = l < v && state[l] == PS_LEAVES;
      key[l] = leaves ? (uint32_t)nbr[l] : 0xffffffffu;
      if (leaves) atomicAdd(&count[nbr[l]], 1);
    }
  }
  int *src_rank = reinterpret_cast<int *>(minpend[0]);   // free now
  if (ITEMS == 1) for (int l = tid; l < v; l += NT) src_rank[l] = 0;
  __syncthreads();
  if (ITEMS == 1) {
    if (my_l < v && key[my_l] != 0xffffffffu && my_begin < my_end) {
      const int c = count_equal_before(key, key[my_l], my_l, my_begin, my_end);
      if (c) atomicAdd(&src_rank[my_l], c);
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int l = k * NT + tid;
    if (l < v && tok[k] >= 0) {
      const uint32_t mine = key[l];
      const bool leaves = mine != 0xffffffffu;
      int c = 0;
      if (leaves) c = ITEMS == 1 ? src_rank[l] : count_equal_before(key, mine, l, 0, v4);
      g.dst[tok[k]] = leaves ? g.win_tokens[off + (int)mine] : -1;
      g.src_rank[tok[k]] = c;
      g.cnt[tok[k]] = count[l];
    }
  }
}

hipError_t launch_pair_select(int n_windows, int max_window, int sum_n, const int32_t *win_offsets,
                              const int32_t *win_tokens, const int32_t *win_remove, const unsigned long long *keys,
                              float *best_fd, int32_t *best_dst, int32_t *dst, int32_t *cnt, int32_t *src_rank,
                              hipStream_t stream) {
  if (n_windows == 0 || sum_n == 0) return hipSuccess;
  PairSelArgs g{};
  g.n_windows = n_windows; g.sum_n = sum_n; g.cap = max_window;
  g.win_offsets = win_offsets; g.win_tokens = win_tokens; g.win_remove = win_remove; g.keys = keys;
  g.best_fd = best_fd; g.best_dst = best_dst; g.dst = dst; g.cnt = cnt; g.src_rank = src_rank;
  const dim3 grid((unsigned)n_windows);
  if (max_window <= 256) hipLaunchKernelGGL((pair_select_kernel<256, 256>), grid, dim3(256), 0, stream, g);
  else if (max_window <= 1024) hipLaunchKernelGGL((pair_select_kernel<1024, 1024>), grid, dim3(1024), 0, stream, g);
  else hipLaunchKernelGGL((pair_select_kernel<1024, PS_MAX>), grid, dim3(1024), 0, stream, g);
  return hipGetLastError();
}

}  // namespace lk
