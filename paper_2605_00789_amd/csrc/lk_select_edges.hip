// Step 2 of the paper's Sec. 3.2.1 read literally: the candidate set T_rho of a window is made of the k lowest-FD EDGES
// of the complete bipartite graph between its node sets A and B -- not one edge per A node.  An A node then owns as
// many edges as rank that low (it is averaged into each of those B nodes with its full weight, Eq. "message-passing"
// with several ones in a row of M) and leaves if it owns at least one, so the number of tokens that go depends on
// the data: between ceil(k / |B|) and min(k, |A|) per window.
//
//   edge_select_kernel : one workgroup per window (body in lk_edge_body.h).  Reads the partial inner-product tiles that
//                        fd_partial_kernel left (lk_score_fd.hip), forms FD of every (a, b) pair into LDS as an
//                        order-preserving integer key, finds the k-th smallest (key, pair index) by LDS histograms
//                        (integer counts, so the result does not depend on the order of the atomics), and writes
//                          dst[a]      the B token of a's lowest selected edge, -1 if a stays
//                          src_rank[a] position of a among the sources of that B token
//                          cnt[b]      number of selected edges into b
//                          best_fd / best_dst  of every A node, as the default selection reports them
//                        plus the window's edge list (a, b, position of a among b's sources) at a fixed offset
//                        (the k of the windows before it); every window writes all of its slots.
//   select_scan_kernel : new_index from dst, grp_offsets from cnt, grp_src[grp_offsets[b] + position] = a for every edge
//                        of the list (lk_select.hip; long lists: edge_fill_kernel behind it).
// With xi requested the same bodies run beside the second xi pass (lk_fused.hip).
//
// Windows of more than 2 * EDGE_MAX_SIDE tokens (up to the library's 4096) do not fit that kernel's LDS; for them
//   edge_keys_kernel       : one workgroup per 32 x 32 partial tile: FD of its pairs as order-preserving keys into a
//                            |A| x |B| matrix per window in the workspace (row-major, pitch |B|)
//   edge_select_big_kernel : one workgroup of 1024 threads per window works on that matrix: the k-th smallest of the
//                            composite keys (FD key, pair index) by a radix select of 11 + 11 + 10 bits over the FD key
//                            and, only if the threshold value is shared by more pairs than are still wanted, 11 + 11 bits
//                            over the pair index (row-major, so a tie at the threshold goes by (A position, B position)
//                            exactly as in the small kernel, without an ordered pass); then one pass by rows (best edge
//                            and lowest selected edge of every A node) and one by columns (sources of every B node, edge
//                            list).  The slots of the edge list are handed out by an LDS counter: the list is scratch,
//                            and what the index scan makes of it does not depend on the slot order.
// The passes re-read the matrix from L2 / memory; one workgroup per window keeps this simple and is adequate for
// the 300- to 600-token windows of the coarse stages (a 2880-token window takes a few hundred microseconds).
#include <atomic>
#include "lk_edge_body.h"

namespace lk {

template <int RECS, int ITEMS>
__global__ __launch_bounds__(EDGE_THREADS, ITEMS == EDGE_ITEMS ? 2 : 3) void edge_select_kernel(FdArgs g, EdgeArgs q) {
  fetch_args<FdArgs, EdgeArgs>();
  extern __shared__ __attribute__((aligned(16))) char edge_lds[];
  edge_select_body<RECS, ITEMS>(g, q, blockIdx.x, edge_lds);
}
__global__ __launch_bounds__(EDGE_THREADS) void edge_keys_kernel(FdArgs g, EdgeArgs q) {
  fetch_args<FdArgs, EdgeArgs>();
  __shared__ __attribute__((aligned(16))) char lds[sizeof(EdgeKeysLds)];
  edge_keys_body(g, q, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------------------------------------------------
// Large windows: FD keys of every pair in a matrix per window (global memory), selection by one workgroup per window.
constexpr int EB_THREADS = 1024;
constexpr int EB_WAVES = EB_THREADS / 64;
constexpr int EB_MAX_SIDE = 2048;   // |A| and |B| of the library's largest window
constexpr int EB_BINS = 2048;       // 11-bit digits

constexpr int EB_LOADS = 16;   // keys a thread keeps in flight per step of the radix and column passes
constexpr int EB_ROWS = 4;     // rows a wave takes at a time in the row pass
__global__ __launch_bounds__(EB_THREADS) void edge_select_big_kernel(FdArgs g, EdgeArgs q) {
  fetch_args<FdArgs, EdgeArgs>();
  __shared__ int hist[EB_BINS];
  __shared__ int tok[2 * EB_MAX_SIDE];
  __shared__ uint16_t selcol[EB_MAX_SIDE];   // lowest selected edge of every A node (0xffff: none)
  __shared__ int wsum[EB_WAVES];
  __shared__ int pick[3];
  __shared__ int slot_counter;
  const int w = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const WinInfo wi = win_info(g, w);
  const int nA = wi.nA, nB = wi.nB;
  if (nA > q.max_a || nB > q.max_b || nA > EB_MAX_SIDE || nB > EB_MAX_SIDE) return;   // refused by the host; left alone
  const int E = nA * nB;
  const int k = edge_count(q.win_remove[w], nA, nB, q.clamp_v);
  for (int i = tid; i < nA + nB; i += EB_THREADS) tok[i] = checked_token(g, wi.off + i);
  if (tid == 0) slot_counter = 0;
  // slots of this window in the edge list (the barriers inside also publish tok[] and the counter)
  int before = edge_slots_before(g, q, w, tid, EB_THREADS);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
  if (lane == 0) wsum[wave] = before;
  __syncthreads();
  int edge_base = 0;
#pragma unroll
  for (int i = 0; i < EB_WAVES; ++i) edge_base += wsum[i];
  __syncthreads();
  if (nB == 0) {   // a window of one token (or none): no pair, nothing leaves
    for (int i = tid; i < nA; i += EB_THREADS) {
      const int t = tok[i];
      if (t >= 0) {
        q.dst[t] = -1; q.cnt[t] = 0; q.src_rank[t] = 0;
        g.best_fd[t] = __uint_as_float(0x7f800000u);
        g.best_dst[t] = -1;
      }
    }
    return;
  }
  const uint32_t *M = q.big_keys + (size_t)w * q.big_stride;

  // ---- the k-th smallest composite key (FD key, pair index): radix select, most significant digit first.
  // Passes 0..2 take the FD key (11, 11, 10 bits), passes 3..4 the pair index (11, 11 bits: E <= 2^22).
  uint32_t kprefix = 0, kmask = 0, eprefix = 0, emask = 0;
  int remaining = k, n_equal = 0;
  for (int pass = 0; pass < 5 && k > 0; ++pass) {   // uniform
    if (pass == 3 && remaining == n_equal) break;   // every pair at the threshold value is wanted: no tie to break
    for (int i = tid; i < EB_BINS; i += EB_THREADS) hist[i] = 0;
    __syncthreads();
    int run_digit = -1, run = 0;   // FD lies in a narrow range: a thread adds a run of equal digits once
    for (int e0 = tid; e0 < E; e0 += EB_LOADS * EB_THREADS) {
      uint32_t key[EB_LOADS];
#pragma unroll
      for (int u = 0; u < EB_LOADS; ++u) { const int e = e0 + u * EB_THREADS; key[u] = M[e < E ? e : E - 1]; }
#pragma unroll
      for (int u = 0; u < EB_LOADS; ++u) {
        const uint32_t e = (uint32_t)(e0 + u * EB_THREADS);
        const bool in = e < (uint32_t)E && (key[u] & kmask) == kprefix && (e & emask) == eprefix;
        int digit;
        if (pass == 0) digit = (int)(key[u] >> 21);
        else if (pass == 1) digit = (int)((key[u] >> 10) & 2047u);
        else if (pass == 2) digit = (int)(key[u] & 1023u);
        else if (pass == 3) digit = (int)((e >> 11) & 2047u);
        else digit = (int)(e & 2047u);
        digit = in ? digit : run_digit;
        if (digit != run_digit) {
          if (run > 0) atomicAdd(&hist[run_digit], run);
          run_digit = digit;
          run = 0;
        }
        run += in ? 1 : 0;
      }
    }
    if (run > 0) atomicAdd(&hist[run_digit], run);
    __syncthreads();
    // the bin that holds the remaining-th key: inclusive scan over the bins, two per thread
    const int h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
    int inc = h0 + h1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    for (int w2 = 0; w2 < wave; ++w2) inc += wsum[w2];
    const int exc = inc - h0 - h1;
    if (exc < remaining && remaining <= exc + h0) { pick[0] = 2 * tid; pick[1] = remaining - exc; pick[2] = h0; }              // exactly one bin
    else if (exc + h0 < remaining && remaining <= inc) { pick[0] = 2 * tid + 1; pick[1] = remaining - exc - h0; pick[2] = h1; }
    __syncthreads();
    const uint32_t digit = (uint32_t)pick[0];
    if (pass == 0) { kprefix |= digit << 21; kmask |= 2047u << 21; }
    else if (pass == 1) { kprefix |= digit << 10; kmask |= 2047u << 10; }
    else if (pass == 2) { kprefix |= digit; kmask |= 1023u; }
    else if (pass == 3) { eprefix |= digit << 11; emask |= 2047u << 11; }
    else { eprefix |= digit; emask |= 2047u; }
    remaining = pick[1];
    n_equal = pick[2];
    __syncthreads();
  }
  const bool any = k > 0;
  const uint32_t T = kprefix;
  const uint32_t Te = emask ? eprefix : 0xffffffffu;   // at the threshold value: the pairs up to this index are taken
  auto selected = [&](uint32_t key, uint32_t e) { return any && (key < T || (key == T && e <= Te)); };

  // ---- by rows: best edge and lowest selected edge of every A node (a wave takes EB_ROWS rows at a time, so that
  // their loads are in flight together; lanes stride the columns)
  for (int la0 = wave * EB_ROWS; la0 < nA; la0 += EB_WAVES * EB_ROWS) {
    unsigned long long best_r[EB_ROWS], best_sel_r[EB_ROWS];   // (key << 32 | column): the minimum is the first minimum
#pragma unroll
    for (int r = 0; r < EB_ROWS; ++r) { best_r[r] = ~0ull; best_sel_r[r] = ~0ull; }
    for (int lb0 = lane; lb0 < nB; lb0 += 4 * 64) {
      uint32_t key[EB_ROWS][4];
#pragma unroll
      for (int r = 0; r < EB_ROWS; ++r) {
        const uint32_t *row = M + (size_t)(la0 + r < nA ? la0 + r : nA - 1) * nB;
#pragma unroll
        for (int u = 0; u < 4; ++u) { const int lb = lb0 + u * 64; key[r][u] = row[lb < nB ? lb : nB - 1]; }
      }
#pragma unroll
      for (int r = 0; r < EB_ROWS; ++r) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int lb = lb0 + u * 64;
          if (lb < nB && la0 + r < nA) {
            const unsigned long long c = ((unsigned long long)key[r][u] << 32) | (unsigned)lb;
            best_r[r] = c < best_r[r] ? c : best_r[r];
            if (selected(key[r][u], (uint32_t)((la0 + r) * nB + lb))) best_sel_r[r] = c < best_sel_r[r] ? c : best_sel_r[r];
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < EB_ROWS; ++r) {
      unsigned long long best = best_r[r], best_sel = best_sel_r[r];
      const int la = la0 + r;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long ob = __shfl_xor(best, o, 64), os = __shfl_xor(best_sel, o, 64);
        best = ob < best ? ob : best;
        best_sel = os < best_sel ? os : best_sel;
      }
      if (lane == 0 && la < nA) {
        const int sel_c = best_sel == ~0ull ? -1 : (int)(best_sel & 0xffffffffu);
        selcol[la] = sel_c < 0 ? (uint16_t)0xffffu : (uint16_t)sel_c;
        const int a_tok = tok[2 * la];
        if (a_tok >= 0) {
          const uint32_t bk = (uint32_t)(best >> 32);
          const uint32_t u = (bk & 0x80000000u) ? (bk & 0x7fffffffu) : ~bk;   // order key back to the float it came from
          g.best_fd[a_tok] = __uint_as_float(u);
          g.best_dst[a_tok] = tok[2 * (int)(best & 0xffffffffu) + 1];
          q.dst[a_tok] = sel_c >= 0 ? tok[2 * sel_c + 1] : -1;
          q.cnt[a_tok] = 0;
          if (sel_c < 0) q.src_rank[a_tok] = 0;   // (a node that leaves gets its rank from the column pass below)
        }
      }
    }
  }
  __syncthreads();
  // ---- by columns: the sources of every B node in ascending A position, edge list, rank of every leaving A node
  for (int lb = tid; lb < nB; lb += EB_THREADS) {
    const int b_tok = tok[2 * lb + 1];
    int pos = 0;
    for (int la0 = 0; la0 < nA; la0 += EB_LOADS) {
      uint32_t key[EB_LOADS];
#pragma unroll
      for (int u = 0; u < EB_LOADS; ++u) { const int la = la0 + u; key[u] = M[(size_t)(la < nA ? la : nA - 1) * nB + lb]; }
#pragma unroll
      for (int u = 0; u < EB_LOADS; ++u) {
        const int la = la0 + u;
        if (la < nA && selected(key[u], (uint32_t)(la * nB + lb))) {
          const int a_tok = tok[2 * la];
          if (selcol[la] == (uint16_t)lb && a_tok >= 0) q.src_rank[a_tok] = pos;
          const int slot = edge_base + atomicAdd(&slot_counter, 1);
          if (slot < q.sum_k) {
            q.edges[slot] = a_tok;
            q.edges[q.sum_k + slot] = b_tok;
            q.edges[2 * q.sum_k + slot] = pos;
          }
          ++pos;
        }
      }
    }
    if (b_tok >= 0) {
      q.dst[b_tok] = -1; q.cnt[b_tok] = pos; q.src_rank[b_tok] = 0;
      g.best_fd[b_tok] = __uint_as_float(0x7f800000u);
      g.best_dst[b_tok] = -1;
    }
  }
}

EdgeArgs make_edge_args(int max_window, int sum_k, const int32_t *win_remove, int32_t *dst, int32_t *cnt, int32_t *src_rank,
                        int32_t *edges, bool device_counts, uint32_t *big_keys) {
  const int maxA = (max_window + 1) / 2, maxB = max_window / 2;
  EdgeArgs q{};
  q.win_remove = win_remove; q.dst = dst; q.cnt = cnt; q.src_rank = src_rank; q.edges = edges; q.sum_k = sum_k;
  q.key_capacity = maxA * (maxB | 1); q.clamp_v = device_counts ? 1 : 0;
  q.big_keys = big_keys; q.big_stride = (size_t)maxA * (size_t)(maxB > 0 ? maxB : 1); q.max_a = maxA; q.max_b = maxB;
  return q;
}

hipError_t launch_edge_select_big(const FdArgs &g, const EdgeArgs &q, hipStream_t stream) {
  if (q.max_a > EB_MAX_SIDE || !q.big_keys || g.group != 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(edge_select_big_kernel, dim3((unsigned)g.n_windows), dim3(EB_THREADS), 0, stream, g, q);
  return hipGetLastError();
}

hipError_t launch_edge_select(const FdArgs &g, const EdgeArgs &q, int dtype, hipStream_t stream) {
  if (g.n_windows == 0 || g.n_tiles == 0) return hipSuccess;
  hipError_t e = launch_fd_partial(g, dtype, stream);
  if (e != hipSuccess) return e;
  if (q.max_a > EDGE_MAX_SIDE) {   // windows beyond the one-kernel path
    if (q.max_a > EB_MAX_SIDE || !q.big_keys || g.group != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(edge_keys_kernel, dim3((unsigned)g.n_tiles), dim3(EDGE_THREADS), 0, stream, g, q);
    e = hipGetLastError();
    return e != hipSuccess ? e : launch_edge_select_big(g, q, stream);
  }
  static std::atomic<bool> allowed[64];   // more dynamic LDS than the 64 KB default, set once per device
  using Kernel = void (*)(FdArgs, EdgeArgs);
  static const Kernel kernels[4][2] = {{edge_select_kernel<1, EDGE_ITEMS_SMALL>, edge_select_kernel<1, EDGE_ITEMS>},
                                       {edge_select_kernel<4, EDGE_ITEMS_SMALL>, edge_select_kernel<4, EDGE_ITEMS>},
                                       {edge_select_kernel<8, EDGE_ITEMS_SMALL>, edge_select_kernel<8, EDGE_ITEMS>},
                                       {edge_select_kernel<16, EDGE_ITEMS_SMALL>, edge_select_kernel<16, EDGE_ITEMS>}};
  static_assert(FD_MAX_RECS == 16, "the last row serves every number of records");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!allowed[dev].load(std::memory_order_acquire)) {
    for (int i = 0; i < 8; ++i) {
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernels[i >> 1][i & 1]), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)edge_lds_bytes(EDGE_MAX_SIDE, EDGE_MAX_SIDE));
      if (e != hipSuccess) return e;
    }
    allowed[dev].store(true, std::memory_order_release);
  }
  const Kernel k = kernels[g.recs == 1 ? 0 : g.recs <= 4 ? 1 : g.recs <= 8 ? 2 : 3][q.max_a * q.max_b > EDGE_ITEMS_SMALL * EDGE_THREADS];
  hipLaunchKernelGGL(k, dim3((unsigned)g.n_windows), dim3(EDGE_THREADS), edge_lds_bytes(q.max_a, q.max_b), stream, g, q);
  return hipGetLastError();
}

size_t edge_big_key_count(int n_windows, int max_window) {
  const int maxA = (max_window + 1) / 2, maxB = max_window / 2;
  if (maxA <= EDGE_MAX_SIDE) return 0;
  return (size_t)n_windows * (size_t)maxA * (size_t)(maxB > 0 ? maxB : 1);
}

}  // namespace lk
