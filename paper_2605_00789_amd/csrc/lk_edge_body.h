// Device-side bodies of the edge selection (lk_select_edges.hip, where the method is described).  They take the window or
// tile and a block of LDS as arguments so that a launch can run them next to the xi passes (lk_fused.hip) as well as on
// their own.
#pragma once
#include "lk_fd_body.h"

namespace lk {

constexpr int EDGE_THREADS = 256;
constexpr int EDGE_WAVES = EDGE_THREADS / 64;
constexpr int EDGE_ITEMS = EDGE_MAX_SIDE * EDGE_MAX_SIDE / EDGE_THREADS;   // keys per thread, at most ...
constexpr int EDGE_ITEMS_SMALL = 4;                                        // ... and in windows of up to 64 tokens
constexpr int EDGE_BINS = 2048;

struct EdgeArgs {
  const int32_t *win_remove;   // k per window
  int32_t *dst, *cnt, *src_rank;
  int32_t *edges;              // [3][sum_k]: A token, B token, position among the B token's sources
  int sum_k;                   // slots of the edge list
  int key_capacity;            // 32-bit keys the launch reserved LDS for
  int clamp_v;                 // counts come from the device alone: a window's k is also bounded by its tokens, so that
                               // sum_k = the tokens of the batch always suffices
  uint32_t *big_keys;          // large windows: [n_windows][big_stride] FD keys
  size_t big_stride;
  int max_a, max_b;            // the caller's bound on the sides of a window
};

// The k a window really gets: what was asked, at most its pairs (and its tokens, see clamp_v).
__device__ __forceinline__ int edge_count(int k_asked, int nA, int nB, int clamp_v) {
  int k = k_asked < 0 ? 0 : k_asked;
  const int E = nA * nB;
  k = k > E ? E : k;
  if (clamp_v && k > nA + nB) k = nA + nB;
  return k;
}
// Slots of the windows before window w.
__device__ __forceinline__ int edge_slots_before(const FdArgs &g, const EdgeArgs &q, int w, int first, int step) {
  int before = 0;
  for (int i = first; i < w; i += step) {
    const int v = g.win_offsets[i + 1] - g.win_offsets[i];
    before += edge_count(q.win_remove[i], side_a(v, 0), side_b(v, 0), q.clamp_v);
  }
  return before;
}

// Fixed part of the LDS of edge_select_body; the keys, [nA][nB | 1], follow.
struct EdgeLds {
  double na2[EDGE_MAX_SIDE], nb2[EDGE_MAX_SIDE];
  int hist[EDGE_BINS];
  int tok[2 * EDGE_MAX_SIDE];   // the window's tokens (checked), in list order: a token lookup inside a loop must not be a
                                // trip to global memory
  uint2 cand[64];               // (key, pair index) of the keys around the threshold
  int wsum[EDGE_WAVES];
  uint32_t wlo[EDGE_WAVES], whi[EDGE_WAVES];
  int pick[3];
  int n_cand, n_slots;
};
__host__ __device__ __forceinline__ size_t edge_lds_bytes(int max_a, int max_b) {
  return sizeof(EdgeLds) + (size_t)max_a * (size_t)(max_b | 1) * sizeof(uint32_t);
}

// Selection of one window of at most 2 * EDGE_MAX_SIDE tokens.  Latency bound: one workgroup per window, a chain of
// memory trips and barriers.  (1) The slices of four neighbouring columns are one 16-byte load each, the first ones in
// flight together with the norms'.  (2) The threshold: one histogram of 2048 bins over the range the keys really span
// leaves a handful of keys in the bin that holds the k-th; these are gathered and ranked by counting with their pair
// index, which settles ties as well.  (Four passes of 8 bits over the raw keys -- the first of them useless, as FD lies
// in [0, 2] -- took 10 of the 25 us of a 55 x 55 window.)  A bin of more than 64 keys is first narrowed by another
// histogram (keys are dense around the median of unrelated tokens: 5184 pairs a window, half of them wanted, counting among up
// to 256 keys in LDS 64 us a call, among up to 64 in registers 46).  With this and the launch shared with the second xi pass, three stages of
// 2880 tokens take 316 us instead of 350.
// RECS: room for the records of a tile, chosen by the launcher (0: here).  Sixteen where one would do are half of the registers,
// and 1024 windows of 36 tokens at d = 1024 beside xi take 26 us instead of 21.  ITEMS: keys per thread, the launcher's bound.
template <int RECS, int ITEMS>
__device__ __forceinline__ void edge_select_body(const FdArgs &g, const EdgeArgs &q, int w, char *lds) {
  EdgeLds &L = *reinterpret_cast<EdgeLds *>(lds);
  uint32_t *keys = reinterpret_cast<uint32_t *>(lds + sizeof(EdgeLds));   // [nA][pitch]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const WinInfo wi = win_info(g, w);
  const int nA = wi.nA, nB = wi.nB;
  // the host refuses such windows, and sizes the LDS from its own bound on the window: a device-side list that breaks
  // either is left alone
  if (nA > EDGE_MAX_SIDE || nB > EDGE_MAX_SIDE || nA * nB > ITEMS * EDGE_THREADS || nA * (nB | 1) > q.key_capacity) return;
  const int E = nA * nB;
  const int k = edge_count(q.win_remove[w], nA, nB, q.clamp_v);

  for (int i = tid; i < nA + nB; i += EDGE_THREADS) L.tok[i] = checked_token(g, wi.off + i);
  // slots of this window in the edge list: the k of the windows before it
  int before = edge_slots_before(g, q, w, tid, EDGE_THREADS);
  if (nB == 0) {   // a window of one token (or none): no pair, nothing leaves
    for (int i = tid; i < nA; i += EDGE_THREADS) {
      const int t = L.tok[i];   // (written by this thread)
      if (t >= 0) {
        q.dst[t] = -1; q.cnt[t] = 0; q.src_rank[t] = 0;
        g.best_fd[t] = __uint_as_float(0x7f800000u);
        g.best_dst[t] = -1;
      }
    }
    return;
  }

  // ---- where the sums of row la, columns 4 c4 .. 4 c4 + 3 lie in the partial tiles
  const int64_t ks_stride = (int64_t)g.n_tiles * FD_TILE_FLOATS;
  const int per = g.mt * g.nt;
  const int row_shift = (g.group > 1) ? (w % g.group) * g.slot : 0;   // rows and columns of this window in a packed tile
  const int tile0 = (g.group > 1) ? w / g.group : w * per;
  auto tile_of = [&](int la, int lb) { return (g.group > 1) ? tile0 : tile0 + (la >> 5) * g.nt + (lb >> 5); };
  auto in_tile = [&](int l) { return (g.group > 1) ? row_shift + l : (l & 31); };
  const int n4 = (nB + 3) >> 2, units = nA * n4;
  auto unit_ptr = [&](int u) {
    u = u < units ? u : units - 1;   // surplus units re-read the last one and are dropped
    const int la = u / n4, lb = (u - la * n4) * 4;
    return g.partial + (int64_t)tile_of(la, lb) * FD_TILE_FLOATS + in_tile(la) * 32 + in_tile(lb);
  };
  const int pitch = nB | 1;   // odd: a thread per row and a thread per column both walk the array without bank conflicts
  int edge_base = 0;
  uint32_t lo = 0xffffffffu, hi = 0u;   // the range the keys span
  auto fill_keys = [&](auto n) {
    constexpr int N = decltype(n)::value;
    f32x4 v[N];
    load_records4(unit_ptr(tid), ks_stride, g.recs, v);
    for (int i = tid; i < nA + nB; i += EDGE_THREADS) {
      const float *p = i < nA ? g.partial + (int64_t)tile_of(i, 0) * FD_TILE_FLOATS + 32 * 32 + in_tile(i)
                              : g.partial + (int64_t)tile_of(0, i - nA) * FD_TILE_FLOATS + 32 * 32 + 32 + in_tile(i - nA);
      const double n2 = sum_records<N>(p, ks_stride, g.recs);
      if (i < nA) L.na2[i] = n2;
      else L.nb2[i - nA] = n2;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
    if (lane == 0) L.wsum[wave] = before;
    if (tid == 0) { L.n_cand = 0; L.n_slots = 0; }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EDGE_WAVES; ++i) edge_base += L.wsum[i];

    // ---- FD of every pair -> order-preserving key in LDS
    for (int u0 = 0; u0 < units; u0 += EDGE_THREADS) {   // uniform
      const int u = u0 + tid;
      double dot[4];
      sum_records4(v, g.recs, dot);
      if (u0 + EDGE_THREADS < units) load_records4(unit_ptr(u + EDGE_THREADS), ks_stride, g.recs, v);
      if (u < units) {
        const int la = u / n4, lb0 = (u - la * n4) * 4;
        const double a2 = L.na2[la];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int lb = lb0 + j;
          if (lb < nB) {
            float f = (float)divergence(g.metric, dot[j], a2, L.nb2[lb]);
            if (!(f >= 0.f)) f = __uint_as_float(0x7f800000u);   // NaN ranks last, like +inf
            const uint32_t key = f32_order_key(f);
            keys[la * pitch + lb] = key;
            lo = key < lo ? key : lo;
            hi = key > hi ? key : hi;
          }
        }
      }
    }
  };
  if constexpr (RECS > 0) fill_keys(std::integral_constant<int, RECS>{});
  else for_records(g.recs, fill_keys);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint32_t l2 = __shfl_xor(lo, o, 64), h2 = __shfl_xor(hi, o, 64);
    lo = l2 < lo ? l2 : lo;
    hi = h2 > hi ? h2 : hi;
  }
  if (lane == 0) { L.wlo[wave] = lo; L.whi[wave] = hi; }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < EDGE_WAVES; ++i) { lo = L.wlo[i] < lo ? L.wlo[i] : lo; hi = L.whi[i] > hi ? L.whi[i] : hi; }

  // ---- every thread takes its keys into registers (pair e = it * EDGE_THREADS + tid): the passes below then touch
  // LDS for the histogram only.  Pair index -> (A position, B position) without a division per pair: a step of
  // EDGE_THREADS pairs moves the position by (step_a, step_b) with at most one carry
  const int step_a = EDGE_THREADS / nB, step_b = EDGE_THREADS - step_a * nB;
  const int la0 = tid / nB, lb0 = tid - la0 * nB;   // this thread's first pair
  uint32_t kreg[ITEMS];
  {
    int la = la0, lb = lb0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      if (it * EDGE_THREADS >= E) break;   // uniform over the workgroup
      kreg[it] = (it * EDGE_THREADS + tid < E) ? keys[la * pitch + lb] : 0u;
      lb += step_b; la += step_a;
      if (lb >= nB) { lb -= nB; ++la; }
    }
  }

  // ---- the k-th smallest (key, pair index)
  int remaining = k;            // how many of the keys in [lo, hi] are wanted
  uint32_t threshold = lo, tie_e = 0xffffffffu;   // at the threshold: the pairs up to this index are taken
  bool ordered_ties = false;
  static_assert(EDGE_THREADS == 256 && EDGE_MAX_SIDE == 128, "a half of the workgroup per node set");
  while (k > 0) {   // uniform; every round narrows [lo, hi] by 11 bits
    const uint32_t width = hi - lo;
    const int shift = width < (uint32_t)EDGE_BINS ? 0 : (32 - __clz((int)width)) - 11;
#pragma unroll
    for (int i = 0; i < EDGE_BINS / EDGE_THREADS / 4; ++i) reinterpret_cast<uint4 *>(L.hist)[i * EDGE_THREADS + tid] = make_uint4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      if (it * EDGE_THREADS >= E) break;
      const uint32_t key = kreg[it];
      if (it * EDGE_THREADS + tid < E && key >= lo && key <= hi) atomicAdd(&L.hist[(key - lo) >> shift], 1);
    }
    __syncthreads();
    // the bin that holds the remaining-th key: inclusive scan, eight bins per thread
    const uint4 h0 = reinterpret_cast<const uint4 *>(L.hist)[2 * tid], h1 = reinterpret_cast<const uint4 *>(L.hist)[2 * tid + 1];
    const int h[8] = {(int)h0.x, (int)h0.y, (int)h0.z, (int)h0.w, (int)h1.x, (int)h1.y, (int)h1.z, (int)h1.w};
    int mine = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) mine += h[i];
    int inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    if (lane == 63) L.wsum[wave] = inc;
    __syncthreads();
    int run = inc - mine;
#pragma unroll
    for (int w2 = 0; w2 < EDGE_WAVES; ++w2) run += (w2 < wave) ? L.wsum[w2] : 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (run < remaining && remaining <= run + h[i]) { L.pick[0] = 8 * tid + i; L.pick[1] = remaining - run; L.pick[2] = h[i]; }   // exactly one bin
      run += h[i];
    }
    __syncthreads();
    lo += (uint32_t)L.pick[0] << shift;
    const uint32_t top = lo + ((1u << shift) - 1u);
    hi = top < hi ? top : hi;
    remaining = L.pick[1];
    const int in_bin = L.pick[2];
    if (shift == 0) {   // one value: `remaining` of its in_bin pairs are wanted, the first ones
      threshold = lo;
      ordered_ties = remaining < in_bin;
      break;
    }
    if (in_bin <= 64) {   // rank the keys of the bin by (key, pair index), in the registers of the first wave
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        if (it * EDGE_THREADS >= E) break;
        const uint32_t key = kreg[it];
        if (it * EDGE_THREADS + tid < E && key >= lo && key <= hi)
          L.cand[atomicAdd(&L.n_cand, 1)] = make_uint2(key, (uint32_t)(it * EDGE_THREADS + tid));
      }
      __syncthreads();
      if (wave == 0) {
        const uint2 me = L.cand[lane < in_bin ? lane : 0];
        int rank = 0;
        for (int i = 0; i < in_bin; ++i) {   // uniform
          const uint32_t ox = (uint32_t)__builtin_amdgcn_readlane((int)me.x, i), oy = (uint32_t)__builtin_amdgcn_readlane((int)me.y, i);
          rank += (ox < me.x || (ox == me.x && oy < me.y)) ? 1 : 0;
        }
        if (lane < in_bin && rank == remaining - 1) { L.pick[0] = (int)me.x; L.pick[1] = (int)me.y; }   // the order is strict: exactly one
      }
      __syncthreads();
      threshold = (uint32_t)L.pick[0];
      tie_e = (uint32_t)L.pick[1];
      break;
    }
    __syncthreads();   // pick and hist are written again
  }
  // k == 0: no key is selected (a flag rather than a sentinel threshold)
  const bool any = k > 0;
  // Pairs at the threshold that are not wanted are pushed past every real key (the largest real key is that of +inf), so
  // that afterwards "selected" simply means key <= threshold.
  if (any && ordered_ties) {   // more equal keys than threads: the wanted ones by an ordered count
    int base = 0;
    int la = la0, lb = lb0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      if (it * EDGE_THREADS >= E) break;
      const bool eq = it * EDGE_THREADS + tid < E && kreg[it] == threshold;
      const unsigned long long bal = __ballot(eq);
      const int in_wave = __popcll(bal & ((1ull << lane) - 1ull));
      __syncthreads();
      if (lane == 0) L.wsum[wave] = __popcll(bal);
      __syncthreads();
      int before_me = base + in_wave, all = 0;
#pragma unroll
      for (int w2 = 0; w2 < EDGE_WAVES; ++w2) {
        before_me += (w2 < wave) ? L.wsum[w2] : 0;
        all += L.wsum[w2];
      }
      if (eq && before_me >= remaining) keys[la * pitch + lb] = 0xffffffffu;
      base += all;
      lb += step_b; la += step_a;
      if (lb >= nB) { lb -= nB; ++la; }
    }
  } else if (any) {
    int la = la0, lb = lb0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      if (it * EDGE_THREADS >= E) break;
      const uint32_t e = (uint32_t)(it * EDGE_THREADS + tid);
      if (e < (uint32_t)E && kreg[it] == threshold && e > tie_e) keys[la * pitch + lb] = 0xffffffffu;
      lb += step_b; la += step_a;
      if (lb >= nB) { lb -= nB; ++la; }
    }
  }
  __syncthreads();

  // ---- lower half of the workgroup, per B node: its selected edges in ascending A position.  The slots of the list are
  // handed out by an LDS counter, once per node (once per edge is a serial chain of as many LDS trips as A nodes); what the
  // index scan makes of the list does not depend on their order.
  if (tid < nB) {
    const int b_tok = L.tok[2 * tid + 1];
    unsigned long long taken[EDGE_MAX_SIDE / 64] = {};   // the A positions of this node's edges
    int pos = 0;
    if (any) {
#pragma unroll
      for (int half = 0; half < EDGE_MAX_SIDE / 64; ++half) {
        const int end = nA < 64 * half + 64 ? nA : 64 * half + 64;
        for (int la8 = 64 * half; la8 < end; la8 += 8) {
          uint32_t key[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) key[i] = keys[(la8 + i < nA ? la8 + i : nA - 1) * pitch + tid];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            taken[half] |= (unsigned long long)(la8 + i < nA && key[i] <= threshold ? 1 : 0) << ((la8 & 63) + i);
        }
      }
      int n = 0;
#pragma unroll
      for (int half = 0; half < EDGE_MAX_SIDE / 64; ++half) n += __popcll(taken[half]);
      const int slot0 = edge_base + (n ? atomicAdd(&L.n_slots, n) : 0);
#pragma unroll
      for (int half = 0; half < EDGE_MAX_SIDE / 64; ++half) {
        for (unsigned long long m = taken[half]; m; m &= m - 1) {
          const int la = 64 * half + __ffsll((long long)m) - 1, slot = slot0 + pos;
          if (slot < q.sum_k) {
            q.edges[slot] = L.tok[2 * la];
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
  // ---- upper half, per A node: lowest selected edge, and the best edge whether selected or not
  if (tid >= EDGE_MAX_SIDE && tid - EDGE_MAX_SIDE < nA) {
    const int la = tid - EDGE_MAX_SIDE;
    uint32_t best = 0xffffffffu, best_sel = 0xffffffffu;
    int best_c = -1, sel_c = -1;
    for (int lb8 = 0; lb8 < nB; lb8 += 8) {
      uint32_t key8[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) key8[i] = keys[la * pitch + (lb8 + i < nB ? lb8 + i : nB - 1)];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int lb = lb8 + i;
        const uint32_t key = key8[i];
        // a key pushed past the threshold above was equal to it before
        const uint32_t real = key == 0xffffffffu ? threshold : key;
        if (lb < nB && real < best) { best = real; best_c = lb; }            // columns ascend: strict < keeps the first minimum
        if (lb < nB && any && key <= threshold && key < best_sel) { best_sel = key; sel_c = lb; }
      }
    }
    int rank = 0;
    if (sel_c >= 0)
      for (int l2 = 0; l2 < la; ++l2) rank += keys[l2 * pitch + sel_c] <= threshold ? 1 : 0;   // sel_c >= 0 implies any
    const int a_tok = L.tok[2 * la];
    if (a_tok >= 0) {
      q.dst[a_tok] = sel_c >= 0 ? L.tok[2 * sel_c + 1] : -1;
      q.src_rank[a_tok] = rank;
      q.cnt[a_tok] = 0;
      // order key back to the float it came from
      const uint32_t u = (best & 0x80000000u) ? (best & 0x7fffffffu) : ~best;
      g.best_fd[a_tok] = __uint_as_float(u);
      g.best_dst[a_tok] = best_c >= 0 ? L.tok[2 * best_c + 1] : -1;
    }
  }
}

// Keys of one 32 x 32 partial tile of a large window (one window per tile: group == 1) -> the window's key matrix.
struct EdgeKeysLds {
  double na2[32], nb2[32];
  int rtok[64];
};
template <int N>
__device__ __forceinline__ void edge_keys_records(const FdArgs &g, const EdgeArgs &q, int tile, char *lds) {
  EdgeKeysLds &L = *reinterpret_cast<EdgeKeysLds *>(lds);
  const int per = g.mt * g.nt;
  const int tid = threadIdx.x;
  const int w = tile / per, rem = tile - w * per, mt = rem / g.nt, nt = rem - mt * g.nt;
  const WinInfo wi = win_info(g, w);
  const int row0 = mt * 32, col0 = nt * 32;
  if (row0 >= wi.nA || col0 >= wi.nB || wi.nA > q.max_a || wi.nB > q.max_b) return;   // uniform
  const int64_t ks_stride = (int64_t)g.n_tiles * FD_TILE_FLOATS;
  const float *base = g.partial + (int64_t)tile * FD_TILE_FLOATS;
  // Four pairs per thread: neighbouring columns of a row where the slices are what takes time (one 16-byte load each).  With a
  // single slice every eighth row of one column, one load a pair, so that a wave writes
  // whole runs of the matrix: 64 windows of 576 tokens at d = 256 33 -> 21 us (sixteen copies of each load before).
  constexpr bool one = N == 1;
  const int r0 = one ? tid >> 5 : tid >> 3, c0 = one ? tid & 31 : (tid & 7) * 4;
  const int dr = one ? 8 : 0, dc = one ? 0 : 1;
  f32x4 v[N];
  if constexpr (one) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[0][j] = base[(r0 + 8 * j) * 32 + c0];
  } else {
    load_records4(base + r0 * 32 + c0, ks_stride, g.recs, v);
  }
  if (tid < 64) {
    // |a|^2 was accumulated by the first tile of this row of tiles, |b|^2 by the first tile of this column of tiles
    const int i = tid & 31;
    if (tid < 32) L.na2[i] = sum_records<N>(g.partial + (int64_t)(w * per + mt * g.nt) * FD_TILE_FLOATS + 32 * 32 + i, ks_stride, g.recs);
    else L.nb2[i] = sum_records<N>(g.partial + (int64_t)(w * per + nt) * FD_TILE_FLOATS + 32 * 32 + 32 + i, ks_stride, g.recs);
    L.rtok[tid] = reinterpret_cast<const int32_t *>(base + FD_TOK_OFFSET)[tid];   // tokens of the 32 rows, then of the 32 columns
  }
  double dot[4];
  sum_records4(v, g.recs, dot);
  __syncthreads();
  uint32_t *M = q.big_keys + (size_t)w * q.big_stride;
  const int pitch = wi.nB;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = r0 + dr * j, c = c0 + dc * j, la = row0 + r, lb = col0 + c;
    float f = (float)divergence(g.metric, dot[j], L.na2[r], L.nb2[c]);
    if (!(f >= 0.f) || L.rtok[r] < 0 || L.rtok[32 + c] < 0) f = __uint_as_float(0x7f800000u);   // NaN ranks last, like +inf
    if (la < wi.nA && lb < wi.nB) M[(size_t)la * pitch + lb] = f32_order_key(f);
  }
}
__device__ __forceinline__ void edge_keys_body(const FdArgs &g, const EdgeArgs &q, int tile, char *lds) {
  if (g.recs > 1) for_records(g.recs, [&](auto n) { edge_keys_records<decltype(n)::value>(g, q, tile, lds); });   // uniform
  else edge_keys_records<1>(g, q, tile, lds);
}

}  // namespace lk
