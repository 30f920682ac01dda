// Device-side bodies of the small-window feature-divergence kernels (paper Sec. 3.2.1 Steps 1-2).  They take the
// workgroup index and a block of LDS as arguments so that a launch can run them next to the bodies of another step
// (lk_fused.hip) as well as on their own (lk_score_fd.hip, where the algorithm is described).
#pragma once
#include <type_traits>
#include "lk_common.h"
#include "lk_launch.h"

namespace lk {


constexpr int FD_THREADS = 256;
constexpr int FD_WAVES = 4;
constexpr int FD_CHUNKS = 4;   // 16-byte chunks per lane and span
constexpr double NORM_EPS = 1e-12;

struct FdArgs {
  const void *X;
  int64_t ldx;
  int d, n_windows, sum_n;
  const int32_t *win_offsets, *win_tokens;
  float *partial;
  float *best_fd;
  int32_t *best_dst;
  int slot, group, mt, nt, n_tiles, ksplit, n_spans, spans_per_wg, chain, recs;
  int metric;   // 0: 1 - cos, 1: |a - b|, 2: |a - b|^2
  int dir;      // 0: even list positions propose, 1: odd ones, PAIR_DIR: all to all others (side_a / pos_a)
  unsigned long long *pair_keys;   // PAIR_DIR: where the epilogue files (FD bits << 32 | neighbour's position) by list
                                   // position; NULL: it writes best_fd / best_dst
};

// Divergence of a pair from its inner product and squared norms (fp64).  The distances use
// |a - b|^2 = |a|^2 + |b|^2 - 2 <a, b>; the three sums of a pair come from the same instruction sequence, so identical
// rows give exactly 0.
__device__ __forceinline__ double divergence(int metric, double dot, double a2, double b2) {
  if (metric == 0) {
    double den;
    if (a2 >= NORM_EPS * NORM_EPS && b2 >= NORM_EPS * NORM_EPS) den = sqrt(a2 * b2);
    else den = fmax(sqrt(a2), NORM_EPS) * fmax(sqrt(b2), NORM_EPS);
    const double fd = 1.0 - dot / den;
    return fd < 0.0 ? 0.0 : fd;   // (a NaN stays a NaN: fmax would turn it into the best possible score)
  }
  const double d2 = a2 + b2 - 2.0 * dot;
  return metric == 1 ? sqrt(d2 < 0.0 ? 0.0 : d2) : (d2 < 0.0 ? 0.0 : d2);
}

// LDS of fd_partial_body: a staged piece of the tile's 64 rows (one 128-byte span per wave and row; the rows padded by 16
// bytes, so that the sixteen lanes of a quarter wave read their 16-byte fragments from 64 different banks), and afterwards
// the four waves' sums.
constexpr int FD_STAGE_BYTES = FD_WAVES * 128;
constexpr int FD_STAGE_PITCH = FD_STAGE_BYTES + 16;
constexpr int FD_RED_LDS = FD_WAVES * (32 * 32 + 2 * 32) * (int)sizeof(double);
constexpr int FD_PARTIAL_LDS = 64 * FD_STAGE_PITCH > FD_RED_LDS ? 64 * FD_STAGE_PITCH : FD_RED_LDS;

struct WinInfo { int off, nA, nB; };

__device__ __forceinline__ WinInfo win_info(const FdArgs &g, int w) {
  WinInfo wi{0, 0, 0};
  if (w < g.n_windows) {
    wi.off = g.win_offsets[w];
    const int v = g.win_offsets[w + 1] - wi.off;
    wi.nA = side_a(v, g.dir);
    wi.nB = side_b(v, g.dir);
  }
  return wi;
}

__device__ __forceinline__ int checked_token(const FdArgs &g, int idx) {
  const int t = g.win_tokens[idx];
  return ((unsigned)t < (unsigned)g.sum_n) ? t : -1;
}

template <typename T>
__device__ __forceinline__ void fd_partial_body(const FdArgs &g, int block_id, char *lds) {
  using E = Elem<T>;
  constexpr int SPAN = 2 * FD_CHUNKS * E::PER_CHUNK;   // elements of a row covered by one span: 64 bytes per half wave

  const int tile = block_id % g.n_tiles;
  const int ks = block_id / g.n_tiles;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 31, half = lane >> 5;

  // rows of this tile
  int a_tok = -1, b_tok = -1;
  bool need_na = true, need_nb = true;
  if (g.group > 1) {
    const int s = r / g.slot, l = r - s * g.slot;
    const WinInfo wi = win_info(g, tile * g.group + s);
    if (l < wi.nA) a_tok = checked_token(g, wi.off + pos_a(l, g.dir));
    if (l < wi.nB) b_tok = checked_token(g, wi.off + pos_b(l, g.dir));
  } else {
    const int per = g.mt * g.nt;
    const int w = tile / per, rem = tile - w * per;
    const int mt = rem / g.nt, nt = rem - mt * g.nt;
    const WinInfo wi = win_info(g, w);
    const int la = mt * 32 + r, lb = nt * 32 + r;
    if (la < wi.nA) a_tok = checked_token(g, wi.off + pos_a(la, g.dir));
    if (lb < wi.nB) b_tok = checked_token(g, wi.off + pos_b(lb, g.dir));
    need_na = (nt == 0);
    need_nb = (mt == 0);
  }
  // slice 0 leaves the tile's token lists (rows, then columns) for the kernel that finishes the tile
  if (ks == 0 && wave == 0)
    reinterpret_cast<int32_t *>(g.partial + (int64_t)tile * FD_TILE_FLOATS + FD_TOK_OFFSET)[lane] = half ? b_tok : a_tok;
  // a tile without A rows or without B rows is never read by the epilogue
  if (__ballot(a_tok >= 0) == 0ull || __ballot(b_tok >= 0) == 0ull) return;

  // The slice travels through LDS in pieces of four spans (one per wave): a wave instruction fetches 512 contiguous bytes
  // of two rows.  Fetched straight into MFMA operands, every lane's 16 bytes lie on a line of their own and the lines of
  // the waves in flight are many times the CU's L1, which costs twice the trips: 2880 tokens in
  // 180 windows 10.6 -> 8.9 us cold, 8.1 -> 6.9 us with X in the caches.
  // Padding rows of the tile read token 0: their products land in rows/columns nobody reads.
  constexpr int ROW_PASSES = 64 / (FD_THREADS / 32);      // 32 threads a row, eight rows per pass
  const int srow = threadIdx.x >> 5, schunk = threadIdx.x & 31;
  const char *rows[ROW_PASSES];
#pragma unroll
  for (int p = 0; p < ROW_PASSES; ++p) {
    const int q = p * (FD_THREADS / 32) + srow;            // rows 0..31: A nodes, 32..63: B nodes
    const int t = __shfl(p < ROW_PASSES / 2 ? a_tok : b_tok, q & 31, 64);
    rows[p] = static_cast<const char *>(g.X) + (int64_t)(t < 0 ? 0 : t) * g.ldx * E::BYTES;
  }
  const int64_t row_bytes = (int64_t)g.d * E::BYTES;
  uint4 st[ROW_PASSES];
  auto load_piece = [&](int s) {   // spans s .. s + 3
    const int64_t o = (int64_t)s * 128 + schunk * 16;
    const bool ok = o + 16 <= row_bytes;
#pragma unroll
    for (int p = 0; p < ROW_PASSES; ++p) {
      const uint4 t = ld16(rows[p] + (ok ? o : row_bytes - 16));   // unconditional load from a clamped address, zeroed
      st[p] = ok ? t : make_uint4(0, 0, 0, 0);
    }
  };
  static_assert(SPAN * E::BYTES == 128, "a span is one 128-byte line of a row");

  // The matrix cores add in fp32.  1 - cos of near-equal rows keeps what those sums lose, so their chains are kept short: in a
  // slice of several chains (`two`, uniform) each goes into an fp64 sum, and the slice's sums leave as two floats.  Error of
  // 1 - cos against 64 bits, rows a few percent apart, rms: 80 tiles, d = 4096, 16 slices 1.4e-8, 4 long ones added in fp32
  // throughout 3.4e-8, so 0.8e-8; 96 tiles, d = 5120, 2.3e-8, 4.3e-8, 1.2e-8.
  const bool two = g.recs > g.ksplit;
  f32x16 acc = {0}, na = {0}, nb = {0};
  double sum[16], sum_a = 0.0, sum_b = 0.0;   // (of the norms this lane's diagonal element (r, r), where it holds one)
#pragma unroll
  for (int i = 0; i < 16; ++i) sum[i] = 0.0;
  auto diagonal = [&](const f32x16 &norms) {
    const int idx = 4 * (r >> 3) + (r & 3);
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) d = (i == idx) ? norms[i] : d;
    return d;
  };
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[i] += (double)acc[i];
    if (need_na) sum_a += (double)diagonal(na);
    if (need_nb) sum_b += (double)diagonal(nb);
  };
  int left = g.chain;
  const int s_begin = ks * g.spans_per_wg;
  const int s_end = min(s_begin + g.spans_per_wg, g.n_spans);
  const char *frag = lds + r * FD_STAGE_PITCH + wave * 128 + half * 64;
  if (s_begin < s_end) load_piece(s_begin);
  for (int s = s_begin; s < s_end; s += FD_WAVES) {   // uniform
    if (s > s_begin) __syncthreads();   // the piece before has been consumed
#pragma unroll
    for (int p = 0; p < ROW_PASSES; ++p)
      *reinterpret_cast<uint4 *>(lds + (p * (FD_THREADS / 32) + srow) * FD_STAGE_PITCH + schunk * 16) = st[p];
    __syncthreads();
    if (s + FD_WAVES < s_end) load_piece(s + FD_WAVES);
    const bool fresh = left == g.chain;   // uniform
    if (s + wave < s_end) {
#pragma unroll
      for (int c = 0; c < FD_CHUNKS; ++c) {
        const uint4 ca = *reinterpret_cast<const uint4 *>(frag + c * 16);
        const uint4 cb = *reinterpret_cast<const uint4 *>(frag + 32 * FD_STAGE_PITCH + c * 16);
        auto multiply = [&](const uint4 &x, const uint4 &y, f32x16 &sum32) {
          if (c == 0 && fresh) {   // a chain begins: zero as the instruction's constant, not 16 registers set to it
            f32x16 begin = {0};
            E::mma32(x, y, begin);
            sum32 = begin;
          } else {
            E::mma32(x, y, sum32);
          }
        };
        multiply(ca, cb, acc);
        if (need_na) multiply(ca, ca, na);
        if (need_nb) multiply(cb, cb, nb);
      }
    } else if (fresh) {   // no span of the last piece for this wave
      acc = f32x16{0}; na = f32x16{0}; nb = f32x16{0};
    }
    if (--left == 0 && two) {   // uniform
      flush();
      left = g.chain;
    }
  }
  if (two && left != g.chain) flush();
  __syncthreads();   // the stage becomes the reduction buffer

  // cross-wave sum through LDS
  float *out = g.partial + ((int64_t)(two ? 2 * ks : ks) * g.n_tiles + tile) * FD_TILE_FLOATS;
  const bool on_diagonal = ((r >> 2) & 1) == half;   // this lane holds the element (r, r)
  auto add_waves = [&](auto zero, auto element, auto norm_a, auto norm_b, auto put) {
    using S = decltype(zero);
    S (*red)[32 * 32] = reinterpret_cast<S (*)[32 * 32]>(lds);                                  // [FD_WAVES][32 * 32]
    S (*rnorm)[2][32] = reinterpret_cast<S (*)[2][32]>(lds + FD_WAVES * 32 * 32 * sizeof(S));   // [FD_WAVES][2][32]
#pragma unroll
    for (int i = 0; i < 16; ++i) red[wave][acc_row(i, lane) * 32 + r] = element(i);
    if (on_diagonal) {
      rnorm[wave][0][r] = norm_a;
      rnorm[wave][1][r] = norm_b;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * 32; e += FD_THREADS) put(e, (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]));
    if (threadIdx.x < 64) {
      const int which = threadIdx.x >> 5, i = threadIdx.x & 31;
      put(32 * 32 + threadIdx.x, (rnorm[0][which][i] + rnorm[1][which][i]) + (rnorm[2][which][i] + rnorm[3][which][i]));
    }
  };
  if (two) {
    float *out_low = out + (int64_t)g.n_tiles * FD_TILE_FLOATS;
    add_waves(0.0, [&](int i) { return sum[i]; }, sum_a, sum_b, [&](int e, double v) {
      // (a sum beyond the type's largest value goes on in the second float, infinities and NaN stay what they are)
      const float high = (float)fmax(fmin(v, 3.4028234663852886e38), -3.4028234663852886e38);
      out[e] = high;
      out_low[e] = (float)(v - (double)high);
    });
  } else {
    add_waves(0.f, [&](int i) { return acc[i]; }, diagonal(na), diagonal(nb), [&](int e, float v) { out[e] = v; });
  }
}

constexpr int FD_MAX_RECS = 16;   // records of partial sums per tile

// f(N) with the smallest N of 4, 8, 16 that covers a tile's records: uniform, so a branch, and ONE for a whole body: an array of
// loads that lives across two such branches ends in scratch memory (80 windows of 30 tokens, d = 4096, 64 prompt rows, scores and
// selection 26.9 us, so 25.8; 20 of 96 tokens 32.6 / 32.0).  Inside it every load is unconditional (surplus records
// re-read the last one and are dropped afterwards), the compiler then issues all of them before the first wait.
template <typename F> __device__ __forceinline__ void for_records(int recs, F f) {
  if (recs > 8) f(std::integral_constant<int, FD_MAX_RECS>{});   // first: it takes the most registers, and two fewer in this place
  else if (recs <= 4) f(std::integral_constant<int, 4>{});
  else f(std::integral_constant<int, 8>{});
}
// Sum of one partial value over the records, in their order (fp64).
template <int N> __device__ __forceinline__ double sum_records(const float *p, int64_t stride, int recs) {
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = p[(i < recs ? i : recs - 1) * stride];
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) s += (i < recs) ? (double)v[i] : 0.0;
  return s;
}
// The same for four neighbouring values: the loads (16 bytes each, all in flight together) and the sums are separate
// calls, so that other loads can be issued between them.
template <int N> __device__ __forceinline__ void load_records4(const float *p, int64_t stride, int recs, f32x4 (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = *reinterpret_cast<const f32x4 *>(p + (i < recs ? i : recs - 1) * stride);
}
template <int N> __device__ __forceinline__ void sum_records4(const f32x4 (&v)[N], int recs, double (&dot)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) dot[j] = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) dot[j] += (i < recs) ? (double)v[i][j] : 0.0;
  }
}

// ---------------------------------------------------------------------------------------------------------
// Windows of more than 64 tokens: best edge of every A node from the partial tiles.  TPR = 8 * min(column tiles, 4)
// threads share an A row, each takes four neighbouring columns of every TPR/8-th column tile: the slices of up to
// 128 columns of a row are one round trip (with eight threads a row, 64 to 255 columns were 2 to 8 trips in a row:
// 16 us for a window of 387 tokens).  A workgroup covers FD_THREADS / TPR rows.  The squared norms of the window's
// columns go to LDS; their loads and those of the first products are in flight together.
constexpr int FD_EPILOGUE_LDS = (FD_MAX_COLS + 32) * (int)sizeof(double);
__host__ __device__ __forceinline__ int fd_epilogue_tpr_shift(int group, int nt) {   // log2 of TPR
  return group > 1 || nt == 1 ? 3 : (nt == 2 ? 4 : 5);
}
__host__ __device__ __forceinline__ int fd_epilogue_blocks(int n_rowblocks, int group, int nt) {
  return n_rowblocks << (fd_epilogue_tpr_shift(group, nt) - 3);
}

template <int N>
__device__ __forceinline__ void fd_epilogue_records(const FdArgs &g, int block_id, char *lds) {
  double *nb2 = reinterpret_cast<double *>(lds);          // [FD_MAX_COLS]
  double *na2 = nb2 + FD_MAX_COLS;                        // [32]
  const int64_t ks_stride = (int64_t)g.n_tiles * FD_TILE_FLOATS;
  const int per = g.mt * g.nt;
  const int tsh = fd_epilogue_tpr_shift(g.group, g.nt);
  const int parts = 1 << (tsh - 3);                       // workgroups per 32-row block
  const int rb = block_id / parts;
  const int row_in_block = (block_id - rb * parts) * (FD_THREADS >> tsh) + ((int)threadIdx.x >> tsh);   // 0..31
  const int sub = (int)threadIdx.x & ((1 << tsh) - 1);

  int tile_row0;            // tile holding the dots of (this row block, column tile 0)
  int tile_col0;            // tile holding |b|^2 of column tile 0
  int w_single = 0, m_single = 0;
  if (g.group > 1) {
    tile_row0 = tile_col0 = rb;
  } else {
    w_single = rb / g.mt;
    m_single = rb - w_single * g.mt;
    tile_row0 = w_single * per + m_single * g.nt;
    tile_col0 = w_single * per;
  }
  const int ncol_tiles = (g.group > 1) ? 1 : g.nt;
  const int t_step = parts;                               // column tiles one sweep of a row's threads covers
  const float *prow = g.partial + (int64_t)tile_row0 * FD_TILE_FLOATS + row_in_block * 32 + (sub & 7) * 4;
  // (a column tile past the window's: clamped, its values are dropped below)
  auto tile_at = [&](int t) { return prow + (int64_t)(t < ncol_tiles ? t : ncol_tiles - 1) * FD_TILE_FLOATS; };
  f32x4 v[N];
  load_records4(tile_at(sub >> 3), ks_stride, g.recs, v);
  for (int c = threadIdx.x; c < ncol_tiles * 32 + 32; c += FD_THREADS) {
    if (c < ncol_tiles * 32)
      nb2[c] = sum_records<N>(g.partial + (int64_t)(tile_col0 + (c >> 5)) * FD_TILE_FLOATS + 32 * 32 + 32 + (c & 31),
                          ks_stride, g.recs);
    else
      na2[c - ncol_tiles * 32] = sum_records<N>(g.partial + (int64_t)tile_row0 * FD_TILE_FLOATS + 32 * 32 + (c - ncol_tiles * 32),
                                            ks_stride, g.recs);
  }
  const int col_cap = (g.group > 1) ? g.slot : g.nt * 32;   // columns this launch really tiled
  WinInfo wi;
  int l, col_base;   // local A position; first tile column of this row's window
  if (g.group > 1) {
    const int s = row_in_block / g.slot;
    l = row_in_block - s * g.slot;
    wi = win_info(g, rb * g.group + s);
    col_base = s * g.slot;
  } else {
    wi = win_info(g, w_single);
    l = m_single * 32 + row_in_block;
    col_base = 0;
  }
  const bool a_valid = l < wi.nA;
  const bool pair = g.dir == PAIR_DIR;
  const int nB = wi.nB < col_cap ? wi.nB : col_cap;
  // the token of this row (and of the B node at the same position): the loads travel with the others
  const int a_tok = a_valid ? checked_token(g, wi.off + pos_a(l, g.dir)) : -1;
  const int b_tok = l < wi.nB ? checked_token(g, wi.off + pos_b(l, g.dir)) : -1;
  __syncthreads();
  double best = __longlong_as_double(0x7ff0000000000000ll);   // +inf
  int best_c = 0x7fffffff;
  const double a2 = na2[row_in_block];
  for (int t0 = 0; t0 < ncol_tiles; t0 += t_step) {   // uniform
    const int t = t0 + (sub >> 3);
    double dot[4];
    sum_records4(v, g.recs, dot);
    if (t0 + t_step < ncol_tiles) load_records4(tile_at(t + t_step), ks_stride, g.recs, v);
    const int tc0 = t * 32 + (sub & 7) * 4;   // first of this thread's columns inside the block's tile row
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = tc0 + j - col_base;   // column inside the window
      if (a_valid && t < ncol_tiles && c >= 0 && c < nB && !(pair && c == l)) {   // no token is its own neighbour
        double fd = divergence(g.metric, dot[j], a2, nb2[tc0 + j]);
        if (pair) fd = (double)(float)fd;   // ranked as the keys will be: equal in fp32 goes to the earlier neighbour
        if (fd < best) { best = fd; best_c = c; }   // columns ascend: strict < keeps the first minimum
      }
    }
  }
  // reduce over the lanes that share this row (at most 32, neighbours)
  for (int m = 1 << (tsh - 1); m >= 1; m >>= 1) {   // uniform
    const double ob = __shfl_xor(best, m, 64);
    const int oc = __shfl_xor(best_c, m, 64);
    if (ob < best || (ob == best && oc < best_c)) { best = ob; best_c = oc; }
  }
  if (pair) {
    if (sub == 0 && a_valid) {
      const bool has = best_c != 0x7fffffff;
      if (g.pair_keys) {
        g.pair_keys[wi.off + l] = has ? ((unsigned long long)__float_as_uint((float)best) << 32) | (unsigned)best_c : ~0ull;
      } else if (a_tok >= 0) {
        const int nb = has ? checked_token(g, wi.off + best_c) : -1;
        g.best_fd[a_tok] = nb >= 0 ? (float)best : __uint_as_float(0x7f800000u);
        g.best_dst[a_tok] = nb;
      }
    }
    return;
  }
  if (sub == 0 && a_tok >= 0) {
    // no finite score at all (NaN rows): propose the first B node with FD = +inf, so that counts stay exact
    const bool has = best_c != 0x7fffffff;
    g.best_fd[a_tok] = has ? (float)best : __uint_as_float(0x7f800000u);
    g.best_dst[a_tok] = (wi.nB > 0) ? checked_token(g, wi.off + pos_b(has ? best_c : 0, g.dir)) : -1;
  }
  if (sub == 1 && b_tok >= 0) {   // B rows carry no proposal
    g.best_fd[b_tok] = __uint_as_float(0x7f800000u);
    g.best_dst[b_tok] = -1;
  }
}

__device__ __forceinline__ void fd_epilogue_body(const FdArgs &g, int block_id, char *lds) {
  for_records(g.recs, [&](auto n) { fd_epilogue_records<decltype(n)::value>(g, block_id, lds); });
}

// ---------------------------------------------------------------------------------------------------------
// Windows that fit one 32 x 32 tile (at most 64 tokens): the epilogue AND the per-window selection (paper Step 2:
// the r A nodes with the lowest FD) in one kernel.  fd_partial_kernel leaves the partial tiles; one workgroup per
// tile sums them in their fixed order and finishes the tile: cosines, first minimum per row, rank of every
// A node among the keys (FD bits, position) of its window, then dst / per-target source counts / rank of each
// source in its group -- exactly what select_window_kernel derives from best_fd and best_dst.
// (Handing the tile to "the last workgroup to arrive" inside fd_partial_kernel was tried and dropped: the
// device-scope fence it needs writes back the L2 of the whole XCD and costs far more than a launch.)
struct SmallSelArgs {
  const int32_t *win_remove;
  int32_t *dst, *cnt, *src_rank;
};

struct SmallTileLds {
  double n2[2][32];             // |a|^2 per tile row, |b|^2 per tile column
  uint32_t row_key[32];         // order-preserving bits of the row's best FD (as stored in fp32)
  int row_col[32];              // best tile column (-1: none)
  int row_tok[32], col_tok[32]; // token of tile row / column, -1 for padding
  int slot_r[32];               // r of the window in slot s (clamped)
  uint32_t col_mask;            // bit c set: tile column c holds a B node
};

// One workgroup per tile: partial tiles summed in slice order, then the tile is finished in registers and LDS.
// Latency bound: every global load of the kernel is independent of the others (the token lists of the tile come from
// the record fd_partial_kernel left with slice 0; a thread's four columns are one 16-byte load per slice), so all of
// them are one trip to memory -- thread-per-value loads were four trips in a row (10 us a launch).
template <int N>
__device__ __forceinline__ void fd_tail_select_records(const FdArgs &g, const SmallSelArgs &q, int tile, char *lds) {
  SmallTileLds &L = *reinterpret_cast<SmallTileLds *>(lds);
  const int tid = threadIdx.x;
  const int64_t ks_stride = (int64_t)g.n_tiles * FD_TILE_FLOATS;
  const float *base = g.partial + (int64_t)tile * FD_TILE_FLOATS;
  const int shift = (g.group > 1) ? (g.slot == 8 ? 3 : 4) : 5;   // tile row or column >> shift = its window slot
  constexpr int TPR = FD_THREADS / 32;   // threads per tile row, four neighbouring columns each
  const int rr0 = tid / TPR, cl = tid % TPR;

  // ---- products (everyone), metadata and squared norms (wave 0)
  // a tile without A rows or without B rows has no sums from fd_partial_kernel: they are not used either
  f32x4 v[N];
  load_records4(base + rr0 * 32 + cl * 4, ks_stride, g.recs, v);
  if (tid < 64) {
    const int m_tok = reinterpret_cast<const int32_t *>(base + FD_TOK_OFFSET)[tid];   // rows 0..31, then columns 0..31
    const int rr = tid & 31;
    const int w = tile * g.group + (rr >> shift);
    const int wc = w < g.n_windows ? w : g.n_windows - 1;
    int m_off = g.win_offsets[wc], m_end = g.win_offsets[wc + 1], m_rem = q.win_remove[wc];
    if (w >= g.n_windows) { m_end = m_off; m_rem = 0; }
    L.n2[tid >> 5][tid & 31] = sum_records<N>(base + 32 * 32 + tid, ks_stride, g.recs);
    if (tid < 32) L.row_tok[tid] = m_tok; else L.col_tok[tid - 32] = m_tok;
    const unsigned long long cm = __ballot(tid >= 32 && m_tok >= 0);
    if (tid == 0) L.col_mask = (uint32_t)(cm >> 32);
    if (tid < 32 && (tid & ((1 << shift) - 1)) == 0) {   // first row of a window slot: its removal count
      const int wv = m_end - m_off;
      const int cap = (g.group > 1) ? g.slot : 32;
      int nA = side_a(wv, g.dir);
      nA = nA < cap ? nA : cap;
      int r = m_rem < 0 ? 0 : (m_rem > nA ? nA : m_rem);
      if (side_b(wv, g.dir) == 0) r = 0;
      L.slot_r[tid >> shift] = r;
    }
  }
  double dots[4];
  sum_records4(v, g.recs, dots);
  __syncthreads();

  // ---- FD and first minimum per row
  {
    const int rr = rr0;
    const int ta = L.row_tok[rr];
    const int sw = rr >> shift;
    const uint32_t cols = L.col_mask & ((shift == 5) ? 0xffffffffu : (((1u << (1 << shift)) - 1u) << (sw << shift)));
    double best = __longlong_as_double(0x7ff0000000000000ll);
    int best_c = 0x7fffffff;
    const double a2 = L.n2[0][rr];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = cl * 4 + k;
      const double fd = divergence(g.metric, dots[k], a2, L.n2[1][c]);
      const bool live = ta >= 0 && ((cols >> c) & 1u);
      if (live && fd < best) { best = fd; best_c = c; }   // columns ascend: strict < keeps the first minimum
    }
#pragma unroll
    for (int m = TPR / 2; m >= 1; m >>= 1) {
      const double ob = __shfl_xor(best, m, 64);
      const int oc = __shfl_xor(best_c, m, 64);
      if (ob < best || (ob == best && oc < best_c)) { best = ob; best_c = oc; }
    }
    if (cl == 0) {
      const bool has = best_c != 0x7fffffff;
      float f = has ? (float)best : __uint_as_float(0x7f800000u);
      // a row without any finite score falls back to the first B node of its window
      const int first_c = cols ? __ffs((int)cols) - 1 : -1;
      const int bc = has ? best_c : first_c;
      if (!(f >= 0.f)) f = __uint_as_float(0x7f800000u);
      L.row_key[rr] = f32_order_key(f);
      L.row_col[rr] = bc;
      if (ta >= 0) {
        g.best_fd[ta] = f;
        g.best_dst[ta] = bc >= 0 ? L.col_tok[bc] : -1;
      }
    }
    if (cl == 1 && L.col_tok[rr] >= 0) {   // B rows carry no proposal
      g.best_fd[L.col_tok[rr]] = __uint_as_float(0x7f800000u);
      g.best_dst[L.col_tok[rr]] = -1;
    }
  }
  __syncthreads();

  // ---- selection by wave 0, row data in registers: lanes 0..31 act for the tile rows (A nodes), lanes 32..63
  // for the tile columns (B nodes).  Values of other rows are read with constant-lane broadcasts.
  if (tid < 64) {
    const int rr = tid & 31;
    const int tok = L.row_tok[rr], col = L.row_col[rr];
    const uint32_t key = L.row_key[rr];
    const int win = rr >> shift;
    const int valid = tok >= 0 ? 1 : 0;
    int rank = 0;
#pragma unroll
    for (int o = 0; o < 32; ++o) {
      const uint32_t ko = (uint32_t)__builtin_amdgcn_readlane((int)key, o);
      const int vo = __builtin_amdgcn_readlane(valid, o);
      rank += (vo && (o >> shift) == win && (ko < key || (ko == key && o < rr))) ? 1 : 0;
    }
    const bool sel = valid && col >= 0 && rank < L.slot_r[win];
    const uint32_t selmask = (uint32_t)__ballot(sel);   // lanes 0..31
    // rows: rank among the earlier sources of the same destination; columns: number of sources
    const bool is_col = tid >= 32;
    const int target = is_col ? rr : col;
    const int limit = is_col ? 32 : rr;
    int n = 0;
#pragma unroll
    for (int o = 0; o < 32; ++o) {
      const int co = __builtin_amdgcn_readlane(col, o);
      n += (((selmask >> o) & 1u) && (o >> shift) == win && co == target && o < limit) ? 1 : 0;
    }
    if (!is_col) {
      if (tok >= 0) {
        q.dst[tok] = sel ? L.col_tok[col] : -1;
        q.src_rank[tok] = sel ? n : 0;
        q.cnt[tok] = 0;
      }
    } else {
      const int tb = L.col_tok[rr];
      if (tb >= 0) {
        q.dst[tb] = -1;
        q.src_rank[tb] = 0;
        q.cnt[tb] = n;
      }
    }
  }
}

__device__ __forceinline__ void fd_tail_select_body(const FdArgs &g, const SmallSelArgs &q, int tile, char *lds) {
  for_records(g.recs, [&](auto n) { fd_tail_select_records<decltype(n)::value>(g, q, tile, lds); });
}

// Arguments of the small-window kernels from a plan and the caller's tensors (host side).
inline FdArgs make_fd_args(const FdPlan &plan, int dtype, const void *X, int64_t ldx, int d, int n_windows, int sum_n,
                           const int32_t *win_offsets, const int32_t *win_tokens, float *partial, float *best_fd,
                           int32_t *best_dst) {
  FdArgs g{};
  g.X = X; g.ldx = ldx; g.d = d; g.n_windows = n_windows; g.sum_n = sum_n;
  g.win_offsets = win_offsets; g.win_tokens = win_tokens;
  g.partial = partial; g.best_fd = best_fd; g.best_dst = best_dst;
  g.slot = plan.slot; g.group = plan.group; g.mt = plan.mt; g.nt = plan.nt;
  g.n_tiles = plan.n_tiles; g.ksplit = plan.ksplit; g.recs = plan.recs; g.metric = plan.metric; g.dir = plan.dir;
  const int span = (dtype == 1) ? 64 : 32;
  g.n_spans = (d + span - 1) / span;
  g.spans_per_wg = plan.spans_per_wg; g.chain = plan.chain;
  return g;
}

}  // namespace lk
