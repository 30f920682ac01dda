// Feature divergence and the best edge of every A node (paper Sec. 3.2.1 Steps 1-2, Eq. "similarity").
//
// For every window the |A| x |B| block of inner products <x_a, x_b> is a dense contraction over the
// hidden dimension and runs on the matrix cores (bf16 -> v_mfma_f32_32x32x16_bf16, fp32 ->
// v_mfma_f32_32x32x2_f32), fp32 accumulation.  The squared norms come from the same instruction
// (a tile times itself: the diagonal is |x|^2), so a token identical to another one gets cos == 1 exactly.
// The FD matrix is never written: an epilogue reduces each A row to (min FD, arg min) directly.
//
//   fd_partial_kernel : one workgroup = one 32x32 tile x one slice of the hidden axis; the tile's rows are staged through
//                       LDS in coalesced pieces, the four waves of the workgroup take interleaved 128-byte runs of
//                       them as MFMA operands, are summed through LDS and stored as a partial tile.
//   fd_epilogue_kernel: sums the partial tiles over the slices in a fixed order (fp64), forms
//                       cos = dot / sqrt(|a|^2 |b|^2), FD = max(1 - cos, 0) and keeps the first minimum per row.
#include "lk_fd_body.h"

namespace lk {

template <typename T>
__global__ __launch_bounds__(FD_THREADS, 3) void fd_partial_kernel(FdArgs g) {
  fetch_args<FdArgs>();
  __shared__ __attribute__((aligned(16))) char lds[FD_PARTIAL_LDS];
  fd_partial_body<T>(g, blockIdx.x, lds);
}

__global__ __launch_bounds__(FD_THREADS) void fd_tail_select_kernel(FdArgs g, SmallSelArgs q) {
  fetch_args<FdArgs, SmallSelArgs>();
  __shared__ __attribute__((aligned(16))) char lds[sizeof(SmallTileLds)];
  fd_tail_select_body(g, q, blockIdx.x, lds);
}

__global__ __launch_bounds__(FD_THREADS) void fd_epilogue_kernel(FdArgs g) {
  fetch_args<FdArgs>();
  __shared__ __attribute__((aligned(16))) char lds[FD_EPILOGUE_LDS];
  fd_epilogue_body(g, blockIdx.x, lds);
}

FdPlan make_fd_small_fused_plan(int n_windows, int max_window_tokens, int d, int dtype_bytes) {
  FdPlan p{};
  const int maxA = (max_window_tokens + 1) / 2;
  if (maxA > 32) return p;   // n_tiles == 0: not applicable
  return make_fd_plan(n_windows, max_window_tokens, d, dtype_bytes);   // single-tile windows: mt == nt == 1
}

hipError_t launch_fd_select_small(const FdPlan &plan, int dtype, const void *X, int64_t ldx, int d, int n_windows,
                                  int sum_n, const int32_t *win_offsets, const int32_t *win_tokens,
                                  const int32_t *win_remove, float *partial, float *best_fd, int32_t *best_dst,
                                  int32_t *dst, int32_t *cnt, int32_t *src_rank, hipStream_t stream) {
  if (n_windows == 0 || plan.n_tiles == 0) return hipSuccess;
  const FdArgs g = make_fd_args(plan, dtype, X, ldx, d, n_windows, sum_n, win_offsets, win_tokens, partial, best_fd, best_dst);
  const dim3 grid((unsigned)(plan.n_tiles * plan.ksplit));
  if (dtype == 1) hipLaunchKernelGGL(fd_partial_kernel<bf16_t>, grid, dim3(FD_THREADS), 0, stream, g);
  else hipLaunchKernelGGL(fd_partial_kernel<float>, grid, dim3(FD_THREADS), 0, stream, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  SmallSelArgs q{win_remove, dst, cnt, src_rank};
  hipLaunchKernelGGL(fd_tail_select_kernel, dim3((unsigned)plan.n_tiles), dim3(FD_THREADS), 0, stream, g, q);
  return hipGetLastError();
}

// Workgroups of the partial tiles.  The fine split of the hidden axis goes on until there are four workgroups for every CU.  Long
// slices of bf16 rows: split only until there is one for every CU, and on while a slice is longer than five pieces.  Beside xi's row
// statistics (768 workgroups fit the chip at a time, three a CU) each further one waits for a slot, and a slice of several pieces has
// the next one in flight while it multiplies.  Scores and selection, fine / long slices, us alone and with xi of 64 prompt rows: 20
// windows of 96 tokens (80 tiles), d = 4096, 28.3 / 27.8 and 34.0 / 33.8; 96 of 36, d = 5120, 29.4 / 27.5 and 44.2 / 40.0; 300 of
// 36, d = 1280, 43.0 / 40.2 and 55.7 / 51.3; 200 of 36, d = 2048, 32.3 / 30.3 and 45.6 / 47.4.  Eight pieces: 144 of 36, d = 3712,
// 29.5 / 30.9 and 46.4 / 46.6.  Not where the two records of a long slice make as many as the fine split has: 180 of 16, d = 4096,
// 22.2 / 23.5 and 29.4 / 31.0, 80 of 30 20.8 / 21.7 and 27.3 / 26.8.  fp32 products take sixteen times as long, a piece of them is
// 1.3 us of a matrix pipe: always fine (3 x 513 tokens, d = 1024: 85.0 us with slices of one piece, 87.1 of two).
constexpr int FD_TARGET_WGS = 256, FD_FINE_WGS = 1024, FD_SLICE_PIECES = 5;

static FdPlan plan_tiles(int n_windows, int maxA, int maxB, int d, int dtype_bytes) {
  FdPlan p{};
  if (maxA <= 16) {
    p.slot = maxA <= 8 ? 8 : 16;
    p.group = 32 / p.slot;
    p.mt = p.nt = 1;
    p.n_tiles = (n_windows + p.group - 1) / p.group;
    p.n_rowblocks = p.n_tiles;
  } else {
    p.slot = 0;
    p.group = 1;
    p.mt = (maxA + 31) / 32;
    p.nt = maxB > 0 ? (maxB + 31) / 32 : 1;
    p.n_tiles = n_windows * p.mt * p.nt;
    p.n_rowblocks = n_windows * p.mt;
  }
  const int span = (dtype_bytes == 2) ? 64 : 32;
  const int n_spans = (d + span - 1) / span;
  const int max_ks = n_spans / FD_WAVES > 0 ? n_spans / FD_WAVES : 1;
  const int pieces = (n_spans + FD_WAVES - 1) / FD_WAVES;
  auto split = [&](int target, int longest) {
    int ks = 1;
    while (((int64_t)p.n_tiles * ks < target || ((int64_t)p.n_tiles * ks < FD_FINE_WGS && pieces > longest * ks)) &&
           ks * 2 <= max_ks && ks * 2 <= FD_MAX_RECS)
      ks *= 2;
    return ks;
  };
  const int fine = split(FD_FINE_WGS, pieces);
  const int ks = dtype_bytes == 2 ? split(FD_TARGET_WGS, FD_SLICE_PIECES) : fine;
  if (2 * ks >= fine) {
    p.ksplit = p.recs = fine;
    p.spans_per_wg = (n_spans + fine - 1) / fine;
    p.chain = pieces;
  } else {
    // A slice of several pieces adds no more products in fp32 than one of the finer split would, and hands the rest on as two
    // floats: two records per workgroup, at most as many as the finer split has (ks <= fine / 2).
    const int per = (pieces + ks - 1) / ks;   // a workgroup stages FD_WAVES spans at a time: a slice is a whole number of pieces
    p.ksplit = (pieces + per - 1) / per;
    p.recs = 2 * p.ksplit;
    p.spans_per_wg = per * FD_WAVES;
    const int fine_pieces = (n_spans + fine - 1) / fine / FD_WAVES;   // whole pieces of a slice of the finer split
    p.chain = fine_pieces > 0 ? fine_pieces : 1;
  }
  // The room for the records stays that of the finer split: a workspace has to serve plans with a smaller window bound as well,
  // which can be split further.
  p.partial_floats = (size_t)p.n_tiles * fine * FD_TILE_FLOATS;
  return p;
}

FdPlan make_fd_plan(int n_windows, int max_window_tokens, int d, int dtype_bytes) {
  return plan_tiles(n_windows, (max_window_tokens + 1) / 2, max_window_tokens / 2, d, dtype_bytes);
}

// Full pairwise matching cut into 32 x 32 tiles with the hidden axis split over workgroups, instead of 192 x 192 tiles
// whose workgroup walks the whole hidden axis: a launch of the large tiles takes 78 us however few of them there are (64
// dependent k-steps at d = 4096), and a window of 36 tokens fills 4 % of one.  The small tiles fetch 512 KB each at
// d = 4096, so their time grows with their number.  Scores alone, d = 4096, large -> small tiles: 180 windows of 16 tokens
// 79.7 -> 17.8 us, one window of 576 tokens (324 small tiles) 78.6 -> 41.4, of 800 (625) 79.7 -> 59.9, of 1024 (1024) 80.3 ->
// 83.9; 64 windows of 128 (1024) 87.9 -> 94.8.  The line lies at 768 tiles.
FdPlan make_fd_pair_plan(int n_windows, int max_window_tokens, int d) {
  const int64_t side = (max_window_tokens + 31) / 32;
  if (max_window_tokens > 2 * 32 * PAIR_SMALL_MAX_TILES || n_windows <= 0) return FdPlan{};
  const int64_t tiles = max_window_tokens <= 16 ? n_windows : side * side * (int64_t)n_windows;
  if (tiles > PAIR_SMALL_MAX_TILES) return FdPlan{};
  FdPlan p = plan_tiles(n_windows, max_window_tokens, max_window_tokens, d, 2);
  p.dir = PAIR_DIR;
  return p;
}

size_t pair_partial_floats(int n_windows, int max_window_tokens, int d) {
  size_t most = 0;
  // a plan changes with the bound only where a tile side does (8, 16, then every 32 tokens), and its tiles only grow in number
  for (int side = 8;; side = side < 32 ? 2 * side : side + 32) {
    const FdPlan p = make_fd_pair_plan(n_windows, side < max_window_tokens ? side : max_window_tokens, d);
    most = p.partial_floats > most ? p.partial_floats : most;
    if (side >= max_window_tokens || p.n_tiles == 0) break;
  }
  return most;
}

hipError_t launch_fd_pair_small(const FdPlan &plan, const void *X, int64_t ldx, int d, int n_windows, int sum_n,
                                const int32_t *win_offsets, const int32_t *win_tokens, float *partial,
                                unsigned long long *keys, float *best_fd, int32_t *best_dst, hipStream_t stream) {
  if (n_windows == 0 || plan.n_tiles == 0) return hipSuccess;
  FdArgs g = make_fd_args(plan, 1, X, ldx, d, n_windows, sum_n, win_offsets, win_tokens, partial, best_fd, best_dst);
  g.pair_keys = keys;
  hipLaunchKernelGGL(fd_partial_kernel<bf16_t>, dim3((unsigned)(plan.n_tiles * plan.ksplit)), dim3(FD_THREADS), 0, stream, g);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fd_epilogue_kernel, dim3((unsigned)fd_epilogue_blocks(plan.n_rowblocks, plan.group, plan.nt)),
                     dim3(FD_THREADS), 0, stream, g);
  return hipGetLastError();
}

hipError_t launch_fd_partial(const FdArgs &g, int dtype, hipStream_t stream) {
  if (g.n_windows == 0 || g.n_tiles == 0) return hipSuccess;
  const dim3 grid((unsigned)(g.n_tiles * g.ksplit));
  if (dtype == 1) hipLaunchKernelGGL(fd_partial_kernel<bf16_t>, grid, dim3(FD_THREADS), 0, stream, g);
  else hipLaunchKernelGGL(fd_partial_kernel<float>, grid, dim3(FD_THREADS), 0, stream, g);
  return hipGetLastError();
}

hipError_t launch_fd(const FdPlan &plan, int dtype, const void *X, int64_t ldx, int d, int n_windows, int sum_n,
                     const int32_t *win_offsets, const int32_t *win_tokens, float *partial, float *best_fd,
                     int32_t *best_dst, hipStream_t stream) {
  if (n_windows == 0 || plan.n_tiles == 0) return hipSuccess;
  const FdArgs g = make_fd_args(plan, dtype, X, ldx, d, n_windows, sum_n, win_offsets, win_tokens, partial, best_fd, best_dst);
  const dim3 grid((unsigned)(plan.n_tiles * plan.ksplit));
  if (dtype == 1) hipLaunchKernelGGL(fd_partial_kernel<bf16_t>, grid, dim3(FD_THREADS), 0, stream, g);
  else hipLaunchKernelGGL(fd_partial_kernel<float>, grid, dim3(FD_THREADS), 0, stream, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fd_epilogue_kernel, dim3((unsigned)fd_epilogue_blocks(plan.n_rowblocks, plan.group, plan.nt)),
                     dim3(FD_THREADS), 0, stream, g);
  return hipGetLastError();
}

}  // namespace lk
