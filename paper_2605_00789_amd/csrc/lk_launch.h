// Host-side launch plans and launcher declarations (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

struct lightkv_problem;

namespace lk {

// The bipartite split of a window's list (Sec. 3.2.1 Step 1) and the direction of the merge (message-passing
// paragraph: the reverse direction is defined analogously).  dir 0: the tokens at list positions 0, 2, 4, ... propose
// and merge into the tokens at positions 1, 3, 5, ...; dir 1: the odd positions propose, the even ones receive.  In
// the kernels "A" is always the proposing side and "B" the receiving side.
// dir 2 (PAIR_DIR): no split -- every token proposes to every other one (full pairwise matching): both sides are the
// whole list.
constexpr int PAIR_DIR = 2;
__host__ __device__ __forceinline__ int side_a(int v, int dir) { return dir == PAIR_DIR ? v : (v + 1 - dir) >> 1; }
__host__ __device__ __forceinline__ int side_b(int v, int dir) { return dir == PAIR_DIR ? v : (v + dir) >> 1; }
__host__ __device__ __forceinline__ int pos_a(int i, int dir) { return dir == PAIR_DIR ? i : 2 * i + dir; }
__host__ __device__ __forceinline__ int pos_b(int j, int dir) { return dir == PAIR_DIR ? j : 2 * j + 1 - dir; }

// ---- feature divergence (Steps 1-2) ------------------------------------------------------
// The |A_w| x |B_w| cosine blocks are cut into 32x32 tiles.  Small windows are packed several to
// a tile (block diagonal): `slot` rows/cols per window, `group` windows per tile.  Large windows
// get mt x nt tiles each.  The d axis is split over `ksplit` workgroups (and the 4 waves of each) that leave `recs`
// records of partial sums per tile; these are summed in a fixed order by the epilogue.
struct FdPlan {
  int slot;         // rows (and cols) reserved per window in a packed tile; 0 when group == 1
  int group;        // windows per tile
  int mt, nt;       // tiles per window along A and B (group == 1)
  int n_tiles;      // tile jobs
  int n_rowblocks;  // epilogue jobs (one per 32 A rows)
  int ksplit;
  int spans_per_wg;        // spans of the hidden axis per workgroup
  int chain;               // pieces of FD_WAVES spans that are added in fp32 before the sum goes on in fp64
  int recs;                // ksplit, or 2 * ksplit: every sum as two floats
  size_t partial_floats;   // room for the records: n_tiles * FD_TILE_FLOATS for at least recs of them
  int metric;              // 0 cosine FD, 1 Euclidean, 2 squared L2 (set by the caller after planning)
  int dir;                 // 0: even list positions propose, 1: odd ones (set by the caller after planning; a plan for
                           // dir 1 is made with the window bound rounded up to even, so that both sides fit)
};
constexpr int FD_TOK_OFFSET = 32 * 32 + 32 + 32;    // dots, |a|^2 partials, |b|^2 partials ...
constexpr int FD_TILE_FLOATS = FD_TOK_OFFSET + 64;  // ... then (slice 0 only) the tokens of the 32 rows and 32 columns
constexpr int FD_MAX_COLS = 2048;                   // |B| of the largest supported window

FdPlan make_fd_plan(int n_windows, int max_window_tokens, int d, int dtype_bytes);
// The same for full pairwise matching (every window's whole v x v matrix in 32 x 32 tiles); n_tiles == 0: the 192 x 192
// tiles of launch_fd_pair are the better cut.
constexpr int PAIR_SMALL_MAX_TILES = 768;
FdPlan make_fd_pair_plan(int n_windows, int max_window_tokens, int d);
// The most floats the partial tiles take under this window bound or a smaller one: a step may be planned with a smaller
// bound than its workspace was sized for, and the plans are not monotone in it.
size_t pair_partial_floats(int n_windows, int max_window_tokens, int d);

// The partition of one stage's tokens and, optionally, the per-window counts that go with it (host struct).
struct WinArgs;
struct WinSpec {
  int tiles, grid_h, grid_w, w;
  int32_t *win_offsets, *win_tokens;
  int count_mode;             // -1: no counts; otherwise a mode of launch_window_counts
  double rho;
  int dir, n_windows;         // (with counts)
  const int32_t *cu_target;
  int32_t *win_remove, *status;
};
// new_index / cu_out: the "next stage" form.  *counts_done says whether the counts were part of the launch (the kernel
// that sorts leaves them to the caller).
hipError_t launch_build_windows(const WinSpec &spec, const int32_t *cu_vis, const int32_t *pos, const int32_t *new_index,
                                const int32_t *cu_out, int batch, int max_seq, bool *counts_done, hipStream_t stream);
// arguments and LDS bytes of the same partition as a guest of another launch; 0 bytes: not possible
size_t make_win_args(const WinSpec &spec, const int32_t *cu_vis, const int32_t *pos, const int32_t *new_index,
                     const int32_t *cu_out, int batch, int max_seq, WinArgs *out);

// Windows + their counts (lk_api.hip), and the fused merge with the next stage's windows beside it; a lightkv_status
int build_windows_with_counts(int32_t batch, const int32_t *h_cu_vis, const int32_t *cu_vis, const int32_t *pos,
                              const int32_t *new_index, const int32_t *cu_vis_out, const WinSpec &spec, void *stream);
// Whether the windows of the stage behind p fit into the launch of p's merge (false for descriptors that the calls refuse).
bool windows_ride(const lightkv_problem *p, const WinSpec &next);
int aggregate_compact_with_windows(const lightkv_problem *p, const int32_t *new_index, const int32_t *grp_offsets,
                                   const int32_t *grp_src, const float *xi, const void *X, int64_t ldx, const void *K,
                                   int64_t ldk, const void *V, int64_t ldv, const int32_t *pos, void *X_out, void *K_out,
                                   void *V_out, int32_t *pos_out, float *x_sqnorm_out, int64_t out_rows,
                                   const int32_t *cu_vis_out, const WinSpec *next, unsigned long long *publish,
                                   unsigned publish_tag, void *stream);

// per-window counts from a ratio (mode 0: tokens, 1: edges) or from per-sequence target lengths (mode 2)
hipError_t launch_window_counts(int batch, int win_per_seq, const int32_t *win_offsets, int mode, int dir, double rho,
                                const int32_t *cu_vis, const int32_t *cu_target, int32_t *win_remove, int32_t *status,
                                hipStream_t stream);

hipError_t launch_fd(const FdPlan &plan, int dtype, const void *X, int64_t ldx, int d, int n_windows, int sum_n,
                     const int32_t *win_offsets, const int32_t *win_tokens, float *partial, float *best_fd,
                     int32_t *best_dst, hipStream_t stream);

// Full pairwise matching on the small tiles: one packed key per list position in `keys`, as launch_fd_pair leaves them,
// or best_fd / best_dst if keys is NULL.
hipError_t launch_fd_pair_small(const FdPlan &plan, const void *X, int64_t ldx, int d, int n_windows, int sum_n,
                                const int32_t *win_offsets, const int32_t *win_tokens, float *partial,
                                unsigned long long *keys, float *best_fd, int32_t *best_dst, hipStream_t stream);

// Windows of at most 64 tokens: partial tiles, then epilogue + per-window selection in one kernel
// (n_tiles == 0: not applicable).
FdPlan make_fd_small_fused_plan(int n_windows, int max_window_tokens, int d, int dtype_bytes);
hipError_t launch_fd_select_small(const FdPlan &plan, int dtype, const void *X, int64_t ldx, int d, int n_windows,
                                  int sum_n, const int32_t *win_offsets, const int32_t *win_tokens,
                                  const int32_t *win_remove, float *partial, float *best_fd, int32_t *best_dst,
                                  int32_t *dst, int32_t *cnt, int32_t *src_rank, hipStream_t stream);

// Step 2 read literally (lk_select_edges.hip): the k lowest-FD edges of every window.  Windows of at most
// 2 * EDGE_MAX_SIDE tokens are ranked in LDS by one kernel; larger ones through a key matrix in `big_keys`.
// `edges` is scratch of 3 * sum_k ints (sum_k = the k of all windows, or a bound on it with device_counts, where a
// window's k is also bounded by its tokens).
constexpr int EDGE_MAX_SIDE = 128;
struct FdArgs;
struct EdgeArgs;
EdgeArgs make_edge_args(int max_window, int sum_k, const int32_t *win_remove, int32_t *dst, int32_t *cnt, int32_t *src_rank,
                        int32_t *edges, bool device_counts, uint32_t *big_keys);
hipError_t launch_fd_partial(const FdArgs &g, int dtype, hipStream_t stream);
hipError_t launch_edge_select(const FdArgs &g, const EdgeArgs &q, int dtype, hipStream_t stream);
hipError_t launch_edge_select_big(const FdArgs &g, const EdgeArgs &q, hipStream_t stream);   // behind the keys of every pair
// the FD keys of every pair of every window, for windows beyond the one-kernel path: 32-bit keys (0 if not needed)
size_t edge_big_key_count(int n_windows, int max_window);
// The edge list as the index scan takes it: [3][sum_k] (A token, B token, position); slots beyond the edges there are
// (grp_offsets[sum_n]) are not read.  A list of more than scan_max slots gets a launch of its own behind the scan.
struct EdgeList { const int32_t *edges; int sum_k, scan_max; };
// The line: one workgroup of the scan takes 1024 edges a trip, a launch costs 1-2 us.  Score-select calls at d = 512, list in
// the scan -> of its own, us: 1024 edges 21.7 -> 23.3, 3104 24.6 -> 24.4, 5184 24.2 -> 22.5, 663552 303 -> 75 (d = 1024).  Where
// only a bound is known (one slot per token): 2880 tokens 20.5 -> 21.6, 16384 with 1536 edges 51.0 -> 51.5, with 8192 56.7 ->
// 53.4, 65536 tokens with 6144 edges 97.7 -> 90.4.
constexpr int EDGE_SCAN_MAX_KNOWN = 2048;    // slots where the host knows the counts
constexpr int EDGE_SCAN_MAX_BOUND = 16384;   // ... where it knows a bound

// Debug dump of the FD of every pair (lk_fd_dump.hip); at most 65535 windows.
hipError_t launch_fd_dump(int dtype, const void *X, int64_t ldx, int d, int n_windows, int max_window, int sum_n,
                          int metric, int dir, const int32_t *win_offsets, const int32_t *win_tokens, float *out,
                          long long capacity, hipStream_t stream);

// Large windows (compute bound): LDS-tiled MFMA GEMM with the row arg-min fused into its epilogue.
struct FdBigPlan {
  int wb;            // MFMA blocks (16 x 16) per edge of the workgroup tile
  int mt, nt;        // workgroup tiles per window along A and B
  int max_window;    // the caller's bound on the tokens of a window
  size_t norm_floats;   // |x|^2 per token (used when the caller does not hand them in)
  int nt_store;      // column tiles that keep keys of their own: nt, or 1 (all tiles of a window share one key per row)
  size_t key_bytes;  // [nt_store][sum_n] packed keys (FD bits << 32 | B token): per column tile, the best key of the A
                     // row at every position of the window lists; all-ones where nothing was offered
  int metric;        // as in FdPlan
  int dir;           // as in FdPlan
};
constexpr int FD_BIG_TILE = 96;            // rows and columns of a workgroup tile
constexpr int FD_BIG_KEYS_PER_TILE_MAX_NT = 4;   // up to this many column tiles per window, each keeps keys of its own
constexpr int FD_BIG_MIN_WINDOW = 128;   // windows bounded by fewer tokens use the small-tile path, and so do
constexpr int FD_BIG_MIN_TILES = 32;     // problems that make up fewer workgroup tiles than this
FdBigPlan make_fd_big_plan(int n_windows, int max_window_tokens, int sum_n);
hipError_t launch_fd_big(const FdBigPlan &plan, const void *X, int64_t ldx, int d, int n_windows, int sum_n,
                         const int32_t *win_offsets, const int32_t *win_tokens, const float *x_sqnorm, float *sq_ws,
                         unsigned long long *keys, float *best_fd, int32_t *best_dst, bool finalize,
                         hipStream_t stream);
// Full pairwise matching (every two tokens of a window): one packed key per list position in `keys`
// (FD bits << 32 | position of the nearest neighbour in the window list).  bf16, d a multiple of 64.
// best_fd / best_dst: written from the keys if not NULL (every token's nearest neighbour).
hipError_t launch_fd_pair(const void *X, int64_t ldx, int d, int n_windows, int max_window, int sum_n, int metric,
                          const int32_t *win_offsets, const int32_t *win_tokens, const float *x_sqnorm, float *sq_ws,
                          unsigned long long *keys, float *best_fd, int32_t *best_dst, hipStream_t stream);
// ... and the selection on those keys (lk_select_pair.hip): dst, source counts and ranks, best_fd / best_dst
hipError_t launch_pair_select(int n_windows, int max_window, int sum_n, const int32_t *win_offsets,
                              const int32_t *win_tokens, const int32_t *win_remove, const unsigned long long *keys,
                              float *best_fd, int32_t *best_dst, int32_t *dst, int32_t *cnt, int32_t *src_rank,
                              hipStream_t stream);

// The smallest workspace the calls take for a problem (lightkv_workspace_size may ask for more: lk_api.hip); a lightkv_status.
int least_workspace(const lightkv_problem *p, size_t *bytes);

// Whether lightkv_score_select with xi requested runs this step on the caller's stream alone (lk_api.hip).
bool score_select_one_stream(const lightkv_problem *p);

// ---- xi and FD on one stream, the k-th kernels of the two chains sharing a launch (lk_fused.hip): pass 1 of xi beside
// the partial tiles, pass 2 beside what finishes them -- FUSED_TAIL: epilogue and selection of windows of at most 64
// tokens, FUSED_EPILOGUE: best edges of larger ones (keys instead of best_fd / best_dst if pair_keys is given).  The
// caller goes on with the selection and launch_select_scan_heads, which sums the heads of xi, or launch_xi_heads.
// FUSED_EDGES: the k lowest edges of every window (of at most 2 * EDGE_MAX_SIDE tokens), or the keys of every pair of larger
// ones (launch_edge_select_big goes on).
enum FusedFinish { FUSED_TAIL = 0, FUSED_EPILOGUE = 1, FUSED_EDGES = 2 };
struct XiArgs;
struct XiPlan;
struct FdArgs;
struct SmallSelArgs;
hipError_t launch_xi_fd_fused(const XiArgs &x, const XiPlan &xp, const FdArgs &f, const SmallSelArgs &q, const EdgeArgs *edges,
                              FusedFinish finish, int n_rowblocks, int dtype, int head_dim, hipStream_t stream);
hipError_t launch_xi_heads(const XiArgs &x, hipStream_t stream);   // the head sum alone (scores without a selection)
// index scan with the head sum of xi in the same launch (x: arguments of the xi passes)
hipError_t launch_select_scan_heads(int batch, int sum_n, const int32_t *cu_vis, const int32_t *dst, int32_t *new_index,
                                    int32_t *grp_offsets, int32_t *grp_src, int32_t *cu_vis_out, const int32_t *cnt,
                                    const int32_t *src_rank, const EdgeList *edges, const XiArgs &x, hipStream_t stream);

// ---- prompt-guidance weight xi (Step 3) ----------------------------------------------------
struct XiPlan {
  int max_text_tiles;  // ceil(max T_b / 32)
  int max_vis_blocks;  // ceil(max N_b / 128): pass 1 leaves one (max, sum) pair per prompt row and block
  size_t stat_floats;  // pass-1 partial (max, sum) pairs: heads * sumT * max_vis_blocks * 2
  size_t part_floats;  // per-head partial xi: heads * sumN
};
XiPlan make_xi_plan(int batch, const int32_t *h_cu_vis, const int32_t *h_cu_txt, int heads, int xi_mode);

hipError_t launch_xi(const XiPlan &plan, int dtype, int xi_mode, int batch, int heads, int head_dim, int sum_n,
                     int sum_t, const int32_t *cu_vis, const int32_t *cu_txt, const void *Q, int64_t q_tok_stride,
                     int64_t q_head_stride, const void *K, int64_t k_tok_stride, int64_t k_head_stride,
                     const float *lse, float scale, float *stats, float *xi_part, float *xi, hipStream_t stream);

// Batches: one workgroup per (sequence, head) pair, both softmax sweeps in one launch (lk_xi_seq.hip).  Applies to
// text-query mode without a given lse, prompts of at most 256 tokens and at least XI_SEQ_MIN_PAIRS pairs.
constexpr int XI_SEQ_MIN_PAIRS = 256;
bool xi_seq_applies(const XiPlan &plan, int xi_mode, const float *lse, int batch, int heads);
hipError_t launch_xi_seq(const XiArgs &g, int dtype, int head_dim, hipStream_t stream);

// ---- selection (Step 2) ----------------------------------------------------------------------
// keys == nullptr: best_fd / best_dst are the inputs.  Otherwise the packed keys of launch_fd_big(..., finalize = false)
// are (planned with key_mt row tiles and key_nt stored column tiles per window), and best_fd / best_dst are written from them on the way (one
// launch less than finalizing first).
hipError_t launch_select(int n_windows, int max_window_tokens, int batch, int sum_n, const int32_t *cu_vis,
                         const int32_t *win_offsets, const int32_t *win_tokens, const int32_t *win_remove,
                         const unsigned long long *keys, int key_mt, int key_nt, float *best_fd, int32_t *best_dst, int32_t *dst,
                         int32_t *new_index, int32_t *grp_offsets, int32_t *grp_src, int32_t *cu_vis_out, int32_t *cnt,
                         int32_t *src_rank, int dir, hipStream_t stream);

// the window half of lightkv_select alone: dst, cnt, src_rank from the scores
hipError_t launch_select_windows(int n_windows, int max_window_tokens, int sum_n, const int32_t *win_offsets,
                                 const int32_t *win_tokens, const int32_t *win_remove, const unsigned long long *keys,
                                 int key_mt, int key_nt, float *best_fd, int32_t *best_dst, int32_t *dst, int32_t *cnt,
                                 int32_t *src_rank, int dir, hipStream_t stream);

// the scan half of lightkv_select alone (dst, cnt, src_rank already written); edges: the sources come from an edge list
hipError_t launch_select_scan(int batch, int sum_n, const int32_t *cu_vis, const int32_t *dst, int32_t *new_index,
                              int32_t *grp_offsets, int32_t *grp_src, int32_t *cu_vis_out, const int32_t *cnt,
                              const int32_t *src_rank, const EdgeList *edges, hipStream_t stream);

// ---- message passing + compaction (Steps 3-5) ---------------------------------------------------
struct RowTensors {
  const void *in[3];
  void *out[3];
  int64_t ld_in[3];
  int64_t ld_out[3];
};
// mode 0: aggregate in place (out == in, only rows with sources are written)
// mode 1: compact (copy staying rows to new_index)      mode 2: aggregate + compact
// x_sqnorm_out (optional, modes 1 and 2): |x|^2 of every output row of the first tensor, fp32
// tail_rows (modes 1 and 2): rows behind the vision span, input row sum_n + j -> output row cu_vis_out[batch] + j
// win (mode 2, optional): the next stage's windows, built by `batch` workgroups of the same launch with win_lds bytes of
// LDS each (at most ROWS_WIN_LDS_MAX: the row workgroups of the launch reserve them too)
// publish (mode 2, optional): host memory of batch + 1 words that receive (publish_tag << 32 | cu_vis_out[i])
constexpr size_t ROWS_WIN_LDS_MAX = 32 * 1024;
hipError_t launch_rows(int mode, int dtype, int d, int sum_n, int batch, const RowTensors &t, const int32_t *new_index,
                       const int32_t *grp_offsets, const int32_t *grp_src, const float *xi, const int32_t *pos,
                       int32_t *pos_out, float *x_sqnorm_out, int64_t out_rows, int64_t tail_rows,
                       const int32_t *cu_vis_out, const WinArgs *win, size_t win_lds, unsigned long long *publish,
                       unsigned publish_tag, hipStream_t stream);

}  // namespace lk
