// The hierarchical schedule (paper Sec. 3.2.2) as one call: every stage's windows, scores, selection and merge are
// enqueued through the library's own entry points, arranged so that
//   - xi (needs only Q and the stage's K rows) runs next to the feature-divergence chain and the selection: in the same
//     launches where lightkv_score_select can do that, on a helper stream otherwise,
//   - the next stage's windows (need only pos and the selection) are built by workgroups of the merge's launch, or beside
//     the merge on a second helper stream (NextWindows below).
// Nothing here launches a kernel itself or allocates device memory.  lightkv_compress_schedule never synchronises;
// lightkv_compress_schedule_ratio (token counts that depend on the data) waits once per stage for the sequence offsets the
// stage leaves, and for the stream before it returns.
#include "../../include/lightkv.h"

#include "lk_helpers.h"
#include "lk_launch.h"

#include <hip/hip_runtime.h>
#include <mutex>
#include <algorithm>

namespace {

// The helper streams (0 runs xi, 1 builds windows) and the fork and join events of one call.  Sets come from a per-device
// pool (lk_helpers.h), distinct from the one lightkv_score uses for its own fork.
using Helpers = lk::HelperSet<2, 4, 1>;
enum { EV_FORK_XI = 0, EV_JOIN_XI = 1, EV_FORK_WIN = 2, EV_JOIN_WIN = 3 };

// a stage's windows, with the counts that go with them in a schedule
lk::WinSpec windows_of(const lightkv_stage &st, int32_t tiles, int32_t grid_h, int32_t grid_w, int count_mode, double rho) {
  lk::WinSpec s{};
  s.tiles = tiles; s.grid_h = grid_h; s.grid_w = grid_w; s.w = st.w;
  s.win_offsets = st.win_offsets; s.win_tokens = st.win_tokens;
  s.count_mode = count_mode; s.rho = rho; s.dir = st.problem.direction; s.n_windows = st.problem.n_windows;
  s.cu_target = st.cu_vis_target; s.win_remove = st.win_remove; s.status = count_mode == LIGHTKV_COUNT_TARGET ? st.status : nullptr;
  return s;
}

int count_mode_of(const lightkv_stage &st) {
  return st.problem.match == LIGHTKV_MATCH_EDGE_TOPK ? LIGHTKV_COUNT_EDGES : LIGHTKV_COUNT_RATIO;
}

// Waits for the words a kernel on `stream` writes under the mailbox's last tag.  The wait ends with the stream at the
// latest: once everything enqueued has finished (or failed), the words are there or never will be.
bool read_mailbox(const lk::Mailbox &box, int n, int32_t *out, hipStream_t stream) {
  int have = 0;
  for (unsigned spin = 1;; ++spin) {
    bool last_look = false;
    if ((spin & 0xfff) == 0) {
      last_look = hipStreamQuery(stream) != hipErrorNotReady;
      (void)hipGetLastError();   // "not ready" is no error of a later launch
    }
    while (have < n) {
      const unsigned long long w = __atomic_load_n(&box.words[have], __ATOMIC_ACQUIRE);
      if ((unsigned)(w >> 32) != box.tag) break;
      out[have++] = (int32_t)(unsigned)(w & 0xffffffffu);
    }
    if (have == n) return true;
    if (last_look) return false;
    __builtin_ia32_pause();
  }
}

// `to` waits for everything enqueued on `from` so far
bool order_after(hipStream_t to, hipStream_t from, hipEvent_t ev) {
  return hipEventRecord(ev, from) == hipSuccess && hipStreamWaitEvent(to, ev, 0) == hipSuccess;
}

// The helpers of a call, taken when a stage first forks.
struct CallHelpers {
  hipStream_t main;
  std::unique_lock<std::mutex> guard;
  Helpers *h = nullptr;
  bool tried = false;
  explicit CallHelpers(hipStream_t m) : main(m) {}
  Helpers *get() {
    if (!tried) { tried = true; h = lk::acquire_helpers<2, 4, 1>(main, guard); }
    return h;
  }
};

// The next stage's windows, once the selection has been enqueued on the caller's stream: guests of the merge's launch
// (`ride`, the merge then takes the spec), or a launch of their own on the second helper stream.
struct NextWindows {
  bool forked = false;
  // true: the merge has to take them along
  bool enqueue(CallHelpers &helpers, bool ride, const lightkv_problem *p, const int32_t *pos, const lightkv_stage &st,
               const lk::WinSpec &spec, lightkv_status &rc) {
    forked = false;
    Helpers *h = ride ? nullptr : helpers.get();
    if (!h) return true;
    if (!order_after(h->stream[1], helpers.main, h->event[EV_FORK_WIN])) { (void)hipGetLastError(); return true; }
    forked = true;
    rc = (lightkv_status)lk::build_windows_with_counts(p->batch, p->h_cu_vis, p->cu_vis, pos, st.new_index, st.cu_vis_out, spec, h->stream[1]);
    if (hipEventRecord(h->event[EV_JOIN_WIN], h->stream[1]) != hipSuccess && rc == LIGHTKV_OK) rc = LIGHTKV_ERR_LAUNCH;
    return false;
  }
  void join(CallHelpers &helpers, lightkv_status &rc) {
    if (forked && hipStreamWaitEvent(helpers.main, helpers.h->event[EV_JOIN_WIN], 0) != hipSuccess && rc == LIGHTKV_OK) rc = LIGHTKV_ERR_LAUNCH;
    forked = false;
  }
};

}  // namespace

extern "C" lightkv_status lightkv_compress_schedule(const lightkv_stage *stages, int32_t n_stages,
                                                    int32_t tiles, int32_t grid_h, int32_t grid_w,
                                                    const void *X, int64_t ldx, const void *K, int64_t ldk,
                                                    const void *V, int64_t ldv, const int32_t *pos,
                                                    const void *Q, int64_t q_tok_stride, int64_t q_head_stride,
                                                    float softmax_scale, void *ws, size_t ws_bytes, void *stream) {
  if (!stages || !X || !K || !V || !pos || !Q) return LIGHTKV_ERR_NULL;
  if (n_stages < 1) return LIGHTKV_ERR_SHAPE;
  for (int s = 0; s < n_stages; ++s) {
    const lightkv_stage &st = stages[s];
    if (st.reserved != 0 || st.problem.match != LIGHTKV_MATCH_BEST_PER_A) return LIGHTKV_ERR_UNSUPPORTED;
    if (!st.win_offsets || !st.win_tokens || !st.xi || !st.best_fd || !st.best_dst || !st.dst || !st.new_index ||
        !st.grp_offsets || !st.grp_src || !st.cu_vis_out || !st.X_out || !st.K_out || !st.V_out || !st.pos_out)
      return LIGHTKV_ERR_NULL;
    if (st.problem.win_offsets != st.win_offsets || st.problem.win_tokens != st.win_tokens) return LIGHTKV_ERR_SHAPE;
    if (!st.problem.h_cu_vis || !st.problem.cu_vis) return LIGHTKV_ERR_NULL;
    if (st.problem.batch != stages[0].problem.batch || st.problem.d != stages[0].problem.d) return LIGHTKV_ERR_SHAPE;
    if (st.cu_vis_target) {   // counts from the token budget: the schedule writes the array the descriptor points to
      if (!st.win_remove) return LIGHTKV_ERR_NULL;
      if (st.problem.win_remove != st.win_remove || st.problem.n_windows % st.problem.batch != 0) return LIGHTKV_ERR_SHAPE;
    }
    size_t need = 0;
    const lightkv_status ws_st = lightkv_workspace_size(&st.problem, &need);
    if (ws_st != LIGHTKV_OK) return ws_st;
    if (!ws || ws_bytes < need) return LIGHTKV_ERR_WORKSPACE;
  }
  hipStream_t main = static_cast<hipStream_t>(stream);
  CallHelpers helpers(main);
  NextWindows next_windows;

  const int d = stages[0].problem.d, head_dim = stages[0].problem.head_dim;
  const void *Xi = X, *Ki = K, *Vi = V;
  int64_t ldxi = ldx, ldki = ldk, ldvi = ldv;
  const int32_t *posi = pos;
  const float *sq = nullptr;          // squared norms of Xi, once a stage has produced them
  bool windows_ready = false;         // this stage's windows were built beside the previous stage's merge
  lightkv_status rc = LIGHTKV_OK;
  for (int s = 0; s < n_stages && rc == LIGHTKV_OK; ++s) {
    const lightkv_stage &st = stages[s];
    const lightkv_problem *p = &st.problem;
    const bool one_stream = lk::score_select_one_stream(p);
    // ---- xi on the helper stream (or, if there is none, first on the caller's)
    bool xi_forked = false;
    if (!one_stream) {
      hipStream_t xs = main;
      Helpers *h = helpers.get();
      if (h && order_after(h->stream[0], main, h->event[EV_FORK_XI])) { xs = h->stream[0]; xi_forked = true; }
      else if (h) (void)hipGetLastError();
      rc = lightkv_score(p, nullptr, 0, nullptr, Q, q_tok_stride, q_head_stride, Ki, ldki, head_dim, LIGHTKV_XI_TEXT_QUERY,
                         nullptr, softmax_scale, st.xi, nullptr, nullptr, nullptr, 0, ws, ws_bytes, xs);
      if (xi_forked && hipEventRecord(h->event[EV_JOIN_XI], h->stream[0]) != hipSuccess) rc = rc == LIGHTKV_OK ? LIGHTKV_ERR_LAUNCH : rc;
    }
    // ---- windows (and their counts from the stage's token budget), unless they were built beside the previous stage's merge
    next_windows.join(helpers, rc);
    if (!windows_ready && rc == LIGHTKV_OK)
      rc = (lightkv_status)lk::build_windows_with_counts(
          p->batch, p->h_cu_vis, p->cu_vis, posi, nullptr, nullptr,
          windows_of(st, tiles, grid_h, grid_w, st.cu_vis_target ? LIGHTKV_COUNT_TARGET : -1, 0.0), main);
    // ---- feature divergence + selection
    if (rc == LIGHTKV_OK) {
      if (one_stream)
        rc = lightkv_score_select(p, Xi, ldxi, sq, Q, q_tok_stride, q_head_stride, Ki, ldki, head_dim,
                                  LIGHTKV_XI_TEXT_QUERY, nullptr, softmax_scale, st.xi, st.best_fd, st.best_dst, st.dst,
                                  st.new_index, st.grp_offsets, st.grp_src, st.cu_vis_out, ws, ws_bytes, main);
      else
        rc = lightkv_score_select(p, Xi, ldxi, sq, nullptr, 0, 0, nullptr, 0, 0, LIGHTKV_XI_GIVEN, nullptr, softmax_scale,
                                  st.xi, st.best_fd, st.best_dst, st.dst, st.new_index, st.grp_offsets, st.grp_src,
                                  st.cu_vis_out, ws, ws_bytes, main);
    }
    // ---- the next stage's windows follow from pos and the selection alone (cu_vis_out of this stage is the next stage's
    // cu_vis).  They ride in the merge's launch if they fit there: a queue crossing costs more than they add to it (three eager
    // stages of 2880 tokens, d = 1024, 158 us riding, 182 forked; of 8192, d = 4096, 468 and 494; of 16384, d = 1024, 516 and
    // 457: the other way round where the partition outlives the rows).
    lk::WinSpec next{};
    bool ride = false;
    if (rc == LIGHTKV_OK && s + 1 < n_stages) {
      next = windows_of(stages[s + 1], tiles, grid_h, grid_w, stages[s + 1].cu_vis_target ? LIGHTKV_COUNT_TARGET : -1, 0.0);
      ride = next_windows.enqueue(helpers, lk::windows_ride(p, next), p, posi, st, next, rc);
    }
    // ---- join xi (whatever happened: nothing stays forked), merge and compact
    if (xi_forked && hipStreamWaitEvent(main, helpers.h->event[EV_JOIN_XI], 0) != hipSuccess) rc = rc == LIGHTKV_OK ? LIGHTKV_ERR_LAUNCH : rc;
    if (rc == LIGHTKV_OK)
      rc = (lightkv_status)lk::aggregate_compact_with_windows(p, st.new_index, st.grp_offsets, st.grp_src, st.xi, Xi, ldxi, Ki,
                                                              ldki, Vi, ldvi, posi, st.X_out, st.K_out, st.V_out, st.pos_out,
                                                              st.x_sqnorm_out, st.out_rows, st.cu_vis_out,
                                                              ride ? &next : nullptr, nullptr, 0, main);
    windows_ready = true;
    Xi = st.X_out; Ki = st.K_out; Vi = st.V_out;
    ldxi = ldki = ldvi = d;
    posi = st.pos_out;
    sq = st.x_sqnorm_out;
  }
  next_windows.join(helpers, rc);   // after an error
  return rc;
}

// The schedule when a stage's token count depends on the data (the k lowest edges of a window, the full pairwise
// visit, or any matching driven by the ratio of Sec. 3.2.2 instead of fixed budgets): per-window counts come from the
// window sizes on the device, and the batch + 1 sequence offsets a stage leaves are read back before the next stage is
// laid out.  A copy and a synchronisation behind the merge left the device idle for 50-70 us a stage (copy, wake-up, planning,
// first launch); the offsets are known once the selection has run, so the merge's launch writes them to pinned host
// memory as it starts: three stages of 2880 tokens 444 -> 350 us.
extern "C" lightkv_status lightkv_compress_schedule_ratio(const lightkv_stage *stages, int32_t n_stages, const double *rho,
                                                          int32_t tiles, int32_t grid_h, int32_t grid_w,
                                                          const void *X, int64_t ldx, const void *K, int64_t ldk,
                                                          const void *V, int64_t ldv, const int32_t *pos,
                                                          const void *Q, int64_t q_tok_stride, int64_t q_head_stride,
                                                          float softmax_scale, void *ws, size_t ws_bytes,
                                                          int32_t *h_cu_vis_out, void *stream) {
  if (!stages || !rho || !X || !K || !V || !pos || !Q || !h_cu_vis_out) return LIGHTKV_ERR_NULL;
  if (n_stages < 1) return LIGHTKV_ERR_SHAPE;
  const int batch = stages[0].problem.batch;
  if (batch < 1) return LIGHTKV_ERR_SHAPE;
  for (int s = 0; s < n_stages; ++s) {
    const lightkv_stage &st = stages[s];
    if (st.reserved != 0 || st.cu_vis_target) return LIGHTKV_ERR_UNSUPPORTED;
    if (!st.win_offsets || !st.win_tokens || !st.win_remove || !st.xi || !st.best_fd || !st.best_dst || !st.dst ||
        !st.new_index || !st.grp_offsets || !st.grp_src || !st.cu_vis_out || !st.X_out || !st.K_out || !st.V_out ||
        !st.pos_out)
      return LIGHTKV_ERR_NULL;
    if (st.problem.win_offsets != st.win_offsets || st.problem.win_tokens != st.win_tokens ||
        st.problem.win_remove != st.win_remove)
      return LIGHTKV_ERR_SHAPE;
    // counts and window sizes are the device's alone here
    if (st.problem.h_win_offsets || st.problem.h_win_remove) return LIGHTKV_ERR_UNSUPPORTED;
    if (st.problem.batch != batch || st.problem.d != stages[0].problem.d || st.problem.max_window_tokens <= 0 ||
        st.problem.n_windows % batch != 0)
      return LIGHTKV_ERR_SHAPE;
    if (!(rho[s] >= 0.0 && rho[s] <= 1e6)) return LIGHTKV_ERR_SHAPE;
  }
  if (!stages[0].problem.h_cu_vis || !stages[0].problem.cu_vis) return LIGHTKV_ERR_NULL;
  hipStream_t main = static_cast<hipStream_t>(stream);
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(main, &cs) != hipSuccess) { (void)hipGetLastError(); return LIGHTKV_ERR_LAUNCH; }
  if (cs != hipStreamCaptureStatusNone) return LIGHTKV_ERR_UNSUPPORTED;   // the call waits for the stream: not capturable

  const int d = stages[0].problem.d, head_dim = stages[0].problem.head_dim;
  const void *Xi = X, *Ki = K, *Vi = V;
  int64_t ldxi = ldx, ldki = ldk, ldvi = ldv;
  const int32_t *posi = pos;
  const float *sq = nullptr;
  const int32_t *h_cu = stages[0].problem.h_cu_vis;   // offsets of the stage's input: on the host ...
  const int32_t *d_cu = stages[0].problem.cu_vis;     // ... and on the device
  bool windows_ready = false;
  CallHelpers helpers(main);
  NextWindows next_windows;
  std::unique_lock<std::mutex> box_guard;
  lk::Mailbox *box = lk::acquire_mailbox(batch + 1, box_guard);
  lightkv_status rc = LIGHTKV_OK;
  for (int s = 0; s < n_stages && rc == LIGHTKV_OK; ++s) {
    const lightkv_stage &st = stages[s];
    lightkv_problem q = st.problem;
    q.h_cu_vis = h_cu;
    q.cu_vis = d_cu;
    int max_seq = 0;
    for (int b = 0; b < batch; ++b) max_seq = std::max(max_seq, h_cu[b + 1] - h_cu[b]);
    // a window holds no more tokens than its sequence: the tighter bound picks the cheaper launch plans; the plans are
    // not monotone in it, so if that one wants more workspace than there is, the stage's own bound is used
    const int bound = st.problem.max_window_tokens;
    q.max_window_tokens = std::max(1, std::min(bound, max_seq));
    size_t need = 0;
    rc = (lightkv_status)lk::least_workspace(&q, &need);
    if (rc == LIGHTKV_OK && (!ws || ws_bytes < need) && q.max_window_tokens != bound) {
      q.max_window_tokens = bound;
      rc = (lightkv_status)lk::least_workspace(&q, &need);
    }
    if (rc == LIGHTKV_OK && (!ws || ws_bytes < need)) rc = LIGHTKV_ERR_WORKSPACE;
    // ---- windows and their counts, unless they were built beside the previous stage's merge
    next_windows.join(helpers, rc);
    if (!windows_ready && rc == LIGHTKV_OK)
      rc = (lightkv_status)lk::build_windows_with_counts(batch, h_cu, d_cu, posi, nullptr, nullptr,
                                                         windows_of(st, tiles, grid_h, grid_w, count_mode_of(st), rho[s]), main);
    // ---- scores (xi and feature divergence) and selection
    if (rc == LIGHTKV_OK)
      rc = lightkv_score_select(&q, Xi, ldxi, sq, Q, q_tok_stride, q_head_stride, Ki, ldki, head_dim, LIGHTKV_XI_TEXT_QUERY,
                                nullptr, softmax_scale, st.xi, st.best_fd, st.best_dst, st.dst, st.new_index, st.grp_offsets,
                                st.grp_src, st.cu_vis_out, ws, ws_bytes, main);
    // ---- merge and compact, the next stage's windows and counts beside it (they follow from the selection alone)
    lk::WinSpec next{};
    bool ride = false;
    if (rc == LIGHTKV_OK && s + 1 < n_stages) {
      next = windows_of(stages[s + 1], tiles, grid_h, grid_w, count_mode_of(stages[s + 1]), rho[s + 1]);
      ride = next_windows.enqueue(helpers, lk::windows_ride(&q, next), &q, posi, st, next, rc);
    }
    if (rc == LIGHTKV_OK)
      rc = (lightkv_status)lk::aggregate_compact_with_windows(&q, st.new_index, st.grp_offsets, st.grp_src, st.xi, Xi, ldxi, Ki,
                                                              ldki, Vi, ldvi, posi, st.X_out, st.K_out, st.V_out, st.pos_out,
                                                              st.x_sqnorm_out, st.out_rows, st.cu_vis_out,
                                                              ride ? &next : nullptr, box ? box->words : nullptr,
                                                              box ? box->next_tag() : 0u, main);
    windows_ready = true;
    // ---- the offsets the stage left: the next stage's descriptor
    int32_t *h_out = h_cu_vis_out + (size_t)s * (batch + 1);
    if (rc == LIGHTKV_OK) {
      bool got;
      if (box) {
        // the merge's first workgroup has written them to the mailbox: the next stage is laid out and enqueued while the
        // rows still move
        got = read_mailbox(*box, batch + 1, h_out, main);
      } else {
        got = hipMemcpyAsync(h_out, st.cu_vis_out, sizeof(int32_t) * (batch + 1), hipMemcpyDeviceToHost, main) == hipSuccess &&
              hipStreamSynchronize(main) == hipSuccess;
      }
      if (!got) {
        (void)hipGetLastError();
        rc = LIGHTKV_ERR_LAUNCH;
      }
    }
    if (rc == LIGHTKV_OK) {
      // a sequence never grows, and everything that stays must have found room in the stage's outputs
      bool ok = h_out[0] == 0;
      for (int b = 0; ok && b < batch; ++b) {
        const int n = h_out[b + 1] - h_out[b];
        ok = n >= 0 && n <= h_cu[b + 1] - h_cu[b];
      }
      if (!ok || h_out[batch] > st.out_rows) rc = LIGHTKV_ERR_SHAPE;
    }
    Xi = st.X_out; Ki = st.K_out; Vi = st.V_out;
    ldxi = ldki = ldvi = d;
    posi = st.pos_out;
    sq = st.x_sqnorm_out;
    h_cu = h_out;
    d_cu = st.cu_vis_out;
  }
  next_windows.join(helpers, rc);   // after an error
  // what was enqueued has finished when the call returns, whatever it returns
  if (hipStreamSynchronize(main) != hipSuccess) {
    (void)hipGetLastError();
    if (rc == LIGHTKV_OK) rc = LIGHTKV_ERR_LAUNCH;
  }
  return rc;
}
