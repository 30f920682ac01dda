// Window partition of the vision tokens (paper Sec. 3.2 and Sec. 3.2.2 "Window partitioning"):
// every token is assigned to a window by its cell in the original image grid, and the tokens of
// each window are listed in ascending sequence order (CSR).  One workgroup per sequence.
//
// Fast path (count table fits LDS): a stable multi-bin partition.  Every wave-sized run of 64
// consecutive tokens counts its tokens per window with ballots; a prefix over the runs and a scan
// over the windows give each token its slot directly -- no sort, no atomics, order preserved.
// Fallback: LDS bitonic sort of (window id, local index) keys.
#include <atomic>
#include "lk_win_body.h"

namespace lk {

constexpr int WIN_THREADS = 1024;
constexpr int LOCAL_BITS = 14;             // local token index < 16384
// Bytes of LDS the partition may take: all that a workgroup can have, as sorting 16384 tokens takes 127 us and counting them
// into 256 windows 35.
constexpr size_t WIN_TABLE_LDS_MAX = 152 * 1024;
constexpr int WIN_KEEP = 4;                // passes of 1024 tokens whose window and rank stay in registers between phases

__global__ __launch_bounds__(WIN_THREADS) void build_windows_table_kernel(WinArgs g) {
  fetch_args<WinArgs>();
  extern __shared__ __attribute__((aligned(16))) char win_lds[];
  build_windows_body<WIN_THREADS, WIN_KEEP>(g, blockIdx.x, win_lds);
}

__global__ __launch_bounds__(WIN_THREADS) void build_windows_sort_kernel(WinArgs g) {
  extern __shared__ uint32_t keys[];
  const int b = blockIdx.x;
  const int base = g.cu_vis[b];
  const int n_all = g.cu_vis[b + 1] - base;                            // tokens looked at
  const int out_base = g.cu_out ? g.cu_out[b] : base;
  const int n = g.cu_out ? g.cu_out[b + 1] - out_base : n_all;         // tokens that take part: they sort to the front
  const int wbase = b * g.win_per_seq;
  const int p2 = next_pow2(n_all > 1 ? n_all : 1);
  for (int i = threadIdx.x; i < p2; i += blockDim.x) {
    const bool in = i < n_all && listed_as(g, base + (i < n_all ? i : 0)) >= 0;
    keys[i] = in ? (((uint32_t)window_of(g, g.pos[base + i]) << LOCAL_BITS) | (uint32_t)i) : 0xffffffffu;
  }
  bitonic_sort_lds(keys, p2);
  // sorted position k holds the k-th token of the window-major order
  for (int k = threadIdx.x; k <= n; k += blockDim.x) {
    const int prev = (k == 0) ? -1 : (int)(keys[k - 1] >> LOCAL_BITS);
    int cur;
    if (k < n) {
      cur = (int)(keys[k] >> LOCAL_BITS);
      g.win_tokens[out_base + k] = listed_as(g, base + (int)(keys[k] & ((1u << LOCAL_BITS) - 1u)));
    } else {
      cur = (b == g.batch - 1) ? g.win_per_seq : g.win_per_seq - 1;   // the next sequence writes its own first offset
    }
    for (int id = prev + 1; id <= cur; ++id) g.win_offsets[wbase + id] = out_base + k;
  }
}

// ---- per-window counts (Sec. 3.2.1 Step 2, Sec. 3.2.2: the ratios P of the schedule) -----------------------------
// One workgroup per sequence.  mode 0: r_w = min(floor(rho v_w), ceil(v_w / 2)) tokens; mode 1: k_w = min(floor(rho v_w / 2),
// |A_w| |B_w|) edges; mode 2: the sequence has to go from its current length to a target length, and the difference
// is spread over its windows as evenly as their sizes allow (no window gives more than its set A): with q the largest
// level for which sum_w min(cap_w, q) stays within the budget, window w gives min(cap_w, q), and the first windows
// that can give more than q give one more until the budget is met.  Integer work throughout; rho is a double so that
// the floor is taken in the precision a host program would use.
constexpr int CNT_THREADS = 256;
constexpr int CNT_CACHE = 8192;   // window sizes kept in LDS (32 KB)

struct CountArgs {
  const int32_t *win_offsets, *cu_vis, *cu_target;
  int32_t *win_remove, *status;
  int win_per_seq, mode, dir;
  double rho;
};

__global__ __launch_bounds__(CNT_THREADS) void window_counts_kernel(CountArgs g) {
  fetch_args<CountArgs>();
  __shared__ int size_lds[CNT_CACHE];
  __shared__ long long scratch[CNT_THREADS / 64];
  const int b = blockIdx.x, W = g.win_per_seq, w0 = b * W;
  const int tid = threadIdx.x;
  auto size_mem = [&](int w) { return g.win_offsets[w0 + w + 1] - g.win_offsets[w0 + w]; };
  if (g.mode != 2) {
    for (int w = tid; w < W; w += CNT_THREADS) g.win_remove[w0 + w] = count_from_ratio(g.mode, g.rho, size_mem(w), g.dir);
    if (g.status && tid == 0) g.status[b] = 0;
    return;
  }
  const int budget = (g.cu_vis[b + 1] - g.cu_vis[b]) - (g.cu_target[b + 1] - g.cu_target[b]);
  // the sizes are looked at several times: the first CNT_CACHE of them are kept in LDS (one trip to memory instead of
  // one per pass, which is what this small kernel's time consists of); longer lists re-read the rest
  for (int w = tid; w < W && w < CNT_CACHE; w += CNT_THREADS) size_lds[w] = size_mem(w);
  __syncthreads();
  auto size_of = [&](int w) { return w < CNT_CACHE ? size_lds[w] : size_mem(w); };
  int32_t *status = g.status ? g.status + b : nullptr;
  if (W > COUNTS_WAVE_MAX) counts_target<CNT_THREADS / 64>(W, budget, g.dir, size_of, g.win_remove + w0, status, scratch);
  else if (tid < 64) counts_target<1>(W, budget, g.dir, size_of, g.win_remove + w0, status, nullptr);
}

hipError_t launch_window_counts(int batch, int win_per_seq, const int32_t *win_offsets, int mode, int dir, double rho,
                                const int32_t *cu_vis, const int32_t *cu_target, int32_t *win_remove, int32_t *status,
                                hipStream_t stream) {
  CountArgs g{};
  g.win_offsets = win_offsets; g.cu_vis = cu_vis; g.cu_target = cu_target; g.win_remove = win_remove; g.status = status;
  g.win_per_seq = win_per_seq; g.mode = mode; g.dir = dir; g.rho = rho;
  hipLaunchKernelGGL(window_counts_kernel, dim3(batch), dim3(CNT_THREADS), 0, stream, g);
  return hipGetLastError();
}

static WinArgs win_args(const WinSpec &spec, const int32_t *cu_vis, const int32_t *pos, const int32_t *new_index,
                        const int32_t *cu_out, int batch) {
  WinArgs g{};
  g.cu_vis = cu_vis; g.pos = pos; g.new_index = new_index; g.cu_out = cu_out; g.batch = batch;
  g.tiles = spec.tiles; g.grid_h = spec.grid_h; g.grid_w = spec.grid_w; g.w = spec.w;
  g.win_per_seq = (spec.w == 0) ? 1 : spec.tiles * spec.w * spec.w;
  g.by_cells = make_fast_div((uint32_t)(spec.grid_h * spec.grid_w));
  g.by_grid_h = make_fast_div((uint32_t)spec.grid_h);
  g.by_grid_w = make_fast_div((uint32_t)spec.grid_w);
  g.win_offsets = spec.win_offsets; g.win_tokens = spec.win_tokens;
  g.count_mode = spec.count_mode; g.rho = spec.rho; g.cu_target = spec.cu_target; g.win_remove = spec.win_remove;
  g.status = spec.status; g.dir = spec.dir;
  return g;
}

// more dynamic LDS than the 64 KB default, set once per device
static hipError_t allow_table_lds() {
  static std::atomic<bool> done[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (done[dev].load(std::memory_order_acquire)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(build_windows_table_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)WIN_TABLE_LDS_MAX);
  if (e == hipSuccess) done[dev].store(true, std::memory_order_release);
  return e;
}

hipError_t launch_build_windows(const WinSpec &spec, const int32_t *cu_vis, const int32_t *pos, const int32_t *new_index,
                                const int32_t *cu_out, int batch, int max_seq, bool *counts_done, hipStream_t stream) {
  WinArgs g = win_args(spec, cu_vis, pos, new_index, cu_out, batch);
  const size_t lds = win_table_bytes(max_seq, g.win_per_seq);
  if (lds <= WIN_TABLE_LDS_MAX) {
    const hipError_t e = allow_table_lds();
    if (e != hipSuccess) return e;
    *counts_done = spec.count_mode >= 0;
    hipLaunchKernelGGL(build_windows_table_kernel, dim3(batch), dim3(WIN_THREADS), lds, stream, g);
  } else {
    *counts_done = false;   // the sort leaves the counts to the caller
    const int p2 = next_pow2(max_seq > 1 ? max_seq : 1);
    hipLaunchKernelGGL(build_windows_sort_kernel, dim3(batch), dim3(WIN_THREADS), p2 * sizeof(uint32_t), stream, g);
  }
  return hipGetLastError();
}

size_t make_win_args(const WinSpec &spec, const int32_t *cu_vis, const int32_t *pos, const int32_t *new_index,
                     const int32_t *cu_out, int batch, int max_seq, WinArgs *out) {
  *out = win_args(spec, cu_vis, pos, new_index, cu_out, batch);
  const size_t lds = win_table_bytes(max_seq, out->win_per_seq);
  return lds <= ROWS_WIN_LDS_MAX ? lds : 0;
}

}  // namespace lk
