// Scores and selection of one step in three launches on ONE stream (paper Sec. 3.2.1 Steps 1-3).
//
// The prompt-guidance weight xi (two passes over the keys, then a sum over heads) and the feature divergence with
// its selection (partial tiles, tile tail, index scan) are two chains of three short kernels each; neither depends
// on the other until the merge.  Run on two streams they overlap, but every fork and join of the streams costs about
// as much as one of these kernels.  Here the k-th kernels of the two chains share a launch instead: the first
// workgroups of a launch run the xi pass, the rest the FD step (device bodies from lk_xi_body.h / lk_fd_body.h;
// the LDS block is the larger of the two needs, registers likewise).
//
//   launch 1   xi pass 1 (row statistics)      |  FD partial tiles               (workgroups of the two kinds alternate)
//   launch 2   xi pass 2 (column sums)         |  windows of at most 64 tokens: tile tail (epilogue + per-window
//                                              |  selection); larger ones: epilogue                (FD workgroups first)
//                                              |  k lowest edges: the selection of every window, or the keys of
//                                              |  large windows' pairs
//   (larger windows: the per-window selection, a launch or two of its own)
//   last       xi heads summed                 |  index scan                     (select_scan_kernel<true, ...>)
//
// Results are bit-identical to the separate kernels.  On two streams the chains overlap as well, but every crossing
// between hardware queues costs 9-15 us (eager calls: an event record, a wait and the start behind it), two of them on
// the critical path of every stage: three stages of 576 tokens 175 -> 124 us,
// of 2880 tokens 261 -> 229 us (graph replay 241 -> 220), of 3 x 513 fp32 tokens 125 -> 87 us.
#include <atomic>
#include "lk_edge_body.h"
#include "lk_xi_body.h"

namespace lk {

template <int A, int B> struct MaxOf { static constexpr int value = A > B ? A : B; };

template <typename T, int DH, int RW>
__global__ __launch_bounds__(XI_THREADS, 3) void rowstat_partial_kernel(XiArgs x, int n_xi_blocks, FdArgs f) {
  fetch_args<XiArgs, int, FdArgs>();
  static_assert(XI_THREADS == FD_THREADS, "both bodies are written for 256 threads");
  __shared__ __attribute__((aligned(16))) char lds[MaxOf<XiStage<T, DH, RW>::LDS_ROWSTAT, FD_PARTIAL_LDS>::value];
  // the two kinds of workgroup alternate, so that both chains get the chip from the start of the launch
  const int n_fd_blocks = f.n_tiles * f.ksplit;
  const int paired = 2 * (n_xi_blocks < n_fd_blocks ? n_xi_blocks : n_fd_blocks);
  const int i = blockIdx.x;
  bool is_xi;
  int id;
  if (i < paired) { is_xi = (i & 1) == 0; id = i >> 1; }
  else { is_xi = n_xi_blocks > n_fd_blocks; id = i - paired / 2; }
  if (is_xi) xi_rowstat_body<T, DH, RW>(x, id, lds);
  else fd_partial_body<T>(f, id, lds);
}

// TAIL: tile tails (windows of at most 64 tokens); otherwise the epilogue of larger windows
template <typename T, int DH, int RW, bool VISION_LSE, bool TAIL>
__global__ __launch_bounds__(XI_THREADS) void colsum_tail_kernel(XiArgs x, int n_fd_blocks, FdArgs f, SmallSelArgs q) {
  fetch_args<XiArgs, int, FdArgs, SmallSelArgs>();
  constexpr int FD_LDS = TAIL ? (int)sizeof(SmallTileLds) : FD_EPILOGUE_LDS;
  __shared__ __attribute__((aligned(16))) char lds[MaxOf<XiStage<T, DH, RW>::LDS_COLSUM, FD_LDS>::value];
  // the few FD workgroups go first: they are the longer dependency chain and must not wait for a free slot
  if ((int)blockIdx.x < n_fd_blocks) {
    if (TAIL) fd_tail_select_body(f, q, blockIdx.x, lds);
    else fd_epilogue_body(f, blockIdx.x, lds);
  } else {
    xi_colsum_body<T, DH, RW, VISION_LSE>(x, blockIdx.x - n_fd_blocks, lds);
  }
}

// The same beside the edge selection; dynamic LDS, as the keys of a window may need more than the column sums do.
template <typename T, int DH, int RW, bool VISION_LSE>
__global__ __launch_bounds__(XI_THREADS) void colsum_edges_kernel(XiArgs x, int n_fd_blocks, FdArgs f, EdgeArgs q) {
  fetch_args<XiArgs, int, FdArgs, EdgeArgs>();
  extern __shared__ __attribute__((aligned(16))) char dyn_lds[];
  if ((int)blockIdx.x >= n_fd_blocks) xi_colsum_body<T, DH, RW, VISION_LSE>(x, blockIdx.x - n_fd_blocks, dyn_lds);
  else if (q.max_a > EDGE_MAX_SIDE) edge_keys_body(f, q, blockIdx.x, dyn_lds);
  else edge_select_body<0, EDGE_ITEMS>(f, q, blockIdx.x, dyn_lds);
}

template <typename T, int DH, int RW, bool VISION_LSE>
static hipError_t launch_colsum_edges(const XiArgs &x, int n_xi_blocks, const FdArgs &f, const EdgeArgs &q, hipStream_t stream) {
  const bool keys_only = q.max_a > EDGE_MAX_SIDE;
  const size_t need = keys_only ? sizeof(EdgeKeysLds) : edge_lds_bytes(q.max_a, q.max_b);
  constexpr size_t colsum = XiStage<T, DH, RW>::LDS_COLSUM;
  const size_t lds = need > colsum ? need : colsum;
  static std::atomic<bool> allowed[64];   // more dynamic LDS than the 64 KB default, set once per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!allowed[dev].load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(colsum_edges_kernel<T, DH, RW, VISION_LSE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)edge_lds_bytes(EDGE_MAX_SIDE, EDGE_MAX_SIDE));
    if (e != hipSuccess) return e;
    allowed[dev].store(true, std::memory_order_release);
  }
  const int n_fd_blocks = keys_only ? f.n_tiles : f.n_windows;
  hipLaunchKernelGGL((colsum_edges_kernel<T, DH, RW, VISION_LSE>), dim3((unsigned)(n_xi_blocks + n_fd_blocks)), dim3(XI_THREADS),
                     lds, stream, x, n_fd_blocks, f, q);
  return hipGetLastError();
}

template <typename T, int DH, int RW, bool VISION_LSE>
static hipError_t launch_two(const XiArgs &x, int n_xi_blocks, bool pass1, bool tail, int n_fd_blocks, const FdArgs &f,
                             const SmallSelArgs &q, const EdgeArgs *edges, hipStream_t stream) {
  const unsigned g1 = (unsigned)((pass1 ? n_xi_blocks : 0) + f.n_tiles * f.ksplit);
  hipLaunchKernelGGL((rowstat_partial_kernel<T, DH, RW>), dim3(g1), dim3(XI_THREADS), 0, stream, x,
                     pass1 ? n_xi_blocks : 0, f);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (edges) return launch_colsum_edges<T, DH, RW, VISION_LSE>(x, n_xi_blocks, f, *edges, stream);
  const unsigned g2 = (unsigned)(n_xi_blocks + n_fd_blocks);
  if (tail)
    hipLaunchKernelGGL((colsum_tail_kernel<T, DH, RW, VISION_LSE, true>), dim3(g2), dim3(XI_THREADS), 0, stream, x, n_fd_blocks, f, q);
  else
    hipLaunchKernelGGL((colsum_tail_kernel<T, DH, RW, VISION_LSE, false>), dim3(g2), dim3(XI_THREADS), 0, stream, x, n_fd_blocks, f, q);
  return hipGetLastError();
}

template <typename T, int DH>
static hipError_t launch_two_t(const XiArgs &x, int n_xi_blocks, bool pass1, bool vision_lse, int max_t, bool tail,
                               int n_fd_blocks, const FdArgs &f, const SmallSelArgs &q, const EdgeArgs *edges,
                               hipStream_t stream) {
  if constexpr (xi_long_chunks_fit<T, DH>()) {
    if (max_t > 64) {
      if (vision_lse) return launch_two<T, DH, 128, true>(x, n_xi_blocks, pass1, tail, n_fd_blocks, f, q, edges, stream);
      return launch_two<T, DH, 128, false>(x, n_xi_blocks, pass1, tail, n_fd_blocks, f, q, edges, stream);
    }
  }
  if (vision_lse) return launch_two<T, DH, 64, true>(x, n_xi_blocks, pass1, tail, n_fd_blocks, f, q, edges, stream);
  return launch_two<T, DH, 64, false>(x, n_xi_blocks, pass1, tail, n_fd_blocks, f, q, edges, stream);
}

hipError_t launch_xi_fd_fused(const XiArgs &x, const XiPlan &xp, const FdArgs &f, const SmallSelArgs &q, const EdgeArgs *edges,
                              FusedFinish finish, int n_rowblocks, int dtype, int head_dim, hipStream_t stream) {
  if ((finish == FUSED_EDGES) != (edges != nullptr)) return hipErrorInvalidValue;
  const int n_xi_blocks = x.batch * x.heads * xp.max_vis_blocks;
  const bool vision_lse = x.lse_per_vision != 0;
  const bool pass1 = !vision_lse && x.lse == nullptr;
  const int max_t = xp.max_text_tiles * 32;
  const bool tail = finish == FUSED_TAIL;
  const int n_fd_blocks = tail ? f.n_tiles : fd_epilogue_blocks(n_rowblocks, f.group, f.nt);
#define LK_CASE(TT, DHV) return launch_two_t<TT, DHV>(x, n_xi_blocks, pass1, vision_lse, max_t, tail, n_fd_blocks, f, q, edges, stream)
  if (dtype == 1) {
    if (head_dim == 128) LK_CASE(bf16_t, 128);
    if (head_dim == 64) LK_CASE(bf16_t, 64);
    if (head_dim == 32) LK_CASE(bf16_t, 32);
  } else {
    if (head_dim == 128) LK_CASE(float, 128);
    if (head_dim == 64) LK_CASE(float, 64);
    if (head_dim == 32) LK_CASE(float, 32);
  }
#undef LK_CASE
  return hipErrorInvalidValue;
}

}  // namespace lk
