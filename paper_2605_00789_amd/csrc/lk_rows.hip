// Message passing (paper Sec. 3.2.1 Step 3, Eq. "message-passing") and delete + reorder (Steps 4-5)
// on the row tensors X, K, V.  Pure HBM streaming: one wave per (token, tensor) row, 16-byte
// loads and stores, fp32 arithmetic, round-to-nearest-even on store.
//
// A token b with sources a_1..a_m becomes  y_b + sum_a w_a (y_a - y_b),  w_a = xi_a / (xi_b + sum xi_a),
// which equals the xi-weighted mean of the equation and returns y_b bit for bit when all rows are equal.
// Sources are visited in ascending token order (grp_src), so results are reproducible run to run.
#include <type_traits>
#include "lk_win_body.h"

namespace lk {

constexpr int ROW_THREADS = 256;

struct RowArgs {
  RowTensors t;
  const int32_t *new_index, *grp_offsets, *grp_src, *pos;
  int32_t *pos_out;
  float *x_sqnorm_out;   // optional: |x|^2 of every output row of tensor 0 (as stored), fp32
  const float *xi;
  int d, sum_n, batch;
  int64_t out_rows;   // capacity of the compacted outputs; rows beyond it are dropped
  int64_t tail_rows;  // rows behind the vision span (modes 1 and 2)
  const int32_t *cu_vis_out;   // with tail_rows: cu_vis_out[batch] vision rows stay
  unsigned long long *publish;   // host memory, or NULL: (publish_tag << 32 | cu_vis_out[i]) for i = 0 .. batch
  unsigned publish_tag;
  int n_guest_blocks; // workgroups in front of the row workgroups: the windows', then the publishing one
  int n_win_blocks;   // workgroups in front of the row workgroups that build the next stage's windows
  int segs;           // segments per row
};

template <typename T> struct RowIO;
template <> struct RowIO<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(const uint4 &v, float (&f)[8]) {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
  }
  static __device__ __forceinline__ uint4 pack(const float (&f)[8]) {
    uint4 v;
    v.x = f32_to_bf16_rne(f[0]) | (f32_to_bf16_rne(f[1]) << 16);
    v.y = f32_to_bf16_rne(f[2]) | (f32_to_bf16_rne(f[3]) << 16);
    v.z = f32_to_bf16_rne(f[4]) | (f32_to_bf16_rne(f[5]) << 16);
    v.w = f32_to_bf16_rne(f[6]) | (f32_to_bf16_rne(f[7]) << 16);
    return v;
  }
};
template <> struct RowIO<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(const uint4 &v, float (&f)[4]) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  static __device__ __forceinline__ uint4 pack(const float (&f)[4]) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
  }
};

// One wave = one segment of one row of one tensor (4 rows per workgroup): U chunks of 16 bytes per lane, so that the
// whole segment is in flight before anything is consumed.  A merged row of more than 8 chunks per lane (8 KB; 5 KB in a short
// launch) is cut into equal segments for as many waves: two passes of one wave over a 10 KB row are two trips to memory in a
// row (2304 rows of 5120 bf16 and 200 text rows: 52 + 6 us in two launches -> 41 us).  A row that is only moved has nothing to
// wait for between its passes: one wave takes them in turn (9216 rows of 16 KB 153 us in segments, 146 so).  All loads are
// unconditional (clamped addresses) so that the compiler never has to wait inside a branch.
constexpr int ROWS_PER_WG = ROW_THREADS / WAVE;
// 16-byte chunks per lane and segment, at most.  Launches of few rows leave waves idle and want more of them with shorter
// lives; longer ones pay for them.  us, 8 KB rows in segments of 4 / whole: merge of three tensors 144 rows 4.9 / 6.4, 2000
// rows 19.8 / 20.6, 4096 rows 35.6 / 34.8; of one tensor 1100 rows 6.9 / 7.5, 2880 rows 13.0 / 12.5, 16384 rows 58.8 / 49.2.
// With squared norms, whose segments wait for one another, three tensors, inputs from memory: 2880 rows 29.8 / 31.8, 5400 48.6 /
// 50.8, 6100 53.2 / 53.1, 7000 59.7 / 59.5, 9216 75.7 / 75.6.
constexpr int ROW_MAX_U = 8, ROW_MAX_U_SHORT = 5;
constexpr int64_t ROWS_SHORT_MAX = 2048, ROWS_SHORT_MAX_SQ = 6144;
constexpr int64_t ROWS_STREAM_OUT_BYTES = 128ll << 20;   // inputs beyond this: nontemporal output stores
constexpr int ROWS_WIN_KEEP = 12;   // passes of 256 tokens the window partition keeps in registers (3072 tokens)

// MODE 0: aggregate in place   1: compact   2: aggregate + compact
//
// Dependent loads are what this kernel waits for, so they are arranged in as few rounds as possible:
//   round 1  the row itself, xi of the row, new_index and the group bounds (all depend on the row number only)
//   round 2  the source list of the group
//   round 3  xi of the sources and the rows of the first two sources, together
// A row without sources is stored after round 1.  Later sources come in pairs: groups of 5 to 11 sources exist in every
// launch, and the last of their waves is what a short launch waits for (three stages of 576 tokens 123.9 -> 120.2 us, with the
// arguments fetched at once; one by one before, and still where addresses are in vector registers, which have no room for two).
//
// Guests share the launch, because a launch or a stream fork of their own costs as much as they do:
//   rows behind the vision span (the prompt's text, Steps 4-5): rows sum_n .. sum_n + tail_rows of the inputs move to
//   output row n' + j, n' = cu_vis_out[batch] being read from the device;
//   the next stage's windows: the first n_win_blocks workgroups build them (they need pos and new_index only);
//   the sequence offsets the step leaves, for a host that has to lay the next stage out: one workgroup writes them to
//   host memory at the start of the launch, so the host works while the rows move.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <bool STREAM>
__device__ __forceinline__ void store16(char *p, const uint4 &v) {
  const u32x4 t4 = {v.x, v.y, v.z, v.w};
  if (STREAM) __builtin_nontemporal_store(t4, reinterpret_cast<u32x4 *>(p));
  else *reinterpret_cast<u32x4 *>(p) = t4;
}

// v of a lane that is the same for the whole wave, in a scalar register or in a vector one
template <bool SCALAR> __device__ __forceinline__ int lane_value(int v, int lane) {
  return SCALAR ? __builtin_amdgcn_readlane(v, lane) : __shfl(v, lane, 64);
}
template <bool SCALAR> __device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(lane_value<SCALAR>(__float_as_int(v), lane));
}

// Registers: 8 chunks a lane fit three waves per SIMD (166; 179 = two waves left alone, merge of 21312 rows 230 us against 199),
// 4 take 134 with row addresses in vector registers and 128 = four waves with scalar ones, 5 chunks 122 and 112.  Rows that are only
// moved keep vector addresses: scalar ones took 24 registers more than eight waves have, the last three loads of an 8 KB row were
// parked in scratch memory (2880 rows and 128 text rows 27.6 -> 35.2 us, 9216 72 -> 86).
//
// STREAM: the output rows are stored nontemporally (a template parameter: as a run-time choice between two stores of
// the same value the compiler merges them into one plain store)
template <typename T, int MODE, bool STREAM, int U, bool SCALAR>
__global__ __launch_bounds__(ROW_THREADS, MODE == 1 ? 8 : (U > 5 || U == 4 ? 3 : 4)) void rows_kernel(RowArgs g, WinArgs wn) {
  using IO = RowIO<T>;
  constexpr int N = IO::N;
  constexpr int BYTES = Elem<T>::BYTES;
  constexpr int HU = U > 4 ? (U + 1) / 2 : U;   // chunks of a merge in flight per source
  const int which = blockIdx.z;   // tensor
  const char *in = static_cast<const char *>(g.t.in[which]);
  char *out = static_cast<char *>(g.t.out[which]);
  const int64_t ld_in = g.t.ld_in[which] * BYTES, ld_out = g.t.ld_out[which] * BYTES;
  fetch_now(in, ld_in, g.new_index, g.grp_offsets, g.xi, g.d, g.sum_n, g.tail_rows, g.n_guest_blocks, g.segs);
  if constexpr (MODE == 2) {
    if ((int)blockIdx.x < g.n_win_blocks) {
      if (blockIdx.y + blockIdx.z > 0) return;
      extern __shared__ __attribute__((aligned(16))) char win_lds[];
      build_windows_body<ROW_THREADS, ROWS_WIN_KEEP>(wn, blockIdx.x, win_lds);
      return;
    }
    if ((int)blockIdx.x < g.n_guest_blocks) {
      if (blockIdx.y + blockIdx.z > 0) return;
      // every word carries the tag, so the host needs no order between them
      for (int i = threadIdx.x; i <= g.batch; i += ROW_THREADS)
        __hip_atomic_store(&g.publish[i], ((unsigned long long)g.publish_tag << 32) | (unsigned)g.cu_vis_out[i],
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      return;
    }
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // SCALAR: the row is the same for all lanes, and the compiler is told: row addresses then live in scalar registers
  const int row_wave = SCALAR ? wave : (int)(threadIdx.x >> 6);
  using Offset = std::conditional_t<SCALAR, uint32_t, int64_t>;
  int64_t b = (int64_t)((int)blockIdx.x - g.n_guest_blocks) * ROWS_PER_WG + row_wave;
  int seg = blockIdx.y;
  // |x|^2 needs all segments of a row: two or four of them are waves of one workgroup then (ROWS_PER_WG / segs rows each).  Other
  // numbers (three: bf16 rows of 10 to 15 KB in short launches) don't fill a workgroup and are taken in turn by one wave.
  const bool sq_split = MODE == 2 && which == 0 && g.x_sqnorm_out != nullptr && (g.segs == 2 || g.segs == ROWS_PER_WG);
  if (sq_split) {
    const int sh = g.segs == 2 ? 1 : 2;
    b = (((int64_t)((int)blockIdx.x - g.n_guest_blocks) * g.segs + blockIdx.y) * ROWS_PER_WG + row_wave) >> sh;
    seg = wave & (g.segs - 1);
  }
  if (b >= g.sum_n + g.tail_rows) return;
  const int n_chunks = g.d / N;
  const char *row_in = in ? in + b * ld_in : nullptr;
  // |x|^2 of the row as it is stored (tensor 0 only, on request): the next stage's feature divergence wants it, and
  // here the row is in registers anyway.  Same order of summation as the stand-alone pass over X: a lane's sum goes on from
  // segment to segment, through LDS where they are waves of one workgroup, in one wave that takes them in turn otherwise (in
  // turn at two segments as well, three stages of 576 tokens took 115.5 us instead of 107.7).
  const bool want_sq = MODE != 0 && which == 0 && g.x_sqnorm_out != nullptr && b < g.sum_n;
  if (want_sq && !sq_split && seg > 0) return;
  const int seg_end = (want_sq && !sq_split) || MODE == 1 ? g.segs : seg + 1;   // (a launch of mode 1 has one workgroup per four rows)

  // round 1 (the in-place mode touches few rows: it looks at the group bounds first instead of fetching every row)
  if (MODE == 0 && g.grp_offsets[b + 1] == g.grp_offsets[b]) return;
  // A row that is merged away is fetched by its own wave as well as by its target's (8-11 % more bytes read): looking
  // at new_index first would save those bytes but puts one more dependent load in front of every row, and the longer
  // life of every wave costs more than the bytes (single launch on 2880 tokens: 26.8 -> 23.9 us without the look).
  // Large outputs are stored nontemporally: they cannot stay cached until the next stage reads them, and kept out of
  // the caches they leave them to the kernels that run next (batch of 16: step -3.6 %; on the cache-resident sizes the
  // same stores cost +2.4 %: the next stage's kernels then find their inputs in HBM).
  uint4 v[U];
  auto load_row = [&](const char *row, int sg, uint4 (&dst)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = (sg * U + u) * WAVE + lane;
      dst[u] = ld16(row + (Offset)((c < n_chunks ? c : n_chunks - 1) * 16));
    }
  };
  if (in != nullptr) load_row(row_in, seg, v);
  if (MODE != 0 && b >= g.sum_n) {   // a row behind the vision span
    int n_keep = g.cu_vis_out[g.batch];
    n_keep = n_keep < 0 ? 0 : (n_keep > g.sum_n ? g.sum_n : n_keep);
    const int64_t out_row = n_keep + (b - g.sum_n);
    if (out_row >= g.out_rows) return;   // no room in the output: dropped, never written out of bounds
    if (which == 0 && seg == 0 && lane == 0 && g.pos && g.pos_out) g.pos_out[out_row] = g.pos[b];
    if (in == nullptr) return;
    char *row_out = out + out_row * ld_out;
    for (int sg = seg; sg < seg_end; ++sg) {
      if (sg > seg) load_row(row_in, sg, v);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = (sg * U + u) * WAVE + lane;
        if (c < n_chunks) store16<STREAM>(row_out + (Offset)(c * 16), v[u]);
      }
    }
    return;
  }
  float xb = 0.f;
  if (MODE != 1) xb = g.xi[b];
  int out_row = (int)b, s0 = 0, s1 = 0;
  if (MODE != 0) out_row = g.new_index[b];
  if (MODE != 1) { s0 = g.grp_offsets[b]; s1 = g.grp_offsets[b + 1]; }
  const int m = s1 - s0;
  if (MODE != 0 && (out_row < 0 || out_row >= g.out_rows)) return;   // merged away, or no room in the output
  if (MODE == 0 && m == 0) return;                                    // in place: nothing to do for this row
  if (MODE != 0 && which == 0 && seg == 0 && lane == 0 && g.pos && g.pos_out) g.pos_out[out_row] = g.pos[b];
  if (in == nullptr) return;
  char *row_out = out + (int64_t)out_row * ld_out;

  // rounds 2 and 3: lane s holds source s and its weight (groups beyond 64 sources take the slow loop)
  int a_l = (int)b;
  float w_l = 0.f, w0 = 0.f, w1 = 0.f;
  const char *row_a0 = row_in, *row_a1 = row_in;
  if (MODE != 1 && m > 0) {
    const int mm = m < WAVE ? m : WAVE;
    a_l = g.grp_src[s0 + (lane < mm ? lane : mm - 1)];
    row_a0 = in + (int64_t)lane_value<SCALAR>(a_l, 0) * ld_in;
    row_a1 = in + (int64_t)lane_value<SCALAR>(a_l, mm > 1 ? 1 : 0) * ld_in;
  }

  float sq = 0.f;
  bool first = true;
  for (; seg < seg_end; ++seg) {
    if (!first) load_row(row_in, seg, v);
    if (MODE != 1 && m > 0) {
      // first half of the segment: its source chunks go out together with the xi loads below
      uint4 va0[HU], va1[HU];
      auto load_source = [&](const char *row, int hb, uint4 (&dst)[HU]) {
#pragma unroll
        for (int u = 0; u < HU; ++u) {
          if (hb + u < U) {
            const int c = (seg * U + hb + u) * WAVE + lane;
            dst[u] = ld16(row + (Offset)((c < n_chunks ? c : n_chunks - 1) * 16));
          }
        }
      };
      auto load_first_two = [&](int hb) {   // chunk by chunk: the sums start with the first of both
#pragma unroll
        for (int u = 0; u < HU; ++u) {
          if (hb + u < U) {
            const int c = (seg * U + hb + u) * WAVE + lane;
            const Offset o = (Offset)((c < n_chunks ? c : n_chunks - 1) * 16);
            va0[u] = ld16(row_a0 + o);
            va1[u] = ld16(row_a1 + o);
          }
        }
      };
      auto source_row = [&](int s) {   // source s of the group (groups of more than 64: from memory)
        return in + (int64_t)(m <= WAVE ? lane_value<SCALAR>(a_l, s) : g.grp_src[s0 + s]) * ld_in;
      };
      auto weight = [&](int s) { return m <= WAVE ? lane_value<SCALAR>(w_l, s) : g.xi[g.grp_src[s0 + s]] * lane_value<SCALAR>(w_l, 0); };
      auto add = [&](const uint4 (&src)[HU], float w, int hb, float (&acc)[HU][N]) {
#pragma unroll
        for (int u = 0; u < HU; ++u) {
          if (hb + u < U) {
            float ya[N], yb[N];
            IO::unpack(src[u], ya);
            IO::unpack(v[hb + u], yb);
#pragma unroll
            for (int e = 0; e < N; ++e) acc[u][e] = fmaf(w, ya[e] - yb[e], acc[u][e]);
          }
        }
      };
      load_first_two(0);
      if (first) {
        const int mm = m < WAVE ? m : WAVE;
        float x_l = g.xi[a_l];
        x_l = lane < mm ? x_l : 0.f;
        float den = x_l;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) den += __shfl_xor(den, o, 64);   // fixed butterfly: reproducible
        den += xb;
        for (int s = s0 + WAVE; s < s1; ++s) den += g.xi[g.grp_src[s]];
        w_l = x_l / den;
        if (m > WAVE) w_l = 1.f / den;   // slow path keeps 1/den instead
        w0 = weight(0);
        w1 = (m <= 1) ? 0.f : weight(1);
      }
#pragma unroll
      for (int hb = 0; hb < U; hb += HU) {
        if (hb > 0) load_first_two(hb);
        float acc[HU][N];   // y_b stays packed in v[] and is unpacked where it is used
#pragma unroll
        for (int u = 0; u < HU; ++u) {
          if (hb + u < U) {
            float y0[N], y1[N], yb[N];
            IO::unpack(v[hb + u], yb);
            IO::unpack(va0[u], y0);
            IO::unpack(va1[u], y1);
#pragma unroll
            for (int e = 0; e < N; ++e) acc[u][e] = fmaf(w1, y1[e] - yb[e], fmaf(w0, y0[e] - yb[e], yb[e]));
          }
        }
        if constexpr (SCALAR) {
          for (int s = 2; s < m; s += 2) {   // later sources, two in flight
            load_source(source_row(s), hb, va0);
            if (s + 1 < m) load_source(source_row(s + 1), hb, va1);   // uniform
            add(va0, weight(s), hb, acc);
            if (s + 1 < m) add(va1, weight(s + 1), hb, acc);
          }
        } else {
          for (int s = 2; s < m; ++s) {   // one by one
            load_source(source_row(s), hb, va0);
            add(va0, weight(s), hb, acc);
          }
        }
#pragma unroll
        for (int u = 0; u < HU; ++u)
          if (hb + u < U) v[hb + u] = IO::pack(acc[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = (seg * U + u) * WAVE + lane;
      if (c < n_chunks) store16<STREAM>(row_out + (Offset)(c * 16), v[u]);
    }
    if (want_sq) {
      float t[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        t[u] = BYTES == 2 ? sumsq_chunk_bf16(v[u]) : sumsq_chunk_f32(v[u]);
        t[u] = (seg * U + u) * WAVE + lane < n_chunks ? t[u] : 0.f;
      }
      if constexpr (MODE == 2) {
        if (sq_split) {   // wait for the sum of the segments before (waves whose rows end early are not waited for)
          __shared__ float before[ROWS_PER_WG][WAVE];
          for (int k = 1; k <= seg; ++k) lds_barrier();
          if (seg > 0) sq = before[wave - 1][lane];
#pragma unroll
          for (int u = 0; u < U; ++u) sq += t[u];
          if (seg + 1 < g.segs) {
            before[wave][lane] = sq;
            for (int k = seg + 1; k < g.segs; ++k) lds_barrier();
            return;
          }
          break;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) sq += t[u];
    }
    first = false;
  }
  if (want_sq) {
    sq = wave_sum_butterfly(sq);
    if (lane == 0) g.x_sqnorm_out[out_row] = sq;
  }
}

template <typename T, int U>
static void launch_rows_u(int mode, bool stream_out, bool scalar, const dim3 &grid, size_t lds, hipStream_t stream, const RowArgs &g,
                          const WinArgs &wn) {
  const dim3 block(ROW_THREADS);
  if constexpr (U <= ROW_MAX_U_SHORT) {
    if (scalar && mode == 0) { hipLaunchKernelGGL((rows_kernel<T, 0, false, U, true>), grid, block, lds, stream, g, wn); return; }
    if constexpr (U == 2 || U == 4) {
      if (scalar && stream_out) { hipLaunchKernelGGL((rows_kernel<T, 2, true, U, true>), grid, block, lds, stream, g, wn); return; }
    }
    if (scalar && mode == 2) { hipLaunchKernelGGL((rows_kernel<T, 2, false, U, true>), grid, block, lds, stream, g, wn); return; }
  }
  if (mode == 0) hipLaunchKernelGGL((rows_kernel<T, 0, false, U, false>), grid, block, lds, stream, g, wn);
  else if (mode == 1 && stream_out) hipLaunchKernelGGL((rows_kernel<T, 1, true, U, false>), grid, block, lds, stream, g, wn);
  else if (mode == 1) hipLaunchKernelGGL((rows_kernel<T, 1, false, U, false>), grid, block, lds, stream, g, wn);
  else if (stream_out) hipLaunchKernelGGL((rows_kernel<T, 2, true, U, false>), grid, block, lds, stream, g, wn);
  else hipLaunchKernelGGL((rows_kernel<T, 2, false, U, false>), grid, block, lds, stream, g, wn);
}

hipError_t launch_rows(int mode, int dtype, int d, int sum_n, int batch, const RowTensors &t, const int32_t *new_index,
                       const int32_t *grp_offsets, const int32_t *grp_src, const float *xi, const int32_t *pos,
                       int32_t *pos_out, float *x_sqnorm_out, int64_t out_rows, int64_t tail_rows,
                       const int32_t *cu_vis_out, const WinArgs *win, size_t win_lds, unsigned long long *publish,
                       unsigned publish_tag, hipStream_t stream) {
  if (mode == 0) tail_rows = 0;
  if (sum_n + tail_rows == 0 && !win && !publish) return hipSuccess;
  RowArgs g{};
  g.x_sqnorm_out = x_sqnorm_out;
  g.t = t; g.new_index = new_index; g.grp_offsets = grp_offsets; g.grp_src = grp_src; g.pos = pos;
  g.pos_out = pos_out; g.xi = xi; g.d = d; g.sum_n = sum_n; g.out_rows = out_rows;
  g.tail_rows = tail_rows; g.cu_vis_out = cu_vis_out; g.batch = batch;
  g.n_win_blocks = win ? batch : 0;
  g.publish = publish; g.publish_tag = publish_tag;
  g.n_guest_blocks = g.n_win_blocks + (publish ? 1 : 0);
  int n_tensors = 0;
  for (int i = 0; i < 3; ++i) n_tensors += t.in[i] != nullptr;
  // nontemporal output stores once the tensors are far beyond what stays cached until the next stage reads them
  const bool stream_out = mode != 0 && (int64_t)sum_n * d * (dtype == 1 ? 2 : 4) * n_tensors > ROWS_STREAM_OUT_BYTES;
  // chunks per lane of a whole row; rows beyond max_u are taken in equal segments, rounded up to a size there is
  const int per_lane = (d * (dtype == 1 ? 2 : 4) / 16 + WAVE - 1) / WAVE;
  const bool is_short = !stream_out && sum_n + tail_rows <= (x_sqnorm_out ? ROWS_SHORT_MAX_SQ : ROWS_SHORT_MAX);
  const int max_u = mode != 1 && is_short ? ROW_MAX_U_SHORT : ROW_MAX_U;
  g.segs = (per_lane + max_u - 1) / max_u;
  const int u = (per_lane + g.segs - 1) / g.segs;
  const dim3 grid((unsigned)(g.n_guest_blocks + (sum_n + tail_rows + ROWS_PER_WG - 1) / ROWS_PER_WG),
                  (unsigned)(mode == 1 ? 1 : g.segs), 3u);
  // Row addresses in scalar registers and later sources in pairs: the last waves of a short launch are what it waits for.  In a
  // longer one the bytes are, and vector addresses keep more of them in flight (2772 rows of 8960 bytes and 197 text rows 33.0 us
  // against 33.4; 16000 of 1 KB 26.8 / 29.3, of 8 KB 121.6 / 122.0; 9216 in place 43.0 / 43.6), except for bf16 rows of two to four
  // chunks a lane, where they cost a wave per SIMD (6400 rows of 3 KB 30.4 against 27.3, 16000 63.2 / 55.9; of 4 KB 33.4 / 31.4 and
  // 69.6 / 64.5; 16000 of 2 KB 38.2 / 37.7).
  const bool scalar = mode != 1 && (is_short || (dtype == 1 && u >= 2 && u <= 4));
  const WinArgs wn = win ? *win : WinArgs{};
  const size_t lds = win ? win_lds : 0;
#define LK_ROWS(TT)                                                                       \
  do {                                                                                    \
    if (u <= 1) launch_rows_u<TT, 1>(mode, stream_out, scalar, grid, lds, stream, g, wn);         \
    else if (u <= 2) launch_rows_u<TT, 2>(mode, stream_out, scalar, grid, lds, stream, g, wn);    \
    else if (u <= 4) launch_rows_u<TT, 4>(mode, stream_out, scalar, grid, lds, stream, g, wn);    \
    else if (u <= 5) launch_rows_u<TT, 5>(mode, stream_out, scalar, grid, lds, stream, g, wn);    \
    else launch_rows_u<TT, 8>(mode, stream_out, scalar, grid, lds, stream, g, wn);                \
  } while (0)
  if (dtype == 1) LK_ROWS(bf16_t);
  else LK_ROWS(float);
#undef LK_ROWS
  return hipGetLastError();
}

}  // namespace lk
