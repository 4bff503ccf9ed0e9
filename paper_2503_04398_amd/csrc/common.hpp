// Shared host/device helpers of the library: status handling, config validation, workspace carving,
// bf16 conversion.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <stddef.h>
#include <type_traits>

#include "semmoe.h"

namespace semmoe {

// ---- status -------------------------------------------------------------------------------------
void set_last_hip_error(hipError_t e);

#define SEMMOE_HIP(expr)                                  \
  do {                                                    \
    hipError_t _e = (expr);                               \
    if (_e != hipSuccess) {                               \
      ::semmoe::set_last_hip_error(_e);                   \
      return SEMMOE_EHIP;                                 \
    }                                                     \
  } while (0)

#define SEMMOE_LAUNCH_CHECK() SEMMOE_HIP(hipGetLastError())

// Facts about the current device, looked up once per device and kept (device ids below 64; thread-safe).
struct DeviceInfo {
  int num_cu;   // compute units
  int max_lds;  // most LDS a workgroup can ask for, bytes
};
int32_t device_info(DeviceInfo* out);

// Raises a kernel's dynamic-LDS limit to the device's maximum, once per device: `done` is the call site's own flag
// word (bit = device id), so every kernel and every device is handled exactly once, from whichever thread comes first.
int32_t allow_max_dynamic_lds(std::atomic<uint64_t>* done, const void* kernel);

// Shape rules every call shares.  `need_ffn`: d and F are used; `need_T`: cfg->T is used.
int32_t validate_config(const semmoe_config* cfg, bool need_T, bool need_rows, bool need_ffn);

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Threads of a workgroup that walks one row of `row_chunks` 16-byte chunks, a chunk per thread and pass: whole waves,
// at most 512 threads, and the count that leaves the fewest lanes without a chunk (896 chunks: 448 threads x 2 passes
// instead of 256 x 3.5; 360 chunks: 384 x 1 instead of 256 x 1.4).
inline int row_walk_threads(int row_chunks) {
  int best = 256, best_waste = 1 << 30;
  for (int passes = 1; passes <= 8; ++passes) {
    int th = cdiv(cdiv(row_chunks, passes), 64) * 64;
    if (th > 512) continue;
    if (th < 64) th = 64;
    const int waste = th * passes - row_chunks;
    if (waste < best_waste) {
      best_waste = waste;
      best = th;
    }
  }
  return best;
}
inline size_t act_bytes(const semmoe_config* cfg) { return cfg->dtype == SEMMOE_BF16 ? 2 : 4; }

// Sequential carving of the caller's workspace.
struct Carver {
  char* base;
  size_t size, off;
  bool ok;
  Carver(void* ws, size_t bytes) : base(static_cast<char*>(ws)), size(bytes), off(0), ok(ws != nullptr) {}
  template <typename T>
  T* take(size_t n) {
    size_t start = align_up(off, 256);
    size_t end = start + n * sizeof(T);
    if (!ok || end > size) {
      ok = false;
      off = end;
      return nullptr;
    }
    off = end;
    return reinterpret_cast<T*>(base + start);
  }
};

// Workspace needs per call (bytes), shared by semmoe_workspace_bytes and the calls themselves.
constexpr int kTokBlock = 256;  // tokens per workgroup in the index kernels
bool index_small(const semmoe_config* cfg, int path);  // reshuffle, dispatch_index: one workgroup, a thread a token
int route_max_parts(const semmoe_config* cfg);  // fused bf16 router: parts of K whose sums the workspace holds, at most
size_t ws_route(const semmoe_config* cfg);
size_t ws_reshuffle(const semmoe_config* cfg);
size_t ws_dispatch(const semmoe_config* cfg);
size_t ws_ffn(const semmoe_config* cfg);
size_t ws_request(const semmoe_config* cfg);
int tuning_value(int key);  // current value of a SEMMOE_TUNE_* knob (-1: default)

// ---- device helpers -----------------------------------------------------------------------------
typedef uint16_t bf16_t;  // storage of a bf16 value

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(static_cast<uint32_t>(v) << 16); }

// round to nearest, ties to even (inputs are finite)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<bf16_t>(u >> 16);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
}

// The k expert ids of a token: KU >= k registers, positions from k on repeat earlier ids (map_ids masks them).  No load sits
// behind a branch, so they all go out together.  quads (k a multiple of four, rows 16-byte aligned): a quarter of the
// instructions; a wave's 64 rows lie anywhere, and each 4-byte instruction costs the address unit as much as a 16-byte one.
// `row` must be readable for k entries even for a token that is not there (callers pass the row of one that is).
typedef __attribute__((ext_vector_type(4))) int32_t i32x4_t;

__host__ __device__ inline bool id_quads(const int32_t* ids, int k) {
  return k % 4 == 0 && (reinterpret_cast<uintptr_t>(ids) & 15u) == 0;
}

// calls f with the register width for k ids as a compile-time constant: loops over 16 positions for 4 experts a token spend
// most of their time on positions that are not there
template <typename F>
inline int32_t with_id_width(int k, F f) {
  if (k <= 4) return f(std::integral_constant<int, 4>{});
  if (k <= 8) return f(std::integral_constant<int, 8>{});
  static_assert(SEMMOE_MAX_K == 16, "the widths here");
  return f(std::integral_constant<int, 16>{});
}

template <int KU>
__device__ __forceinline__ void load_id_row(const int32_t* __restrict__ row, int k, bool quads, int (&e)[KU]) {
  static_assert(KU % 4 == 0, "whole quads");
  if (quads) {
#pragma unroll
    for (int j = 0; j < KU; j += 4) {
      const i32x4_t v = *reinterpret_cast<const i32x4_t*>(row + min(j, k - 4));
#pragma unroll
      for (int x = 0; x < 4; ++x) e[j + x] = v[x];
    }
  } else {
#pragma unroll
    for (int j = 0; j < KU; ++j) e[j] = row[min(j, k - 1)];
  }
}

// r[j] = map[e[j]] for j < k when the token is there and the expert lies in [0,E), else -1.  The map (expert -> rank, or
// expert -> physical position; -1: outside its range) lies in LDS: gathered from memory it is a second exposed latency.
template <int KU>
__device__ __forceinline__ void map_ids(const int (&e)[KU], bool have, int k, int E, const int32_t* map, int (&r)[KU]) {
#pragma unroll
  for (int j = 0; j < KU; ++j) {
    const bool ok = have && j < k && (unsigned)e[j] < (unsigned)E;
    const int m = map[ok ? e[j] : 0];
    r[j] = ok ? m : -1;
  }
}

// The k experts of a token mapped through a table (expert -> rank, or expert -> physical position):
//   r[j] = map[row[j]] for j < k when the token is there, the expert lies in [0,E) and the mapped value in [0,limit),
//   else -1 (also for j >= k).
// No load sits behind a branch: indices are clamped and the result is masked afterwards, so the k id loads go out
// together and then the k table loads - two exposed latencies.  Written per element with a test in front of each load,
// the compiler waits for every load before it issues the next: 2k latencies, 3-4 us of an index kernel.
// `row` must be readable for k entries even when `have` is false (callers pass the row of a token that exists).
template <int KU>
__device__ __forceinline__ void load_mapped_ids_n(const int32_t* __restrict__ row, bool have, int k, int E,
                                                  const int32_t* __restrict__ map, int limit,
                                                  int (&r)[SEMMOE_MAX_K]) {
  int e[KU], m[KU];
#pragma unroll
  for (int j = 0; j < KU; ++j) e[j] = row[min(j, k - 1)];
#pragma unroll
  for (int j = 0; j < KU; ++j) {
    const bool ok = have && j < k && (unsigned)e[j] < (unsigned)E;
    e[j] = ok ? e[j] : -1;
  }
#pragma unroll
  for (int j = 0; j < KU; ++j) m[j] = map[max(e[j], 0)];
#pragma unroll
  for (int j = 0; j < SEMMOE_MAX_K; ++j) r[j] = -1;
#pragma unroll
  for (int j = 0; j < KU; ++j) r[j] = (e[j] >= 0 && (unsigned)m[j] < (unsigned)limit) ? m[j] : -1;
}

__device__ __forceinline__ void load_mapped_ids(const int32_t* __restrict__ row, bool have, int k, int E,
                                                const int32_t* __restrict__ map, int limit, int (&r)[SEMMOE_MAX_K]) {
  static_assert(SEMMOE_MAX_K == 16, "the two widths below");
  if (k <= 8) load_mapped_ids_n<8>(row, have, k, E, map, limit, r);  // k is uniform: a scalar branch
  else load_mapped_ids_n<16>(row, have, k, E, map, limit, r);
}

// Number of bits below position t in a bitmap of WORDS 32-bit words in LDS (16-byte aligned): whole words masked by their
// place, four a load, no loop over the words before t that every lane leaves somewhere else.
template <int WORDS>
__device__ __forceinline__ int bits_below(const uint32_t* words, int t) {
  static_assert(WORDS % 4 == 0, "whole quads");
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  const int w = t >> 5;
  const uint32_t below = (1u << (t & 31)) - 1u;
  int n = 0;
#pragma unroll
  for (int x = 0; x < WORDS; x += 4) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(words + x);
#pragma unroll
    for (int y = 0; y < 4; ++y) n += __popc(x + y < w ? v[y] : (x + y == w ? v[y] & below : 0u));
  }
  return n;
}

// Column sums of a [n_rows][n_cols] table of counts: tot[c] += all rows, pre[c] += the rows before `b` (both in LDS,
// zeroed by the caller, who also places the barriers).  Every workgroup of the index kernels reads the whole table, so
// the time is the number of loads a thread waits for one after the other.  With n_cols a multiple of four a thread owns
// four columns (one 16-byte load) of every (threads / (n_cols / 4))-th row, eight loads in flight: a 64 x 256 table is
// two such batches a thread (as single columns it was eight: 16.4 us for dp_fused_kernel on 16384 tokens of 256 experts;
// a 64 x 288 table, with more columns than the 256 threads and so an atomic per element, 19.4 us for rs_fused_kernel).
// The first eight loads can be requested ahead of time (`column_sums_first`), before other work that has its own chain
// of dependent loads.
struct ColumnBatch {
  i32x4_t v[8];
};

__device__ __forceinline__ bool column_quads(int n_cols) { return n_cols % 4 == 0 && n_cols / 4 <= int(blockDim.x); }

__device__ __forceinline__ ColumnBatch column_sums_first(const int32_t* __restrict__ table, int n_rows, int n_cols) {
  ColumnBatch f;
  const int t = threadIdx.x, nt = blockDim.x, nq = n_cols / 4;
  const bool quads = column_quads(n_cols);
  const int rpp = quads ? nt / nq : 0;  // rows covered per pass
  const int c = quads ? t % nq : 0, r0 = quads ? t / nq : 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int bb = r0 + u * rpp;
    f.v[u] = (r0 < rpp && bb < n_rows) ? reinterpret_cast<const i32x4_t*>(table)[size_t(bb) * nq + c] : i32x4_t{0, 0, 0, 0};
  }
  return f;
}

__device__ __forceinline__ void column_sums_before(const int32_t* __restrict__ table, int n_rows, int n_cols, int b,
                                                   int32_t* tot, int32_t* pre, const ColumnBatch* first = nullptr) {
  const int t = threadIdx.x, nt = blockDim.x;
  if (column_quads(n_cols)) {
    const int nq = n_cols / 4, rpp = nt / nq;
    const int c = t % nq, r0 = t / nq;
    if (r0 >= rpp) return;
    i32x4_t s = {0, 0, 0, 0}, sb = {0, 0, 0, 0};
    for (int bb0 = r0; bb0 < n_rows; bb0 += 8 * rpp) {
      i32x4_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int bb = bb0 + u * rpp;
        if (first && bb0 == r0) v[u] = first->v[u];
        else v[u] = bb < n_rows ? reinterpret_cast<const i32x4_t*>(table)[size_t(bb) * nq + c] : i32x4_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s += v[u];
        sb += (bb0 + u * rpp < b) ? v[u] : i32x4_t{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {  // integer sums: the order does not matter
      if (s[x]) atomicAdd(&tot[4 * c + x], s[x]);
      if (sb[x]) atomicAdd(&pre[4 * c + x], sb[x]);
    }
    return;
  }
  for (int c0 = 0; c0 < n_cols; c0 += nt) {  // a column a thread; few columns: several threads share one
    const int nc = min(nt, n_cols - c0), rpp = nt / nc;
    const int c = t % nc, r0 = t / nc;
    if (r0 >= rpp) continue;
    int s = 0, sb = 0;
    for (int bb0 = r0; bb0 < n_rows; bb0 += 8 * rpp) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int bb = bb0 + u * rpp;
        v[u] = bb < n_rows ? table[size_t(bb) * n_cols + c0 + c] : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s += v[u];
        sb += (bb0 + u * rpp < b) ? v[u] : 0;
      }
    }
    if (s) atomicAdd(&tot[c0 + c], s);
    if (sb) atomicAdd(&pre[c0 + c], sb);
  }
}

}  // namespace semmoe
