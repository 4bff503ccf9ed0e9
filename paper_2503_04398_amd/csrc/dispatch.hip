// dispatch: the dispatch all2all of expert parallelism (Sec. 1) as a single-device permutation.
// Index half: a stable counting sort of the P = T*k (token, expert) pairs by physical expert, pairs
// taken in shuffled-token order.  A token's k experts are distinct, so inside a 256-token workgroup the
// rank of a pair among equal keys is the popcount of the key's token bitmap below that token; across
// workgroups an exclusive scan over (expert, workgroup).  Row half: each token row is read once and
// written to its k slots with 16-byte accesses.
#include "common.hpp"
#include "scan_util.hpp"

namespace semmoe {

constexpr int kWords = kTokBlock / 32;

struct DispatchWs {
  int32_t* cnt;        // [NB][E]    per-block pair counts per physical expert -> base slot after the scan
  uint32_t* send_part; // [NB][D*D]  per-block send matrices
  uint32_t* remote_part;  // [NB]    per-block pairs whose expert sits on another rank than the token
};

// A workgroup's token chain: its token (shf), then in one go the token's ids and its rank; the expert -> physical position
// table and everything else a workgroup has to set up are requested and done while the chain runs.  The map entry of an
// expert is its position | its rank << 16 (-1: outside the range), so that no pair divides by the experts per rank.
__device__ __forceinline__ int token_at(int T, int pos, const int32_t* __restrict__ shf) {
  const int tok = pos < T ? shf[pos] : -1;
  return (unsigned)tok < (unsigned)T ? tok : -1;
}

__device__ __forceinline__ void load_phys_map(int E, int m, const int32_t* __restrict__ phys, int32_t* map) {
  for (int x = threadIdx.x; x < E; x += blockDim.x) {
    const int q = phys[x];
    map[x] = (unsigned)q < (unsigned)E ? (q | (q / m) << 16) : -1;
  }
}

__device__ __forceinline__ void zero_quads(void* lds, int n_quads) {
  for (int x = threadIdx.x; x < n_quads; x += blockDim.x) reinterpret_cast<uint4*>(lds)[x] = make_uint4(0, 0, 0, 0);
}

// Pairs of a workgroup's tokens per (rank of the token, rank of the expert).  The tokens of a workgroup sit on one rank or
// two, so its pairs fall on few entries, and LDS adds to one address run one after the other: every entry has several
// copies side by side (in neighbouring banks), and neighbouring lanes add to different ones.
__host__ __device__ inline int send_copies(int D) { return D <= 8 ? 8 : (D <= 32 ? 2 : 1); }

template <int KU>
__device__ __forceinline__ int count_send(int D, int s, const int (&q)[KU], uint32_t* send, int copies) {
  int remote = 0;
  if ((unsigned)s >= (unsigned)D) return 0;
  const int mine = int(threadIdx.x) & (copies - 1);
#pragma unroll
  for (int j = 0; j < KU; ++j)
    if (q[j] >= 0) {
      const int r = q[j] >> 16;
      atomicAdd(&send[(s * D + r) * copies + mine], 1u);
      remote += r != s;
    }
  return remote;
}

__device__ __forceinline__ uint32_t send_total(const uint32_t* send, int x, int copies) {
  uint32_t v = 0;
  for (int c = 0; c < copies; ++c) v += send[x * copies + c];
  return v;
}

template <int KU, int WORDS>
__device__ __forceinline__ void set_bits(const int (&q)[KU], uint32_t* bm) {
  const int t = threadIdx.x;
#pragma unroll
  for (int j = 0; j < KU; ++j)
    if (q[j] >= 0) atomicOr(&bm[(q[j] & 0xffff) * WORDS + (t >> 5)], 1u << (t & 31));
}

template <int WORDS>
__device__ __forceinline__ int bits_of(const uint32_t* words) {
  int c = 0;
#pragma unroll
  for (int y = 0; y < WORDS; y += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(words + y);
    c += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
  }
  return c;
}

// slot_of_pair of a token's k pairs (a run of 4k bytes) and its inverse.  slot[j] < 0: no pair
template <int KU>
__device__ __forceinline__ void store_slots(int tok, int k, const int (&slot)[KU], bool quads,
                                            int32_t* __restrict__ slot_of_pair, int32_t* __restrict__ pair_of_slot) {
  const int pair0 = tok * k;
  if (quads) {
#pragma unroll
    for (int j = 0; j < KU; j += 4)
      if (j < k) {
        if (slot[j] >= 0 && slot[j + 1] >= 0 && slot[j + 2] >= 0 && slot[j + 3] >= 0) {
          *reinterpret_cast<i32x4_t*>(slot_of_pair + size_t(pair0) + j) = i32x4_t{slot[j], slot[j + 1], slot[j + 2], slot[j + 3]};
        } else {
#pragma unroll
          for (int x = 0; x < 4; ++x)
            if (slot[j + x] >= 0) slot_of_pair[pair0 + j + x] = slot[j + x];
        }
      }
  } else {
#pragma unroll
    for (int j = 0; j < KU; ++j)
      if (slot[j] >= 0) slot_of_pair[pair0 + j] = slot[j];
  }
#pragma unroll
  for (int j = 0; j < KU; ++j)
    if (slot[j] >= 0) pair_of_slot[slot[j]] = pair0 + j;
}

// D1: per-block counts per physical expert and per-block send matrix
template <int KU>
__global__ __launch_bounds__(kTokBlock) void dp_count_kernel(int T, int k, int E, int D,
                                                             const int32_t* __restrict__ ids,
                                                             const int32_t* __restrict__ token_rank,
                                                             const int32_t* __restrict__ shf,
                                                             const int32_t* __restrict__ phys, DispatchWs w) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  // [E][kWords] bitmaps | [D*D][copies] send counts + remote pairs, whole quads | [E] map
  const int copies = send_copies(D), n_send = D * D * copies, send_quads = (n_send + 1 + 3) / 4;
  uint32_t* bm = reinterpret_cast<uint32_t*>(lds_raw);
  uint32_t* send = bm + E * kWords;
  int32_t* map = reinterpret_cast<int32_t*>(send + send_quads * 4);
  const int tok = token_at(T, blockIdx.x * kTokBlock + threadIdx.x, shf);
  load_phys_map(E, E / D, phys, map);
  zero_quads(bm, E * kWords / 4 + send_quads);
  int e[KU], q[KU];
  load_id_row(ids + size_t(max(tok, 0)) * k, k, id_quads(ids, k), e);
  const int s = token_rank[max(tok, 0)];
  __syncthreads();
  map_ids(e, tok >= 0, k, E, map, q);
  set_bits<KU, kWords>(q, bm);
  int remote = count_send(D, tok >= 0 ? s : -1, q, send, copies);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) remote += __shfl_xor(remote, o);
  if ((threadIdx.x & 63) == 0 && remote) atomicAdd(&send[n_send], (uint32_t)remote);
  __syncthreads();
  for (int x = threadIdx.x; x < E; x += kTokBlock) w.cnt[size_t(blockIdx.x) * E + x] = bits_of<kWords>(bm + x * kWords);
  for (int x = threadIdx.x; x < D * D; x += kTokBlock) w.send_part[size_t(blockIdx.x) * D * D + x] = send_total(send, x, copies);
  if (threadIdx.x == 0) w.remote_part[blockIdx.x] = send[n_send];
}

// D2: expert_offsets, rank_offsets, slot base of (block, expert) relative to the expert's first slot,
// send_matrix, remote_pairs (one workgroup, all threads busy: see column_prefix)
__global__ __launch_bounds__(kScanThreads) void dp_scan_kernel(int NB, int E, int D,
                                                                int32_t* __restrict__ expert_offsets,
                                                                int32_t* __restrict__ rank_offsets,
                                                                uint32_t* __restrict__ send_matrix,
                                                                unsigned long long* __restrict__ remote_pairs,
                                                                DispatchWs w) {
  __shared__ int32_t tot[SEMMOE_MAX_E + 1];
  __shared__ int32_t send_tot[SEMMOE_MAX_D * SEMMOE_MAX_D];
  __shared__ int32_t scratch[kScanThreads];
  __shared__ unsigned long long remote_sh;
  const int tid = threadIdx.x;
  if (tid == 0) remote_sh = 0ull;
  column_prefix(w.cnt, E, [](int c) { return c; }, E, NB, w.cnt, E, tot, scratch);
  wave_exclusive_scan_lds(tot, E);
  const int m = E / D;
  for (int q = tid; q <= E; q += blockDim.x) {
    expert_offsets[q] = tot[q];
    if (q % m == 0) rank_offsets[q / m] = tot[q];
  }
  column_prefix(reinterpret_cast<const int32_t*>(w.send_part), D * D, [](int c) { return c; }, D * D, NB,
                static_cast<int32_t*>(nullptr), 0, send_tot, scratch);
  unsigned long long remote = 0;
  for (int x = tid; x < D * D; x += blockDim.x) {
    send_matrix[x] = (uint32_t)send_tot[x];
    if (x / D != x % D) remote += (uint32_t)send_tot[x];
  }
  if (remote) atomicAdd(&remote_sh, remote);
  __syncthreads();
  if (tid == 0) *remote_pairs = remote_sh;
}

// D3: slot of every pair and its inverse
template <int KU>
__global__ __launch_bounds__(kTokBlock) void dp_slot_kernel(int T, int k, int E, int D, const int32_t* __restrict__ ids,
                                                            const int32_t* __restrict__ shf,
                                                            const int32_t* __restrict__ phys,
                                                            int32_t* __restrict__ slot_of_pair,
                                                            int32_t* __restrict__ pair_of_slot,
                                                            const int32_t* __restrict__ expert_offsets, DispatchWs w) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];  // [E][kWords] bitmaps | [E] map
  uint32_t* bm = reinterpret_cast<uint32_t*>(lds_raw);
  int32_t* map = reinterpret_cast<int32_t*>(bm + E * kWords);
  const int tok = token_at(T, blockIdx.x * kTokBlock + threadIdx.x, shf);
  load_phys_map(E, E / D, phys, map);
  zero_quads(bm, E * kWords / 4);
  int e[KU], q[KU];
  load_id_row(ids + size_t(max(tok, 0)) * k, k, id_quads(ids, k), e);
  __syncthreads();
  map_ids(e, tok >= 0, k, E, map, q);
  set_bits<KU, kWords>(q, bm);
  __syncthreads();
  if (tok < 0) return;
  int slot[KU];
#pragma unroll
  for (int j = 0; j < KU; ++j) {
    const int at = max(q[j], 0) & 0xffff;
    slot[j] = q[j] < 0 ? -1
                       : expert_offsets[at] + w.cnt[size_t(blockIdx.x) * E + at] +
                             bits_below<kWords>(bm + at * kWords, threadIdx.x);
  }
  store_slots(tok, k, slot, id_quads(slot_of_pair, k), slot_of_pair, pair_of_slot);
}

// Columns c_lo .. c_lo + n_cols - 1 of a [n_rows][stride] table summed into acc (LDS, zeroed by the caller) by all threads:
// with V = 4 whole quads (c_lo, n_cols and stride multiples of four), four loads a thread in flight.
template <int V>
__device__ __forceinline__ void sum_some_columns(const uint32_t* __restrict__ table, int n_rows, int stride, int c_lo,
                                                 int n_cols, uint32_t* acc) {
  typedef __attribute__((ext_vector_type(V))) uint32_t vec_t;
  const int t = threadIdx.x, nt = blockDim.x;
  for (int c0 = 0; c0 < n_cols; c0 += nt * V) {
    const int nv = min(nt, (n_cols - c0) / V), rpp = nt / nv;  // columns (of V) in this pass, rows at a time
    const int c = c0 + t % nv * V, r0 = t / nv;
    if (r0 >= rpp) continue;
    vec_t s = {};
    for (int r = r0; r < n_rows; r += 4 * rpp) {
      vec_t x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        x[u] = r + u * rpp < n_rows ? *reinterpret_cast<const vec_t*>(table + size_t(r + u * rpp) * stride + c_lo + c) : vec_t{};
#pragma unroll
      for (int u = 0; u < 4; ++u) s += x[u];
    }
#pragma unroll
    for (int x = 0; x < V; ++x)
      if (s[x]) atomicAdd(&acc[c + x], s[x]);
  }
}

// D2 + D3 in one launch: every workgroup sums the [NB][E] count table itself (column totals -> expert offsets,
// prefix over the workgroups before it -> its base inside each expert) instead of waiting for a scan kernel; the entries
// of the send matrix are dealt out to the workgroups in runs, summed by all threads of each (an entry a wave, as it was
// before, took 1024 entries on 8 workgroups 32 rounds of exposed latency: 2048 tokens of 32 ranks as two launches 29 us, now 13).  The chain of dependent loads, the
// tables and the LDS set-up all start together, and there are three barriers (16384 tokens, 256 experts: 13.2 -> 9.4 us);
// workgroup 0 writes the offsets and the remote-pair count.
template <int KU>
__global__ __launch_bounds__(kTokBlock) void dp_fused_kernel(int T, int k, int E, int D, int NB,
                                                             const int32_t* __restrict__ ids,
                                                             const int32_t* __restrict__ shf,
                                                             const int32_t* __restrict__ phys,
                                                             int32_t* __restrict__ slot_of_pair,
                                                             int32_t* __restrict__ pair_of_slot,
                                                             int32_t* __restrict__ expert_offsets,
                                                             int32_t* __restrict__ rank_offsets,
                                                             uint32_t* __restrict__ send_matrix,
                                                             unsigned long long* __restrict__ remote_pairs,
                                                             DispatchWs w) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  // [E][kWords] bitmaps | off[E+4] | pre[E] | send sums of this workgroup | remote (u64) | [E] map; all but the map zeroed
  const int Ep = (E + 3) / 4 * 4, DD = D * D;
  const int my_cols = DD % 4 == 0 ? (DD / 4 + NB - 1) / NB * 4 : (DD + NB - 1) / NB, colsp = (my_cols + 3) / 4 * 4;
  uint32_t* bm = reinterpret_cast<uint32_t*>(lds_raw);
  int32_t* off = reinterpret_cast<int32_t*>(bm + E * kWords);
  int32_t* pre = off + Ep + 4;
  uint32_t* send = reinterpret_cast<uint32_t*>(pre + Ep);
  unsigned long long* remote_sh = reinterpret_cast<unsigned long long*>(send + colsp);
  int32_t* map = reinterpret_cast<int32_t*>(send + colsp + 4);
  const int t = threadIdx.x, b = blockIdx.x;
  const int tok = token_at(T, b * kTokBlock + t, shf);
  const ColumnBatch first = column_sums_first(w.cnt, NB, E);
  load_phys_map(E, E / D, phys, map);
  zero_quads(bm, (E * kWords + Ep + 4 + Ep + colsp + 4) / 4);
  int e[KU], q[KU];
  load_id_row(ids + size_t(max(tok, 0)) * k, k, id_quads(ids, k), e);
  __syncthreads();
  const int c_lo = b * my_cols, c_n = max(0, min(my_cols, DD - c_lo));  // a last run that is cut short is whole quads too
  if (c_n > 0) {
    if (DD % 4 == 0) sum_some_columns<4>(w.send_part, NB, DD, c_lo, c_n, send);
    else sum_some_columns<1>(w.send_part, NB, DD, c_lo, c_n, send);
  }
  column_sums_before(w.cnt, NB, E, b, off, pre, &first);
  map_ids(e, tok >= 0, k, E, map, q);
  set_bits<KU, kWords>(q, bm);
  if (b == 0) {  // remote pairs: sum of the workgroups' counts
    unsigned long long part = 0;
    for (int bb = t; bb < NB; bb += kTokBlock) part += w.remote_part[bb];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) part += __shfl_xor(part, o);
    if ((t & 63) == 0 && part) atomicAdd(remote_sh, part);
  }
  __syncthreads();
  first_wave_exclusive_scan(off, E);
  for (int x = t; x < c_n; x += kTokBlock) send_matrix[c_lo + x] = send[x];
  __syncthreads();
  if (b == 0) {
    const int m = E / D;
    for (int x = t; x <= E; x += kTokBlock) {
      expert_offsets[x] = off[x];
      if (x % m == 0) rank_offsets[x / m] = off[x];
    }
    if (t == 0) *remote_pairs = *remote_sh;
  }
  if (tok < 0) return;
  int slot[KU];
#pragma unroll
  for (int j = 0; j < KU; ++j) {
    const int at = max(q[j], 0) & 0xffff;
    slot[j] = q[j] < 0 ? -1 : off[at] + pre[at] + bits_below<kWords>(bm + at * kWords, t);
  }
  store_slots(tok, k, slot, id_quads(slot_of_pair, k), slot_of_pair, pair_of_slot);
}

static size_t dp_count_lds(int E, int D) {
  return size_t(E) * kWords * 4 + size_t(cdiv(D * D * send_copies(D) + 1, 4)) * 16 + size_t(E) * 4;
}
static size_t dp_fused_lds(int E, int D, int NB) {
  const size_t Ep = align_up(E, 4), cols = align_up(size_t(cdiv(cdiv(D * D, 4), NB)) * 4, 4);
  return size_t(E) * kWords * 4 + (2 * Ep + 4 + cols + 4) * 4 + size_t(E) * 4;
}
constexpr int kFusedMaxNB = 512;  // beyond, every block reading the whole table costs more than the scan kernel

// One workgroup for everything, a thread a token (T <= BLK): one launch, no tables.  A small kernel's time is its chain of
// dependent loads and barriers: one pass over the tokens, four barriers.  The bits below a token's place: with 8 words a
// key (and with 32, for up to 4 pairs a token) they are counted in the bitmap, with 16 they come from a prefix over the words.
template <int KU, int BLK>
__global__ __launch_bounds__(BLK) void dp_small_kernel(int T, int k, int E, int D, const int32_t* __restrict__ ids,
                                                       const int32_t* __restrict__ token_rank,
                                                       const int32_t* __restrict__ shf,
                                                       const int32_t* __restrict__ phys,
                                                       int32_t* __restrict__ slot_of_pair,
                                                       int32_t* __restrict__ pair_of_slot,
                                                       int32_t* __restrict__ expert_offsets,
                                                       int32_t* __restrict__ rank_offsets,
                                                       uint32_t* __restrict__ send_matrix,
                                                       unsigned long long* __restrict__ remote_pairs) {
  constexpr int W = BLK / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  // [E][W] bitmaps | [D*D][copies] send counts + remote pairs, whole quads | off[E+4] | [E] map | [E][W] word prefix (u16)
  const int copies = send_copies(D), n_send = D * D * copies, send_quads = (n_send + 1 + 3) / 4;
  const int Ep = (E + 3) / 4 * 4;
  uint32_t* bm = reinterpret_cast<uint32_t*>(lds_raw);
  uint32_t* send = bm + E * W;
  int32_t* off = reinterpret_cast<int32_t*>(send + send_quads * 4);
  int32_t* map = off + Ep + 4;
  uint16_t* wpre = reinterpret_cast<uint16_t*>(map + E);
  const int t = threadIdx.x, m = E / D;
  const int tok = token_at(T, t, shf);
  load_phys_map(E, m, phys, map);
  zero_quads(bm, E * W / 4 + send_quads + Ep / 4 + 1);
  int e[KU], q[KU];
  int s = -1;
  if (T > 0) {  // a token that is not there reads token 0's row
    load_id_row(ids + size_t(max(tok, 0)) * k, k, id_quads(ids, k), e);
    s = token_rank[max(tok, 0)];
  } else {
#pragma unroll
    for (int j = 0; j < KU; ++j) e[j] = -1;
  }
  __syncthreads();
  map_ids(e, tok >= 0, k, E, map, q);
  set_bits<KU, W>(q, bm);
  int remote = count_send(D, tok >= 0 ? s : -1, q, send, copies);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) remote += __shfl_xor(remote, o);
  if ((t & 63) == 0 && remote) atomicAdd(&send[n_send], (uint32_t)remote);
  __syncthreads();
  if constexpr (W != 16) {
    for (int x = t; x < E; x += BLK) off[x] = bits_of<W>(bm + x * W);
  } else {  // a key's words are a row of 16 lanes
    const int w = t & 15;
    for (int key = t >> 4; key < Ep; key += BLK / 16) {  // four keys a wave: all or none of them below Ep
      const int c = key < E ? __popc(bm[key * W + w]) : 0;
      int incl = c;
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, false);
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, false);
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, false);
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, false);
      if (key < E) {
        wpre[key * W + w] = uint16_t(incl - c);
        if (w == W - 1) off[key] = incl;
      }
    }
  }
  for (int x = t; x < D * D; x += BLK) send_matrix[x] = send_total(send, x, copies);
  if (t == 0) *remote_pairs = send[n_send];
  __syncthreads();
  first_wave_exclusive_scan(off, E);
  __syncthreads();
  for (int x = t; x <= E; x += BLK) {
    expert_offsets[x] = off[x];
    if (x % m == 0) rank_offsets[x / m] = off[x];
  }
  if (tok < 0) return;
  int slot[KU];
#pragma unroll
  for (int j = 0; j < KU; ++j) {
    const int at = max(q[j], 0) & 0xffff;
    int below;
    if constexpr (W != 16) below = bits_below<W>(bm + at * W, t);
    else below = wpre[at * W + (t >> 5)] + __popc(bm[at * W + (t >> 5)] & ((1u << (t & 31)) - 1u));
    slot[j] = q[j] < 0 ? -1 : off[at] + below;
  }
  store_slots(tok, k, slot, id_quads(slot_of_pair, k), slot_of_pair, pair_of_slot);
}

static size_t dp_small_lds(int E, int D, int blk) {
  const size_t W = blk / 32, Ep = align_up(E, 4);
  return size_t(E) * W * 4 + size_t(cdiv(D * D * send_copies(D) + 1, 4)) * 16 + (Ep + 4) * 4 + size_t(E) * 4 +
         (blk == 512 ? size_t(E) * W * 2 : 0);
}

// D4: move rows.  One workgroup per token; each thread owns 16-byte chunks of the row.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

template <int K_UNROLL>
__global__ __launch_bounds__(512) void dp_rows_kernel(int k, int row_chunks, int P, const u32x4_t* __restrict__ X,
                                                      const int32_t* __restrict__ slot_of_pair,
                                                      u32x4_t* __restrict__ X_perm) {
  const int tok = blockIdx.x;
  const int32_t* sl = slot_of_pair + size_t(tok) * k;
  for (int c = threadIdx.x; c < row_chunks; c += blockDim.x) {
    const u32x4_t v = X[size_t(tok) * row_chunks + c];
    if constexpr (K_UNROLL > 0) {
#pragma unroll
      for (int j = 0; j < K_UNROLL; ++j) {
        const int s = sl[j];
        if ((unsigned)s < (unsigned)P) __builtin_nontemporal_store(v, &X_perm[size_t(s) * row_chunks + c]);
      }
    } else {
      for (int j = 0; j < k; ++j) {
        const int s = sl[j];
        if ((unsigned)s < (unsigned)P) __builtin_nontemporal_store(v, &X_perm[size_t(s) * row_chunks + c]);
      }
    }
  }
}

static bool carve_dispatch(const semmoe_config* cfg, void* ws, size_t bytes, DispatchWs* w) {
  const size_t NB = cdiv(cfg->T, kTokBlock);
  Carver c(ws, bytes);
  w->cnt = c.take<int32_t>(NB * cfg->E);
  w->send_part = c.take<uint32_t>(NB * cfg->D * cfg->D);
  w->remote_part = c.take<uint32_t>(NB);
  return c.ok;
}

size_t ws_dispatch(const semmoe_config* cfg) {
  const size_t NB = cdiv(cfg->T, kTokBlock);
  return align_up(NB * cfg->E * 4, 256) + align_up(NB * cfg->D * cfg->D * 4, 256) + align_up(NB * 4, 256) + 512;
}

}  // namespace semmoe

using namespace semmoe;

static int32_t dispatch_index_impl(const semmoe_config* cfg, hipStream_t s, const int32_t* topk_ids,
                                   const int32_t* token_rank, const int32_t* shf, const int32_t* phys_of_expert,
                                   int32_t* slot_of_pair, int32_t* pair_of_slot, int32_t* expert_offsets,
                                   int32_t* rank_offsets, uint32_t* send_matrix, uint64_t* remote_pairs, void* ws,
                                   size_t ws_bytes) {
  if (!topk_ids || !token_rank || !shf || !phys_of_expert || !slot_of_pair || !pair_of_slot || !expert_offsets ||
      !rank_offsets || !send_matrix || !remote_pairs)
    return SEMMOE_EINVAL;
  DispatchWs w;
  if (!carve_dispatch(cfg, ws, ws_bytes, &w)) return SEMMOE_EWORKSPACE;
  const int T = cfg->T, k = cfg->k, E = cfg->E, D = cfg->D;
  const int NB = cdiv(T, kTokBlock);
  const int path = tuning_value(SEMMOE_TUNE_INDEX_PATH);
  unsigned long long* remote = reinterpret_cast<unsigned long long*>(remote_pairs);
  return with_id_width(k, [&](auto ku) -> int32_t {  // KU: registers for a token's k experts
    constexpr int KU = decltype(ku)::value;
    if (index_small(cfg, path)) {
      const int form = T <= 256 ? 0 : (T <= 512 ? 1 : 2), blk = 256 << form;
      auto kern = form == 0 ? dp_small_kernel<KU, 256> : dp_small_kernel<KU, 512>;
      if constexpr (KU == 4)
        if (form == 2) kern = dp_small_kernel<KU, 1024>;
      const size_t lds = dp_small_lds(E, D, blk);
      static std::atomic<uint64_t> lds_allowed[3];  // one flag word per kernel, a bit per device
      const int32_t as = allow_max_dynamic_lds(&lds_allowed[form], reinterpret_cast<const void*>(kern));
      if (as != SEMMOE_OK) return as;
      hipLaunchKernelGGL(kern, dim3(1), dim3(blk), lds, s, T, k, E, D, topk_ids, token_rank, shf,
                         phys_of_expert, slot_of_pair, pair_of_slot, expert_offsets, rank_offsets, send_matrix, remote);
      SEMMOE_LAUNCH_CHECK();
      return SEMMOE_OK;
    }
    if (NB > 0) {
      hipLaunchKernelGGL(dp_count_kernel<KU>, dim3(NB), dim3(kTokBlock), dp_count_lds(E, D), s, T, k, E, D, topk_ids,
                         token_rank, shf, phys_of_expert, w);
      SEMMOE_LAUNCH_CHECK();
    }
    if (NB > 0 && ((path != 1 && NB <= kFusedMaxNB) || path == 3)) {
      hipLaunchKernelGGL(dp_fused_kernel<KU>, dim3(NB), dim3(kTokBlock), dp_fused_lds(E, D, NB), s, T, k, E, D, NB,
                         topk_ids, shf, phys_of_expert, slot_of_pair, pair_of_slot, expert_offsets, rank_offsets,
                         send_matrix, remote, w);
      SEMMOE_LAUNCH_CHECK();
      return SEMMOE_OK;
    }
    hipLaunchKernelGGL(dp_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, NB, E, D, expert_offsets, rank_offsets,
                       send_matrix, remote, w);
    SEMMOE_LAUNCH_CHECK();
    if (NB > 0) {
      hipLaunchKernelGGL(dp_slot_kernel<KU>, dim3(NB), dim3(kTokBlock), size_t(E) * (kWords + 1) * 4, s, T, k, E, D,
                         topk_ids, shf, phys_of_expert, slot_of_pair, pair_of_slot, expert_offsets, w);
    }
    SEMMOE_LAUNCH_CHECK();
    return SEMMOE_OK;
  });
}

static int32_t dispatch_rows_impl(const semmoe_config* cfg, hipStream_t s, const void* X,
                                  const int32_t* slot_of_pair, void* X_perm) {
  if (!X || !X_perm || !slot_of_pair || !aligned16(X) || !aligned16(X_perm)) return SEMMOE_EINVAL;
  const int T = cfg->T, k = cfg->k;
  if (T == 0) return SEMMOE_OK;
  const int row_chunks = int(size_t(cfg->d) * act_bytes(cfg) / 16);
  const u32x4_t* Xv = static_cast<const u32x4_t*>(X);
  u32x4_t* Xp = static_cast<u32x4_t*>(X_perm);
  const int P = T * k;
  // long rows: four waves, however many chunks the last pass leaves idle (rows of 896 chunks, 16384 tokens x 8: 435 us
  // with 448 threads, 424 with 256; up to 512 chunks no difference)
  const int threads = row_chunks > 512 ? 256 : row_walk_threads(row_chunks);
  switch (k) {
    case 1: hipLaunchKernelGGL(dp_rows_kernel<1>, dim3(T), dim3(threads), 0, s, k, row_chunks, P, Xv, slot_of_pair, Xp); break;
    case 2: hipLaunchKernelGGL(dp_rows_kernel<2>, dim3(T), dim3(threads), 0, s, k, row_chunks, P, Xv, slot_of_pair, Xp); break;
    case 4: hipLaunchKernelGGL(dp_rows_kernel<4>, dim3(T), dim3(threads), 0, s, k, row_chunks, P, Xv, slot_of_pair, Xp); break;
    case 8: hipLaunchKernelGGL(dp_rows_kernel<8>, dim3(T), dim3(threads), 0, s, k, row_chunks, P, Xv, slot_of_pair, Xp); break;
    default: hipLaunchKernelGGL(dp_rows_kernel<0>, dim3(T), dim3(threads), 0, s, k, row_chunks, P, Xv, slot_of_pair, Xp); break;
  }
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

extern "C" int32_t semmoe_dispatch_index(const semmoe_config* cfg, void* stream, const int32_t* topk_ids,
                                         const int32_t* token_rank, const int32_t* shf,
                                         const int32_t* phys_of_expert, int32_t* slot_of_pair, int32_t* pair_of_slot,
                                         int32_t* expert_offsets, int32_t* rank_offsets, uint32_t* send_matrix,
                                         uint64_t* remote_pairs, void* ws, size_t ws_bytes) {
  int32_t st = validate_config(cfg, true, false, false);
  if (st != SEMMOE_OK) return st;
  return dispatch_index_impl(cfg, static_cast<hipStream_t>(stream), topk_ids, token_rank, shf, phys_of_expert,
                             slot_of_pair, pair_of_slot, expert_offsets, rank_offsets, send_matrix, remote_pairs, ws,
                             ws_bytes);
}

extern "C" int32_t semmoe_dispatch_rows(const semmoe_config* cfg, void* stream, const void* X,
                                        const int32_t* slot_of_pair, void* X_perm) {
  int32_t st = validate_config(cfg, true, true, false);
  if (st != SEMMOE_OK) return st;
  return dispatch_rows_impl(cfg, static_cast<hipStream_t>(stream), X, slot_of_pair, X_perm);
}

extern "C" int32_t semmoe_dispatch(const semmoe_config* cfg, void* stream, const void* X, const int32_t* topk_ids,
                                   const int32_t* token_rank, const int32_t* shf, const int32_t* phys_of_expert,
                                   void* X_perm, int32_t* slot_of_pair, int32_t* pair_of_slot,
                                   int32_t* expert_offsets, int32_t* rank_offsets, uint32_t* send_matrix,
                                   uint64_t* remote_pairs, void* ws, size_t ws_bytes) {
  int32_t st = validate_config(cfg, true, X != nullptr, false);
  if (st != SEMMOE_OK) return st;
  if (X && (!X_perm || !aligned16(X) || !aligned16(X_perm))) return SEMMOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  st = dispatch_index_impl(cfg, s, topk_ids, token_rank, shf, phys_of_expert, slot_of_pair, pair_of_slot,
                           expert_offsets, rank_offsets, send_matrix, remote_pairs, ws, ws_bytes);
  if (st != SEMMOE_OK || !X) return st;
  return dispatch_rows_impl(cfg, s, X, slot_of_pair, X_perm);
}
