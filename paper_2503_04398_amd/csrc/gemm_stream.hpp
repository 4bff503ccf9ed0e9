// Grouped GEMM for few rows per group (and for fp32): every weight row streams through the chip once.
//
// What bounds it: with at most 64 token rows per tile a bf16 weight row costs more time in HBM than in the matrix
// cores, so the kernel is a read stream with MFMAs attached, and its speed is the bytes every compute unit keeps in
// flight.  Hence:
//   * a workgroup's NW waves (four; eight below) share one tile (16*TW weight rows x 16*TT tokens) and cut K between them, 128
//     bytes of every row at a time (wave w takes slices w, w+NW, ...): the workgroup reads NW * 128 consecutive bytes per row
//     and step, and no wave needs another's operands, so there is no barrier inside a tile and no wave ever waits for the
//     slowest line of a slice that all of them share;
//   * a load instruction covers 8 rows x 128 bytes (four neighbouring lanes in one 64-byte segment; loading MFMA
//     fragments directly puts them into four rows, and the address unit then passes 16 bytes a cycle instead of 64),
//     one step ahead into registers; waits are counted by the compiler per register;
//   * a step's registers go through a few KB of LDS that belong to the wave alone, to change from load layout to
//     fragment layout (16-byte chunks swizzled by the row: no bank conflicts);
//   * eight waves (bf16, one set of weights) where the tiles are so few that each compute unit gets one: then the waves of one
//     workgroup are all that is in flight;
//   * the load stream does not stop at a tile's end: the steps past it are the first ones of the workgroup's next
//     tile, so the epilogue (partial sums of the waves through LDS) runs under loads in flight.
// fp32 (v_mfma_f32_16x16x4_f32: full fp32 products and sums): a lane's 16 bytes are four k of its row, used by four
// MFMAs in turn - any order of k will do as long as both operands use the same one.
#pragma once
#include "gemm_core.hpp"
#include "gemm_w4.hpp"

namespace semmoe {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

template <int MODE, int TW, int TT, int NWAVES = 4>
struct StreamCfg {
  static constexpr int NW = NWAVES, kThreads = 64 * NW;
  static constexpr int BT = 16 * TT;
  static constexpr int FEAT = (MODE == kModeSwiglu) ? TW * 8 : TW * 16;
  static constexpr int kStgWave = (TW + TT) * 2048;  // one step of one wave
  static constexpr int kRedBytes = NW * TW * TT * 1024;
  static constexpr int kTileBytes = NW * kStgWave > kRedBytes ? NW * kStgWave : kRedBytes;  // the two share their place
  static size_t lds_bytes(int nq) { return size_t(kTileBytes) + (size_t(nq) * 4 + 1) * 4; }  // + tile prefix + group table
  static_assert(MODE != kModeSwiglu || TW % 2 == 0, "gate and up tiles in pairs");
};

// 16 bytes at uniform base + per-lane offset + uniform offset.  A buffer load and not a plain one: whether it passes by
// the caches (nt) is part of the instruction, and where one branch loads with and the other without it the compiler
// folds two plain loads into one and drops the hint.
template <bool NT>
__device__ __forceinline__ u32x4_t stream_load(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, int(voff), int(soff), NT ? 2 : 0));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const unsigned char* base) {
  // no bound of its own (offsets are clamped before the load); 32-bit offsets, raw addressing
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(scalar_ptr(base)), 0, -1, 0x00027000);
}

template <bool F32>
__device__ __forceinline__ f32x4_t stream_mfma(u32x4_t w, u32x4_t x, f32x4_t c) {
  if constexpr (F32) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[j]), __uint_as_float(x[j]), c, 0, 0, 0);
    return c;
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c,
                                                   0, 0, 0);
  }
}

// KTAIL: K is not a multiple of a slice (128 bytes of a row) or gives some wave no slice at all: addresses are clamped
// into the row and what lies behind its end counts as zero.  WIDE: rows so long, or so many, that 32-bit offsets from the
// panels' first rows do not reach them all (64-bit addresses per lane; with KTAIL only).
template <int MODE, bool F32, int TW, int TT, bool KTAIL, bool WIDE = false, bool SIZED = false, int NWAVES = 4>
__device__ __forceinline__ void gemm_stream_body(const GemmArgs& a, unsigned char* lds_raw, int skip = 0) {
  static_assert(KTAIL || !WIDE, "the wide form clamps every address");
  using C = StreamCfg<MODE, TW, TT, NWAVES>;
  constexpr int NW = C::NW;
  using off_t = std::conditional_t<WIDE, uint64_t, uint32_t>;
  constexpr int ES = F32 ? 4 : 2;          // bytes of an element
  f32x4_t* red = reinterpret_cast<f32x4_t*>(lds_raw);  // [wave][weight tile][token tile][lane]
  int* pre = reinterpret_cast<int*>(lds_raw + C::kTileBytes);
  int* gtab = pre + a.nq + 1;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;         // MFMA fragment: row l16, 16 bytes of k at g
  const int l_row = lane >> 3, l_chunk = lane & 7;  // load: row l_row of 8, 16 bytes at l_chunk of 128

  for (int q = tid; q < a.nq; q += C::kThreads) {
    gtab[3 * q] = a.offsets ? a.offsets[a.q_lo + q] : 0;
    gtab[3 * q + 1] = a.offsets ? a.offsets[a.q_lo + q + 1] : a.n_rows_single;
    gtab[3 * q + 2] = a.group_to_weight ? a.group_to_weight[a.q_lo + q] : a.q_lo + q;
  }
  const int n_ftiles = (a.N + C::FEAT - 1) / C::FEAT;
  const int total = __builtin_amdgcn_readfirstlane(build_tile_prefix<SIZED>(a, n_ftiles, pre, C::BT));  // ends with a barrier
  const ItemWalk my = xcd_share(total, true, skip);  // neighbours share a weight tile: token tile fastest
  int round = 0;
  if (my.count == 0) return;  // the whole workgroup leaves, before any further barrier

  struct Tile {
    int row_lo, n_tok, f0, widx;
    bool once;  // the group has one token tile: nobody else reads these weights
  };
  auto locate = [&](int t) __attribute__((always_inline)) {
    const int q = __builtin_amdgcn_readfirstlane(find_group(pre, a.nq, t));
    const int local = t - __builtin_amdgcn_readfirstlane(pre[q]);
    const int g_lo = __builtin_amdgcn_readfirstlane(gtab[3 * q]);
    const int row_hi = __builtin_amdgcn_readfirstlane(gtab[3 * q + 1]);
    const int n_tt = (row_hi - g_lo + C::BT - 1) / C::BT;
    const int ft = __builtin_amdgcn_readfirstlane(local / n_tt), tt = local - ft * n_tt;
    Tile r;
    r.row_lo = g_lo + tt * C::BT;
    r.n_tok = min(C::BT, row_hi - r.row_lo);
    r.f0 = ft * C::FEAT;
    r.widx = __builtin_amdgcn_readfirstlane(gtab[3 * q + 2]);
    r.once = n_tt == 1;
    return r;
  };

  // ---- load side: the tile whose slices are being requested, and the byte offset inside its rows.  An address is
  // uniform base + min(row offset of the lane, offset of the last row there is): rows outside the matrix are read
  // from its last row and never stored.
  const uint32_t row_bytes = uint32_t(a.K) * ES;  // below 2^32 (checked by the launcher)
  const int nst = int((row_bytes + 127ull) / 128);
  const int n = max(1, (nst - wave + NW - 1) / NW);  // slices of this wave per tile
  const off_t w_ld = off_t(a.ldw) * ES, x_ld = off_t(a.ldx) * ES;
  const uint32_t lane_k = KTAIL ? 0u : uint32_t(l_chunk * 16);
  const off_t w_lane = off_t(l_row) * w_ld + lane_k, w_last = off_t(a.N - 1) * w_ld + lane_k;
  const off_t x_lane = off_t(l_row) * x_ld + lane_k;
  const unsigned char *wbase, *xbase;
  off_t w_first = 0, x_last = 0;
  int l_round = 0, l_left = n, l_at = 0, l_ntt = 0, f_ntt = 0;  // l_at: which of the wave's slices is next
  bool l_once = true;
  uint32_t koff = 0;
  auto aim = [&](int t) __attribute__((always_inline)) {
    const Tile r = locate(t);
    wbase = static_cast<const unsigned char*>(a.W) + size_t(r.widx) * a.w_group_stride * ES;
    xbase = static_cast<const unsigned char*>(a.X) + size_t(r.row_lo) * a.ldx * ES;
    w_first = off_t(r.f0) * w_ld;
    x_last = off_t(r.n_tok - 1) * x_ld + lane_k;
    l_ntt = (r.n_tok + 15) >> 4;
    l_once = r.once;
    // where K is cut evenly (what a last, partial slice holds is masked by its place in the walk)
    l_at = KTAIL || nst % NW != 0 ? 0 : first_step(a, r.widx, ES, n);
    koff = wave * 128 + l_at * (NW * 128);
  };
  u32x4_t wb[2 * TW], xb[2 * TT];
  auto fetch = [&]() __attribute__((always_inline)) {
    const uint32_t at = KTAIL ? 0u : koff;
    const uint32_t lane_at = KTAIL ? uint32_t(min(koff + uint32_t(l_chunk) * 16, uint32_t(row_bytes - 16))) : 0u;
    const unsigned char* const ubase = wbase + size_t(a.N) * w_ld;
    if constexpr (WIDE) {
#pragma unroll
      for (int i = 0; i < 2 * TW; ++i) {
        const int wt = i >> 1;
        const int row = ((MODE == kModeSwiglu) ? (wt >> 1) * 16 : wt * 16) + (i & 1) * 8;
        wb[i] = *reinterpret_cast<const u32x4_t*>(((MODE == kModeSwiglu && (wt & 1)) ? ubase : wbase) +
                                                  (min(w_first + off_t(row) * w_ld + w_lane, w_last) + lane_at));
      }
#pragma unroll
      for (int j = 0; j < 2 * TT; ++j)
        if ((j >> 1) < l_ntt)
          xb[j] = *reinterpret_cast<const u32x4_t*>(xbase + (min(off_t(j * 8) * x_ld + x_lane, x_last) + lane_at));
    } else {
      const __amdgpu_buffer_rsrc_t wr = stream_rsrc(wbase), ur = stream_rsrc(ubase), xr = stream_rsrc(xbase);
      auto weights = [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2 * TW; ++i) {
          const int wt = i >> 1;  // gate and up tiles alternate
          const int row = ((MODE == kModeSwiglu) ? (wt >> 1) * 16 : wt * 16) + (i & 1) * 8;
          wb[i] = stream_load<decltype(nt)::value>((MODE == kModeSwiglu && (wt & 1)) ? ur : wr,
                                                   min(w_first + uint32_t(row) * w_ld + w_lane, w_last) + lane_at, at);
        }
      };
      // weights that no other tile reads pass by the caches (a plain read stream: 6.9 TB/s with nt, 6.4 without); those of
      // a group with several token tiles are read again by the neighbouring workgroup
      // (nor where slices straddle cache lines: a line's other half is another wave's)
      if (l_once && !KTAIL) weights(std::true_type{}); else weights(std::false_type{});
#pragma unroll
      for (int j = 0; j < 2 * TT; ++j)
        if ((j >> 1) < l_ntt) xb[j] = stream_load<false>(xr, min(uint32_t(j * 8) * x_ld + x_lane, x_last) + lane_at, at);
    }
    f_ntt = l_ntt;
    koff += NW * 128;
    if (++l_at == n) {
      l_at = 0;
      koff = wave * 128;
    }
    if (--l_left == 0) {
      l_left = n;
      if (l_round + 1 < my.count) ++l_round;  // past the last tile: its slices once more, which nobody uses
      aim(my.item(l_round));
    }
  };

  f32x4_t acc[TW][TT];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  };

  // accumulator of (weight tile, token tile): lane holds weight rows 4*(lane/16) + 0..3 for token lane%16
  auto finish = [&](int t) __attribute__((always_inline)) {
    const Tile r = locate(t);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // every wave is through with its staging area
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j) red[((wave * TW + i) * TT + j) * 64 + lane] = acc[i][j];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    auto total_of = [&](int i, int j) __attribute__((always_inline)) {
      f32x4_t v = red[(i * TT + j) * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += red[((w * TW + i) * TT + j) * 64 + lane];
      return v;
    };
    constexpr int FT = (MODE == kModeSwiglu) ? TW / 2 : TW;  // 16-feature tiles of the output
    for (int unit = wave; unit < FT * TT; unit += NW) {
      const int j = unit / FT, p = unit - j * FT;
      const int tok = j * 16 + l16, feat = r.f0 + p * 16 + g * 4;
      if (j * 16 >= r.n_tok) break;
      f32x4_t v;
      if constexpr (MODE == kModeSwiglu) {
        const f32x4_t gt = total_of(2 * p, j), up = total_of(2 * p + 1, j);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = F32 ? gt[e] / (1.0f + expf(-gt[e])) * up[e] : silu_mul(gt[e], up[e]);
      } else {
        v = total_of(p, j);
      }
      if (tok >= r.n_tok || feat >= a.N) continue;
      const size_t row = size_t(r.row_lo) + tok;
      if constexpr (MODE == kModeLogits) {  // N need not be a multiple of four
        const int cls = a.token_class ? a.token_class[row] : -1;
        const float* cb = (cls >= 0 && cls < a.n_classes && a.class_bias) ? a.class_bias + size_t(cls) * a.N : nullptr;
        float* o = static_cast<float*>(a.out) + row * size_t(a.N);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (feat + e < a.N) {
            float s = v[e];
            if (a.b_g) s += a.b_g[feat + e];
            if (cb) s += cb[feat + e];
            o[feat + e] = s;
          }
      } else if constexpr (F32) {
        *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out) + row * a.ldo + feat) = v;
      } else {
        *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.out) + row * a.ldo + feat) =
            make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // the sums have been read: their place is staging area again
  };

  // rows of 128 bytes; chunk c of row r lies at position c ^ (r/2 % 8)
  unsigned char* const stg = lds_raw + wave * C::kStgWave;
  const int swz = (l16 >> 1) & 7;
  unsigned char* const put0 = stg + l_row * 128 + ((l_chunk ^ ((l_row >> 1) & 7)) * 16);        // rows 0..7 of a tile
  unsigned char* const put1 = stg + l_row * 128 + ((l_chunk ^ (((l_row >> 1) + 4) & 7)) * 16);  // rows 8..15
  const unsigned char* const get = stg + l16 * 128;

  aim(my.item(0));
  fetch();
  clear();
  int slice = wave;  // of the tile being computed
  for (;;) {
    const bool in = !KTAIL || uint32_t(slice) * 128 + uint32_t(l_chunk) * 16 < row_bytes;
    const int ntt = f_ntt;
#pragma unroll
    for (int i = 0; i < 2 * TW; ++i)
      *reinterpret_cast<u32x4_t*>((i & 1 ? put1 : put0) + i * 1024) = in ? wb[i] : u32x4_t{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 2 * TT; ++j)
      if (j < 2 || (j >> 1) < ntt)  // a tile has at least one token
        *reinterpret_cast<u32x4_t*>((j & 1 ? put1 : put0) + (2 * TW + j) * 1024) = in ? xb[j] : u32x4_t{0, 0, 0, 0};
    __builtin_amdgcn_sched_barrier(0);
    fetch();  // every register of the step has been written down
    __builtin_amdgcn_sched_barrier(0);
    // the wave's own LDS operations complete in order: no wait between its writes and its reads
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4_t wf[TW];
      const unsigned char* from = get + ((h * 4 + g) ^ swz) * 16;
#pragma unroll
      for (int i = 0; i < TW; ++i) wf[i] = *reinterpret_cast<const u32x4_t*>(from + i * 2048);
#pragma unroll
      for (int j = 0; j < TT; ++j)
        if (j == 0 || j < ntt) {  // the first without a test: its MFMAs then wait for one fragment at a time
          const u32x4_t xf = *reinterpret_cast<const u32x4_t*>(from + (TW + j) * 2048);
#pragma unroll
          for (int i = 0; i < TW; ++i) acc[i][j] = stream_mfma<F32>(wf[i], xf, acc[i][j]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    slice += NW;
    if (slice >= nst) {  // also where this wave has no slice of its own (KTAIL): it has added zeros once
      finish(my.item(round));
      if (++round == my.count) break;
      slice = wave;
      clear();
    }
  }
}

template <int MODE, bool F32, int TW, int TT, bool KTAIL, bool WIDE = false, int NW = 4>
__global__ __launch_bounds__(64 * NW, 2) void gemm_stream_kernel(const GemmArgs a) {
  static_assert(NW == 4 || NW == 8, "two workgroups of four waves a compute unit, or one of eight: at least two waves a SIMD");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  gemm_stream_body<MODE, F32, TW, TT, KTAIL, WIDE, false, NW>(a, lds_raw);
}

// The rows of each group live on the device, and the mean the host expects can be far off: the ranks of an affinity
// placement, one hot expert.  So the groups of more than many.rows_min rows run as 128 x 64 tiles with the LDS ring, which
// reads a weight tile once for every 64 tokens at a better pace (8 experts of 316 rows each where the host expects 19:
// 809 us streamed, 435 so), and the others as above.  Few large tiles get workgroups of their own, at most half of the
// grid; else every workgroup takes its share of both.  The two write disjoint rows; only the workgroup's own LDS is
// waited for in between.
template <int MODE, int TW, int TT, bool KTAIL>
__global__ __launch_bounds__(256, 2) void gemm_stream_ring_kernel(const GemmArgs few, const GemmArgs many) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  // a launch without large groups does not build their list
  int* any = reinterpret_cast<int*>(lds_raw);
  if (threadIdx.x == 0) *any = 0;
  __syncthreads();
  for (int q = threadIdx.x; q < many.nq; q += 256)
    if (listed_rows<true>(many, q)) *any = 1;  // any number of threads write the same value
  __syncthreads();
  const bool some = __builtin_amdgcn_readfirstlane(*any) != 0;
  __syncthreads();
  int large = 0;
  if (some) {
    large = __builtin_amdgcn_readfirstlane(gemm_bf16_dma_body<MODE, 2, 2, 2, 1, 64, 3, true>(many, lds_raw));
    __syncthreads();
  }
  gemm_stream_body<MODE, false, TW, TT, KTAIL, false, true>(few, lds_raw, side_workgroups(large, int(gridDim.x)));
}

}  // namespace semmoe
