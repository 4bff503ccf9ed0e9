// Kernel instantiations and the host launcher of the grouped GEMM core.
#include "gemm_core.hpp"
#include "gemm_w4.hpp"
#include "gemm_stream.hpp"

namespace semmoe {

// Tuning knobs (semmoe_set_tuning): process-wide, read by every call from every thread; meant for tests and sweeps.
static std::atomic<int> g_tune[8] = {{-1}, {-1}, {-1}, {-1}, {-1}, {-1}, {-1}, {-1}};

// compute units / LDS limit of the current device (looked up once per device; 256 / 64 KB if the lookup fails)
static int num_cu() {
  DeviceInfo d;
  return device_info(&d) == SEMMOE_OK ? d.num_cu : 256;
}
static int max_lds() {
  DeviceInfo d;
  return device_info(&d) == SEMMOE_OK ? d.max_lds : 65536;
}

int tuning_value(int key) { return (key >= 0 && key < 8) ? g_tune[key].load(std::memory_order_relaxed) : -1; }

static int grid_for(long long tile_bound, long long cap) {
  if (tuning_value(SEMMOE_TUNE_GRID_CAP) > 0 && cap > tuning_value(SEMMOE_TUNE_GRID_CAP)) cap = tuning_value(SEMMOE_TUNE_GRID_CAP);
  tile_bound = (tile_bound + 7) / 8 * 8;  // whole rounds over the XCDs: the kernels split their list among these
  return (int)(tile_bound < cap ? tile_bound : cap);
}

template <int MODE, int NWF, int NWT, int TF, int TT, int BK, int MINW = 1>
static int32_t launch_bf16(const GemmArgs& a, int max_rows, int blocks_per_cu, hipStream_t stream) {
  using C = Bf16Cfg<MODE, NWF, NWT, TF, TT, BK>;
  const int n_ftiles = cdiv(a.N, C::FEAT);
  const long long bound = (long long)(max_rows / C::BT + a.nq) * n_ftiles;
  if (bound <= 0) return SEMMOE_OK;
  const int grid = grid_for(bound, (long long)num_cu() * blocks_per_cu);
  auto kern = gemm_bf16_kernel<MODE, NWF, NWT, TF, TT, BK, MINW>;
  if (C::kLdsBytes > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  if (C::kLdsBytes > 48 * 1024) {
    static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
    {
      const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
      if (as != SEMMOE_OK) return as;
    }
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), C::kLdsBytes, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

template <int MODE, int NWF, int NWT, int TF, int TT, int BK, int NSTAGE, int MINW = 1>
static int32_t launch_dma(const GemmArgs& a, int max_rows, int blocks_per_cu, hipStream_t stream) {
  using C = DmaCfg<MODE, NWF, NWT, TF, TT, BK, NSTAGE>;
  const int n_ftiles = cdiv(a.N, C::FEAT);
  const long long bound = (long long)(max_rows / C::BT + a.nq) * n_ftiles;
  if (bound <= 0) return SEMMOE_OK;
  const int grid = grid_for(bound, (long long)num_cu() * blocks_per_cu);
  auto kern = gemm_bf16_dma_kernel<MODE, NWF, NWT, TF, TT, BK, NSTAGE, MINW>;
  if (C::kLdsBytes > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  if (C::kLdsBytes > 48 * 1024) {
    static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
    {
      const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
      if (as != SEMMOE_OK) return as;
    }
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), C::kLdsBytes, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

// Four-wave 256 x 256 kernel; shapes it does not take are reported with SEMMOE_EUNSUPPORTED before any launch.
template <int MODE, int BK, int NSTAGE, int DMA_EVERY, int TJ = 4>
static int32_t launch_w4(const GemmArgs& a, int max_rows, hipStream_t stream) {
  using C = W4Cfg<MODE, BK, NSTAGE, DMA_EVERY, TJ>;
  const int w_rows = (MODE == kModeSwiglu) ? 2 * a.N : a.N;
  if (a.K % BK != 0 || a.K / BK < NSTAGE) return SEMMOE_EUNSUPPORTED;
  if ((unsigned long long)w_rows * a.ldw * 2 >= (1ull << 32) || (unsigned long long)C::BT * a.ldx * 2 >= (1ull << 32))
    return SEMMOE_EUNSUPPORTED;  // per-lane row offsets are 32-bit
  const size_t lds = TJ == 4 ? C::kLdsBytes : C::lds_bytes(a.nq);
  if (lds > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  const int n_ftiles = cdiv(a.N, C::FEAT);
  const long long bound = (long long)(max_rows / C::BT + a.nq) * n_ftiles;
  if (bound <= 0) return SEMMOE_OK;
  const int grid = grid_for(bound, num_cu());
  auto kern = gemm_bf16_w4_kernel<MODE, BK, NSTAGE, DMA_EVERY, TJ>;
  static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
  {
    const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
    if (as != SEMMOE_OK) return as;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), lds, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

// Tail launch of a head/tail split: the parent tiles (256 x 256) the head launch left over, cut into 128 x 64
// pieces (weight rows x tokens: 2 along the features, 4 along the tokens), two workgroups per CU with a ring of 3.
// A piece is a long, thin K loop with little arithmetic per slice: its speed is the bytes it keeps in flight over
// the latency of a load.  One workgroup per CU with a ring of 6 is faster when few parent tiles are left (config 2:
// 28 tiles, FFN 256 -> 246 us) and slower when many are (configs 3 and 4: +5 %); the count is only known on the device.
template <int MODE, int RING, int PER_CU>
static int32_t launch_tail_as(GemmArgs a, int max_rows, int head_grid, hipStream_t stream) {
  using C = DmaCfg<MODE, 2, 2, 2, 1, 64, RING>;
  constexpr int kSubT = 256 / C::BT, kSubF = 256 / C::BW;
  const int n_ftiles_p = cdiv(a.N, kSubF * C::FEAT);
  const long long bound_p = (long long)(max_rows / 256 + a.nq) * n_ftiles_p;  // parent tiles, at most
  const long long left_p = bound_p < head_grid ? bound_p : (long long)head_grid * a.sched_thr / 16;  // ... left over
  if (left_p <= 0) return SEMMOE_OK;
  a.sched_mode = 2;
  a.sched_g = head_grid;
  a.sched_sub_t = kSubT;
  a.sched_sub_f = kSubF;
  const int grid = grid_for(left_p * kSubT * kSubF, (long long)num_cu() * PER_CU);
  auto kern = gemm_bf16_dma_kernel<MODE, 2, 2, 2, 1, 64, RING, 1>;
  if (C::kLdsBytes > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
  {
    const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
    if (as != SEMMOE_OK) return as;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), C::kLdsBytes, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

// Tail launch with 128 x 128 pieces (four per parent tile), one workgroup per compute unit: the K loop of the
// four-wave kernel in small.  K must be a multiple of 64 with at least a ring of slices.
template <int MODE, int NSTAGE>
static int32_t launch_tail_pieces(GemmArgs a, int max_rows, int head_grid, hipStream_t stream) {
  using C = DmaCfg<MODE, 2, 2, 2, 2, 64, NSTAGE>;
  const int w_rows = (MODE == kModeSwiglu) ? 2 * a.N : a.N;
  if (a.K % 64 != 0 || a.K / 64 < NSTAGE) return SEMMOE_EUNSUPPORTED;
  if ((unsigned long long)w_rows * a.ldw * 2 >= (1ull << 32) || (unsigned long long)C::BT * a.ldx * 2 >= (1ull << 32))
    return SEMMOE_EUNSUPPORTED;  // per-lane row offsets are 32-bit
  if (C::kLdsBytes > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  constexpr int kSubT = 256 / C::BT, kSubF = 256 / C::BW;
  const int n_ftiles_p = cdiv(a.N, kSubF * C::FEAT);
  const long long bound_p = (long long)(max_rows / 256 + a.nq) * n_ftiles_p;  // parent tiles, at most
  const long long left_p = bound_p < head_grid ? bound_p : (long long)head_grid * a.sched_thr / 16;  // ... left over
  if (left_p <= 0) return SEMMOE_OK;
  a.sched_mode = 2;
  a.sched_g = head_grid;
  a.sched_sub_t = kSubT;
  a.sched_sub_f = kSubF;
  const int grid = grid_for(left_p * kSubT * kSubF, num_cu());
  auto kern = gemm_bf16_piece_kernel<MODE, NSTAGE>;
  static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
  {
    const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
    if (as != SEMMOE_OK) return as;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), C::kLdsBytes, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

// Every tile as 128 x 128 pieces with the loads placed between the MFMAs (the tail's piece kernel with nothing left
// to a head launch): for problems whose 256 x 256 tiles would leave most compute units idle, such as the shared
// expert on one rank's shard of tokens.
template <int MODE>
static int32_t launch_all_pieces(GemmArgs a, int max_rows, hipStream_t stream) {
  using C = DmaCfg<MODE, 2, 2, 2, 2, 64, 3>;
  const int w_rows = (MODE == kModeSwiglu) ? 2 * a.N : a.N;
  if (a.K % 64 != 0 || a.K / 64 < 3) return SEMMOE_EUNSUPPORTED;
  if ((unsigned long long)w_rows * a.ldw * 2 >= (1ull << 32) || (unsigned long long)C::BT * a.ldx * 2 >= (1ull << 32))
    return SEMMOE_EUNSUPPORTED;  // per-lane row offsets are 32-bit
  if (C::kLdsBytes > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  const long long bound_p = (long long)(max_rows / 256 + a.nq) * cdiv(a.N, 2 * C::FEAT);  // parent tiles, at most
  if (bound_p <= 0) return SEMMOE_OK;
  a.sched_mode = 2;
  a.sched_g = 1 << 24;  // no head launch: more workgroups than there can be tiles, so the cut falls at tile 0
  a.sched_thr = 16;
  a.sched_sub_t = 2;
  a.sched_sub_f = 2;
  a.sched_fine = 1;  // 128 x 64 pieces when the 128 x 128 ones would leave half the compute units idle
  const int grid = grid_for(bound_p * 8, num_cu());
  auto kern = gemm_bf16_piece_kernel<MODE, 3>;
  static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
  {
    const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
    if (as != SEMMOE_OK) return as;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), C::kLdsBytes, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

// Head (four-wave 256 x 256 tiles, K slices of 64, ring of 2) and tail (128 x 128 pieces, ring of 3) in one launch.
// SEMMOE_EUNSUPPORTED when either half does not take the shape: the caller then launches them one after the other.
template <int MODE, int NSTAGE = 2, int TJ = 4>
static int32_t launch_w4_split(const GemmArgs& h, int max_rows, hipStream_t stream) {
  using CH = W4Cfg<MODE, 64, NSTAGE, 2, TJ>;
  using CP = DmaCfg<MODE, 2, 2, 2, 2, 64, 3>;
  const int w_rows = (MODE == kModeSwiglu) ? 2 * h.N : h.N;
  if (h.K % 64 != 0 || h.K / 64 < 3) return SEMMOE_EUNSUPPORTED;
  if ((unsigned long long)w_rows * h.ldw * 2 >= (1ull << 32) || (unsigned long long)CH::BT * h.ldx * 2 >= (1ull << 32))
    return SEMMOE_EUNSUPPORTED;  // per-lane row offsets are 32-bit
  const size_t head_lds = TJ == 4 ? CH::kLdsBytes : CH::lds_bytes(h.nq);
  const size_t lds = head_lds > CP::kLdsBytes ? head_lds : CP::kLdsBytes;
  if (lds > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  const int n_ftiles = cdiv(h.N, CH::FEAT);
  const long long bound = (long long)(max_rows / CH::BT + h.nq) * n_ftiles;
  if (bound <= 0) return SEMMOE_OK;
  const int grid = grid_for(bound, num_cu());
  GemmArgs t = h;  // the tail's view of the same problem: the tiles the head's `grid` workgroups leave over, in pieces
  t.sched_mode = 2;
  t.sched_g = grid;
  t.sched_sub_t = CH::BT / CP::BT;
  t.sched_sub_f = CH::BW / CP::BW;
  t.sched_fine = tuning_value(SEMMOE_TUNE_TAIL_RING) == 2 ? 0 : 1;
  auto kern = gemm_bf16_w4_split_kernel<MODE, 64, NSTAGE, 2, 3, TJ>;
  static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
  {
    const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
    if (as != SEMMOE_OK) return as;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, stream, h, t);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

template <int MODE>
static int32_t launch_tail(const GemmArgs& a, int max_rows, int head_grid, hipStream_t stream) {
  const int ring = tuning_value(SEMMOE_TUNE_TAIL_RING);
  if (ring == 6) return launch_tail_as<MODE, 6, 1>(a, max_rows, head_grid, stream);
  if (ring == 3) return launch_tail_as<MODE, 3, 2>(a, max_rows, head_grid, stream);
  // 128 x 128 pieces as a launch of their own (the default runs them inside the head's launch: launch_w4_split)
  const int32_t st = launch_tail_pieces<MODE, 3>(a, max_rows, head_grid, stream);  // a ring of 4 gains nothing
  if (st != SEMMOE_EUNSUPPORTED) return st;
  return launch_tail_as<MODE, 3, 2>(a, max_rows, head_grid, stream);
}

// grid of a launch with 256 x 256 tiles and one workgroup per compute unit (the head launch of a split)
static int big_tile_grid(const GemmArgs& a, int max_rows, int feat) {
  const long long bound = (long long)(max_rows / 256 + a.nq) * cdiv(a.N, feat);
  return grid_for(bound, num_cu());
}

template <int MODE, bool F32, int TW, int TT, bool KTAIL, bool WIDE, int NW = 4>
static int32_t launch_stream_as(const GemmArgs& a, int max_rows, int per_cu, hipStream_t stream) {
  using C = StreamCfg<MODE, TW, TT, NW>;
  const long long bound = (long long)(max_rows / C::BT + a.nq) * cdiv(a.N, C::FEAT);
  if (bound <= 0) return SEMMOE_OK;
  const size_t lds = C::lds_bytes(a.nq);
  const int grid = grid_for(bound, (long long)num_cu() * per_cu);
  auto kern = gemm_stream_kernel<MODE, F32, TW, TT, KTAIL, WIDE, NW>;
  if (lds > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  if (lds > 48 * 1024) {
    static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
    const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
    if (as != SEMMOE_OK) return as;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::kThreads), lds, stream, a);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

// SEMMOE_EUNSUPPORTED where 32-bit offsets do not reach every row: fp32 then takes the wide form, bf16 another tile
template <int MODE, bool F32, int TW, int TT, int NW = 4>
static int32_t launch_stream(const GemmArgs& a, int max_rows, int per_cu, hipStream_t stream) {
  const unsigned long long es = F32 ? 4 : 2, row_bytes = a.K * es;
  const unsigned long long w_rows = (MODE == kModeSwiglu) ? 2ull * a.N : a.N, x_rows = StreamCfg<MODE, TW, TT>::BT;
  if (w_rows * a.ldw * es >= (1ull << 31) || x_rows * a.ldx * es >= (1ull << 31)) return SEMMOE_EUNSUPPORTED;
  if (row_bytes % 128 == 0 && row_bytes >= 128 * NW)
    return launch_stream_as<MODE, F32, TW, TT, false, false, NW>(a, max_rows, per_cu, stream);
  return launch_stream_as<MODE, F32, TW, TT, true, false, NW>(a, max_rows, per_cu, stream);
}

// Groups of up to `few_rows` rows streamed, the others as 128 x 64 tiles, in one launch
template <int MODE, int TW, int TT, bool KTAIL>
static int32_t launch_stream_ring_as(const GemmArgs& a, int max_rows, int few_rows, int per_cu, hipStream_t stream) {
  using CS = StreamCfg<MODE, TW, TT>;
  using CD = DmaCfg<MODE, 2, 2, 2, 1, 64, 3>;
  const long long bound_s = (long long)(max_rows / CS::BT + a.nq) * cdiv(a.N, CS::FEAT);
  const long long bound_d = (long long)(max_rows / CD::BT + a.nq) * cdiv(a.N, CD::FEAT);
  // room for workgroups that keep to the large tiles (at most half of the grid) beside those that keep to the others
  const long long bound = bound_s + (max_rows > few_rows ? 2 * bound_d : 0);
  if (bound <= 0) return SEMMOE_OK;
  const size_t lds = CS::lds_bytes(a.nq) > CD::kLdsBytes ? CS::lds_bytes(a.nq) : CD::kLdsBytes;
  if (lds > size_t(max_lds())) return SEMMOE_EUNSUPPORTED;
  const int grid = grid_for(bound, (long long)num_cu() * per_cu);
  auto kern = gemm_stream_ring_kernel<MODE, TW, TT, KTAIL>;
  static std::atomic<uint64_t> lds_allowed{0};  // one flag word per instantiation, a bit per device
  const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
  if (as != SEMMOE_OK) return as;
  GemmArgs few = a, many = a;
  few.rows_max = few_rows;
  many.rows_min = few_rows;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, stream, few, many);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

template <int MODE, int TW, int TT>
static int32_t launch_stream_ring(const GemmArgs& a, int max_rows, int few_rows, int per_cu, hipStream_t stream) {
  const unsigned long long row_bytes = a.K * 2ull, w_rows = (MODE == kModeSwiglu) ? 2ull * a.N : a.N;
  if (w_rows * a.ldw * 2 >= (1ull << 31) || StreamCfg<MODE, TW, TT>::BT * 2ull * a.ldx >= (1ull << 31))
    return SEMMOE_EUNSUPPORTED;  // 32-bit offsets do not reach every row
  if (row_bytes % 128 == 0 && row_bytes >= 512) return launch_stream_ring_as<MODE, TW, TT, false>(a, max_rows, few_rows, per_cu, stream);
  return launch_stream_ring_as<MODE, TW, TT, true>(a, max_rows, few_rows, per_cu, stream);
}

// Workgroups per compute unit: a tile's walk over K is a few steps (K 512: four a wave) with a sum over the waves behind them, and
// only other workgroups fill the time between.  As many as the registers (2 x 4: three, 4 x 4: two) and the LDS hold, and no more: the
// shares of the persistent workgroups are fixed, one that starts late ends late.
template <int MODE, int TW, int TT>
static int f32_per_cu(int nq) {
  const int fit = max_lds() / int(StreamCfg<MODE, TW, TT>::lds_bytes(nq)), most = TT == 4 ? (TW == 2 ? 3 : 2) : 4;
  return fit < most ? (fit < 1 ? 1 : fit) : most;
}

// fp32: 32 weight rows x 32 tokens with four workgroups a compute unit, 16 tokens where the mean is no more or the tiles are
// few; 64 x 64 with two a compute unit (half the operand bytes a product) where there are so many tiles that the last
// round does not matter.  From how many a compute unit on, by rows and K (of the time as smaller tiles; 1600 FFNs of 2 to 256 experts,
// 3 to 400 rows each, skewed by 0 to 1.0):
//   * more than 32 rows, K of 3600 and more: 4 (4 to 6: gate/up 0.93 to 0.95, down 0.98; 2 to 4: level with single shapes at 1.2)
//   * more than 8 rows, K of 1024 and more: 6 (6 to 8: 9 to 32 rows 0.97 to 1.00, more rows 0.90 to 0.98; 4 to 6: 0.98 to 1.03)
//   * more than 48 rows, shorter K: 12 (0.96 from there on, 6 to 12: 0.99 to 1.07); 9 to 48 rows 8, where one tile a group along the
//     tokens reads the weights once (128 experts of 37 rows, d 1000, F 504: 288 against 259 us; skewed by 0.8, 1.07 with 8 to 10)
//   * 4 to 8 rows: 8 from K 1024 on (8 to 12: 0.99), 16 below (level; 8 to 16: 1.01 to 1.02).  The mean says nothing about a hot
//     expert (512 experts, d = F = 512, mean 11, nearly all rows on one: 212 us on 16 tokens a tile, 140 so)
//   * one set of weights, whose last tile alone is ragged, more than 32 rows: 3.5 (d 3064, F 1504: 1200 tokens 321 against 361 us, 600
//     tokens 170 each; d 904, F 1792: 600 tokens 91 against 78)
// With a line at 12 for all of K below 4096 the calls of more than 32 rows were 0.995 of the time with two workgroups a compute unit and
// tiles that followed the mean alone, a third of them more than 3 % behind.
// Against plain FMAs on 64 x 64 tiles that share every slice: 0.41 of the time over 834 random shapes; behind by 10 to 36 %
// only where a row is two slices (K up to 96) and 128 experts or more make the sum over the waves the most of the work
// (leaving the waves without a slice out of that sum changed nothing).
// id: a shape by its tuning id; others are for bf16 and leave the choice here.
template <int MODE>
static int32_t launch_f32(int id, const GemmArgs& a, int max_rows, int est_rows_per_group, hipStream_t stream) {
  const bool rows_reachable = (unsigned long long)a.K * 4 < (1ull << 32) - 1024;  // a row below 4 GB
  switch (id) {
    case 30: return launch_stream<MODE, true, 2, 2>(a, max_rows, f32_per_cu<MODE, 2, 2>(a.nq), stream);
    case 31: return launch_stream<MODE, true, 2, 4>(a, max_rows, f32_per_cu<MODE, 2, 4>(a.nq), stream);
    case 32: return launch_stream<MODE, true, 4, 4>(a, max_rows, 2, stream);
    case 36: return launch_stream<MODE, true, 2, 1>(a, max_rows, f32_per_cu<MODE, 2, 1>(a.nq), stream);
    case 37: return rows_reachable ? launch_stream_as<MODE, true, 2, 1, true, true>(a, max_rows, f32_per_cu<MODE, 2, 1>(a.nq), stream) : SEMMOE_EUNSUPPORTED;
    default: break;
  }
  const int est = est_rows_per_group < 1 ? 1 : est_rows_per_group;
  auto items = [&](int tw, int tt) {
    return (long long)a.nq * cdiv(est, 16 * tt) * cdiv(a.N, (MODE == kModeSwiglu) ? 8 * tw : 16 * tw);
  };
  const long long cus = num_cu();
  int32_t st;
  const bool deep = a.K >= 1024;
  // 64 x 64 tiles from so many half tiles a compute unit on
  const int line = !a.offsets && est > 32      ? 7
                   : est > 32 && a.K >= 3600   ? 8
                   : est > 48                  ? (deep ? 12 : 24)
                   : est > 8                   ? (deep ? 12 : 16)
                                               : (deep ? 16 : 32);
  if (est >= 4 && items(4, 4) * 2 >= line * cus)
    st = launch_stream<MODE, true, 4, 4>(a, max_rows, 2, stream);
  else if (est > 16 && items(2, 2) >= 2 * cus)
    st = launch_stream<MODE, true, 2, 2>(a, max_rows, f32_per_cu<MODE, 2, 2>(a.nq), stream);
  else
    st = launch_stream<MODE, true, 2, 1>(a, max_rows, f32_per_cu<MODE, 2, 1>(a.nq), stream);
  if (st != SEMMOE_EUNSUPPORTED) return st;
  if (!rows_reachable) return SEMMOE_EUNSUPPORTED;
  return launch_stream_as<MODE, true, 2, 1, true, true>(a, max_rows, f32_per_cu<MODE, 2, 1>(a.nq), stream);
}

// left-over share of a round (in sixteenths) up to which the split happens
static int split_threshold() {
  const int t = tuning_value(SEMMOE_TUNE_HEAD_TAIL);
  return (t >= 1 && t <= 16) ? t : 8;
}

// 256 weight rows x 128 tokens, ring of 3, left-over tiles as pieces in the same launch
template <int MODE>
static int32_t launch_w4_128(const GemmArgs& a, int max_rows, hipStream_t stream) {
  if (tuning_value(SEMMOE_TUNE_HEAD_TAIL) == 0) return launch_w4<MODE, 64, 3, 2, 2>(a, max_rows, stream);  // no pieces
  GemmArgs h = a;
  h.sched_mode = 1;
  h.sched_thr = split_threshold();
  return launch_w4_split<MODE, 3, 2>(h, max_rows, stream);
}

// tile shapes: id -> (waves along weight rows, waves along tokens, MFMA tiles per wave, K slice)
template <int MODE>
static int32_t launch_bf16_tile(int id, const GemmArgs& a, int max_rows, int bpc, hipStream_t s) {
  switch (id) {
    case 0: return launch_bf16<MODE, 2, 2, 2, 2, 64>(a, max_rows, bpc > 0 ? bpc : 2, s);  // 128 x 128, 4 waves
    case 3: return launch_bf16<MODE, 2, 4, 4, 2, 64>(a, max_rows, bpc > 0 ? bpc : 1, s);  // 256 x 256, 8 waves
    case 4: return launch_bf16<MODE, 4, 2, 2, 4, 64>(a, max_rows, bpc > 0 ? bpc : 1, s);  // 256 x 256, 8 waves
    case 6: return launch_bf16<MODE, 2, 4, 2, 2, 64>(a, max_rows, bpc > 0 ? bpc : 1, s);  // 128 x 256, 8 waves
    case 11: return launch_dma<MODE, 2, 4, 4, 2, 32, 4>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 256 x 256, 8 waves
    case 12: return launch_dma<MODE, 4, 2, 2, 4, 32, 4>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 256 x 256, 8 waves
    case 14: return launch_dma<MODE, 2, 4, 2, 2, 32, 4>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 128 x 256, 8 waves
    case 15: return launch_dma<MODE, 2, 4, 4, 2, 32, 3>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 256 x 256, ring of 3
    case 16: return launch_dma<MODE, 2, 4, 4, 2, 64, 2>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 256 x 256, K 64 x 2
    case 17: return launch_bf16<MODE, 4, 1, 2, 1, 64>(a, max_rows, bpc > 0 ? bpc : 2, s);       // 256 x 32 (decode)
    case 18: return launch_bf16<MODE, 4, 1, 2, 2, 64>(a, max_rows, bpc > 0 ? bpc : 2, s);       // 256 x 64
    case 19: return launch_dma<MODE, 4, 1, 2, 1, 64, 4>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 256 x 32, ring of 4 (decode)
    case 25: return launch_dma<MODE, 4, 1, 2, 2, 64, 3>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 256 x 64, ring of 3
    case 26: return launch_dma<MODE, 2, 2, 2, 1, 64, 3>(a, max_rows, bpc > 0 ? bpc : 2, s);     // 128 x 64, ring of 3, two per CU
    case 27: return launch_dma<MODE, 2, 2, 2, 1, 64, 4>(a, max_rows, bpc > 0 ? bpc : 1, s);     // 128 x 64, ring of 4
    // weights streamed through registers: 16 x TW weight rows, 16 x TT tokens
    case 30: case 31: case 32: {
      const int32_t st = id == 30   ? launch_stream<MODE, false, 2, 2>(a, max_rows, bpc > 0 ? bpc : 2, s)
                         : id == 31 ? launch_stream<MODE, false, 2, 4>(a, max_rows, bpc > 0 ? bpc : 2, s)
                                    : launch_stream<MODE, false, 4, 4>(a, max_rows, bpc > 0 ? bpc : 2, s);
      if (st != SEMMOE_EUNSUPPORTED) return st;
      return launch_bf16_tile<MODE>(26, a, max_rows, 0, s);  // panels beyond 32-bit offsets
    }
    // ... with eight waves a workgroup, one workgroup a compute unit
    case 38: case 39: case 40: {
      const int32_t st = id == 38   ? launch_stream<MODE, false, 2, 2, 8>(a, max_rows, bpc > 0 ? bpc : 1, s)
                         : id == 39 ? launch_stream<MODE, false, 4, 2, 8>(a, max_rows, bpc > 0 ? bpc : 1, s)
                                    : launch_stream<MODE, false, 4, 4, 8>(a, max_rows, bpc > 0 ? bpc : 1, s);
      if (st != SEMMOE_EUNSUPPORTED) return st;
      return launch_bf16_tile<MODE>(26, a, max_rows, 0, s);
    }
    // streamed up to so many rows per group that the ring of case 26 reads the weights less often
    case 34: case 35: {
      const int32_t st = id == 34 ? launch_stream_ring<MODE, 2, 4>(a, max_rows, 64, bpc > 0 ? bpc : 2, s)
                                  : launch_stream_ring<MODE, 4, 4>(a, max_rows, 64, bpc > 0 ? bpc : 2, s);
      if (st != SEMMOE_EUNSUPPORTED) return st;
      return launch_bf16_tile<MODE>(26, a, max_rows, 0, s);
    }
    case 33: {  // four waves, 256 x 128
      const int32_t st = launch_w4_128<MODE>(a, max_rows, s);
      if (st != SEMMOE_EUNSUPPORTED) return st;
      return launch_bf16_tile<MODE>(26, a, max_rows, 0, s);  // K not a multiple of 64 or short, or too many groups
    }
    case 28: {  // 128 x 128 pieces, loads between the MFMAs
      const int32_t st = launch_all_pieces<MODE>(a, max_rows, s);
      if (st != SEMMOE_EUNSUPPORTED) return st;
      return launch_bf16<MODE, 2, 2, 2, 2, 64>(a, max_rows, bpc > 0 ? bpc : 2, s);  // K not a multiple of 64, or short
    }
    default: break;
  }
  if (id >= 20 && id <= 22) {  // four waves, 256 x 256, loads interleaved with the MFMAs
    int32_t st;
    switch (id) {
      case 20: st = launch_w4<MODE, 32, 4, 4>(a, max_rows, s); break;  // K slices of 32, ring of 4, a load every 4th MFMA
      case 21: st = launch_w4<MODE, 32, 4, 2>(a, max_rows, s); break;  // ... every 2nd MFMA
      default: st = launch_w4<MODE, 64, 2, 2>(a, max_rows, s); break;  // K slices of 64, ring of 2 (the fastest measured)
    }
    if (st != SEMMOE_EUNSUPPORTED) return st;
    return launch_bf16_tile<MODE>(16, a, max_rows, bpc, s);  // K not a multiple of the slice, or too short
  }
  return SEMMOE_EINVAL;
}

// Default tile shape from the mean rows per group that the caller expects (the true, ragged row counts live on the
// device), the depth K and the number of tiles.  Whole FFNs (gate/up + down) on cold weights, us; group sizes spread
// lognormally by 0.3:
//   A: 128 experts, d 2048, F 768;  B: 16 experts, d 4096, F 1536;  C: 8 experts, d 7168, F 2048
//          streamed alone             streamed up to 64 rows        128 x 64 (26)    256 x 128 (33)   256 x 256 (22)
//   rows   32 x 32 (30) 64 x 64 (32)  32 x 64 (34) 64 x 64 (35)
//   8      199 103 120  210 111 121   210 105 122  212 112 122      241 126 133
//   16     218 107 123  218 112 131   228 111 125  220 114 132      243 128 134      258 133 163
//   32     295 135 165  242 116 137   272 124 142  244 118 138      248 132 136      265 135 170
//   48                  285 146 170                286 143 162      263 139 179      275 139 177      309 168 232
//   64                  326 165 183                318 173 181      288 162 187      285 142 186      318 172 238
//   110                                                             370 190 234      308 158 202      341 179 251
//   160                                                             453 227 257      367 192 217      376 198 256
//   300                                                                              517 264 300      534 299 322
//   400                                                                              630 311 355      656 339 344
// (as 128 x 128 tiles (0): 379 204 298 at 110 rows; as pieces (28): 946 414 435 at 400).  30 and 32 have no answer to a
// hot expert, so what runs is 34 or 35: groups beyond 64 rows take the 128 x 64 tiles in the same launch, which costs
// 1 to 5 % where there is none.  34 against 35: 105 122 to 112 122 us at 8 rows; at 16 rows 34 is still ahead on B and C
// (111 125 to 114 132) and 35 on A (220 to 228), at 32 rows 35 throughout.
// The mean is that of all experts: it is the launch's own only where the launch has all of them, a rank that an affinity
// placement loads may have several times as many rows.  So the lines lie lower for one rank's experts (16 experts,
// d 4096, F 1536, 93 rows each where 23 are expected: 190 us, streamed 205; d 2048, F 768, 1040 rows where 260 are
// expected: 203 us as 256 x 256 tiles, 208 as 256 x 128).
// K and the number of tiles, over 6000 random shapes (d, F 64 to 7168, 2 to 512 experts; a product's gain or loss as a
// share of its FFN, against the 128 x 64 tiles):
//   * a streamed tile ends with a sum over four waves, which a short K does not repay, least of all with many tiles:
//     up to 9 rows, 32 x 64: K below 192 +88 % beyond 2048 tiles, +24 % at 256 to 512, +3 % up to 64; K 384 to 639 +14,
//     +3, -14 %; K 1400 to 2100 -4, -5, -27 %.  Few tiles wait for one walk over K, which the four waves share: the line
//     lies at K 192 up to a tile per four compute units (-6 % above it), 384 up to one per two, 960 beyond.  64 x 64 has
//     half the sums: from K 640 on where there are more than two tiles a compute unit (K 640 to 959: -4 % where 32 x 64
//     has +5).  10 to 19 rows, 64 x 64: -2 to -8 % from K 960, with few tiles from 640; where the 128 x 64 tiles just
//     have a compute unit each from K 2560 (-1 to -3 %; up to 1408 +3 to +6 %).  20 to 39 rows: from K 1408 on, not with a
//     compute unit each (+1 to +10 %), and up to fewer tiles the more rows it drags along: K 1408 to 2099 20 to 24 rows -3 % up
//     to 2048 tiles, +1 % beyond, 25 to 29 rows level up to 1024, +1 % beyond, 30 to 39 rows -2 % up to 512, +4 % beyond.
//   * K 2048 and 4096: rows a power of two apart, where one slice of the 128 x 64 tile, 128 bytes of each of 192 rows, falls on
//     few memory channels; a streamed step reads 512 consecutive bytes of a row.  With a common start of all walks 64 x 64 was ahead
//     at any number of tiles (10 to 19 rows 4 to 20 %, 20 to 39 rows 2 to 13 %); with the starts spread over the groups it
//     still is 3 to 11 % at 10 to 24 rows; from 34 on, next point.
//   * 256 x 128 tiles need work for every compute unit: 40 to 95 rows, fewer than 96 of them +10 to +20 %, half of the
//     compute units +1 % at K 1000 and -3 % from K 1400, all of them +6 % below K 384 and 0 to -7 % from 640, two rounds -7 %.
//     One rank's launch counts the tiles of three times the mean: a loaded rank has that many, and if it has not the loss is
//     smaller than the gain (5995 random shapes with half to eight times the mean on the rank; 40 to 95 rows expected and 8 times
//     as many there: 5 % over counting the mean's, even loads: 1 % behind it).
//     From 20 rows expected on one rank's launch takes them where, one per group along the tokens, they are one round of five
//     eighths of the compute units or more, K 2560 and above (K 2880, 180 of them: 0.95 of 128 x 64 with the rows it expects, 0.88
//     with twice as many, 1.01 at worst; K 4096, 192: 0.98, 0.85 and 1.01).  Half the compute units (K 7168): 4 % behind with the rows
//     it expects, 17 ahead with twice as many; beyond one round 3 to 12 % behind (K 1408 to 2880, 250 to 360 tiles).  A launch
//     with all experts from 34 rows (128 experts of 39 rows, d 2048: 262 -> 240 us, 64 of d 4096, F 1536: 453 -> 438; at 30 rows 4 %
//     behind 64 x 64 streamed, at 32 level) and as many tiles as K asks for.  Of the 128 x 64 tiles' time, with one to two a compute
//     unit, two to four, more: K 1024 to 1407 1.04 to 1.09, 1.00 to 1.06, 0.95 to 0.99; K from 1408 on 1.01 to 1.03, 0.98 to 1.02,
//     0.98 to 0.99; K 4096 0.95 to 1.01 from one on.  Where it is not taken K 4096, and K 2048 with a tile a compute unit or
//     more, keep 64 x 64 streamed: 0.94 and 0.96 of the 128 x 64 tiles.
//     384 experts and more leave no room in its LDS for their table (512 experts, d 1024, F 512, 300 rows: 776 us as
//     256 x 256 tiles, 1134 as 128 x 64).
// Rows that are no whole 128 bytes: neighbouring slices share cache lines, and from about ten rows on the staged tiles
// read them at the better rate (10 rows of d 2832: 191 against 208).
// One set of weights (the shared expert) on few rows has so few tiles that a compute unit gets one, and its speed is what
// the waves of that one keep in flight: eight waves a workgroup, each an eighth of K, and the smallest tile that still
// leaves one a compute unit (38: 32 x 32, 39: 64 x 32, 40: 64 x 64; each step halves or so the operand bytes that all
// tiles draw from L2, 15 TB/s of which is what they then wait for).  Four waves -> eight, FFN in us: C 16 rows 37 -> 28, 64
// rows 42 -> 35; 64 x 64 against 32 x 32 with four waves: C 256 rows 68 -> 54, B 300 rows 48 -> 36, against 128 x 64 pieces A 300
// rows 29 -> 21, d 4096, F 256, 512 rows 39 -> 20.  Sixteen waves have fewer registers each than the loads need (C 16 rows
// 33); K below 1024 is three steps a wave or less (d 640, F 384: 11.0 with four waves, 12.4 with eight).  Beyond
// one tile a compute unit: up to 128 rows four waves on 32 x 32, two workgroups a compute unit; else 128 x 128 pieces as long as
// they are one round (C, down, 640 rows: 140 tiles of 256 x 128 are 8 % ahead of two rounds of pieces; B, 1024 rows: 128
// tiles 15 % behind one); 64 x 64 with four waves where K is 4096 or a larger power of two, whose weight rows all start on the same memory
// channels (one set has no starts to spread), and there are twice as many weight rows as tokens (B, gate/up, 640 rows: 63 us with pieces,
// 53 so; K 12288, rows 24 KB apart, was not measured and keeps the pieces).  188 shapes (d, F 256 to 20000, 1 to 2048 rows): 0.83 of the time before.  2000 rows of
// it: 45 83 179 as 256 x 128 tiles, 66 112 236 as 256 x 256, 37 105 234 as pieces.  256 x 256 tiles are ahead of 256 x 128
// from three fifths of the compute units on (170 to 190 of them: 2 to 4 %; 130 to 150: 2 % behind); 2514 rows of d 6968,
// F 1312, gate/up without whole slices: 248 us for the FFN with pieces, 331 with 256 x 256 tiles on less than half of the chip.
static int default_tile(const GemmArgs& a, int max_rows, int est_rows_per_group, int w_rows) {
  const int est = est_rows_per_group, t256 = cdiv(w_rows, 256);
  const long long cus = num_cu();
  const bool whole_slices = a.K % 64 == 0 && a.K / 64 >= 3;  // what the tiles with a running load stream need
  const int big_tile = (long long)(max_rows / 256 + a.nq) * t256 * 2 >= cus ? 22 : 28;
  if (!a.offsets) {
    auto tiles = [&](int w, int t) { return (long long)cdiv(w_rows, w) * cdiv(est, t); };
    if (tiles(32, 32) <= cus) return a.K >= 1024 ? 38 : 30;
    if (tiles(64, 32) <= cus) return 39;
    if (tiles(64, 64) <= cus) return 40;
    if (tiles(64, 64) <= 2 * cus && a.K >= 4096 && (a.K & (a.K - 1)) == 0 && w_rows >= 2 * est) return 32;
    if (est <= 128 && t256 * 4 < 3 * cus) return 30;
    if (tiles(256, 128) * 2 <= cus) return est <= 256 && !whole_slices ? 31 : 28;
    if (!whole_slices) return est < 96 ? 26 : (est < 192 ? 0 : big_tile);
    return est < 384 || (long long)cdiv(est, 256) * t256 * 5 < 3 * cus ? 33 : 22;
  }
  const bool all_rows = (long long)a.nq * (est + 1) >= max_rows;
  const long long ring = (long long)a.nq * cdiv(w_rows, 128);  // 128 x 64 tiles, one per group along the tokens
  if (est < 10) {
    if (ring * 2 <= cus) return a.K >= (ring * 4 <= cus ? 192 : 384) ? 34 : 26;
    if (ring > 2 * cus && a.K < 1536) return a.K >= 640 ? 35 : 26;
    return a.K >= 960 ? 34 : 26;
  }
  const bool w4_room = W4Cfg<kModeStore, 64, 3, 2, 2>::lds_bytes(a.nq) <= size_t(max_lds());
  if (est < 40) {
    const long long mid = (long long)a.nq * w_rows / 256;  // 256 x 128 tiles, one per group along the tokens
    const bool pow2 = a.K >= 2048 && (a.K & (a.K - 1)) == 0;
    const int full = a.K < 1408 ? 4 : (pow2 && a.K >= 4096 ? 1 : 2);  // tiles a compute unit
    if (whole_slices && w4_room && (all_rows ? est >= 34 && a.K >= 1024 && mid >= full * cus
                                             : est >= 20 && mid * 8 >= 5 * cus && mid <= cus && a.K >= 2560))
      return 33;
    if (!whole_slices || (est >= 20 && !all_rows)) return 26;
    if (pow2 && (est < 34 || a.K >= 4096 || mid >= cus)) return 35;
    const bool one_each = ring * 2 > cus && ring <= cus;
    if (est < 20) return a.K >= (ring * 2 <= cus ? 640 : (one_each ? 2560 : 960)) ? 35 : 26;
    return a.K >= 1408 && !one_each && ring <= (est < 25 ? 8 : est < 30 ? 4 : 2) * cus ? 35 : 26;
  }
  if (whole_slices && est < 384 && w4_room) {
    // 256 x 128 tiles, as full ones
    const long long mid = (long long)a.nq * w_rows * cdiv(all_rows ? est : 3 * est, 128) / 256;
    if (est < 192) return mid * 2 >= 3 * cus || (mid >= cus && a.K >= 640) || (mid * 2 >= cus && a.K >= 1408) ? 33 : 26;
    if (all_rows && a.K >= 640 && mid * 2 >= cus) return 33;
  }
  if (est < 192) return est < 96 ? 26 : 0;
  return big_tile;
}

// Head/tail split: for the tile shapes of 256 x 256 with a persistent grid of one workgroup per compute unit.
static bool split_launch(int id) {
  const bool big = id == 16 || (id >= 20 && id <= 22);
  const int t = tuning_value(SEMMOE_TUNE_HEAD_TAIL);
  return big && t != 0;
}

int32_t launch_ksplit_gemm(const void* X, const void* W, int T, int N, int d, int n_parts, float* partial,
                           hipStream_t stream) {
  if (T <= 0 || N <= 0 || n_parts < 1 || n_parts > 64 || N % 4 != 0) return SEMMOE_EUNSUPPORTED;
  if (d % (64 * n_parts) != 0 || (long long)T * n_parts > 0x3fffffffLL) return SEMMOE_EUNSUPPORTED;
  GemmArgs a{};
  a.X = X; a.ldx = d;
  a.W = W; a.ldw = d; a.w_group_stride = size_t(d / n_parts);
  a.N = N; a.K = d / n_parts;
  a.offsets = nullptr; a.q_lo = 0; a.nq = n_parts; a.n_rows_single = T;
  a.group_to_weight = nullptr;
  a.out = partial; a.ldo = N;
  a.ksplit_rows = T;
  return launch_w4<kModeLogits, 64, 2, 2>(a, T * n_parts, stream);
}

int32_t launch_gemm(int mode, int dtype, const GemmArgs& a, int max_rows, int est_rows_per_group,
                    hipStream_t stream) {
  if (a.nq <= 0 || max_rows <= 0) return SEMMOE_OK;
  if (a.nq > 512) return SEMMOE_EUNSUPPORTED;
  if (dtype == SEMMOE_BF16) {
    const int bpc = tuning_value(SEMMOE_TUNE_BLOCKS_PER_CU);
    switch (mode) {
      case kModeLogits: return launch_bf16<kModeLogits, 2, 2, 2, 1, 64>(a, max_rows, 2, stream);  // 128 experts x 64 tokens
      case kModeSwiglu: {
        const int id = tuning_value(SEMMOE_TUNE_GATEUP_TILE) >= 0
                           ? tuning_value(SEMMOE_TUNE_GATEUP_TILE)
                           : default_tile(a, max_rows, est_rows_per_group, 2 * a.N);
        if (!split_launch(id)) return launch_bf16_tile<kModeSwiglu>(id, a, max_rows, bpc, stream);
        GemmArgs h = a;
        h.sched_mode = 1;
        h.sched_thr = split_threshold();
        if (id == 22 && (tuning_value(SEMMOE_TUNE_TAIL_RING) < 0 || tuning_value(SEMMOE_TUNE_TAIL_RING) == 2)) {  // both halves in one launch
          const int32_t sm = launch_w4_split<kModeSwiglu>(h, max_rows, stream);
          if (sm != SEMMOE_EUNSUPPORTED) return sm;
        }
        const int32_t st = launch_bf16_tile<kModeSwiglu>(id, h, max_rows, 1, stream);
        if (st != SEMMOE_OK) return st;
        return launch_tail<kModeSwiglu>(h, max_rows, big_tile_grid(a, max_rows, 128), stream);
      }
      default: {
        const int id = tuning_value(SEMMOE_TUNE_DOWN_TILE) >= 0
                           ? tuning_value(SEMMOE_TUNE_DOWN_TILE)
                           : default_tile(a, max_rows, est_rows_per_group, a.N);
        if (!split_launch(id)) return launch_bf16_tile<kModeStore>(id, a, max_rows, bpc, stream);
        GemmArgs h = a;
        h.sched_mode = 1;
        h.sched_thr = split_threshold();
        if (id == 22 && (tuning_value(SEMMOE_TUNE_TAIL_RING) < 0 || tuning_value(SEMMOE_TUNE_TAIL_RING) == 2)) {
          const int32_t sm = launch_w4_split<kModeStore>(h, max_rows, stream);
          if (sm != SEMMOE_EUNSUPPORTED) return sm;
        }
        const int32_t st = launch_bf16_tile<kModeStore>(id, h, max_rows, 1, stream);
        if (st != SEMMOE_OK) return st;
        return launch_tail<kModeStore>(h, max_rows, big_tile_grid(a, max_rows, 256), stream);
      }
    }
  }
  const int gate_id = tuning_value(SEMMOE_TUNE_GATEUP_TILE), down_id = tuning_value(SEMMOE_TUNE_DOWN_TILE);
  switch (mode) {
    case kModeLogits: return launch_f32<kModeLogits>(gate_id, a, max_rows, est_rows_per_group, stream);
    case kModeSwiglu: return launch_f32<kModeSwiglu>(gate_id, a, max_rows, est_rows_per_group, stream);
    default: return launch_f32<kModeStore>(down_id, a, max_rows, est_rows_per_group, stream);
  }
}

}  // namespace semmoe

extern "C" int32_t semmoe_set_tuning(int32_t key, int32_t value) {
  if (key < 0 || key >= 8) return SEMMOE_EINVAL;
  semmoe::g_tune[key].store(value, std::memory_order_relaxed);
  return SEMMOE_OK;
}

extern "C" int32_t semmoe_get_tuning(int32_t key, int32_t* value_out) {
  if (key < 0 || key >= 8 || !value_out) return SEMMOE_EINVAL;
  *value_out = semmoe::tuning_value(key);
  return SEMMOE_OK;
}
