// route: router GEMM (grouped-GEMM core, logits epilogue) + wavefront-level top-k selection.
// Gating function of Sec. 3.2: G(h) = top-k(softmax(W_g h + b_g)); the group-limited sigmoid router is
// the variant the DeepSeek-V3-shaped workload names.
#include "gemm_core.hpp"

namespace semmoe {

// Sigmoid as a fixed sequence of individually rounded fp32 operations (no contraction), so that any
// implementation of the same sequence gives the same bits.  Plain operators: the pragma does not reach into __fmul_rn and
// __fadd_rn, inline functions that are compiled with contraction, and a product and a sum of theirs became one FMA (one value
// in 80 was off by an ulp or two).
__device__ __forceinline__ float sigmoid_exact_seq(float x) {
#pragma clang fp contract(off)
  x = fminf(fmaxf(x, -30.0f), 30.0f);
  const float t = -x * 1.4426950408889634f;
  const float n = rintf(t);
  const float f = t - n;
  float p = 0.00015403530393381608f;
  p = p * f + 0.0013333558146428443f;
  p = p * f + 0.009618129107628477f;
  p = p * f + 0.05550410866482158f;
  p = p * f + 0.2402265069591007f;
  p = p * f + 0.6931471805599453f;
  p = p * f + 1.0f;
  const float q = 1.0f + ldexpf(p, static_cast<int>(n));
  // 1 / q rounded to nearest: the hardware's reciprocal and two Newton steps with fused residuals, five instructions where the
  // division takes a dozen.  q lies in [1, 2^44), where nothing underflows and the steps scale exactly, so every q of one binade
  // stands for all.  An error of 1 ulp in the first value would not do (from 0.5 for q = 2 - 2^-23 the steps end at 0.5): it is
  // gfx950's values for which the result is that of the division, q by q.
  float r = __builtin_amdgcn_rcpf(q);
  r = __builtin_fmaf(__builtin_fmaf(-q, r, 1.0f), r, r);
  return __builtin_fmaf(__builtin_fmaf(-q, r, 1.0f), r, r);
}

// ---- wave-wide reductions through DPP row shifts / broadcasts (no LDS permutes) ---------------------------
// After the four row_shr steps lane 15 of every 16-lane row holds the row's result; row_bcast:15 folds row r
// into row r+1, row_bcast:31 folds rows 0-1 into rows 2-3; lane 63 then holds the result of the wave.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f32(float old, float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

// Selection scores are compared as integers: key(x) orders like x (and -0 like +0), integer max needs no NaN
// canonicalisation, and the row-shift folds into the max instruction.  key is its own inverse.
__device__ __forceinline__ int to_key(float x) {
  const int b = __float_as_int(x + 0.0f);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float from_key(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i32(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, 0xf, false);
}

// One instruction per step: v_max_i32 with the row shift / broadcast applied to its first source.  Lanes
// whose shifted source does not exist are disabled by the DPP rules and keep their value.  The two wait states
// that a DPP read needs after a vector-ALU write of the same register are written out (s_nop 1).
#define SEMMOE_DPP_MAX(ctrl) \
  asm volatile("s_nop 1\n\tv_max_i32_dpp %0, %0, %0 " ctrl " row_mask:0xf bank_mask:0xf" : "+v"(v))
__device__ __forceinline__ int wave_max_key(int v) {
  SEMMOE_DPP_MAX("row_shr:1");
  SEMMOE_DPP_MAX("row_shr:2");
  SEMMOE_DPP_MAX("row_shr:4");
  SEMMOE_DPP_MAX("row_shr:8");
  SEMMOE_DPP_MAX("row_bcast:15");
  SEMMOE_DPP_MAX("row_bcast:31");
  asm volatile("s_nop 1" ::: "memory");
  return __builtin_amdgcn_readlane(v, 63);
}
#undef SEMMOE_DPP_MAX

__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f32<0x111, 0xf>(0.0f, v);
  v += dpp_f32<0x112, 0xf>(0.0f, v);
  v += dpp_f32<0x114, 0xf>(0.0f, v);
  v += dpp_f32<0x118, 0xf>(0.0f, v);
  v += dpp_f32<0x142, 0xa>(0.0f, v);  // rows 1 and 3 take the sum of the row before
  v += dpp_f32<0x143, 0xc>(0.0f, v);  // rows 2 and 3 take the sum of rows 0-1
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

constexpr int kNoExpert = 0x7fffffff;

// Selection for NT tokens by one wavefront, the NT dependent chains of wave-wide reductions interleaved in one
// instruction stream (a single chain leaves the vector ALU idle most of the time).  rows[t] points at token t's
// E fp32 logits (global or LDS), nullptr = no token.  Lane l holds experts l, l+64, l+128, ...
template <int NC, int NT>
__device__ __forceinline__ void select_rows(const semmoe_config& cfg, const float* const (&rows)[NT],
                                            const float* __restrict__ sel_bias, int lane,
                                            int32_t* const (&ids_out)[NT], float* const (&w_out)[NT]) {
  const int E = cfg.E, k = cfg.k;
  const float NEG = -__builtin_inff();
  const int NEGK = to_key(NEG);

  int val[NT][NC];    // key of the selection score (logit, or s' in sigmoid mode)
  float aux[NT][NC];  // softmax: logit; sigmoid: s
  uint32_t live[NT];  // bit c: entry c may still be selected
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    live[t] = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int e = lane + 64 * c;
      val[t][c] = NEGK;
      aux[t][c] = 0.0f;
      if (e < E && rows[t]) {
        const float x = rows[t][e];
        if (cfg.score == SEMMOE_SIGMOID) {
          const float sg = sigmoid_exact_seq(x);
          aux[t][c] = sg;
          val[t][c] = to_key(__fadd_rn(sg, sel_bias ? sel_bias[e] : 0.0f));
        } else {
          aux[t][c] = x;
          val[t][c] = to_key(x);
        }
        live[t] |= 1u << c;
      }
    }
  }

  // arg-max over the entries whose bit is set in mask[t]: largest value, equal values -> lowest expert id.
  // Expert id = lane + 64*c, so among equal values the lowest slot c wins, then the lowest lane.
  // No entry at all: kNoExpert and -inf.
  auto wave_argmax = [&](const uint32_t(&mask)[NT], int(&vmax)[NT], int(&arg)[NT]) {
    int m[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      m[t] = NEGK;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if ((mask[t] >> c) & 1u) m[t] = max(m[t], val[t][c]);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) vmax[t] = wave_max_key(m[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      int e = kNoExpert;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const unsigned long long hit = __ballot(((mask[t] >> c) & 1u) && val[t][c] == vmax[t]);
        if (e == kNoExpert && hit != 0ull) e = (__ffsll((long long)hit) - 1) + 64 * c;
      }
      arg[t] = e;
    }
  };

  if (cfg.score == SEMMOE_SIGMOID && cfg.n_group > 1) {
    // group score = sum of the group's two largest s'; keep the topk_group best groups
    const int gs = E / cfg.n_group;
    int my_gscore[NT];  // lane g holds the key of the score of group g
#pragma unroll
    for (int t = 0; t < NT; ++t) my_gscore[t] = NEGK;
    for (int g = 0; g < cfg.n_group; ++g) {
      uint32_t in_g[NT];
      uint32_t base = 0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int e = lane + 64 * c;
        if (e < E && e / gs == g) base |= 1u << c;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) in_g[t] = base & live[t];
      int v1[NT], v2[NT];
      int e1[NT], e2[NT];
      wave_argmax(in_g, v1, e1);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (e1[t] != kNoExpert && (e1[t] & 63) == lane) in_g[t] &= ~(1u << (e1[t] >> 6));
      wave_argmax(in_g, v2, e2);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float sc = (e2[t] == kNoExpert) ? from_key(v1[t]) : __fadd_rn(from_key(v1[t]), from_key(v2[t]));
        if (lane == g) my_gscore[t] = to_key(sc);
      }
    }
    // the topk_group best groups: lanes hold one group score each (slot 0 only)
    unsigned long long keep[NT];
    bool taken[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      keep[t] = 0;
      taken[t] = false;
    }
    for (int r = 0; r < cfg.topk_group; ++r) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bool cand = lane < cfg.n_group && !taken[t];
        const int wm = wave_max_key(cand ? my_gscore[t] : NEGK);
        const unsigned long long hit = __ballot(cand && my_gscore[t] == wm);
        const int g = __ffsll((long long)hit) - 1;
        keep[t] |= 1ull << g;
        if (lane == g) taken[t] = true;
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      uint32_t allowed = 0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int e = lane + 64 * c;
        if (e < E && ((keep[t] >> (e / gs)) & 1ull)) allowed |= 1u << c;
      }
      live[t] &= allowed;
    }
  }

  // k rounds of wave-wide arg-max; lane j keeps the j-th winner
  int my_id[NT];
  float my_val[NT];  // softmax: winning logit; sigmoid: s of the winner
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    my_id[t] = 0;
    my_val[t] = 0.0f;
  }
  for (int j = 0; j < k; ++j) {
    int vm[NT];
    int e[NT];
    wave_argmax(live, vm, e);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int owner = e[t] & 63, slot = e[t] >> 6;
      float a = 0.0f;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c == slot) a = aux[t][c];
      a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), owner));
      if (lane == owner) live[t] &= ~(1u << slot);
      if (lane == j) {
        my_id[t] = e[t];
        my_val[t] = a;
      }
    }
  }

#pragma unroll
  for (int t = 0; t < NT; ++t) {
    float w;
    if (cfg.score == SEMMOE_SOFTMAX) {
      const float mx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_val[t]), 0));  // first winner = row max
      float part = 0.0f;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (lane + 64 * c < E) part += expf(aux[t][c] - mx);
      const float denom = wave_sum(part);
      w = (lane < k) ? expf(my_val[t] - mx) / denom : 0.0f;
      if (cfg.renorm) w = w / wave_sum(w);
    } else {
      w = (lane < k) ? my_val[t] : 0.0f;
      if (cfg.renorm) w = w / wave_sum(w);
      w *= cfg.routed_scale;
    }
    if (lane < k && rows[t]) {
      ids_out[t][lane] = my_id[t];
      w_out[t][lane] = w;
    }
  }
}

// NC = experts per lane, chosen from E so that the unrolled loops carry no dead slots
template <int NT>
__device__ __forceinline__ void select_rows_any(const semmoe_config& cfg, const float* const (&rows)[NT],
                                                const float* __restrict__ sel_bias, int lane,
                                                int32_t* const (&ids_out)[NT], float* const (&w_out)[NT]) {
  if (cfg.E <= 64) select_rows<1, NT>(cfg, rows, sel_bias, lane, ids_out, w_out);
  else if (cfg.E <= 128) select_rows<2, NT>(cfg, rows, sel_bias, lane, ids_out, w_out);
  else if (cfg.E <= 256) select_rows<4, NT>(cfg, rows, sel_bias, lane, ids_out, w_out);
  else select_rows<8, NT>(cfg, rows, sel_bias, lane, ids_out, w_out);
}

// ---- selection with one token per 16-lane row ---------------------------------------------------------------
// A wave-wide arg-max spends 64 lanes and a scalar round trip (readlane, ballot, find-first) on one token's
// few experts per lane.  Here a token lives in one DPP row of 16 lanes (expert id = slot*16 + lane-in-row), so one
// instruction stream serves four tokens, and a reduction is four row-local steps (xor 1 and xor 2 inside a quad,
// then the two mirrors) after which every lane of the row holds the result: no broadcast, no scalar registers.
// NCH independent groups of four tokens are interleaved to fill the dependent-issue gaps.
#define SEMMOE_ROW_STEP(op, ctrl, x) \
  asm volatile("s_nop 1\n\t" op " %0, %0, %0 " ctrl " row_mask:0xf bank_mask:0xf" : "+v"(x))
#define SEMMOE_ROW_REDUCE(op, arr)                                                               \
  do {                                                                                           \
    _Pragma("unroll") for (int c_ = 0; c_ < NCH; ++c_) SEMMOE_ROW_STEP(op, "quad_perm:[1,0,3,2]", arr[c_]); \
    _Pragma("unroll") for (int c_ = 0; c_ < NCH; ++c_) SEMMOE_ROW_STEP(op, "quad_perm:[2,3,0,1]", arr[c_]); \
    _Pragma("unroll") for (int c_ = 0; c_ < NCH; ++c_) SEMMOE_ROW_STEP(op, "row_half_mirror", arr[c_]);     \
    _Pragma("unroll") for (int c_ = 0; c_ < NCH; ++c_) SEMMOE_ROW_STEP(op, "row_mirror", arr[c_]);          \
  } while (0)

// ---- the largest k of a row ------------------------------------------------------------------------------------
// Every lane sorts its own entries, then lanes merge their lists with those of other lanes, four levels, until all 16 hold
// the row's KEEP largest in order: no round per winner and no search for the slot that holds it.  An entry is one 64-bit
// word, the order-preserving key above, the expert below (the lower id is the larger word), laid out as a positive finite
// double, so that a comparator is v_max_f64 and v_min_f64: two instructions for key and id together.  8 of 128 experts for
// four tokens: about 280 instructions, where 8 rounds of arg-max took 860.
__device__ __forceinline__ double pack_entry(int key, int id) {
  const uint32_t u = uint32_t(key) ^ 0x80000000u;
  return __hiloint2double(int(u >> 2), int((u << 30) | uint32_t(255 - id)));
}
__device__ __forceinline__ int entry_key(double v) {
  return int(((uint32_t(__double2hiint(v)) << 2) | (uint32_t(__double2loint(v)) >> 30)) ^ 0x80000000u);
}
__device__ __forceinline__ int entry_id(double v) { return 255 - (__double2loint(v) & 255); }

// inline assembly: the library's fmax / fmin canonicalise every operand whose bits came from elsewhere
__device__ __forceinline__ double max64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double min64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int N>
__device__ __forceinline__ void order_pair(double (&v)[N], int i, int j) {  // the larger one to i
  const double a = v[i], b = v[j];
  v[i] = max64(a, b);
  v[j] = min64(a, b);
}

// Batcher's odd-even merge sort of v[LO .. LO + LEN - 1], largest first
template <int LO, int LEN, int R, int N>
__device__ __forceinline__ void odd_even_merge(double (&v)[N]) {
  if constexpr (2 * R < LEN) {
    odd_even_merge<LO, LEN, 2 * R>(v);
    odd_even_merge<LO + R, LEN, 2 * R>(v);
#pragma unroll
    for (int i = LO + R; i + R < LO + LEN; i += 2 * R) order_pair(v, i, i + R);
  } else {
    order_pair(v, LO, LO + R);
  }
}
template <int LO, int LEN, int N>
__device__ __forceinline__ void sort_entries(double (&v)[N]) {
  if constexpr (LEN > 1) {
    sort_entries<LO, LEN / 2>(v);
    sort_entries<LO + LEN / 2, LEN / 2>(v);
    odd_even_merge<LO, LEN, 1>(v);
  }
}
// v[0 .. LEN - 1] first falls and then rises (or the other way round): into falling order
template <int LEN, int N>
__device__ __forceinline__ void order_bitonic(double (&v)[N]) {
#pragma unroll
  for (int half = LEN / 2; half > 0; half /= 2)
#pragma unroll
    for (int i = 0; i < LEN; ++i)
      if ((i & half) == 0) order_pair(v, i, i + half);
}

// the entries v[0 .. M - 1] of another lane of the row.  The two wait states that a DPP read needs after a vector-ALU write of
// its source are written out once for the block.
enum : int { kXor1 = 0, kXor2 = 1, kHalfMirror = 2, kMirror = 3 };
#define SEMMOE_MOVE2(ctrl)                                                                                             \
  asm("s_nop 1\n\tv_mov_b32_dpp %0, %4 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %1, %5 " ctrl                \
      " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %2, %6 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %3, %7 " \
      ctrl " row_mask:0xf bank_mask:0xf"                                                                               \
      : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3])                                                             \
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]))
#define SEMMOE_MOVE4(ctrl)                                                                                             \
  asm("s_nop 1\n\tv_mov_b32_dpp %0, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %1, %9 " ctrl                \
      " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %2, %10 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %3, %11 " \
      ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %4, %12 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %5, %13 " \
      ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %6, %14 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_mov_b32_dpp %7, %15 " \
      ctrl " row_mask:0xf bank_mask:0xf"                                                                               \
      : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7])         \
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]))
template <int STEP, int M, int N>
__device__ __forceinline__ void entries_of_partner(const double (&v)[N], double (&b)[M]) {
  constexpr int G = M >= 4 ? 4 : 2;  // entries per block; a single one is moved twice
#pragma unroll
  for (int g = 0; g < M; g += G) {
    int x[2 * G], o[2 * G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const double e = v[M == 1 ? 0 : g + i];
      x[2 * i] = __double2loint(e);
      x[2 * i + 1] = __double2hiint(e);
    }
    if constexpr (G == 4) {
      if constexpr (STEP == kXor1) SEMMOE_MOVE4("quad_perm:[1,0,3,2]");
      else if constexpr (STEP == kXor2) SEMMOE_MOVE4("quad_perm:[2,3,0,1]");
      else if constexpr (STEP == kHalfMirror) SEMMOE_MOVE4("row_half_mirror");
      else SEMMOE_MOVE4("row_mirror");
    } else {
      if constexpr (STEP == kXor1) SEMMOE_MOVE2("quad_perm:[1,0,3,2]");
      else if constexpr (STEP == kXor2) SEMMOE_MOVE2("quad_perm:[2,3,0,1]");
      else if constexpr (STEP == kHalfMirror) SEMMOE_MOVE2("row_half_mirror");
      else SEMMOE_MOVE2("row_mirror");
    }
#pragma unroll
    for (int i = 0; i < G; ++i)
      if (g + i < M) b[g + i] = __hiloint2double(o[2 * i + 1], o[2 * i]);
  }
}
#undef SEMMOE_MOVE2
#undef SEMMOE_MOVE4

// v[0 .. M - 1], in order, becomes the merger with the partner's list: twice as long while that is at most KEEP, else the
// KEEP largest.  Both lanes of a pair end with the same list.
template <int STEP, int M, int KEEP>
__device__ __forceinline__ void merge_with_partner(double (&v)[KEEP]) {
  double b[M];
  entries_of_partner<STEP, M>(v, b);
  if constexpr (2 * M <= KEEP) {
#pragma unroll
    for (int i = 0; i < M; ++i) v[M + i] = b[M - 1 - i];
    order_bitonic<2 * M>(v);
  } else {
#pragma unroll
    for (int i = 0; i < M; ++i) v[i] = max64(v[i], b[M - 1 - i]);
    order_bitonic<M>(v);
  }
}

// a lane's NS entries -> the row's KEEP largest, in order, in every lane
template <int NS, int KEEP>
__device__ __forceinline__ void largest_of_row(const double (&all)[NS], double (&v)[KEEP]) {
  constexpr int M0 = NS < KEEP ? NS : KEEP;
  double u[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) u[i] = all[i];
  sort_entries<0, M0>(u);
#pragma unroll
  for (int i = 0; i < M0; ++i) v[i] = u[i];
  if constexpr (NS > KEEP) {  // the lane's further runs of KEEP entries
#pragma unroll
    for (int r = KEEP; r < NS; r += KEEP) {
      double w[KEEP];
#pragma unroll
      for (int i = 0; i < KEEP; ++i) w[i] = u[r + i];
      sort_entries<0, KEEP>(w);
#pragma unroll
      for (int i = 0; i < KEEP; ++i) v[i] = max64(v[i], w[KEEP - 1 - i]);
      order_bitonic<KEEP>(v);
    }
  }
  constexpr int M1 = 2 * M0 <= KEEP ? 2 * M0 : KEEP, M2 = 2 * M1 <= KEEP ? 2 * M1 : KEEP, M3 = 2 * M2 <= KEEP ? 2 * M2 : KEEP;
  merge_with_partner<kXor1, M0>(v);
  merge_with_partner<kXor2, M1>(v);
  merge_with_partner<kHalfMirror, M2>(v);
  merge_with_partner<kMirror, M3>(v);
}

// Group-limited selection with 8 groups of whole slots (SPG each): the entries of groups that are not among the best
// topk_group get the key of -inf.  A group's score is the sum of its two largest.  The lanes of a row halve the groups
// between them level by level (lane bit 3, then 1, then 0 decides which half a lane goes on with and which it hands to its
// partner), so that a level merges half the pairs of the one before, and the last one merges a single pair over lane
// bit 2; each group then sits in two lanes, and its place among the 8 is a count over seven moves.  A loop over the groups with
// four levels each, and another over the winners, took 12 us of dependent instructions (one wave: 16.7 us, a softmax 4.5).
template <int SPG, int NS, int NCH>
__device__ __forceinline__ void keep_best_of_8_groups(int (&val)[NCH][NS], int topk_group, int lane) {
  static_assert(NS == 8 * SPG && (SPG == 1 || SPG == 2), "8 groups");
  const int NEGK = to_key(-__builtin_inff());
  const bool b0 = lane & 1, b1 = lane & 2, b3 = lane & 8;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    int p1[8], p2[8];  // the two largest keys of each group, of the lanes merged so far
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const int x = val[ch][g * SPG], y = SPG == 2 ? val[ch][g * SPG + 1] : NEGK;
      p1[g] = max(x, y);
      p2[g] = SPG == 2 ? min(x, y) : NEGK;
    }
#define SEMMOE_HALVE(N, bit, ctrl)                                            \
  _Pragma("unroll") for (int i = 0; i < N; ++i) {                             \
    const int k1 = bit ? p1[N + i] : p1[i], k2 = bit ? p2[N + i] : p2[i];     \
    const int s1 = bit ? p1[i] : p1[N + i], s2 = bit ? p2[i] : p2[N + i];     \
    const int r1 = dpp_i32<ctrl, 0xf>(s1, s1), r2 = dpp_i32<ctrl, 0xf>(s2, s2); \
    p1[i] = max(k1, r1);                                                      \
    p2[i] = max(min(k1, r1), max(k2, r2));                                    \
  }
    SEMMOE_HALVE(4, b3, 0x128)  // row_ror:8
    SEMMOE_HALVE(2, b1, 0x4E)
    SEMMOE_HALVE(1, b0, 0xB1)
#undef SEMMOE_HALVE
    {  // lane bit 2: half mirror (all three low bits), then the two lowest back
      const int h1 = dpp_i32<0x141, 0xf>(p1[0], p1[0]), h2 = dpp_i32<0x141, 0xf>(p2[0], p2[0]);
      const int r1 = dpp_i32<0x1B, 0xf>(h1, h1), r2 = dpp_i32<0x1B, 0xf>(h2, h2);
      const int k1 = p1[0], k2 = p2[0];
      p1[0] = max(k1, r1);
      p2[0] = max(min(k1, r1), max(k2, r2));
    }
    const float sc = p2[0] == NEGK ? from_key(p1[0]) : __fadd_rn(from_key(p1[0]), from_key(p2[0]));
    const int mine = to_key(sc);
    // groups ahead of this lane's, number 4 b3 + 2 b1 + b0: a larger score, or the same one and a lower number, which is
    // where the highest differing bit is set here
    const int m0 = mine - int(b0), m1 = mine - int(b1), m3 = mine - int(b3);
    const int o8 = dpp_i32<0x128, 0xf>(mine, mine);
    const int ahead = int(dpp_i32<0xB1, 0xf>(mine, mine) > m0) + int(dpp_i32<0x4E, 0xf>(mine, mine) > m1) +
                      int(dpp_i32<0x1B, 0xf>(mine, mine) > m1) + int(o8 > m3) + int(dpp_i32<0xB1, 0xf>(o8, o8) > m3) +
                      int(dpp_i32<0x4E, 0xf>(o8, o8) > m3) + int(dpp_i32<0x1B, 0xf>(o8, o8) > m3);
    const unsigned long long kept = __ballot(ahead < topk_group && mine >= NEGK);
    const uint32_t mask = (lane < 32 ? uint32_t(kept) : uint32_t(kept >> 32)) >> (lane & 16);
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      const int g = c / SPG, at = (g >> 2) * 8 + ((g >> 1) & 1) * 2 + (g & 1);
      val[ch][c] = (mask >> at) & 1u ? val[ch][c] : NEGK;
    }
  }
}

// rowp[ch] / idp[ch] / wp[ch]: this lane's token of group ch (the same for the 16 lanes of a row), nullptr = none.
// Same selection rule as select_rows: the k largest in order, equal values -> lowest expert id.  KEEP >= k: 2, 4, 8 or 16.
// KEYED: the keys of the selection scores have been formed already and lie `key_off` words behind the logits.
template <int NS, int KEEP, int NCH, bool SIG, bool KEYED>
__device__ __forceinline__ void select_rows16(const semmoe_config& cfg, const float* const (&rowp)[NCH],
                                              const float* __restrict__ sel_bias, int lane,
                                              int32_t* const (&idp)[NCH], float* const (&wp)[NCH], int key_off) {
  static_assert(SIG || !KEYED, "a softmax key is its logit");
  const int E = cfg.E, k = cfg.k, l16 = lane & 15;
  constexpr bool sigmoid = SIG;  // compile-time: the softmax form carries none of the sigmoid form's bookkeeping
  const int NEGK = to_key(-__builtin_inff());

  // rowp[ch] is always readable (the callers point the rows of absent tokens at a present one) and the expert index
  // is clamped, so the loads carry no branch and go out together; what is absent is masked afterwards.  A token is
  // present when it has somewhere to write (idp[ch]).
  int val[NCH][NS];    // key of the selection score
  float x[NCH][NS], sb[NS];
#pragma unroll
  for (int c = 0; c < NS; ++c) {
    const int e = min(c * 16 + l16, E - 1);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) x[ch][c] = KEYED ? rowp[ch][key_off + e] : rowp[ch][e];
    sb[c] = (SIG && !KEYED && sel_bias) ? sel_bias[e] : 0.0f;
  }
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      const bool there = c * 16 + l16 < E && idp[ch] != nullptr;
      if (KEYED) {
        val[ch][c] = there ? __float_as_int(x[ch][c]) : NEGK;
      } else if (sigmoid) {
        const float sg = sigmoid_exact_seq(x[ch][c]);
        val[ch][c] = there ? to_key(__fadd_rn(sg, sb[c])) : NEGK;
      } else {
        val[ch][c] = there ? to_key(x[ch][c]) : NEGK;
      }
    }
  }

  if (sigmoid && NS >= 8 && cfg.n_group == 8 && E == 16 * NS) {
    if constexpr (NS >= 8) keep_best_of_8_groups<NS / 8>(val, cfg.topk_group, lane);
  } else if (sigmoid && cfg.n_group > 1) {
    // group score = sum of the group's two largest s'; lane g of a row keeps the score of group g
    const int gs = E / cfg.n_group;
    int grp[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) grp[c] = (c * 16 + l16) / gs;
    int gkey[NCH];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) gkey[ch] = NEGK;
    const bool whole_slots = gs % 16 == 0;  // a group is a run of gs/16 slots, the same for every lane
    const int spg = whole_slots ? gs / 16 : 0;
    for (int g = 0; g < cfg.n_group; ++g) {
      int a1[NCH], a2[NCH];  // the two largest keys seen so far (with multiplicity)
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        a1[ch] = NEGK;
        a2[ch] = NEGK;
      }
      auto take = [&](int ch, int v) {  // an absent entry has the lowest key: it changes neither
        a2[ch] = max(a2[ch], min(a1[ch], v));
        a1[ch] = max(a1[ch], v);
      };
      if (whole_slots) {  // a uniform test skips the slots of the other groups
#pragma unroll
        for (int c = 0; c < NS; ++c) {
          if (c < g * spg || c >= (g + 1) * spg) continue;
#pragma unroll
          for (int ch = 0; ch < NCH; ++ch) take(ch, val[ch][c]);
        }
      } else {  // every lane tests its own entry: a select, not a branch, of which there would be one per entry and group (26 tokens
        // of 96 experts in 16 groups, 4 a token: 19.2 us with branches, 10.1 so; whole slots in a loop of their own, 192
        // in 4: 13.3 -> 9.2)
#pragma unroll
        for (int c = 0; c < NS; ++c) {
          const bool in = grp[c] == g;
#pragma unroll
          for (int ch = 0; ch < NCH; ++ch) take(ch, in ? val[ch][c] : NEGK);
        }
      }
      // merge the sorted pairs of disjoint lane sets: xor 1, xor 2, half mirror, mirror
#define SEMMOE_PAIR_MERGE(CTRL)                                                    \
  _Pragma("unroll") for (int ch = 0; ch < NCH; ++ch) {                             \
    const int b1 = dpp_i32<CTRL, 0xf>(a1[ch], a1[ch]);                             \
    const int b2 = dpp_i32<CTRL, 0xf>(a2[ch], a2[ch]);                             \
    a2[ch] = max(min(a1[ch], b1), max(a2[ch], b2));                                \
    a1[ch] = max(a1[ch], b1);                                                      \
  }
      SEMMOE_PAIR_MERGE(0xB1)
      SEMMOE_PAIR_MERGE(0x4E)
      SEMMOE_PAIR_MERGE(0x141)
      SEMMOE_PAIR_MERGE(0x140)
#undef SEMMOE_PAIR_MERGE
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const float sc = (a2[ch] == NEGK) ? from_key(a1[ch]) : __fadd_rn(from_key(a1[ch]), from_key(a2[ch]));
        if (l16 == g) gkey[ch] = to_key(sc);
      }
    }
    uint32_t keep[NCH];
    bool taken[NCH];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      keep[ch] = 0;
      taken[ch] = false;
    }
    for (int r = 0; r < cfg.topk_group; ++r) {
      int m[NCH], g[NCH];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) m[ch] = (l16 < cfg.n_group && !taken[ch]) ? gkey[ch] : NEGK;
      int top[NCH];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) top[ch] = m[ch];
      SEMMOE_ROW_REDUCE("v_max_i32_dpp", top);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
        g[ch] = (l16 < cfg.n_group && !taken[ch] && m[ch] == top[ch]) ? l16 : kNoExpert;
      SEMMOE_ROW_REDUCE("v_min_i32_dpp", g);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        keep[ch] |= 1u << (g[ch] & 31);
        if (l16 == g[ch]) taken[ch] = true;
      }
    }
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
      for (int c = 0; c < NS; ++c) val[ch][c] = ((keep[ch] >> (grp[c] & 31)) & 1u) ? val[ch][c] : NEGK;
    }
  }

  // lane j of the row keeps the j-th winner
  int my_id[NCH];
  float my_val[NCH], mx[NCH];
  if constexpr (KEEP == 2) {
    // one or two winners: a round each, the row's largest key and the lowest expert that holds it.  The shortest list costs more
    // than that (8192 tokens of 256 experts, softmax, 1 a token: lists 3.98 us, so 3.41; 128 experts in 4 groups, sigmoid, 2 a
    // token 8.40 and 7.39)
    for (int j = 0; j < k; ++j) {
      int top[NCH], arg[NCH];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        top[ch] = NEGK;  // keys below -inf's (NaN) are out
#pragma unroll
        for (int c = 0; c < NS; ++c) top[ch] = max(top[ch], val[ch][c]);
      }
      SEMMOE_ROW_REDUCE("v_max_i32_dpp", top);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        arg[ch] = kNoExpert;
#pragma unroll
        for (int c = NS - 1; c >= 0; --c) arg[ch] = val[ch][c] == top[ch] ? c * 16 + l16 : arg[ch];
      }
      SEMMOE_ROW_REDUCE("v_min_i32_dpp", arg);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        if (j == 0) mx[ch] = from_key(top[ch]);
        if (j == 0 || l16 == j) {
          my_id[ch] = top[ch] == NEGK ? kNoExpert : arg[ch];
          my_val[ch] = from_key(top[ch]);
        }
#pragma unroll
        for (int c = 0; c < NS; ++c) val[ch][c] = arg[ch] == c * 16 + l16 ? NEGK : val[ch][c];
      }
    }
  } else {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      double all[NS], top[KEEP];
#pragma unroll
      for (int c = 0; c < NS; ++c) all[c] = pack_entry(max(val[ch][c], NEGK), c * 16 + l16);  // keys below -inf's (NaN): out too
      largest_of_row(all, top);
      double mine = top[0];
#pragma unroll
      for (int j = 1; j < KEEP; ++j) mine = l16 == j ? top[j] : mine;
      const int key = entry_key(mine);
      my_id[ch] = key == NEGK ? kNoExpert : entry_id(mine);
      my_val[ch] = from_key(key);
      mx[ch] = from_key(entry_key(top[0]));  // row maximum
    }
  }
  if constexpr (SIG) {
    // the weight is s without the selection bias.  Lane j forms it once more from its winner's logit: carrying s along
    // per slot costs a move per slot and round and a reduction per round, this one load and one sigmoid.
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const bool won = l16 < k && my_id[ch] != kNoExpert;
      const float s = sigmoid_exact_seq(rowp[ch][won ? my_id[ch] : 0]);
      my_val[ch] = won ? s : 0.0f;
    }
  }

  float w[NCH];
  if (!sigmoid) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) w[ch] = (l16 < k) ? expf(my_val[ch] - mx[ch]) : 0.0f;
    if (!cfg.renorm) {  // softmax over all experts; with renormalisation its denominator cancels and is not formed
      float part[NCH];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        part[ch] = 0.0f;
#pragma unroll
        for (int c = 0; c < NS; ++c)
          if (c * 16 + l16 < E) part[ch] += expf(x[ch][c] - mx[ch]);
      }
      SEMMOE_ROW_REDUCE("v_add_f32_dpp", part);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) w[ch] = w[ch] / part[ch];
    }
  } else {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) w[ch] = (l16 < k) ? my_val[ch] : 0.0f;
  }
  if (cfg.renorm) {
    float tot[NCH];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) tot[ch] = w[ch];
    SEMMOE_ROW_REDUCE("v_add_f32_dpp", tot);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) w[ch] = w[ch] / tot[ch];
  }
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    if (sigmoid) w[ch] *= cfg.routed_scale;
    if (l16 < k && idp[ch]) {
      idp[ch][l16] = my_id[ch];
      wp[ch][l16] = w[ch];
    }
  }
}
#undef SEMMOE_ROW_REDUCE
#undef SEMMOE_ROW_STEP

constexpr int kRowChains = 2;                   // interleaved groups of four tokens
constexpr int kRowTokens = 4 * kRowChains;      // tokens a wave selects for per call of the row form

// the row form holds E <= 256 experts (16 slots per lane), k <= 16 winners and 16 group scores per row
__host__ __device__ inline bool select_by_rows(const semmoe_config& cfg) {
  return cfg.E <= 256 && cfg.k <= 16 && (cfg.score != SEMMOE_SIGMOID || cfg.n_group <= 16);
}

// Which selection code a kernel instantiation carries.  The host picks it from E, k, the score function and the group
// count, so that a kernel holds one form instead of all of them (a fused router with every form in it was 150 KB of
// code: its prologue alone, hoisted set-up of forms it never ran, took 3 us of instruction fetch per workgroup).
// SLOTS: 0 any E, k and number of groups; else the row form with up to 4, 8 or 16 slots per lane.  KEEP: length of the lists
// of the row form, 4, 8 or 16 (>= k), or 2: no lists, a round per winner.
template <int SLOTS, int KEEP>
struct SelForm {
  static constexpr int kSlots = SLOTS, kKeep = KEEP;
  static constexpr bool kRows = SLOTS > 0;
};
using SelAny = SelForm<0, 0>;
inline int select_slots(const semmoe_config& cfg) {
  if (!select_by_rows(cfg)) return 0;
  return cfg.E <= 64 ? 4 : (cfg.E <= 128 ? 8 : 16);
}
// f(form, sigmoid) with the form of the configuration, of those with SLOTS slots, and the score function as types
template <int SLOTS, typename F>
inline int32_t with_select_form(const semmoe_config& cfg, F f) {
  auto with_score = [&](auto form) -> int32_t {
    return cfg.score == SEMMOE_SIGMOID ? f(form, std::true_type{}) : f(form, std::false_type{});
  };
  // two by softmax: lists of 4 are level with two rounds or 2 % ahead
  if (cfg.k == 1 || (cfg.k == 2 && cfg.score == SEMMOE_SIGMOID)) return with_score(SelForm<SLOTS, 2>{});
  if (cfg.k <= 4) return with_score(SelForm<SLOTS, 4>{});
  if (cfg.k <= 8) return with_score(SelForm<SLOTS, 8>{});
  return with_score(SelForm<SLOTS, 16>{});
}

// Tokens base .. base + kRowTokens - 1 (those below n_tok) by one wave: token = base + ch*4 + row.
// row_of(token) -> pointer to its E logits; ids / weights are written to topk_ids / topk_w at tok_global0 + token.
template <typename FORM, bool SIG, int NCH = kRowChains, bool KEYED = false, typename RowOf>
__device__ __forceinline__ void select_tokens_by_rows(const semmoe_config& cfg, int base, int n_tok, RowOf row_of,
                                                      int tok_global0, const float* __restrict__ sel_bias, int lane,
                                                      int32_t* __restrict__ topk_ids, float* __restrict__ topk_w,
                                                      int key_off = 0) {
  static_assert(FORM::kRows, "a row form");
  constexpr int KEEP = FORM::kKeep;
  const float* rowp[NCH];
  int32_t* idp[NCH];
  float* wp[NCH];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const int tl = base + ch * 4 + (lane >> 4);
    const bool ok = tl < n_tok && tok_global0 + tl < cfg.T;
    rowp[ch] = row_of(min(tl, n_tok - 1));  // an absent token reads a present one's row and writes nothing
    idp[ch] = ok ? topk_ids + size_t(tok_global0 + tl) * cfg.k : nullptr;
    wp[ch] = ok ? topk_w + size_t(tok_global0 + tl) * cfg.k : nullptr;
  }
  if constexpr (FORM::kSlots > 4) {
    select_rows16<FORM::kSlots, KEEP, NCH, SIG, KEYED>(cfg, rowp, sel_bias, lane, idp, wp, key_off);
  } else {
    if (cfg.E <= 16) select_rows16<1, KEEP, NCH, SIG, KEYED>(cfg, rowp, sel_bias, lane, idp, wp, key_off);
    else if (cfg.E <= 32) select_rows16<2, KEEP, NCH, SIG, KEYED>(cfg, rowp, sel_bias, lane, idp, wp, key_off);
    else select_rows16<4, KEEP, NCH, SIG, KEYED>(cfg, rowp, sel_bias, lane, idp, wp, key_off);
  }
}

constexpr int kSelTokens = 2;  // tokens a wave selects for at a time (four gain nothing: the selection is bound by instruction issue)

__global__ __launch_bounds__(256) void select_topk_kernel(semmoe_config cfg, const float* __restrict__ logits,
                                                          const float* __restrict__ sel_bias,
                                                          int32_t* __restrict__ topk_ids,
                                                          float* __restrict__ topk_w) {
  const int lane = threadIdx.x & 63;
  const int token0 = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * kSelTokens;
  if (token0 >= cfg.T) return;  // whole wave leaves together
  const float* rows[kSelTokens];
  int32_t* ids_out[kSelTokens];
  float* w_out[kSelTokens];
#pragma unroll
  for (int t = 0; t < kSelTokens; ++t) {
    const int token = token0 + t;
    const bool ok = token < cfg.T;
    rows[t] = ok ? logits + size_t(token) * cfg.E : nullptr;
    ids_out[t] = ok ? topk_ids + size_t(token) * cfg.k : nullptr;
    w_out[t] = ok ? topk_w + size_t(token) * cfg.k : nullptr;
  }
  select_rows_any<kSelTokens>(cfg, rows, sel_bias, lane, ids_out, w_out);
}

// Fused router for bf16: logits of TT*32 tokens x all experts, then the selection, in one kernel.
//   X and W_r slices of 64 K-elements are brought into an NSTAGE ring in LDS by direct global->LDS loads
//   (each wave instruction moves 8 rows x 128 contiguous bytes), chunk-swizzled as in the grouped GEMM.
//   4 waves; wave w owns expert tiles w*TF .. w*TF+TF-1 (32 experts each) for all TT token tiles.
//   MFMA A operand = W_r rows (experts), B operand = X rows (tokens): a lane ends with 4 consecutive experts
//   of one token per register group.  After the K loop the fp32 logits (+ bias terms) are parked in LDS and
//   each wave selects for its share of the tokens.
template <int TF, int TT, int NSTAGE>
struct RouteCfg {
  static constexpr int BW = 4 * TF * 32;   // expert rows per stage
  static constexpr int BT = TT * 32;       // token rows per stage
  static constexpr int ROWS = BW + BT;
  static constexpr int BK = 64, RB = 128, CPR = 8, RPI = 8, RPB = 2;
  static constexpr int IPS = ROWS / RPI;   // wave instructions per stage
  static constexpr int IPW = IPS / 4;
  static constexpr int kStageBytes = ROWS * RB;
  static_assert(IPS % 4 == 0, "instructions divide over the waves");
  static_assert((NSTAGE - 1) * IPW < 64, "vmcnt range");
};

// PARTS (the token tiles alone would leave much of the chip idle): a workgroup takes (token tile, tile of 128 TF experts,
// part of K) and writes its raw fp32 sums to partial[part][token][expert]; a second kernel adds the parts up in order, adds the
// bias terms and selects.
// A kernel of its own without the selection, and one tile a workgroup: a short kernel waits for its code, and a loop over
// tiles has the compiler set up in front of it what the selection behind it needs (spilled scalars and all).
template <int TF, int TT, int NSTAGE, typename FORM, bool SIG, bool PARTS>
__global__ __launch_bounds__(256) void route_fused_kernel(semmoe_config cfg, const bf16_t* __restrict__ X,
                                                          const bf16_t* __restrict__ W_r,
                                                          const float* __restrict__ b_g,
                                                          const int32_t* __restrict__ token_class,
                                                          const float* __restrict__ class_bias,
                                                          const float* __restrict__ sel_bias,
                                                          float* __restrict__ logits_out,
                                                          int32_t* __restrict__ topk_ids,
                                                          float* __restrict__ topk_w, int n_parts,
                                                          float* __restrict__ partial) {
  using C = RouteCfg<TF, TT, NSTAGE>;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const unsigned lds_base = static_cast<unsigned>(reinterpret_cast<size_t>(lds_raw));
  float* lg = reinterpret_cast<float*>(lds_raw);  // [BT][E + 4] after the K loop
  const int T = cfg.T, E = cfg.E, K = cfg.d;
  const int ldl = E + 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 31, half = lane >> 5;
  const int nk = (K + C::BK - 1) / C::BK;
  const int k_tail = K - (nk - 1) * C::BK;
  const int frag_swz = (lrow / C::RPB) % C::CPR;
  const int d_row = lane / C::CPR, d_pos = lane % C::CPR;

  const int spp = PARTS ? (nk + n_parts - 1) / n_parts : nk;  // slices per part
  const int n_et = PARTS ? (E + C::BW - 1) / C::BW : 1;  // tiles of experts; without PARTS one holds them all
  const int item = PARTS ? int(blockIdx.x) / n_parts : int(blockIdx.x), part = PARTS ? int(blockIdx.x) - item * n_parts : 0;
  const int tile = item / n_et, e0 = (item - tile * n_et) * C::BW;
  const int s_lo = PARTS ? min(part * spp, nk) : 0, n_it = min(nk, s_lo + spp) - s_lo;
  const int tok0 = tile * C::BT;
  const bf16_t* src[C::IPW];
  int src_chunk[C::IPW];
#pragma unroll
  for (int i = 0; i < C::IPW; ++i) {
    const int sr = (wave * C::IPW + i) * C::RPI + d_row;
    const int c = d_pos ^ ((sr / C::RPB) % C::CPR);
    src_chunk[i] = c;
    src[i] = (sr < C::BW) ? W_r + size_t(min(e0 + sr, E - 1)) * K + c * 8
                          : X + size_t(min(tok0 + sr - C::BW, T - 1)) * K + c * 8;
  }
  auto issue = [&](int it_, int stage_at) {  // slice s_lo + it_ of K into the ring stage at that offset
    const int slice = s_lo + it_;
    const unsigned dst0 = lds_base + stage_at + wave * C::IPW * 1024;
    const int k0 = slice * C::BK;
    if (slice + 1 < nk || k_tail == C::BK) {
#pragma unroll
      for (int i = 0; i < C::IPW; ++i) lds_dma16(src[i] + k0, dst0 + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < C::IPW; ++i) {
        if (src_chunk[i] * 8 < k_tail) lds_dma16(src[i] + k0, dst0 + i * 1024);
        else *reinterpret_cast<uint4*>(lds_raw + (dst0 - lds_base) + i * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
      }
    }
  };

  // two accumulator sets (even / odd k-steps): halves the chain of dependent MFMAs inside a slice
  f32x16_t acc[TF][TT], acc2[TF][TT];
#pragma unroll
  for (int i = 0; i < TF; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] = 0.0f;
        acc2[i][j][r] = 0.0f;
      }

  // the tokens' classes are requested before the ring: they have arrived long before the logits need them
  int cls_of[TT];
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    const int tok = tok0 + j * 32 + lrow;
    cls_of[j] = (!PARTS && token_class && tok < T) ? token_class[tok] : -1;
  }
#pragma unroll
  for (int s0 = 0; s0 < NSTAGE - 1; ++s0)
    if (s0 < n_it) issue(s0, s0 * C::kStageBytes);
  // Offsets of the stages of slices it and it + NSTAGE - 1, kept: a slice is one chain of wait, barrier, reads and MFMAs, and
  // it % NSTAGE, formed anew for every address of it, stands in that chain (4097 to 8192 tokens, up to 128 experts, 0.89 of the time
  // from d 2880 on, 0.94 below; more experts, whose slices are longer, 0.99 to 1.00)
  int read_at = 0, fill_at = (NSTAGE - 1) * C::kStageBytes;
  auto next_stage = [](int at) { return at == (NSTAGE - 1) * C::kStageBytes ? 0 : at + C::kStageBytes; };
  for (int it = 0; it < n_it; ++it) {
    const int younger = min(NSTAGE - 2, n_it - 1 - it);
    if (younger >= 4) wait_vmcnt<4 * C::IPW>();
    else if (younger == 3) wait_vmcnt<3 * C::IPW>();
    else if (younger == 2) wait_vmcnt<2 * C::IPW>();
    else if (younger == 1) wait_vmcnt<1 * C::IPW>();
    else wait_vmcnt<0>();
    __syncthreads();
    const unsigned char* Ws = lds_raw + read_at;
    const unsigned char* Xs = Ws + C::BW * C::RB;
    const unsigned char* wrow = Ws + (wave * TF * 32 + lrow) * C::RB;
    const unsigned char* xrow = Xs + lrow * C::RB;
    // all fragment reads of the slice are requested before the first MFMA (the per-slice work is small: the
    // loop is bound by latencies, not by throughput)
    bf16x8_t af[4][TF], bfr[4][TT];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const int off = ((st * 2 + half) ^ frag_swz) * 16;
#pragma unroll
      for (int i = 0; i < TF; ++i) af[st][i] = *reinterpret_cast<const bf16x8_t*>(wrow + i * 32 * C::RB + off);
#pragma unroll
      for (int j = 0; j < TT; ++j) bfr[st][j] = *reinterpret_cast<const bf16x8_t*>(xrow + j * 32 * C::RB + off);
    }
    // the refill of the stage freed by the barrier goes out while the fragment reads are in flight
    __builtin_amdgcn_sched_barrier(0);
    if (it + NSTAGE - 1 < n_it) issue(it + NSTAGE - 1, fill_at);
    __builtin_amdgcn_sched_barrier(0);
    read_at = next_stage(read_at);
    fill_at = next_stage(fill_at);
#pragma unroll
    for (int st = 0; st < 4; st += 2) {
#pragma unroll
      for (int i = 0; i < TF; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[st][i], bfr[st][j], acc[i][j], 0, 0, 0);
          acc2[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[st + 1][i], bfr[st + 1][j], acc2[i][j], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < TF; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] += acc2[i][j];
  if constexpr (PARTS) {  // raw sums of this part of K
#pragma unroll
    for (int j = 0; j < TT; ++j) {
      const int tok = tok0 + j * 32 + lrow;
#pragma unroll
      for (int i = 0; i < TF; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int e = e0 + (wave * TF + i) * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
          if (e < E && tok < T) partial[(size_t(part) * T + tok) * E + e] = acc[i][j][r];
        }
      }
    }
    return;
  }
  __syncthreads();  // every wave is done with the ring: its first bytes now hold the logits

  // A lane holds, per 32 x 32 block, four groups of four consecutive experts of one token.  With E a multiple of
  // four and 16-byte aligned bias arrays a group's bias terms are one 16-byte load each, all requested before the
  // first is used (one exposed latency per token tile instead of one per element), and a group's logits are
  // one 16-byte LDS write and one 16-byte store.
  const bool vec4 = (E & 3) == 0 && ((reinterpret_cast<size_t>(b_g) | reinterpret_cast<size_t>(class_bias) |
                                      reinterpret_cast<size_t>(logits_out)) & 15) == 0;
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    const int tl = j * 32 + lrow;
    const int tok = tok0 + tl;
    const int cls = cls_of[j];
    const float* cb = (cls >= 0 && cls < cfg.num_classes && class_bias) ? class_bias + size_t(cls) * E : nullptr;
    if (vec4) {
      f32x4_t add[TF][4];
#pragma unroll
      for (int i = 0; i < TF; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int e0 = (wave * TF + i) * 32 + g * 8 + half * 4;
          f32x4_t a = {0.0f, 0.0f, 0.0f, 0.0f};
          if (e0 < E) {
            if (b_g) a = *reinterpret_cast<const f32x4_t*>(b_g + e0);
            if (cb) a += *reinterpret_cast<const f32x4_t*>(cb + e0);
          }
          add[i][g] = a;
        }
#pragma unroll
      for (int i = 0; i < TF; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int e0 = (wave * TF + i) * 32 + g * 8 + half * 4;
          if (e0 < E) {
            f32x4_t v = {acc[i][j][g * 4], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]};
            v += add[i][g];
            *reinterpret_cast<f32x4_t*>(lg + tl * ldl + e0) = v;
            if (logits_out && tok < T) *reinterpret_cast<f32x4_t*>(logits_out + size_t(tok) * E + e0) = v;
          }
        }
      continue;
    }
#pragma unroll
    for (int i = 0; i < TF; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int e = (wave * TF + i) * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        if (e < E) {
          float v = acc[i][j][r];
          if (b_g) v += b_g[e];
          if (cb) v += cb[e];
          lg[tl * ldl + e] = v;
          if (logits_out && tok < T) logits_out[size_t(tok) * E + e] = v;
        }
      }
    }
  }
  __syncthreads();
  if constexpr (FORM::kRows) {
    for (int base = wave * kRowTokens; base < C::BT; base += 4 * kRowTokens)
      select_tokens_by_rows<FORM, SIG>(
          cfg, base, C::BT, [&](int tl) { return lg + tl * ldl; }, tok0, sel_bias, lane, topk_ids, topk_w);
  } else {
    for (int tl0 = wave; tl0 < C::BT; tl0 += 4 * kSelTokens) {
      const float* rows[kSelTokens];
      int32_t* ids_out[kSelTokens];
      float* w_out[kSelTokens];
#pragma unroll
      for (int t = 0; t < kSelTokens; ++t) {
        const int tl = tl0 + 4 * t;
        const int tok = tok0 + tl;
        const bool ok = tl < C::BT && tok < T;
        rows[t] = ok ? lg + tl * ldl : nullptr;
        ids_out[t] = ok ? topk_ids + size_t(tok) * cfg.k : nullptr;
        w_out[t] = ok ? topk_w + size_t(tok) * cfg.k : nullptr;
      }
      select_rows_any<kSelTokens>(cfg, rows, sel_bias, lane, ids_out, w_out);
    }
  }
}

template <typename FORM, bool SIG>
__global__ __launch_bounds__(256) void select_topk_rows_kernel(semmoe_config cfg, const float* __restrict__ logits,
                                                               const float* __restrict__ sel_bias,
                                                               int32_t* __restrict__ topk_ids,
                                                               float* __restrict__ topk_w) {
  const int lane = threadIdx.x & 63;
  const int base = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * kRowTokens;
  if (base >= cfg.T) return;  // whole wave leaves together
  select_tokens_by_rows<FORM, SIG>(
      cfg, base, cfg.T, [&](int tl) { return logits + size_t(tl) * cfg.E; }, 0, sel_bias, lane, topk_ids, topk_w);
}

// The two kernels below in one, for the row forms of the selection and E a multiple of four: a wave adds up the parts
// of its four tokens (ascending order, then b_g, then the class bias: the same sums as route_reduce_kernel)
// into LDS with 16-byte loads and selects from there.  The partial sums are read once and never again.
// paired_bias (with both biases): b_g + class bias first and their sum to the logit, as the fused kernel with 16-byte bias
// loads does; for sums that are the fused kernel's own (one part), so that a call gives the same bits by either.
constexpr int kSumSelectMaxE = 256;
constexpr int kSumSelectChains = 1;                       // four tokens a wave: twice the waves to hide the latencies
constexpr int kSumSelectTokens = 4 * kSumSelectChains;
// PB parts of U chunks of four experts are requested before the first is used.
template <typename FORM, bool SIG, int PB, int U>
__global__ __launch_bounds__(256) void route_sum_select_kernel(semmoe_config cfg, int n_parts, bool paired_bias,
                                                               const float* __restrict__ partial,
                                                               const float* __restrict__ b_g,
                                                               const int32_t* __restrict__ token_class,
                                                               const float* __restrict__ class_bias,
                                                               const float* __restrict__ sel_bias,
                                                               float* __restrict__ logits_out,
                                                               int32_t* __restrict__ topk_ids,
                                                               float* __restrict__ topk_w) {
  // logits, and behind them (sigmoid) the keys of the selection scores: formed here, four a loop round, because the sixteen
  // of a lane one after the other in the selection are 3 KB of code that every wave waits for
  __shared__ __attribute__((aligned(16))) float lg_all[4 * kSumSelectTokens * (kSumSelectMaxE + 4) * (SIG ? 2 : 1)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int base = (blockIdx.x * int(blockDim.x >> 6) + wave) * kSumSelectTokens;  // up to four waves per workgroup
  if (base >= cfg.T) return;  // whole wave leaves together (no workgroup barrier below)
  const int E = cfg.E, e4 = E / 4, ld = E + 4;
  float* lg = lg_all + wave * kSumSelectTokens * (kSumSelectMaxE + 4);
  constexpr int kKeyOff = 4 * kSumSelectTokens * (kSumSelectMaxE + 4);
  const int n_tok = min(kSumSelectTokens, cfg.T - base);
  const size_t n = size_t(cfg.T) * E;
  const bool out16 = logits_out && (reinterpret_cast<size_t>(logits_out) & 15) == 0;
  const int n_idx = n_tok * e4;
  for (int idx0 = lane; idx0 < n_idx; idx0 += 64 * U) {
    int tl[U], e[U], cls[U];
    size_t at[U];
    f32x4_t v[U];
#pragma unroll
    for (int c = 0; c < U; ++c) {  // chunks behind the end stand on the last one and are not written
      const int idx = min(idx0 + c * 64, n_idx - 1);
      tl[c] = idx / e4;
      e[c] = (idx - tl[c] * e4) * 4;
      at[c] = size_t(base + tl[c]) * E + e[c];
      cls[c] = token_class ? token_class[base + tl[c]] : -1;
      v[c] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
    for (int p0 = 0; p0 < n_parts; p0 += PB) {
      f32x4_t x[U][PB];
#pragma unroll
      for (int u = 0; u < PB; ++u)
#pragma unroll
        for (int c = 0; c < U; ++c)
          x[c][u] = p0 + u < n_parts
                        ? __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(partial + size_t(p0 + u) * n + at[c]))
                        : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < U; ++c)
#pragma unroll
        for (int u = 0; u < PB; ++u) v[c] += x[c][u];
    }
#pragma unroll
    for (int c = 0; c < U; ++c) {
      if (idx0 + c * 64 >= n_idx) break;
      const bool classed = cls[c] >= 0 && cls[c] < cfg.num_classes && class_bias;
      if (paired_bias && classed) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[c][u] += b_g[e[c] + u] + class_bias[size_t(cls[c]) * E + e[c] + u];
      } else {
        if (b_g) {
#pragma unroll
          for (int u = 0; u < 4; ++u) v[c][u] += b_g[e[c] + u];
        }
        if (classed) {
#pragma unroll
          for (int u = 0; u < 4; ++u) v[c][u] += class_bias[size_t(cls[c]) * E + e[c] + u];
        }
      }
      *reinterpret_cast<f32x4_t*>(lg + tl[c] * ld + e[c]) = v[c];
      if constexpr (SIG) {
        i32x4_t key;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          key[u] = to_key(__fadd_rn(sigmoid_exact_seq(v[c][u]), sel_bias ? sel_bias[e[c] + u] : 0.0f));
        *reinterpret_cast<i32x4_t*>(lg + kKeyOff + tl[c] * ld + e[c]) = key;
      }
      if (out16) {
        *reinterpret_cast<f32x4_t*>(logits_out + at[c]) = v[c];
      } else if (logits_out) {
#pragma unroll
        for (int u = 0; u < 4; ++u) logits_out[at[c] + u] = v[c][u];
      }
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  select_tokens_by_rows<FORM, SIG, kSumSelectChains, SIG>(
      cfg, 0, n_tok, [&](int tl) { return lg + tl * ld; }, base, sel_bias, lane, topk_ids, topk_w, kKeyOff);
}

// launches route_sum_select_kernel when the shape has a row form of the selection and E is a multiple of four;
// false: nothing was launched (the caller runs the two kernels)
static bool launch_sum_select(const semmoe_config* cfg, hipStream_t s, int n_parts, bool paired_bias, const float* partial,
                              const float* b_g, const int32_t* token_class, const float* class_bias,
                              const float* sel_bias, float* logits_out, int32_t* topk_ids, float* topk_w) {
  const int slots = select_slots(*cfg);
  if (slots == 0 || cfg->E > kSumSelectMaxE || cfg->E % 4 != 0) return false;
  // few tokens: a wave a workgroup, so that they spread over as many compute units as there are, and all loads of a wave
  // in flight at once (256 tokens, 128 experts, 16 parts: 18.8 -> 15.2 us for the route); many: the waves hide each
  // other's latencies and registers are what is short (16384 tokens, 256 experts, 4 parts: 111 us so, 114 us with 16
  // loads in flight)
  const int waves = cfg->T <= 2048 ? 1 : 4;
  const dim3 grid(cdiv(cfg->T, waves * kSumSelectTokens)), block(64 * waves);
  auto launch = [&](auto form, auto sig) -> int32_t {
    using FORM = decltype(form);
    constexpr bool SIG = decltype(sig)::value;
    auto kern = waves == 4 ? route_sum_select_kernel<FORM, SIG, 8, 1> : route_sum_select_kernel<FORM, SIG, 16, 2>;
    hipLaunchKernelGGL(kern, grid, block, 0, s, *cfg, n_parts, paired_bias, partial, b_g, token_class, class_bias, sel_bias,
                       logits_out, topk_ids, topk_w);
    return SEMMOE_OK;
  };
  if (slots == 16) with_select_form<16>(*cfg, launch);
  else if (slots == 8) with_select_form<8>(*cfg, launch);
  else with_select_form<4>(*cfg, launch);
  return true;
}

// logits[tok][e] = sum over the parts of K, in ascending order, + b_g[e] + class_bias[token_class[tok]][e]
__global__ __launch_bounds__(256) void route_reduce_kernel(semmoe_config cfg, int n_parts,
                                                           const float* __restrict__ partial,
                                                           const float* __restrict__ b_g,
                                                           const int32_t* __restrict__ token_class,
                                                           const float* __restrict__ class_bias,
                                                           float* __restrict__ logits, float* __restrict__ logits_out) {
  const size_t n = size_t(cfg.T) * cfg.E;
  const size_t idx = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= n) return;
  const int tok = int(idx / cfg.E), e = int(idx - size_t(tok) * cfg.E);
  float v = 0.0f;
  for (int p0 = 0; p0 < n_parts; p0 += 8) {  // eight loads in flight
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = p0 + u < n_parts ? __builtin_nontemporal_load(partial + size_t(p0 + u) * n + idx) : 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) v += x[u];
  }
  if (b_g) v += b_g[e];
  const int cls = token_class ? token_class[tok] : -1;
  if (cls >= 0 && cls < cfg.num_classes && class_bias) v += class_bias[size_t(cls) * cfg.E + e];
  logits[idx] = v;
  if (logits_out) logits_out[idx] = v;
}

// Many tokens and more than 128 experts: the fused kernel's workgroup (64 tokens) streams all of W_r past its tokens,
// five rows of operands per token and slice.  The 256 x 256 tile of the grouped GEMM takes two, with K cut into as
// many parts as fill the chip; the parts are then added in order and the selection runs as a kernel of its own.  Which
// token counts take how many parts decides the order of the sums, and with it which of two groups of experts with nearly
// equal scores a token goes to: half the parts on 256 x 128 tiles are 7 us faster on 16384 tokens (94 -> 87) and 8 of them would
// halve the time of 1024 to 8191, but one token in 16384 then goes elsewhere.
// tune (SEMMOE_TUNE_ROUTE_SPLIT): -1 automatic, 0 never, 100 + n this form with n parts whatever the token count.
static int route_big_parts(const semmoe_config* cfg, int ncu) {
  const int tune = tuning_value(SEMMOE_TUNE_ROUTE_SPLIT);
  if (cfg->dtype != SEMMOE_BF16 || tune == 0 || cfg->E <= 128 || cfg->E % 4 != 0 || cfg->d % 64 != 0) return 0;
  const int nk = cfg->d / 64;
  const long long tiles = (long long)cdiv(cfg->T, 256) * cdiv(cfg->E, 256);
  const int cap = tiles >= 1024 ? 1 : int(1024 / tiles < 8 ? 1024 / tiles : 8);  // what the workspace is sized for
  if (tune >= 100) {
    const int parts = tune - 100;
    return (parts >= 1 && parts <= cap && nk % parts == 0 && nk / parts >= 2) ? parts : 0;
  }
  if (tune > 0) return 0;  // a forced split of the fused kernel
  if (tiles * 8 < ncu) return 0;  // too few tokens to fill the chip with 256-token tiles and K parts of useful depth
  int parts = int(ncu / tiles);
  if (parts < 1) parts = 1;
  if (parts > cap) parts = cap;
  while (parts > 1 && (nk % parts != 0 || nk / parts < 8)) --parts;
  if (tiles * parts * 4 < (long long)ncu * 3) return 0;  // K too short to cut into enough parts: the fused kernel fills the chip
  return nk / parts >= 2 ? parts : 0;
}

// Parts of K for the fused router, 1 = none.  With at most a 32-token tile for every second compute unit the rest of the chip
// takes parts of K: up to 512 tokens at least two slices each; beyond (up to 128 experts) at least 6, and what the walk gets
// shorter by has to repay the second kernel: 20 slices (4096 tokens, two parts: d 2048 15.4 -> 15.8 us, d 2880 18.0 -> 17.1,
// d 4096 23.6 -> 20.1; 1024 tokens: d 2048 15.0 -> 12.3, d 4096 23.5 -> 13.4).
// tune: -1 automatic, 0 never, n > 1 that many parts
static int route_parts(const semmoe_config* cfg, int ncu) {
  const int tune = tuning_value(SEMMOE_TUNE_ROUTE_SPLIT);
  const int n_tiles = cdiv(cfg->T, 32), nk = cdiv(cfg->d, 64);
  const int most = route_max_parts(cfg);
  if (cfg->dtype != SEMMOE_BF16 || tune == 0 || most < 2) return 1;
  const bool forced = tune > 1 && tune < 100, many = cfg->T > 512 && !forced;
  int parts = forced ? tune : ncu / n_tiles;
  if (many && parts > nk / 6) parts = nk / 6;
  if (parts > most) parts = most;
  if (parts > nk / 2) parts = nk / 2;  // at least two slices per part
  if (parts < 2) return 1;
  return many && nk - nk / parts < 20 ? 1 : parts;
}

static int32_t validate_select(const semmoe_config* cfg) {
  int32_t st = validate_config(cfg, true, false, false);
  if (st != SEMMOE_OK) return st;
  if (cfg->k > 64) return SEMMOE_EUNSUPPORTED;
  if (cfg->score == SEMMOE_SIGMOID) {
    if (cfg->n_group < 1 || cfg->topk_group < 1) return SEMMOE_EINVAL;
    if (cfg->n_group > 64) return SEMMOE_EUNSUPPORTED;
    if (cfg->E % cfg->n_group != 0 || cfg->topk_group > cfg->n_group) return SEMMOE_ESHAPE;
    if (cfg->k > cfg->topk_group * (cfg->E / cfg->n_group)) return SEMMOE_ESHAPE;
  }
  return SEMMOE_OK;
}

static int32_t launch_select(const semmoe_config* cfg, hipStream_t stream, const float* logits,
                             const float* sel_bias, int32_t* topk_ids, float* topk_w) {
  if (cfg->T == 0) return SEMMOE_OK;
  const int waves_per_block = 4;
  const int slots = select_slots(*cfg);
  if (slots > 0) {
    const dim3 grid(cdiv(cfg->T, waves_per_block * kRowTokens)), block(64 * waves_per_block);
    auto launch = [&](auto form, auto sig) -> int32_t {
      hipLaunchKernelGGL((select_topk_rows_kernel<decltype(form), decltype(sig)::value>), grid, block, 0, stream, *cfg, logits,
                         sel_bias, topk_ids, topk_w);
      return SEMMOE_OK;
    };
    if (slots == 16) with_select_form<16>(*cfg, launch);
    else if (slots == 8) with_select_form<8>(*cfg, launch);
    else with_select_form<4>(*cfg, launch);
    SEMMOE_LAUNCH_CHECK();
    return SEMMOE_OK;
  }
  hipLaunchKernelGGL(select_topk_kernel, dim3(cdiv(cfg->T, waves_per_block * kSelTokens)), dim3(64 * waves_per_block), 0, stream,
                     *cfg, logits, sel_bias, topk_ids, topk_w);
  SEMMOE_LAUNCH_CHECK();
  return SEMMOE_OK;
}

}  // namespace semmoe

using namespace semmoe;

extern "C" int32_t semmoe_route_from_logits(const semmoe_config* cfg, void* stream, const float* logits,
                                            const float* sel_bias, int32_t* topk_ids, float* topk_w) {
  int32_t st = validate_select(cfg);
  if (st != SEMMOE_OK) return st;
  if (!logits || !topk_ids || !topk_w) return SEMMOE_EINVAL;
  return launch_select(cfg, static_cast<hipStream_t>(stream), logits, sel_bias, topk_ids, topk_w);
}

extern "C" int32_t semmoe_route(const semmoe_config* cfg, void* stream, const void* X, const void* W_r,
                                const float* b_g, const int32_t* token_class, const float* class_bias,
                                const float* sel_bias, float* logits_out, int32_t* topk_ids, float* topk_w, void* ws,
                                size_t ws_bytes) {
  int32_t st = validate_select(cfg);
  if (st != SEMMOE_OK) return st;
  st = validate_config(cfg, true, true, false);
  if (st != SEMMOE_OK) return st;
  if (!X || !W_r || !topk_ids || !topk_w) return SEMMOE_EINVAL;
  if ((token_class == nullptr) != (class_bias == nullptr)) return SEMMOE_EINVAL;
  if (token_class && cfg->num_classes <= 0) return SEMMOE_EINVAL;
  if (!aligned16(X) || !aligned16(W_r)) return SEMMOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (cfg->T == 0) return SEMMOE_OK;
  if (cfg->dtype == SEMMOE_BF16) {
    const bf16_t* Xb = static_cast<const bf16_t*>(X);
    const bf16_t* Wb = static_cast<const bf16_t*>(W_r);
    const int tf = cfg->E <= 128 ? 1 : (cfg->E <= 256 ? 2 : 4);
    DeviceInfo di;
    st = device_info(&di);
    if (st != SEMMOE_OK) return st;
    const int ncu = di.num_cu;
    if (const int big_parts = route_big_parts(cfg, ncu)) {
      Carver c(ws, ws_bytes);
      float* part = c.take<float>(size_t(big_parts) * cfg->T * cfg->E);
      float* lg = c.take<float>(size_t(cfg->T) * cfg->E);
      if (!c.ok) return SEMMOE_EWORKSPACE;
      st = launch_ksplit_gemm(X, W_r, cfg->T, cfg->E, cfg->d, big_parts, part, s);
      if (st == SEMMOE_OK && launch_sum_select(cfg, s, big_parts, false, part, b_g, token_class, class_bias, sel_bias,
                                               logits_out, topk_ids, topk_w)) {
        SEMMOE_LAUNCH_CHECK();
        return SEMMOE_OK;
      }
      if (st == SEMMOE_OK) {
        const size_t n = size_t(cfg->T) * cfg->E;
        hipLaunchKernelGGL(route_reduce_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, *cfg, big_parts, part,
                           b_g, token_class, class_bias, lg, logits_out);
        SEMMOE_LAUNCH_CHECK();
        return launch_select(cfg, s, lg, sel_bias, topk_ids, topk_w);
      }
      if (st != SEMMOE_EUNSUPPORTED) return st;
    }
    int n_parts = route_parts(cfg, ncu);
    const int slots = select_slots(*cfg);
    // 129 to 256 experts: two workgroups share a tile of 32 tokens, 128 experts each, while all of them are one round of the
    // chip; the sums stay as they are.  A workgroup then streams 160 rows a slice instead of 288, and the selection's kernel has
    // the whole chip (group-limited sigmoid, d 7168: 16 tokens 16.8 -> 14.1 us, 256 19.8 -> 17.2, 1024 59.5 -> 41.6, 4096 59.7 ->
    // 44.7).  Not with 64 tokens (5000: 60.0 us fused, 68.9 so) or 128 (10000: 95.7, 98.1).  Where K is not in parts the
    // selection's launch comes on top, and the walk has to be long enough to repay it (of the fused kernel's time, 513 to 4096 tokens
    // of 132 to 256 experts: softmax d 512 1.24 to 1.46, d 1536 0.98 to 1.08, d 2048 0.92 to 1.03; sigmoid, whose keys the second kernel
    // forms on the whole chip, d 1024 0.97 to 1.10, d 1536 0.92 to 1.02).
    bool split_e = tf == 2 && slots == 16 && cfg->E % 4 == 0 && tuning_value(SEMMOE_TUNE_ROUTE_SPLIT) != 0 &&
                   2 * cdiv(cfg->T, 32) * n_parts <= ncu &&
                   (n_parts > 1 || cdiv(cfg->d, 64) >= (cfg->score == SEMMOE_SIGMOID ? 24 : 32));
    float* partial = nullptr;
    float* logits_ws = nullptr;
    if (n_parts > 1 || split_e) {
      Carver c(ws, ws_bytes);
      partial = c.take<float>(size_t(n_parts) * cfg->T * cfg->E);
      logits_ws = c.take<float>(size_t(cfg->T) * cfg->E);
      if (!c.ok) {  // beyond 512 tokens a second kernel is worth a workspace, but not needed
        if (n_parts > 1 && cfg->T <= 512) return SEMMOE_EWORKSPACE;
        n_parts = 1;
        split_e = false;
        partial = nullptr;
      }
    }
    // tokens per workgroup: 32 while that is one round of the chip, then 64 (up to 256 experts), and 128 (up to 128 experts) from
    // where that still gives every compute unit a tile: every workgroup streams all of W_r past its tokens, and a second
    // round of it costs more than the wider tile (10000 tokens, d 2048, 128 experts: 28 us as 32, 24 as 64)
    const bool wide = n_parts == 1 && cdiv(cfg->T, 32) > ncu && tf <= 2;
    const bool wider = wide && tf == 1 && cdiv(cfg->T, 128) >= 256;
    const int bt = wider ? 128 : (wide ? 64 : 32);
    const int items = cdiv(cfg->T, bt) * n_parts * (split_e ? 2 : 1);
    // TF x 128 experts and TT x 32 tokens a workgroup, a ring of NS
    auto launch = [&](auto tf_, auto tt_, auto ns_, auto form, auto sig, auto in_parts) -> int32_t {
      constexpr int TF = decltype(tf_)::value, TT = decltype(tt_)::value, NS = decltype(ns_)::value;
      using RC = RouteCfg<TF, TT, NS>;
      auto kern = route_fused_kernel<TF, TT, NS, decltype(form), decltype(sig)::value, decltype(in_parts)::value>;
      size_t lds = size_t(NS) * RC::kStageBytes;
      const size_t lg_bytes = partial ? 0 : size_t(RC::BT) * (cfg->E + 4) * 4;
      if (lg_bytes > lds) lds = lg_bytes;
      static std::atomic<uint64_t> lds_allowed{0};  // one per instantiation
      const int32_t as = allow_max_dynamic_lds(&lds_allowed, reinterpret_cast<const void*>(kern));
      if (as != SEMMOE_OK) return as;
      hipLaunchKernelGGL(kern, dim3(items), dim3(256), lds, s, *cfg, Xb, Wb, b_g, token_class, class_bias, sel_bias,
                         logits_out, topk_ids, topk_w, n_parts, partial);
      return SEMMOE_OK;
    };
    // the forms a shape can need: up to 128 experts 4 and 8 slots, up to 256 experts 16, or none of them
    auto launch_128 = [&](auto tf_, auto tt_, auto ns_) -> int32_t {
      auto with = [&](auto form, auto sig) { return launch(tf_, tt_, ns_, form, sig, std::false_type{}); };
      if (slots == 4) return with_select_form<4>(*cfg, with);
      if (slots == 8) return with_select_form<8>(*cfg, with);
      return launch(tf_, tt_, ns_, SelAny{}, std::false_type{}, std::false_type{});
    };
    auto launch_256 = [&](auto tf_, auto tt_, auto ns_) -> int32_t {
      auto with = [&](auto form, auto sig) { return launch(tf_, tt_, ns_, form, sig, std::false_type{}); };
      if (slots == 16) return with_select_form<16>(*cfg, with);
      return launch(tf_, tt_, ns_, SelAny{}, std::false_type{}, std::false_type{});
    };
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    constexpr std::integral_constant<int, 4> c4{};
    constexpr std::integral_constant<int, 5> c5{};
    constexpr std::integral_constant<int, 6> c6{};
    if (partial) {
      auto sums = [&](auto tf_, auto ns_) { return launch(tf_, c1, ns_, SelAny{}, std::false_type{}, std::true_type{}); };
      st = tf == 1 || split_e ? sums(c1, c6) : (tf == 2 ? sums(c2, c4) : sums(c4, c2));
    } else if (tf == 1) {
      st = wider ? launch_128(c1, c4, c4) : (wide ? launch_128(c1, c2, c5) : launch_128(c1, c1, c6));
    } else if (tf == 2) {
      st = wide ? launch_256(c2, c2, c3) : launch_256(c2, c1, c4);
    } else {
      st = launch(c4, c1, c2, SelAny{}, std::false_type{}, std::false_type{});
    }
    if (st != SEMMOE_OK) return st;
    SEMMOE_LAUNCH_CHECK();
    if (partial) {
      // adding the parts and selecting in one kernel where the shape has a row form (256 tokens, 128 experts, 16 parts:
      // 3.4 + 6.2 us as two kernels and the gap between them)
      // (one part: the fused kernel's sums, and its order of the bias terms, which its 16-byte loads add to each other first)
      const bool paired_bias = n_parts == 1 && b_g && class_bias && aligned16(b_g) && aligned16(class_bias) && aligned16(logits_out);
      if (launch_sum_select(cfg, s, n_parts, paired_bias, partial, b_g, token_class, class_bias, sel_bias, logits_out, topk_ids,
                            topk_w)) {
        SEMMOE_LAUNCH_CHECK();
        return SEMMOE_OK;
      }
      const size_t n = size_t(cfg->T) * cfg->E;
      hipLaunchKernelGGL(route_reduce_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, *cfg, n_parts, partial,
                         b_g, token_class, class_bias, logits_ws, logits_out);
      SEMMOE_LAUNCH_CHECK();
      return launch_select(cfg, s, logits_ws, sel_bias, topk_ids, topk_w);
    }
    return SEMMOE_OK;
  }
  // fp32: the streamed GEMM (fp32 MFMAs) into the logits buffer, then the selection kernel
  float* logits = logits_out;
  if (!logits) {
    Carver c(ws, ws_bytes);
    logits = c.take<float>(size_t(cfg->T) * cfg->E);
    if (!c.ok) return SEMMOE_EWORKSPACE;
  }
  GemmArgs a{};
  a.X = X; a.ldx = cfg->d;
  a.W = W_r; a.w_group_stride = 0; a.ldw = cfg->d;
  a.N = cfg->E; a.K = cfg->d;
  a.offsets = nullptr; a.q_lo = 0; a.nq = 1; a.n_rows_single = cfg->T;
  a.group_to_weight = nullptr;
  a.out = logits; a.ldo = cfg->E;
  a.b_g = b_g; a.token_class = token_class; a.class_bias = class_bias; a.n_classes = cfg->num_classes;
  st = launch_gemm(kModeLogits, cfg->dtype, a, cfg->T, cfg->T, s);
  if (st != SEMMOE_OK) return st;
  return launch_select(cfg, s, logits, sel_bias, topk_ids, topk_w);
}
