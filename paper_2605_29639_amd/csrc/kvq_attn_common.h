// Device helpers shared by the attention kernels (kvq_attn.hip, kvq_prefill.hip): vector
// types, stored codes -> f16, the cross-lane pieces of the softmax.
#pragma once

#include <utility>

#include "kvq_internal.h"

namespace kvq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef short short2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr float kPOffset = 10.0f;   // probabilities are scaled by 2^10 (cancels in acc / l)
constexpr float kMinVScale = 7.888609052210118e-31f;  // 2^-100

// Cross-lane scans and reductions on the DPP network (no LDS round trips): Hillis-Steele
// inside each row of 16 lanes (row_shr 1, 2, 4, 8), then the last lane of row 0 / row 2 into
// row 1 / row 3 (row_bcast:15) and lane 31 into rows 2 and 3 (row_bcast:31).  Lanes a step does
// not reach receive the operation's identity.  Lane 63 ends up holding the reduction.
template <class Op>
__device__ inline int dpp_scan_bits(int v, int identity, Op op) {
#define KVQ_DPP_STEP(CTRL, ROWS) \
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, CTRL, ROWS, 0xF, false))
  KVQ_DPP_STEP(0x111, 0xF);  // row_shr:1
  KVQ_DPP_STEP(0x112, 0xF);  // row_shr:2
  KVQ_DPP_STEP(0x114, 0xF);  // row_shr:4
  KVQ_DPP_STEP(0x118, 0xF);  // row_shr:8
  KVQ_DPP_STEP(0x142, 0xA);  // row_bcast:15 into rows 1 and 3
  KVQ_DPP_STEP(0x143, 0xC);  // row_bcast:31 into rows 2 and 3
#undef KVQ_DPP_STEP
  return v;
}
__device__ inline int wave_incl_scan(int v) {
  return dpp_scan_bits(v, 0, [](int a, int b) { return a + b; });
}
__device__ inline int lane_value(int v, int lane_index) {  // lane_index wave-uniform
  return __builtin_amdgcn_readlane(v, lane_index);
}
__device__ inline int wave_sum(int v) { return lane_value(wave_incl_scan(v), 63); }
__device__ inline int wave_min(int v) {
  return lane_value(dpp_scan_bits(v, 0x7FFFFFFF, [](int a, int b) { return a < b ? a : b; }), 63);
}

template <class F, int... Is>
__device__ inline void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}
// value of lane I of the caller's 16-lane row
template <int I>
__device__ inline float row_bcast(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x150 + I, 0xF, 0xF, true));
}

// value of the lane I places before the caller's, around its 16-lane row
template <int I>
__device__ inline float row_ror(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + I, 0xF, 0xF, true));
}

// Over the four lanes that share lane % 16: v_permlane32_swap_b32 and v_permlane16_swap_b32 of a value with
// itself leave it beside the value 32 (16) lanes away, without the round trip through LDS of a shuffle,
// which nothing hides where one or two wavefronts run on a SIMD.
template <class Op>
__device__ inline float xor16_reduce(float v, Op op) {
  const uint32_t u = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t w = __float_as_uint(op(__uint_as_float(h[0]), __uint_as_float(h[1])));
  const auto r = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float xor16_max(float v) {
  return xor16_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ inline float xor16_sum(float v) {
  return xor16_reduce(v, [](float a, float b) { return a + b; });
}

// Four stored code bytes (one dword) -> four f16, in byte order.
template <int MODE>
__device__ inline void cvt4(uint32_t x, half2v& lo, half2v& hi) {
  if constexpr (MODE == KVQ_INT8_TOKEN_HEAD) {
    // stored byte u = code + 128; 0x6400 | u is the f16 1024 + u, so subtracting 1152 gives code
    const uint32_t a = __builtin_amdgcn_perm(0x64646464u, x, 0x04010400u);
    const uint32_t b = __builtin_amdgcn_perm(0x64646464u, x, 0x04030402u);
    const half2v bias = {(_Float16)1152.0f, (_Float16)1152.0f};
    lo = __builtin_bit_cast(half2v, a) - bias;
    hi = __builtin_bit_cast(half2v, b) - bias;
  } else {
    // gfx950's packed e4m3 -> f16 conversion (exact); NaN codes must not reach it as V data
    lo = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x, 1.0f, false);
    hi = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x, 1.0f, true);
  }
}

// Eight stored int4 nibbles (code + 8) of one word -> eight f16 codes; element 2i comes from
// nibble i, element 2i + 1 from nibble i + 4.  An AND-OR drops two nibbles, 16 bits apart,
// into the mantissas of a pair of f16 1024.0: nibbles at bits 0-3 give 1024 + n, nibbles at
// bits 4-7 give 1024 + 16 n; one packed add or fused multiply-add turns either into n - 8.
__device__ inline half8 cvt_int4(uint32_t x) {
  const half2v k1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
  const half2v k16th = {(_Float16)0.0625f, (_Float16)0.0625f};
  const half2v k72 = {(_Float16)72.0f, (_Float16)72.0f};
  const uint32_t y = x >> 8;
  const half2v a = __builtin_bit_cast(half2v, (x & 0x000F000Fu) | 0x64006400u) - k1032;
  const half2v b = __builtin_bit_cast(half2v, (x & 0x00F000F0u) | 0x64006400u) * k16th - k72;
  const half2v c = __builtin_bit_cast(half2v, (y & 0x000F000Fu) | 0x64006400u) - k1032;
  const half2v d = __builtin_bit_cast(half2v, (y & 0x00F000F0u) | 0x64006400u) * k16th - k72;
  half8 r;
  r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
  r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
  return r;
}

template <int MODE>
__device__ inline half8 cvt8(uint32_t x0, uint32_t x1) {
  half2v a, b, c, d;
  cvt4<MODE>(x0, a, b);
  cvt4<MODE>(x1, c, d);
  half8 r;
  r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
  r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
  return r;
}

// Online softmax of one 64-token group for NT tiles of 16 query rows, shared by the streaming
// and the many-row kernels.  In: S, the raw contractions K.q in the accumulator layout (lane
// (row n, sub-block g) holds the 16 tokens of sub-block g); the scales as skp = K scale * softmax
// scale * log2(e), lsv = log2(V scale), rsv = 1 / V scale; pos_lane = position of the lane's first
// token; nrow = causal length of the lane's row per tile.  Token-scaled formats have them in LDS:
// `scales` points at the lane's 16 tokens' skp, then lsv, then rsv, each array 64 floats long.  The 16
// lanes of a row read the same address, a broadcast, so a logit costs one multiply-add (as row
// broadcasts riding on a multiply and an add they cost two instructions of the slower DPP form: the
// many-row kernel 406 -> 396 us int8, 351 -> 341 int4; the two-tile streaming kernel 152 -> 149).  The
// other formats have one skp, lsv, rsv per lane: the maximum is taken of the raw contractions and the exponent is one multiply-add.  Group-scaled int4: S already
// holds the logits (plus lsv), and is left holding the probabilities in fp32 for its caller to scale
// once more.
// Out: pb, the probabilities times the V scale as the B operand of P.V (f16 scaled by 2^10, or two
// bf16 terms for an unquantized cache); the running maximum m_run (of logit + lsv, base 2) and sum
// l_run are updated and acc is rescaled when a maximum moved.
// TAIL: some row's causal length ends inside the group, so positions are masked.
// (An unquantized cache's factor is not negative: its caller puts the sign of the softmax scale into q.
// The test and its branch between QK^T and the softmax cost the two-tile streaming kernel 6 %.)
// The kernel for 256 rows takes its three parts apart: the first runs under its matrix instructions.
template <int MODE, bool TAIL>
struct SoftmaxForm {
  static constexpr bool PLAIN = MODE == KVQ_BF16_PLAIN;
  static constexpr bool FP8 = MODE == KVQ_FP8E4M3_BLOCK_HEAD || MODE == KVQ_FP8E4M3_TENSOR;
  static constexpr bool GROUPED = MODE == KVQ_INT4_GROUP32;
  static constexpr bool TOKEN_SCALE = MODE == KVQ_INT8_TOKEN_HEAD || MODE == KVQ_INT4_TOKEN_HEAD || GROUPED;
  static constexpr bool RAW = !TOKEN_SCALE && !TAIL;  // S stays the raw contraction, its factor >= 0
  static constexpr bool kLogits = TOKEN_SCALE && !GROUPED;  // from S by softmax_logits
};
constexpr int kScalePitch = 16;  // floatx4s per array of scales

// Part 1: quad u of the lane's tokens (its K scales k4, logarithms of the V scales l4): S becomes the
// logits where the format needs it, mx their maximum so far.
template <int MODE, int NT, bool TAIL>
__device__ inline void softmax_logits(floatx4 (&S)[NT][4], int u, const floatx4& k4, const floatx4& l4,
                                      float skp, float lsv, int pos_lane, const int (&nrow)[NT],
                                      float (&mx)[NT]) {
  using F = SoftmaxForm<MODE, TAIL>;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float z = S[nt][u][i];
      if constexpr (F::kLogits) z = __builtin_fmaf(z, k4[i], l4[i]);
      else if constexpr (TAIL && !F::GROUPED) z = __builtin_fmaf(z, skp, lsv);
      if constexpr (TAIL) z = (pos_lane + 4 * u + i < nrow[nt]) ? z : -INFINITY;
      if constexpr (!F::RAW) S[nt][u][i] = z;
      mx[nt] = fmaxf(mx[nt], z);
    }
}

// Part 2: the running maxima, the factors alpha the accumulators shrink by, and what part 3 subtracts.
template <int MODE, int NT, bool TAIL>
__device__ inline void softmax_maxima(const float (&mx)[NT], float skp, float lsv, float (&m_run)[NT],
                                      float (&alpha)[NT], float (&msub)[NT]) {
  using F = SoftmaxForm<MODE, TAIL>;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float m_here = F::RAW ? __builtin_fmaf(mx[nt], skp, lsv) : mx[nt];
    const float m_new = fmaxf(m_run[nt], xor16_max(m_here));
    const float m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
    alpha[nt] = __builtin_amdgcn_exp2f(m_run[nt] - m_safe);
    m_run[nt] = m_new;
    msub[nt] = F::RAW ? lsv - (m_safe - kPOffset) : m_safe - kPOffset;
  }
}

// Part 3: probabilities and sums.  AHEAD: r_all holds the lane's 16 reciprocals of the V scales, else
// they are read from `scales` as they are needed.
template <int MODE, int NT, bool TAIL, bool AHEAD, class Operand, int NP>
__device__ inline void softmax_probabilities(floatx4 (&S)[NT][4], const floatx4* scales, const floatx4 (&r_all)[4],
                                             float skp, float rsv, const float (&alpha)[NT],
                                             const float (&msub)[NT], float (&l_run)[NT], Operand (&pb)[NT][NP]) {
  using F = SoftmaxForm<MODE, TAIL>;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float lsum = 0.0f;
    [[maybe_unused]] uint32_t hi_bits[16];
    [[maybe_unused]] float rest[16];
    [[maybe_unused]] floatx4 r4[2];
    constexpr bool READ = F::TOKEN_SCALE && !AHEAD;
    if constexpr (READ) r4[0] = scales[2 * kScalePitch];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if constexpr (READ) {
        if (u < 3) r4[(u + 1) & 1] = scales[2 * kScalePitch + u + 1];
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tix = 4 * u + i;
        const float pr = __builtin_amdgcn_exp2f(F::RAW ? __builtin_fmaf(S[nt][u][i], skp, msub[nt])
                                                       : S[nt][u][i] - msub[nt]);
        if constexpr (F::TOKEN_SCALE) lsum = __builtin_fmaf(pr, AHEAD ? r_all[u][i] : r4[u & 1][i], lsum);
        else lsum += pr;
        if constexpr (F::PLAIN) {
          // bf16 keeps 8 bits of a probability: it goes in as two terms, the value cut to bf16 and
          // the (exactly representable) rest rounded to bf16, 16 bits in all.  (Rounded, not cut: a
          // row's largest probability comes out a last place below or above 2^10, and cut it would
          // lose up to 2^-16 of itself, which is a peaked row's whole error.)
          hi_bits[tix] = __float_as_uint(pr) & 0xFFFF0000u;
          rest[tix] = pr - __uint_as_float(hi_bits[tix]);
        } else if constexpr (F::GROUPED) {
          S[nt][u][i] = pr;
        } else {
          pb[nt][tix >> 3][tix & 7] = (_Float16)pr;
        }
      }
      if constexpr (READ) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (F::PLAIN) {
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        uintx4 ph, pl;
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // two tokens' bf16 terms to a word
          const int t = 8 * hf + 2 * e;
          ph[e] = __builtin_amdgcn_perm(hi_bits[t + 1], hi_bits[t], 0x07060302u);
          pl[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{rest[t], rest[t + 1]}), bf16x2));
        }
        pb[nt][hf] = __builtin_bit_cast(bf16x8, ph);
        pb[nt][2 + hf] = __builtin_bit_cast(bf16x8, pl);
      }
    }
    if constexpr (F::FP8) lsum *= rsv;  // one scale per lane
    l_run[nt] = __builtin_fmaf(l_run[nt], alpha[nt], lsum);
  }
}

// (per 16-row tile: a tile none of whose rows' maxima moved keeps its accumulators as they are)
template <int NT, int DT>
__device__ inline void softmax_rescale(const float (&alpha)[NT], floatx4 (&acc)[NT][DT]) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (__any(alpha[nt] != 1.0f)) {
#pragma unroll
      for (int tt = 0; tt < DT; ++tt) acc[nt][tt] *= alpha[nt];
    }
  }
}

template <int MODE, int NT, int DT, bool TAIL, class Operand, int NP>
__device__ inline void online_softmax(floatx4 (&S)[NT][4], const floatx4* scales, float skp, float lsv,
                                      float rsv, int pos_lane, const int (&nrow)[NT],
                                      float (&m_run)[NT], float (&l_run)[NT],
                                      floatx4 (&acc)[NT][DT], Operand (&pb)[NT][NP]) {
  using F = SoftmaxForm<MODE, TAIL>;
  float mx[NT], alpha[NT], msub[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) mx[nt] = -INFINITY;
  if constexpr (F::RAW && !F::PLAIN) {
    if (__any(skp < 0.0f)) {  // (a negative softmax scale, or static scale)
      const float sign = skp < 0.0f ? -1.0f : 1.0f;
      skp *= sign;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int u = 0; u < 4; ++u) S[nt][u] *= sign;
    }
  }
  // (the next four tokens' scales are requested while these are used, and no earlier: registers)
  [[maybe_unused]] floatx4 k4[2], l4[2];
  if constexpr (F::kLogits) {
    k4[0] = scales[0];
    l4[0] = scales[kScalePitch];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if constexpr (F::kLogits) {
      if (u < 3) {
        k4[(u + 1) & 1] = scales[u + 1];
        l4[(u + 1) & 1] = scales[kScalePitch + u + 1];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    softmax_logits<MODE, NT, TAIL>(S, u, k4[u & 1], l4[u & 1], skp, lsv, pos_lane, nrow, mx);
    if constexpr (F::kLogits) __builtin_amdgcn_sched_barrier(0);
  }
  softmax_maxima<MODE, NT, TAIL>(mx, skp, lsv, m_run, alpha, msub);
  const floatx4 none[4] = {};
  softmax_probabilities<MODE, NT, TAIL, false>(S, scales, none, skp, rsv, alpha, msub, l_run, pb);
  softmax_rescale<NT, DT>(alpha, acc);
}

}  // namespace
}  // namespace kvq
