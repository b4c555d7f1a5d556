// kv_quant_write kernels (gfx950): bf16 K/V rows -> int8, int4 or fp8-e4m3 codes + fp32 scales
// in the paged cache (Section 7.2.2, on-the-fly quantization with dynamic scaling), or the
// rows themselves for an unquantized cache.
//
// The unit of work is a run: consecutive tokens of the call with consecutive slots that fall into
// one 16-token sub-block (or, block-scaled fp8, into one cache block, whose tokens share a scale).
// One 64-lane wavefront does a run of one kv head, so every output byte and every scale has exactly
// one writer (the one exception, int4 V words, uses integer atomics, see store_v_nibbles).
//   write_window_kernel  prompts: a wavefront per (window of 16 tokens, kv head) does every run that
//                        starts in its window, K and V
//   write_run_kernel     decode steps, small chunks: a wavefront per (token, kv head, K|V); the one
//                        that has a run's first token does the run (unquantized: each its own token)
//   write_fp8_block_kernel  prompts under block-scaled fp8 with blocks above 16 tokens: a workgroup
//                        per (block_size tokens, kv head), a wavefront per sub-block
// A run of one token is done two channels a lane (in the window kernel int4 and unquantized ones only);
// longer ones by sub-block: 16-byte loads, the 16 rows spread over the lanes so that the codes leave
// in 8- and 16-byte stores (see load_subblock).
// The decisions that fix an integer (the rounding of x/scale) equal fp64's: for a bf16 x and an
// fp32 scale the fp64 quotient is either exactly a rounding tie or at least 2^-25 (relative 2^-29
// for the fp8 midpoints) away from one, so rounding it equals rounding the exact quotient.  The
// scale itself is the quotient absmax/qmax rounded once to fp32.
#include "kvq_quant.h"

namespace kvq {
namespace {

constexpr int kWaves = 4;  // wavefronts per workgroup
constexpr int kBulkTokens = 1024;  // calls with at least this many tokens take the window kernel

// value of a lane, wave-uniform
__device__ inline uint32_t lane_u32(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ inline int64_t lane_i64(int64_t v, int lane) {
  return (int64_t)(((uint64_t)lane_u32((uint32_t)((uint64_t)v >> 32), lane) << 32) |
                   lane_u32((uint32_t)v, lane));
}
// maximum over the wavefront, wave-uniform: DPP inside the four rows of 16 lanes, then scalar
__device__ inline uint32_t wave_max_u32(uint32_t v) {
  v = row_max_u32<16>(v);
  return max(max(lane_u32(v, 0), lane_u32(v, 16)), max(lane_u32(v, 32), lane_u32(v, 48)));
}
// this wavefront's index in the workgroup, in a scalar register
__device__ inline int wave_index() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Nearest E4M3 (finite-only) code of the real y: ties to even, saturating at 448.
__device__ inline uint8_t fp8_code(double y) {
  const uint64_t bits = (uint64_t)__double_as_longlong(y);
  const uint32_t sign = (uint32_t)(bits >> 63) << 7;
  const double a = fabs(y);
  if (a >= 448.0) return (uint8_t)(sign | 0x7E);
  int e = (int)((bits >> 52) & 0x7FF) - 1023;  // floor(log2 a) for normal a
  e = e < -6 ? -6 : e;                         // below 2^-6 the spacing stays 2^-9
  const int r = (int)rint(ldexp(a, 3 - e));    // a / 2^(e-3), exact scaling; r in [0, 16]
  return (uint8_t)(sign | (uint32_t)(((e + 7) << 3) + r - 8));
}

__device__ inline double fp8_value(uint32_t c) {
  const int e = (c >> 3) & 15, m = c & 7;
  const double mag = e == 0 ? ldexp((double)m, -9) : ldexp((double)(8 + m), e - 10);
  return (c & 0x80) ? -mag : mag;
}

// ---- a 16-token sub-block in registers ------------------------------------------------------
// A lane's piece of a token row: D / 16 adjacent channels (16 or 8 bytes), 16 lanes to a row.
template <int D>
using Piece = uint32_t __attribute__((ext_vector_type(D / 32)));

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// largest |bf16| bit pattern among a piece's values
template <int D>
__device__ inline uint32_t piece_absmax(const Piece<D>& raw) {
  ushort2v m = {0, 0};
#pragma unroll
  for (int j = 0; j < D / 32; ++j)
    m = __builtin_elementwise_max(m, __builtin_bit_cast(ushort2v, raw[j] & 0x7FFF7FFFu));
  return m[0] > m[1] ? m[0] : m[1];
}
template <int D>
__device__ inline float bf16_of(const Piece<D>& raw, int e) {  // element e of the piece
  const uint32_t w = raw[e >> 1];
  return (e & 1) ? __uint_as_float(w & 0xFFFF0000u) : __uint_as_float(w << 16);
}

// The rows of a sub-block: lane (c = lane % 16, g = lane / 16) holds channels D/16 c .. of four of
// them.  Which four depends on the cache order the codes go into: for K rows 4 i + g (load i), so
// that each store instruction fills whole quads; for V rows 4 g + i, so that the lane's codes of a
// channel are adjacent in that channel's 16-token row.
// Rows r_lo .. r_hi - 1 of the sub-block are the run's tokens (all 16 for a whole sub-block);
// `src` is where row r_lo's token lies; the other rows are not read.  (The prompt kernels read
// every row once: the loads are non-temporal, which makes them 3-4 % faster.)
template <int D>
__device__ inline void load_subblock(const uint16_t* __restrict__ src, size_t tstride, int kv,
                                     int lane, int r_lo, int r_hi, Piece<D> (&raw)[4]) {
  const int c = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = kv ? 4 * g + i : 4 * i + g;
    raw[i] = Piece<D>{};
    if (r >= r_lo && r < r_hi)
      raw[i] = __builtin_nontemporal_load(
          (const Piece<D>*)(src + (size_t)(r - r_lo) * tstride + (D / 16) * c));
  }
}

// v_permlane32_swap_b32 exchanges the upper half of a with the lower half of b,
// v_permlane16_swap_b32 the odd rows of 16 lanes of a with the even ones of b
__device__ inline void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ inline void swap_rows(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// Bytes lo .. hi - 1 (wave-uniform, and 0 .. 16 at most) of the rows of 16 tokens of channels d, d + 4, ..: whole
// words, and the ends in at most two pieces a word; the bytes around them may be another wavefront's and are
// not touched.
template <int ROWS>
__device__ inline void store_row_parts(uint8_t* __restrict__ row, const uint32_t* word, int lo, int hi) {
  const uint32_t bytes = (1u << hi) - (1u << lo);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t here = (bytes >> (4 * j)) & 15u;
    if (here == 15u) {
#pragma unroll
      for (int x = 0; x < ROWS; ++x) *(uint32_t*)(row + 64 * x + 4 * j) = word[4 * x + j];
    } else if (here != 0u) {
#pragma unroll
      for (int n = 0; n < 4; n += 2) {
        const uint32_t two = (here >> n) & 3u;
#pragma unroll
        for (int x = 0; x < ROWS; ++x) {
          uint8_t* at = row + 64 * x + 4 * j + n;
          const uint32_t w = word[4 * x + j];
          if (two == 3u) *(uint16_t*)at = (uint16_t)(w >> (8 * n));
          else if (two == 1u) at[0] = (uint8_t)(w >> (8 * n));
          else if (two == 2u) at[1] = (uint8_t)(w >> (8 * n + 8));
        }
      }
    }
  }
}

// V codes of a sub-block: word[e] holds the bytes of channel D/16 c + e for the lane's four tokens.
// The four rows of lanes exchange a 4 x 4 square of words, after which a lane has all 16 tokens of
// every fourth channel: a channel's row leaves as one 16-byte store, and the four lanes of a
// channel group fill 64 adjacent bytes.  Of a run shorter than the sub-block the row's bytes lo .. hi - 1 leave in a
// few smaller pieces.  (Byte by byte from the words as they were, 32 stores to 16 lines each, the
// ends of 8 sequences of 685 tokens took as long as all the rest: int8 and e4m3 16 us, now 11.6; 688 tokens 8.
// 64 runs of four tokens 6.7 -> 5.6.)
template <int D>
__device__ inline void store_v_codes(uint8_t* __restrict__ tile, uint32_t (&word)[D / 16], int base,
                                     int bs, int lane, int r_lo, int r_hi) {
  constexpr int CH = D / 16;
  const int c = lane & 15, g = lane >> 4;
#pragma unroll
  for (int e = 0; e < CH; e += 4) {
    swap_halves(word[e], word[e + 2]);
    swap_halves(word[e + 1], word[e + 3]);
    swap_rows(word[e], word[e + 1]);
    swap_rows(word[e + 2], word[e + 3]);
  }
  if (r_lo == 0 && r_hi == 16) {
#pragma unroll
    for (int e = 0; e < CH; e += 4)
      *(uint4*)(tile + v_elem(base, CH * c + e + g, bs, D)) =
          make_uint4(word[e], word[e + 1], word[e + 2], word[e + 3]);
  } else {
    store_row_parts<CH / 4>(tile + v_elem(base, CH * c + g, bs, D), word, r_lo, r_hi);
  }
}

// The fast rounding below marks what it cannot decide; those rows are done again by the single-token
// routines, behind a wait for the stores they overwrite: a loop of little code and few registers, so
// that it costs the common path nothing.  marks[i]: this lane's row of load i is to be done again (for
// K row 4 i + g, for V row 4 g + i); `live`: bit mask of the rows there are.
template <class Redo>
__device__ inline void redo_rows(const bool (&marks)[4], int kv, uint32_t live, Redo redo) {
  if (__builtin_expect(!__any(marks[0] || marks[1] || marks[2] || marks[3]), 1)) return;
  uint32_t rows = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t m = __ballot(marks[i]);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if ((m >> (16 * g)) & 0xFFFFu) rows |= 1u << (kv ? 4 * g + i : 4 * i + g);
  }
  rows &= live;
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  while (rows) {
    redo(__builtin_ctz(rows));
    rows &= rows - 1;
  }
}

// channels E lane .. of a token's row (E = D / 64)
template <int D>
__device__ inline void load_token(const uint16_t* __restrict__ row, int lane, uint32_t (&bits)[D / 64]) {
  if constexpr (D == 128) {
    const uint32_t two = ((const uint32_t*)row)[lane];
    bits[0] = two & 0xFFFFu;
    bits[1] = two >> 16;
  } else {
    bits[0] = row[lane];
  }
}
template <int E>
__device__ inline uint32_t token_absmax(const uint32_t (&bits)[E]) {
  uint32_t a = bits[0] & 0x7FFFu;
  if constexpr (E == 2) a = max(a, bits[1] & 0x7FFFu);
  return a;
}
template <int E>
__device__ inline void store_k(uint8_t* p, const uint8_t (&c)[E]) {
  if constexpr (E == 2) *(uint16_t*)p = (uint16_t)(c[0] | (c[1] << 8));
  else p[0] = c[0];
}

// ---- int8, one scale per (token, kv head) -------------------------------------------------
// Rounding x / s, s = absmax / 127 rounded to fp32, by one multiply-add per element.  With x = mx 2^i and
// absmax = ma 2^j (mx, ma of 8 bits) the unrounded 127 x / absmax meets a half-integer (2k + 1) / 2
// either exactly or with a relative distance of at least 1 / (254 * 255) = 1.5e-5, because
// 254 mx 2^(i-j) and (2k + 1) ma are integers up to a power of two.  s is off by 2^-24 at most, so an
// x / s that is not one of those exact hits stays on its side of the half-integer under any factor
// within 1e-5 of 1 / s; and all exact hits of a row lie on the same side of theirs, the one the
// rounding of s put them on: beyond if s was rounded down, short of it if up.  So the row's factor is
// 1 / s moved by 2^-20 towards that side, and fma(x, factor, 1.5 * 2^23 + 128), whose unit in the last
// place is 1, is the exact quotient's rounding plus 128: the low byte of its bit pattern is the stored
// code.  If s is exact (127 divides ma: a power of two) the factor is exact and ties go to even.
// int4 (7 in place of 127): a distance of 2.8e-4 and a shift of 2^-14; s is exact for every ma that 7
// divides, and where its reciprocal is not, ties are found as the elements on which a factor moved up
// and one moved down disagree: the even one of the two.
template <int QMAX>
constexpr float kShift = QMAX == 127 ? 9.5367432e-07f : 6.1035156e-05f;  // 2^-20, 2^-14
// (below it a scale, or its error, need not be a normal number: such rows are marked)
constexpr float kTinyScale = 8.2718061e-25f;  // 2^-80

struct Factors {
  float up, down;  // the same unless the scale is exact
};
template <int QMAX>
__device__ inline Factors row_factors(uint32_t amax, float s) {
  const float r = __builtin_amdgcn_rcpf(s);
  const float inv = __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);  // (exact for a power of two)
  const float error = __builtin_fmaf(-(float)QMAX, s, bf16_bits_to_float(amax)) * inv;  // 0 or >= 2^-24
  const float side = __builtin_amdgcn_fmed3f(error * 16384.0f, -kShift<QMAX>, kShift<QMAX>);
  Factors f;
  f.up = __builtin_fmaf(inv, QMAX == 7 && error == 0.0f ? kShift<QMAX> : side, inv);
  f.down = QMAX == 7 ? __builtin_fmaf(inv, error == 0.0f ? -kShift<QMAX> : side, inv) : f.up;
  return f;
}
// a word whose low bits are the stored code (int8: code + 128, int4: code + 8)
template <int QMAX>
__device__ inline uint32_t rounded(float x, const Factors& f) {
  constexpr float kMagic = 12582912.0f + (QMAX + 1);  // 1.5 * 2^23 + the offset
  const uint32_t t = __float_as_uint(__builtin_fmaf(x, f.up, kMagic));
  if constexpr (QMAX == 127) {
    return t;
  } else {
    const uint32_t u = __float_as_uint(__builtin_fmaf(x, f.down, kMagic));
    return (t & 1u) ? u : t;
  }
}

// One row's piece, its absmax and scale known.  Returns whether the row has to be done again.
template <int D, int QMAX>
__device__ inline bool round_piece(const Piece<D>& raw, uint32_t amax, float s, uint32_t (&t)[D / 16]) {
  // (an all-zero row: s = 0, and any finite factor gives codes of 0)
  const Factors f = row_factors<QMAX>(amax == 0 ? 0x3F80u : amax, amax == 0 ? 1.0f / QMAX : s);
#pragma unroll
  for (int e = 0; e < D / 16; ++e) t[e] = rounded<QMAX>(bf16_of<D>(raw, e), f);
  return s <= kTinyScale && amax != 0;
}

// one token
template <int D>
__device__ inline void int8_token(const uint32_t (&bits)[D / 64], uint8_t* __restrict__ tile,
                                  float* __restrict__ sp, int kv, int off, int bs, int lane) {
  constexpr int E = D / 64;
  const uint32_t amax = wave_max_u32(token_absmax<E>(bits));  // |bf16| orders like its bit pattern
  const float s = quantum<127>(amax);
  uint8_t c[E];
  if (s > kTinyScale) {
    const Factors f = row_factors<127>(amax, s);
#pragma unroll
    for (int e = 0; e < E; ++e) c[e] = (uint8_t)rounded<127>(bf16_bits_to_float(bits[e]), f);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e)
      c[e] = stored_byte(amax == 0 ? (uint8_t)0 : int8_code(bf16_bits_to_float(bits[e]), s), KVQ_INT8_TOKEN_HEAD);
  }
  if (kv == 0) {
    store_k<E>(tile + k_elem(off, lane * E, bs, D), c);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) tile[v_elem(off, lane * E + e, bs, D)] = c[e];
  }
  if (lane == 0) *sp = s;
}

// the low bytes of four words, packed in order
__device__ inline uint32_t low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_amdgcn_perm(b, a, 0x0c0c0400u) | __builtin_amdgcn_perm(d, c, 0x04000c0cu);
}

// `src` is row r_lo's token, as for load_subblock
template <int D>
__device__ inline void int8_subblock(const Piece<D> (&raw)[4], const uint16_t* __restrict__ src,
                                     size_t tstride, uint8_t* __restrict__ tile,
                                     float* __restrict__ srow, int kv, int off0, int bs, int lane,
                                     int r_lo, int r_hi) {
  constexpr int CH = D / 16;  // channels per lane
  const int c = lane & 15, g = lane >> 4;
  uint32_t amax[4];
  float s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) amax[i] = row_max_u32<16>(piece_absmax<D>(raw[i]));
  quanta<127>(amax, s);
  uint32_t v_words[CH];  // V: per channel, the lane's tokens' codes
  bool marks[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t t[CH];
    marks[i] = round_piece<D, 127>(raw[i], amax[i], s[i], t);
    if (kv == 0) {
      Piece<D / 2> words;
#pragma unroll
      for (int n = 0; n < CH / 4; ++n) words[n] = low_bytes(t[4 * n], t[4 * n + 1], t[4 * n + 2], t[4 * n + 3]);
      const int r = 4 * i + g;
      if (r >= r_lo && r < r_hi) *(Piece<D / 2>*)(tile + k_elem(off0 + r, CH * c, bs, D)) = words;
    } else {
      // the low byte of t[e] becomes byte i of the channel's word
      constexpr uint32_t kInsert[4] = {0x0c0c0c04u, 0x03020400u, 0x03040100u, 0x04020100u};
#pragma unroll
      for (int e = 0; e < CH; ++e)
        v_words[e] = __builtin_amdgcn_perm(t[e], i == 0 ? 0u : v_words[e], kInsert[i]);
    }
  }
  // the sub-block's 16 scales in one store: lane (c = i, group g) writes its row i's
  if (c < 4) {
    const int r = kv ? 4 * g + c : 4 * c + g;
    if (r >= r_lo && r < r_hi) srow[r] = c == 0 ? s[0] : c == 1 ? s[1] : c == 2 ? s[2] : s[3];
  }
  if (kv == 1) store_v_codes<D>(tile, v_words, off0, bs, lane, r_lo, r_hi);
  redo_rows(marks, kv, (1u << r_hi) - (1u << r_lo), [&](int r) {
    uint32_t bits[D / 64];
    load_token<D>(src + (size_t)(r - r_lo) * tstride, lane, bits);
    int8_token<D>(bits, tile, srow + r, kv, off0 + r, bs, lane);
  });
}

// ---- int4, head_dim 128 ---------------------------------------------------------------------
// As int8 with 7 in place of 127 and two codes per byte; a code is stored as the nibble code + 8.
// The 32-bit word / nibble a logical element lives in is given by int4_k_word, int4_v_word and
// int4_nibble.  GROUPED: one scale per 32 adjacent channels instead of one per token and head.

// the low nibbles of two words, 16 bits apart
__device__ inline uint32_t nibble_pair(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, 0x05040100u) & 0x000F000Fu;
}
// Tokens r_lo .. r_hi - 1 of the 8-token word whose first token is `first`, as a nibble mask.
__device__ inline uint32_t nibble_mask(int first, int r_lo, int r_hi) {
  uint32_t m = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (first + e >= r_lo && first + e < r_hi) m |= 15u << (4 * int4_nibble(e));
  return m;
}
// A channel's two V words.  A run that does not fill a word clears and sets only its own nibbles with
// integer atomics: other runs of the same call (a skipped token in mid sub-block, tokens not in
// slot order) are handled by other wavefronts and share the word.  The nibbles of different
// tokens are disjoint, so the result does not depend on the order in which the wavefronts arrive.
__device__ inline void store_v_nibbles(uint32_t* __restrict__ words, uint32_t lo, uint32_t hi,
                                       uint32_t mask_lo, uint32_t mask_hi) {
  if ((mask_lo & mask_hi) == ~0u) {
    *(uint2*)words = make_uint2(lo, hi);
    return;
  }
  if (mask_lo != 0) {
    atomicAnd(words, ~mask_lo);
    atomicOr(words, lo & mask_lo);
  }
  if (mask_hi != 0) {
    atomicAnd(words + 1, ~mask_hi);
    atomicOr(words + 1, hi & mask_hi);
  }
}

// One token.  A lane owns channels 2 lane and 2 lane + 1; K: the four lanes of a quad hold the eight
// codes of one word and combine them with two cross-lane ORs.
template <bool GROUPED>
__device__ inline void int4_token(const uint32_t (&bits)[2], uint8_t* __restrict__ tile,
                                  float* __restrict__ sp, int kv, int off, int lane) {
  uint32_t amax = token_absmax<2>(bits);
  amax = GROUPED ? row_max_u32<16>(amax) : wave_max_u32(amax);
  const float s = quantum<7>(amax);
  const uint32_t n0 = (amax == 0) ? 8u : int4_nib(bf16_bits_to_float(bits[0]), s);
  const uint32_t n1 = (amax == 0) ? 8u : int4_nib(bf16_bits_to_float(bits[1]), s);
  if (kv == 0) {
    // channels 2 lane, 2 lane + 1 are elements 2 (lane % 4) and + 1 of their word
    uint32_t word = (n0 << (4 * (lane & 3))) | (n1 << (4 * ((lane & 3) + 4)));
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0xB1, 0xF, 0xF, false);
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0x4E, 0xF, 0xF, false);
    if ((lane & 3) == 0) *(uint32_t*)(tile + int4_k_word(off, 2 * lane)) = word;
  } else {
    const int so = off & 15, sh = 4 * int4_nibble(so & 7);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      uint32_t* word = (uint32_t*)(tile + int4_v_word(off - so, 2 * lane + e)) + (so >> 3);
      atomicAnd(word, ~(15u << sh));
      atomicOr(word, (e ? n1 : n0) << sh);
    }
  }
  if (GROUPED ? (lane & 15) == 0 : lane == 0) sp[GROUPED ? lane >> 4 : 0] = s;
}

// K (tokens 4 i + g): the lane's eight codes of a token are one whole word.  V (tokens 4 g + i): the
// lane's four tokens of a channel are nibbles 2a, 2a+1, 2a+4 and 2a+5, a = g % 2, of the channel's
// word g / 2; the rows of lanes exchange those parts so that a lane ends up with both words of two
// channels.
template <bool GROUPED>
__device__ inline void int4_subblock(const Piece<128> (&raw)[4], const uint16_t* __restrict__ src,
                                     size_t tstride, uint8_t* __restrict__ tile,
                                     float* __restrict__ srow, int kv, int off0, int lane, int r_lo,
                                     int r_hi) {
  constexpr int NG = GROUPED ? 4 : 1;  // scales per token; a group of 32 channels = 4 lanes
  const int c = lane & 15, g = lane >> 4;
  uint32_t amax[4];
  float s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) amax[i] = row_max_u32<GROUPED ? 4 : 16>(piece_absmax<128>(raw[i]));
  quanta<7>(amax, s);
  bool marks[4];
  uint32_t t[4][8];  // [token i][channel e]: the low nibble is code + 8
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tok = kv ? 4 * g + i : 4 * i + g;
    marks[i] = round_piece<128, 7>(raw[i], amax[i], s[i], t[i]);
    if (tok >= r_lo && tok < r_hi) {
      if (kv == 0)
        *(uint32_t*)(tile + int4_k_word(off0 + tok, 8 * c)) =
            nibble_pair(t[i][0], t[i][1]) | nibble_pair(t[i][2], t[i][3]) << 4 |
            nibble_pair(t[i][4], t[i][5]) << 8 | nibble_pair(t[i][6], t[i][7]) << 12;
      if (GROUPED ? (c & 3) == 0 : c == 0) srow[tok * NG + (GROUPED ? c >> 2 : 0)] = s[i];
    }
  }
  if (kv == 1) {
    uint32_t w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      w[e] = (nibble_pair(t[0][e], t[1][e]) | nibble_pair(t[2][e], t[3][e]) << 4) << (8 * (g & 1));
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // row pairs: channel e + 4 (g % 2), its word g / 2 whole
      swap_rows(w[e], w[e + 4]);
      w[e] |= w[e + 4];
    }
    const uint32_t mask_lo = nibble_mask(0, r_lo, r_hi), mask_hi = nibble_mask(8, r_lo, r_hi);
#pragma unroll
    for (int e = 0; e < 2; ++e) {  // wavefront halves: channel e + 2 (g / 2) + 4 (g % 2), both words
      swap_halves(w[e], w[e + 2]);
      const int d = 8 * c + e + 2 * (g >> 1) + 4 * (g & 1);
      store_v_nibbles((uint32_t*)(tile + int4_v_word(off0, d)), w[e], w[e + 2], mask_lo, mask_hi);
    }
  }
  redo_rows(marks, kv, (1u << r_hi) - (1u << r_lo), [&](int r) {
    uint32_t bits[2];
    load_token<128>(src + (size_t)(r - r_lo) * tstride, lane, bits);
    int4_token<GROUPED>(bits, tile, srow + r * NG, kv, off0 + r, lane);
  });
}

// ---- fp8-e4m3 -------------------------------------------------------------------------------
// one token under a given scale (0x00 under a zero scale)
template <int D>
__device__ inline void fp8_token(const uint32_t (&bits)[D / 64], uint8_t* __restrict__ tile, float s,
                                 int kv, int off, int bs, int lane) {
  constexpr int E = D / 64;
  uint8_t c[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
    c[e] = s > 0.0f ? fp8_code((double)bf16_bits_to_float(bits[e]) / (double)s) : (uint8_t)0;
  if (kv == 0) {
    store_k<E>(tile + k_elem(off, lane * E, bs, D), c);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) tile[v_elem(off, lane * E + e, bs, D)] = c[e];
  }
}

// Rounding x / s to E4M3 with the hardware conversion (v_cvt_pk_fp8_f32: nearest, ties to even, exact
// for every |value| <= 448 including the subnormals and the sign of zero; above 464 it gives NaN),
// without a test per element.  A code boundary is an odd number b of at most 5 bits times a power of two,
// and x has 8 bits.  If x / s comes within 2^-19 (relative) of a boundary, s is that close to some
// mx / b; two different such fractions are 1 / (255 * 31) apart at least, so all elements that come that
// close have the same fraction, and the sign of mx / b - s says for all of them whether x / s lies
// beyond its boundary or short of it.  The 16 values of b are tried by 16 lanes:
//   no fraction near s: any factor within 2^-20 of 1 / s rounds every x as the exact quotient;
//   one, not equal to s (a block scale, absmax / 448 rounded, mostly: b = 7): the factor is 1 / s moved
//   by 2^-20 to the right side;
//   one equal to s: those elements are exact ties.  The product is exact if s is a power of two;
//   otherwise the quotient, corrected once by its remainder, is exact where it is a boundary.
// Scales below 2^-80 or near the end of the fp32 range: all rows are marked and done again.
// CLAMP: values beyond 448 s exist (static scales).
// Rows r_lo .. r_hi - 1 of the 16-token sub-block at block offset `base`, held in `raw` in the order
// load_subblock leaves them (`src` is row r_lo's token), encoded under the scale and stored.
template <int D, bool CLAMP>
__device__ inline void fp8_subblock(const Piece<D> (&raw)[4], const uint16_t* __restrict__ src,
                                    size_t tstride, int kv, uint8_t* __restrict__ tile, int base,
                                    int r_lo, int r_hi, float scale, int bs, int lane) {
  constexpr int CH = D / 16;  // channels per lane
  const int c = lane & 15, g = lane >> 4;
  // (the same in every lane)
  const float s = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(scale)));
  auto convert = [](const float (&q)[4]) {
    const int half = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], half, true);
  };
  // words of four codes: K, words W i .. of row i (W = CH / 4 words of four channels); V, word e the
  // four tokens of channel e
  constexpr int W = CH / 4;
  uint32_t word[CH];
  auto encode = [&](auto quotient) {
    Piece<D> rows[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < D / 32; ++j) {
        // (opaque copies, so that the unpacked values are not kept in registers for every use of this)
        uint32_t bits = raw[i][j];
        asm volatile("" : "+v"(bits));
        rows[i][j] = bits;
      }
#pragma unroll
    for (int w = 0; w < CH; ++w) {
      float q[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        q[n] = quotient(kv == 0 ? bf16_of<D>(rows[w / W], 4 * (w % W) + n) : bf16_of<D>(rows[n], w));
        if constexpr (CLAMP) q[n] = __builtin_amdgcn_fmed3f(q[n], -448.0f, 448.0f);
      }
      word[w] = convert(q);
    }
  };
  bool marks[4] = {false, false, false, false};
  if (!(s > 0.0f)) {  // an all-zero run under a zero scale
#pragma unroll
    for (int w = 0; w < CH; ++w) word[w] = 0;
  } else {
    const float r = __builtin_amdgcn_rcpf(s);
    const float inv = __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);  // (exact for a power of two)
    const float b = (float)(2 * c + 1), p = s * b;
    const uint32_t bits = __float_as_uint(p);  // the bf16 number nearest to b s
    const float near = __uint_as_float((bits + 0x7FFFu + ((bits >> 16) & 1u)) & 0xFFFF0000u);
    const float error = __builtin_fmaf(-b, s, near);  // (sign and zero exact)
    const uint32_t found = (uint32_t)__ballot(fabsf(error) <= p * 1.9073486e-06f) & 0xFFFFu;
    const float side = found ? __uint_as_float(lane_u32(__float_as_uint(error), __builtin_ctz(found))) : 0.0f;
    if (found == 0 || side != 0.0f || (__float_as_uint(s) & 0x7FFFFFu) == 0) {
      const float f = __builtin_fmaf(inv, side > 0.0f ? kShift<127> : side < 0.0f ? -kShift<127> : 0.0f, inv);
      encode([&](float x) { return x * f; });
    } else {
      encode([&](float x) {
        const float q = x * inv;
        return __builtin_fmaf(__builtin_fmaf(-q, s, x), inv, q);
      });
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) marks[i] = !(s > kTinyScale && s < 1e36f);
  }
  if (kv == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + g;
      Piece<D / 2> words;
#pragma unroll
      for (int n = 0; n < W; ++n) words[n] = word[W * i + n];
      if (r >= r_lo && r < r_hi) *(Piece<D / 2>*)(tile + k_elem(base + r, CH * c, bs, D)) = words;
    }
  } else {
    store_v_codes<D>(tile, word, base, bs, lane, r_lo, r_hi);
  }
  redo_rows(marks, kv, (1u << r_hi) - (1u << r_lo), [&](int r) {
    uint32_t bits[D / 64];
    load_token<D>(src + (size_t)(r - r_lo) * tstride, lane, bits);
    fp8_token<D>(bits, tile, s, kv, base + r, bs, lane);
  });
}

// the scale of a block after a run whose largest |bf16| is `amax` was added to it
__device__ inline float grown_scale(float s_prev, uint32_t amax) {
  const float s_run = quantum<448>(amax);
  return s_prev > s_run ? s_prev : s_run;
}

// V bytes of consecutive tokens for one channel are adjacent in the sub-block order: a run of
// tokens is gathered per channel into one 16-byte row image and stored once.
struct RowImage {
  unsigned long long lo = 0, hi = 0;  // bytes 0..7 and 8..15 of a 16-token V row
  __device__ void put(int pos, uint8_t b) {
    if (pos < 8) lo |= (unsigned long long)b << (8 * pos);
    else hi |= (unsigned long long)b << (8 * (pos - 8));
  }
  __device__ uint8_t get(int pos) const {
    return (uint8_t)(pos < 8 ? lo >> (8 * pos) : hi >> (8 * (pos - 8)));
  }
};

// The general routine of block-scaled fp8, K or V: one run of `run` tokens starting at token t0,
// slot0 (any length, any start inside the block), the block's older codes re-expressed where its
// scale grows.  A lane owns D/64 channels of every token.  Taken by single tokens and by runs that
// make a scale grow over older codes.  The new code of an old one depends on the code alone, so
// the wavefront works the 256 of them out once, four per lane in fp64, and looks the block's
// bytes up in `table` (256 bytes of LDS of the wavefront's own).
template <int D>
__device__ inline void fp8_run(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                               uint8_t* __restrict__ cache, float* __restrict__ scales, int H,
                               int bs, int kv, int h, int t0, int64_t slot0, int run, int lane,
                               uint32_t* __restrict__ table) {
  constexpr int E = D / 64;
  const int64_t blk = slot0 >> __builtin_ctz(bs);  // block sizes are powers of two
  const int o_min = (int)(slot0 & (bs - 1));
  const uint16_t* src = (kv ? v : k) + ((size_t)t0 * H + h) * D + lane * E;
  const size_t tstride = (size_t)H * D;
  float* sp = scales + ((size_t)blk * 2 + kv) * H + h;
  const float s_prev = o_min > 0 ? *sp : 0.0f;
  uint32_t amax = 0;
  for (int i = 0; i < run; ++i) {
#pragma unroll
    for (int e = 0; e < E; ++e) amax = max(amax, (uint32_t)src[i * tstride + e] & 0x7FFFu);
  }
  amax = wave_max_u32(amax);
  const float s_new = grown_scale(s_prev, amax);
  // the block's scale grew: the codes stored below the run are re-expressed in the new scale
  const bool regrade = o_min > 0 && s_new > s_prev && s_prev > 0.0f;
  if (regrade) {
    uint32_t four = 0;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const uint32_t c = 4 * lane + n;
      const uint32_t to = (c & 0x7F) == 0x7F  // NaN codes stay
                              ? c
                              : fp8_code(fp8_value(c) * (double)s_prev / (double)s_new);
      four |= to << (8 * n);
    }
    table[lane] = four;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  auto regraded = [&](uint32_t c) -> uint8_t { return ((const uint8_t*)table)[c]; };
  auto encoded = [&](int i, int e) -> uint8_t {
    if (!(s_new > 0.0f)) return 0;
    return fp8_code((double)bf16_bits_to_float(src[i * tstride + e]) / (double)s_new);
  };

  uint8_t* tile = cache + tile_offset(blk, kv, h, H, bs, D);
  if (kv == 0) {
    if (regrade) {
      for (int off = 0; off < o_min; ++off) {
        uint8_t* pc = tile + k_elem(off, lane * E, bs, D);
        uint8_t c[E];
#pragma unroll
        for (int e = 0; e < E; ++e) c[e] = regraded(pc[e]);
        store_k<E>(pc, c);
      }
    }
    for (int i = 0; i < run; ++i) {
      uint8_t c[E];
#pragma unroll
      for (int e = 0; e < E; ++e) c[e] = encoded(i, e);
      store_k<E>(tile + k_elem(o_min + i, lane * E, bs, D), c);
    }
  } else {
    // V: sub-block by sub-block, each channel's 16-token row read (if it holds older codes),
    // updated and stored once
    const int first_sb = regrade ? 0 : (o_min >> 4);
    const int last_sb = (o_min + run - 1) >> 4;
    for (int sb = first_sb; sb <= last_sb; ++sb) {
      const int lo = max(o_min - 16 * sb, 0);             // first new position in this row
      const int hi = min(o_min + run - 16 * sb, 16);      // one past the last new position
      const int old_n = regrade ? min(lo, 16) : 0;        // older codes to re-express: [0, old_n)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        uint8_t* row = tile + v_elem(16 * sb, lane * E + e, bs, D);
        RowImage img;
        if (old_n > 0) {
          const uint4 old = *(const uint4*)row;
          const uint32_t w[4] = {old.x, old.y, old.z, old.w};
#pragma unroll
          for (int j = 0; j < 16; ++j)
            if (j < old_n) img.put(j, regraded((w[j >> 2] >> (8 * (j & 3))) & 0xFFu));
        }
        for (int j = lo; j < hi; ++j) img.put(j, encoded(16 * sb + j - o_min, e));
        const int first = old_n > 0 ? 0 : lo;  // older codes, if re-expressed, end where the new begin
        if (hi - first == 16) {
          *(uint4*)row = make_uint4((uint32_t)img.lo, (uint32_t)(img.lo >> 32), (uint32_t)img.hi,
                                    (uint32_t)(img.hi >> 32));
        } else {
          for (int j = first; j < hi; ++j) row[j] = img.get(j);
        }
      }
    }
  }
  if (lane == 0) *sp = s_new;
}

// ---- unquantized cache: the rows are copied to their slots ---------------------------------
// K: a piece goes out as it came.  V: the four tokens of a channel become two words, and one
// v_permlane16_swap_b32 per word pairs them with the neighbour row's four tokens, so that every
// store is a whole 16-byte half-row.
template <int D>
__device__ inline void plain_subblock(const Piece<D> (&raw)[4], uint16_t* __restrict__ tile, int kv,
                                      int base, int lane, int r_lo, int r_hi) {
  constexpr int CH = D / 16;   // channels per lane
  const int c = lane & 15, g = lane >> 4;
  if (kv == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + g;
      if (r >= r_lo && r < r_hi) *(Piece<D>*)(tile + k_elem16(base + r, CH * c, D)) = raw[i];
    }
    return;
  }
  // channel e's tokens 4 g, 4 g + 1 and 4 g + 2, 4 g + 3
  uint32_t lo[CH], hi[CH];
#pragma unroll
  for (int e = 0; e < CH; ++e) {
    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;  // the halves the channel sits in
    lo[e] = __builtin_amdgcn_perm(raw[1][e >> 1], raw[0][e >> 1], sel);
    hi[e] = __builtin_amdgcn_perm(raw[3][e >> 1], raw[2][e >> 1], sel);
  }
  // even g: channels e of the first half of CH with tokens 0-7 of the half-row, odd g: the second
  uint4 piece[CH / 2];
#pragma unroll
  for (int e = 0; e < CH / 2; ++e) {
    swap_rows(lo[e], lo[e + CH / 2]);
    swap_rows(hi[e], hi[e + CH / 2]);
    piece[e] = make_uint4(lo[e], hi[e], lo[e + CH / 2], hi[e + CH / 2]);
  }
  // (half-rows of a channel: the first 8 tokens', and 8 D elements on the others')
  uint16_t* to = tile + v_elem16(base + 8 * (g >> 1), CH * c + (CH / 2) * (g & 1), D);
  if (r_lo == 0 && r_hi == 16) {
#pragma unroll
    for (int e = 0; e < CH / 2; ++e) *(uint4*)(to + 8 * e) = piece[e];
    return;
  }
  // a run shorter than the sub-block: whole words, and a slot alone at its ends; the others keep their contents.
  // (Slot by slot: 30 k tokens of 13 ragged sequences 45.5 us, now 44; 300 runs of 11 tokens 22, now 19.)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t rows = (((1u << r_hi) - (1u << r_lo)) >> (8 * h)) & 0xFFu;  // (wave-uniform)
    if (rows == 0 || (g >> 1) != h) continue;
    if (rows == 0xFFu) {
#pragma unroll
      for (int e = 0; e < CH / 2; ++e) *(uint4*)(to + 8 * e) = piece[e];
      continue;
    }
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      const uint32_t two = (rows >> t) & 3u;
      if (two == 0) continue;
#pragma unroll
      for (int e = 0; e < CH / 2; ++e) {
        const uint32_t w = t == 0 ? piece[e].x : t == 2 ? piece[e].y : t == 4 ? piece[e].z : piece[e].w;
        if (two == 3u) *(uint32_t*)(to + 8 * e + t) = w;
        else if (two == 1u) to[8 * e + t] = (uint16_t)w;
        else to[8 * e + t + 1] = (uint16_t)(w >> 16);
      }
    }
  }
}

// ---- unquantized rows of many runs ---------------------------------------------------------
// A window of many short runs (a decode step of more than a thousand sequences): run after run, each a
// masked sub-block, is a chain of round trips.  Here the window's rows are requested eight at a time, two
// channels a lane, and every row goes to its own slot.  Lane r + 1 holds row r's slot; `rows`: bit mask
// of the rows to store; `src`: row 0's token, of n.  Single tokens of 8 heads x 128: 1024 33 us run
// after run, 14 like this (9 with a wavefront for each token, head and K|V, which takes prompts 2.7
// times as long), 4096 45 and 28 (25).  (All 16 rows at once 12 us, but then the compiler orders the
// common path differently: a prompt of 30000 tokens 46 us instead of 44.7.)
template <int D>
__device__ inline void scatter_plain(const uint16_t* __restrict__ src, size_t tstride, int n,
                                     uint16_t* __restrict__ cache, int64_t slot, uint32_t rows, int kv,
                                     int h, int H, int bs, int lane) {
  constexpr int E = D / 64;
#pragma unroll 1
  for (int r0 = 0; r0 < 16; r0 += 8) {
    uint32_t bits[8][E];
#pragma unroll
    for (int r = 0; r < 8; ++r)
      load_token<D>(src + (size_t)min(r0 + r, n - 1) * tstride, lane, bits[r]);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (!((rows >> (r0 + r)) & 1u)) continue;
      const int64_t to = lane_i64(slot, r0 + r + 1);
      const int off = (int)(to & (bs - 1));
      uint16_t* elems = cache + tile_offset(to >> __builtin_ctz(bs), kv, h, H, bs, D);
      if constexpr (E == 2) {
        if (kv == 0) {
          *(uint32_t*)(elems + k_elem16(off, lane * 2, D)) = bits[r][0] | bits[r][1] << 16;
          continue;
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e)
        elems[kv ? v_elem16(off, lane * E + e, D) : k_elem16(off, lane * E + e, D)] = (uint16_t)bits[r][e];
    }
  }
}

// ---- the kernels ----------------------------------------------------------------------------

// Where a mode's (block, K|V, head) tile starts, and its scales of block offset `off` on.
template <int MODE, int D>
__device__ inline uint8_t* tile_of(uint8_t* cache, int64_t blk, int kv, int h, int H, int bs) {
  constexpr int RB = MODE == KVQ_BF16_PLAIN ? 2 * D
                     : MODE == KVQ_INT4_TOKEN_HEAD || MODE == KVQ_INT4_GROUP32 ? D / 2 : D;
  return cache + tile_offset(blk, kv, h, H, bs, RB);
}
template <int MODE>
__device__ inline float* scales_of(float* scales, int64_t blk, int kv, int h, int H, int bs, int off) {
  if constexpr (MODE == KVQ_FP8E4M3_TENSOR) return scales + kv;
  const size_t tile = ((size_t)blk * 2 + kv) * H + h;
  if constexpr (MODE == KVQ_FP8E4M3_BLOCK_HEAD) return scales + tile;
  return scales + (tile * bs + off) * (MODE == KVQ_INT4_GROUP32 ? 4 : 1);
}

// One sub-block of a run under every format but block-scaled fp8 (whose scale the caller finds).
template <int MODE, int D>
__device__ inline void store_subblock(const Piece<D> (&raw)[4], const uint16_t* __restrict__ src,
                                      uint8_t* __restrict__ cache, float* __restrict__ scales,
                                      int64_t blk, int kv, int h, int H, int bs, int off0, int lane,
                                      int r_lo, int r_hi) {
  const size_t tstride = (size_t)H * D;
  uint8_t* tile = tile_of<MODE, D>(cache, blk, kv, h, H, bs);
  float* sp = scales_of<MODE>(scales, blk, kv, h, H, bs, off0);
  if constexpr (MODE == KVQ_INT8_TOKEN_HEAD) {
    int8_subblock<D>(raw, src, tstride, tile, sp, kv, off0, bs, lane, r_lo, r_hi);
  } else if constexpr (MODE == KVQ_INT4_TOKEN_HEAD || MODE == KVQ_INT4_GROUP32) {
    int4_subblock<MODE == KVQ_INT4_GROUP32>(raw, src, tstride, tile, sp, kv, off0, lane, r_lo, r_hi);
  } else if constexpr (MODE == KVQ_BF16_PLAIN) {
    plain_subblock<D>(raw, (uint16_t*)tile, kv, off0, lane, r_lo, r_hi);
  } else {
    static_assert(MODE == KVQ_FP8E4M3_TENSOR, "");
    fp8_subblock<D, true>(raw, src, tstride, kv, tile, off0, r_lo, r_hi, *sp, bs, lane);
  }
}

// Prompts: a wavefront per (window of 16 consecutive tokens of the call, kv head) does every run that
// starts in its window, K and V alike, so no wavefront is launched only to find that its token is
// not a run's first, the slots are worked out once (one load: lane i holds the slot of token
// window - 1 + i, and runs end within 15 tokens of the window), and V's rows are on their way
// while K's are encoded.  Everything that is the same for the wavefront sits in scalar registers.
// (Block-scaled fp8 comes here with 16-token blocks only.)
// Bound by memory.  30 k tokens of 8 heads x 128, 16-token blocks, in and out at: int8 38 us = 4.9 TB/s,
// fp8 37 us = 5.0, static fp8 39 us = 4.7, int4 34.5 us = 4.5, bf16 52.7 us = 4.7 (a large copy: 5.0).
// With a test per element for near-ties, 4-byte V stores 128 bytes apart and per-lane index
// arithmetic the same took 54, 54, 69, 66 and 152 us (16 to 31 vector instructions per element; now 5).
template <int MODE, int D>
__global__ __launch_bounds__(kWaves * 64) void write_window_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int64_t* __restrict__ slot_mapping, int32_t num_tokens, uint8_t* __restrict__ cache,
    float* __restrict__ scales, int32_t H, int32_t bs) {
  constexpr bool FP8_BLOCK = MODE == KVQ_FP8E4M3_BLOCK_HEAD;
  __shared__ uint32_t table[FP8_BLOCK ? kWaves : 1][64];
  const int lane = threadIdx.x & 63, wv = wave_index();
  const uint32_t unit = blockIdx.x * kWaves + wv;  // (windows x heads: below 2^32 by the launch's check)
  const uint32_t w = unit / (uint32_t)H;
  if (w >= (uint32_t)((num_tokens + 15) >> 4)) return;
  const int h = (int)(unit - w * (uint32_t)H), w0 = (int)w * 16;
  const int t = w0 - 1 + lane;
  const int64_t slot = lane < 32 && t >= 0 && t < num_tokens ? slot_mapping[t] : -1;
  // token t continues the run of token t - 1 (no slot below 1 does, so the first lane does not)
  const int64_t before = __shfl_up((long long)slot, 1, 64);
  const bool cont = lane > 0 && slot > 0 && (slot & 15) != 0 && slot == before + 1;
  const uint32_t conts = (uint32_t)(__ballot(cont) >> 1);
  uint32_t starts = (uint32_t)(__ballot(slot >= 0 && !cont) >> 1) & 0xFFFFu;
  const size_t tstride = (size_t)H * D;
  if constexpr (MODE == KVQ_BF16_PLAIN) {
    if (__builtin_expect(__builtin_popcount(starts) > 2, 0)) {
      // all runs but the last, which may go on behind the window
      const uint32_t last = 1u << (31 - __builtin_clz(starts)), first = starts & -starts;
      const uint32_t rows = (uint32_t)(__ballot(slot >= 0) >> 1) & (last - first);
      const size_t row0 = ((size_t)w0 * H + h) * D;
      const int n = min(16, num_tokens - w0);
      scatter_plain<D>(k + row0, tstride, n, (uint16_t*)cache, slot, rows, 0, h, H, bs, lane);
      scatter_plain<D>(v + row0, tstride, n, (uint16_t*)cache, slot, rows, 1, h, H, bs, lane);
      starts = last;
    }
  }
  while (starts) {
    const int j = __builtin_ctz(starts);
    starts &= starts - 1;
    const int64_t slot0 = lane_i64(slot, j + 1);
    const int run = 1 + __builtin_ctz(~((uint64_t)conts >> (j + 1)));
    const int64_t blk = slot0 >> __builtin_ctz(bs);  // block sizes are powers of two
    const int so = (int)(slot0 & 15), off0 = (int)(slot0 & (bs - 1)) - so;
    const size_t row0 = ((size_t)(w0 + j) * H + h) * D;
    if constexpr (MODE == KVQ_INT4_TOKEN_HEAD || MODE == KVQ_INT4_GROUP32) {
      if (run == 1) {  // (1024 single tokens of 8 heads: 26.6 us, each as a masked sub-block 45)
        uint32_t k_bits[2], v_bits[2];
        load_token<D>(k + row0, lane, k_bits);
        load_token<D>(v + row0, lane, v_bits);
#pragma unroll
        for (int kv = 0; kv < 2; ++kv)
          int4_token<MODE == KVQ_INT4_GROUP32>(kv ? v_bits : k_bits, tile_of<MODE, D>(cache, blk, kv, h, H, bs),
                                               scales_of<MODE>(scales, blk, kv, h, H, bs, off0 + so), kv,
                                               off0 + so, lane);
        continue;
      }
    }
    Piece<D> k_rows[4], v_rows[4];
    load_subblock<D>(k + row0, tstride, 0, lane, so, so + run, k_rows);
    load_subblock<D>(v + row0, tstride, 1, lane, so, so + run, v_rows);
    if constexpr (!FP8_BLOCK) {
      store_subblock<MODE, D>(k_rows, k + row0, cache, scales, blk, 0, h, H, bs, off0, lane, so, so + run);
      store_subblock<MODE, D>(v_rows, v + row0, cache, scales, blk, 1, h, H, bs, off0, lane, so, so + run);
    } else {
      float* sp[2];
      float s_new[2];
      bool grew = false;  // over older codes of the block: they have to be re-expressed
#pragma unroll
      for (int kv = 0; kv < 2; ++kv) {
        uint32_t amax = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) amax = max(amax, piece_absmax<D>(kv ? v_rows[i] : k_rows[i]));
        sp[kv] = scales_of<MODE>(scales, blk, kv, h, H, bs, off0);
        const float s_prev = so > 0 ? *sp[kv] : 0.0f;
        s_new[kv] = grown_scale(s_prev, wave_max_u32(amax));
        grew |= so > 0 && s_new[kv] > s_prev && s_prev > 0.0f;
      }
      if (grew) {
#pragma unroll 1
        for (int kv = 0; kv < 2; ++kv)
          fp8_run<D>(k, v, cache, scales, H, bs, kv, h, w0 + j, slot0, run, lane, table[wv]);
      } else {
        fp8_subblock<D, false>(k_rows, k + row0, tstride, 0, tile_of<MODE, D>(cache, blk, 0, h, H, bs), off0, so, so + run,
                               s_new[0], bs, lane);
        fp8_subblock<D, false>(v_rows, v + row0, tstride, 1, tile_of<MODE, D>(cache, blk, 1, h, H, bs), off0, so, so + run,
                               s_new[1], bs, lane);
        if (lane == 0) {
          *sp[0] = s_new[0];
          *sp[1] = s_new[1];
        }
      }
    }
  }
}

// Decode steps and small chunks: unit = (token, kv head, K|V); the wavefront of a run's first token does the run
// (block-scaled fp8, whose runs are longer than a sub-block: that of a sub-block's first does the sub-block).  A
// decode step is a chain of round trips behind a launch: the token's row is requested together with the slots (lane i
// holds the slot of token t0 - 1 + i).  Most wavefronts of a chunk end there, so what counts is how many are
// resident: eight to a SIMD (64 registers).  Block-scaled fp8 took 72: 225 runs of four tokens 16.9 us, now 11.6.
template <int MODE, int D>
__global__ __launch_bounds__(kWaves * 64, 8) void write_run_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int64_t* __restrict__ slot_mapping, int32_t num_tokens, uint8_t* __restrict__ cache,
    float* __restrict__ scales, int32_t H, int32_t bs) {
  constexpr bool FP8_BLOCK = MODE == KVQ_FP8E4M3_BLOCK_HEAD;
  constexpr int E = D / 64;  // channels per lane of a single token
  __shared__ uint32_t table[FP8_BLOCK ? kWaves : 1][64];
  const int lane = threadIdx.x & 63, wv = wave_index();
  const uint64_t unit = (uint64_t)blockIdx.x * kWaves + wv;
  const uint32_t heads = 2u * (uint32_t)H;
  const uint64_t token = unit / heads;
  if (token >= (uint64_t)num_tokens) return;
  const uint32_t hk = (uint32_t)(unit - token * heads);
  const int t0 = (int)token, kv = (int)(hk & 1), h = (int)(hk >> 1);
  const uint16_t* src = (kv ? v : k) + ((size_t)t0 * H + h) * D;
  uint32_t bits[E];  // the first token
  load_token<D>(src, lane, bits);
  const int t = t0 - 1 + lane;
  const int64_t slot = t >= 0 && t < num_tokens ? slot_mapping[t] : -1;
  const int64_t slot0 = lane_i64(slot, 1);
  if (slot0 < 0) return;
  if constexpr (MODE == KVQ_BF16_PLAIN) {
    // (nothing ties the tokens of a run together: all of them in parallel, 512 tokens 4.5 us, 6.6 by runs)
    const int64_t to = slot0 >> __builtin_ctz(bs);
    const int at = (int)(slot0 & (bs - 1));
    uint16_t* elems = (uint16_t*)tile_of<MODE, D>(cache, to, kv, h, H, bs);
#pragma unroll
    for (int e = 0; e < E; ++e)
      elems[kv ? v_elem16(at, lane * E + e, D) : k_elem16(at, lane * E + e, D)] = (uint16_t)bits[e];
    return;
  }
  const int span = FP8_BLOCK ? bs : 16;  // a run ends with its block / sub-block
  const int at = (int)(slot0 & (span - 1));
  const bool inside = at > 0 && lane_i64(slot, 0) == slot0 - 1;  // not a run's first token
  if (inside && (!FP8_BLOCK || (at & 15) != 0)) return;
  const uint64_t same = __ballot(lane > 0 && lane <= span - at && slot == slot0 + (lane - 1)) >> 1;
  int run = __builtin_ctzll(~same);  // (63 where every lane's token belongs to it)
  if (FP8_BLOCK && run == 63) {      // block sizes reach 256
    for (int base = 63; base < span - at; base += 64) {
      const int j = base + lane;
      const bool in = j < span - at && t0 + j < num_tokens && slot_mapping[t0 + j] == slot0 + j;
      const uint64_t m = __ballot(in);
      const int n = m == ~0ull ? 64 : __builtin_ctzll(~m);
      run += n;
      if (n < 64) break;
    }
  }
  const int64_t blk = slot0 >> __builtin_ctz(bs);
  const int off = (int)(slot0 & (bs - 1));
  const size_t tstride = (size_t)H * D;
  if constexpr (FP8_BLOCK) {
    int back = 0;  // tokens of the run before this one
    if (inside) {
      for (int base = 0; base < at; base += 64) {
        const int j = base + lane + 1;
        const uint64_t m = __ballot(j <= at && j <= t0 && slot_mapping[max(t0 - j, 0)] == slot0 - j);
        const int n = m == ~0ull ? 64 : __builtin_ctzll(~m);
        back += n;
        if (n < 64) break;
      }
    }
    run += back;
    if (run > 1) {
      // A wavefront per sub-block of the run (that of the sub-block's first token), unless the scale grows
      // over older codes.  The scale needs the absmax of the whole run, which each of them takes for itself,
      // two sub-blocks requested at a time: all of it is small, and nobody waits for anybody.  A scale read
      // when another of the run's wavefronts has stored the new one already gives the new one again.  (One
      // wavefront for the run, sub-block after sub-block: 500 tokens of 8 heads x 128 in blocks of 32, 64 and
      // 128 tokens 10.8, 18.6 and 24.5 us, now 9.5, 11.2 and 15.8; 120 tokens 5.8, 9.2 and 13.1, now 4.8, 5.4
      // and 7.4.  Four sub-blocks requested at a time are faster alone, 12.0 for 500 in blocks of 128, and
      // take the registers of a third of the wavefronts: 900 in blocks of 32 10.4 -> 13.6.)
      const int o_min = off - back, first_sb = o_min >> 4, last_sb = (o_min + run - 1) >> 4;
      const uint16_t* run_src = src - (size_t)back * tstride;
      auto rows_of = [&](int sb, Piece<D> (&raw)[4], int& r_lo, int& r_hi) {
        r_lo = max(o_min - 16 * sb, 0);
        r_hi = min(o_min + run - 16 * sb, 16);
        const uint16_t* first = run_src + (size_t)(16 * sb + r_lo - o_min) * tstride;
        load_subblock<D>(first, tstride, kv, lane, r_lo, r_hi, raw);
        return first;
      };
      float* sp = scales_of<MODE>(scales, blk, kv, h, H, bs, off);
      const float s_prev = o_min > 0 ? *sp : 0.0f;  // (a run from offset 0 starts the block afresh)
      Piece<D> raw[4];
      int r_lo, r_hi;
      const int sb = off >> 4;
      const uint16_t* first = rows_of(sb, raw, r_lo, r_hi);
      uint32_t amax = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) amax = max(amax, piece_absmax<D>(raw[i]));
      for (int x = first_sb; x <= last_sb && first_sb < last_sb; x += 2) {
        Piece<D> some[2][4];
        int lo, hi;
#pragma unroll
        for (int n = 0; n < 2; ++n) rows_of(min(x + n, last_sb), some[n], lo, hi);
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int i = 0; i < 4; ++i) amax = max(amax, piece_absmax<D>(some[n][i]));
      }
      const float s_new = grown_scale(s_prev, wave_max_u32(amax));
      if (!(o_min > 0 && s_new > s_prev && s_prev > 0.0f)) {
        fp8_subblock<D, false>(raw, first, tstride, kv, tile_of<MODE, D>(cache, blk, kv, h, H, bs), 16 * sb, r_lo, r_hi,
                               s_new, bs, lane);
        if (!inside && lane == 0) *sp = s_new;
        return;
      }
      if (inside) return;  // (the run's first wavefront does all of it)
    }
    fp8_run<D>(k, v, cache, scales, H, bs, kv, h, t0, slot0, run, lane, table[wv]);
  } else {
    if (run > 1) {
      Piece<D> raw[4];
      load_subblock<D>(src, tstride, kv, lane, at, at + run, raw);
      store_subblock<MODE, D>(raw, src, cache, scales, blk, kv, h, H, bs, off - at, lane, at, at + run);
      return;
    }
    uint8_t* tile = tile_of<MODE, D>(cache, blk, kv, h, H, bs);
    float* sp = scales_of<MODE>(scales, blk, kv, h, H, bs, off);
    if constexpr (MODE == KVQ_INT8_TOKEN_HEAD) {
      int8_token<D>(bits, tile, sp, kv, off, bs, lane);
    } else if constexpr (MODE == KVQ_INT4_TOKEN_HEAD || MODE == KVQ_INT4_GROUP32) {
      int4_token<MODE == KVQ_INT4_GROUP32>(bits, tile, sp, kv, off, lane);
    } else if constexpr (MODE == KVQ_FP8E4M3_TENSOR) {
      fp8_token<D>(bits, tile, *sp, kv, off, bs, lane);
    }
  }
}

// Prompts under one scale per block with blocks of more than 16 tokens: the block's absmax ties its
// sub-blocks together.  A workgroup of bs / 16 wavefronts owns bs consecutive tokens of the call and
// one kv head, and handles the runs that start among them: wavefront j loads sub-block j of the run
// (K and V, kept in registers), the sub-blocks' absmax values meet in LDS, and every wavefront
// encodes its own sub-block under the block's scale.  A run whose scale would grow over older codes of
// the block goes to the general routine (wavefront 0).  The slots are read once: wavefront j takes 32
// of the 2 bs tokens a run can reach and leaves their slots and two bit masks (token starts a run,
// token continues one) in LDS.  64-token blocks, 30 k tokens: 54 -> 44 us, 4.2 TB/s.  Every wavefront
// takes every barrier: the list of runs comes from LDS and the loops over it are uniform.
template <int D>
__global__ __launch_bounds__(1024) void write_fp8_block_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int64_t* __restrict__ slot_mapping, int32_t num_tokens, uint8_t* __restrict__ cache,
    float* __restrict__ scales, int32_t H, int32_t bs) {
  __shared__ int64_t sh_slot[512];
  __shared__ uint32_t sh_start[16], sh_cont[16];
  __shared__ uint32_t sh_amax[2][16];
  __shared__ uint32_t table[64];
  const int lane = threadIdx.x & 63, wv = wave_index();
  const int nw = bs >> 4;  // wavefronts of the workgroup = sub-blocks of a block
  const int h = (int)(blockIdx.x % (uint32_t)H);
  const int g0 = (int)(blockIdx.x / (uint32_t)H) * bs;  // the workgroup's first token
  {
    const int t = g0 + 32 * wv - 1 + lane;  // (bs <= 256 and g0 < num_tokens: below 2^31)
    const int64_t slot = lane < 33 && t >= 0 && t < num_tokens ? slot_mapping[t] : -1;
    const int64_t before = __shfl_up((long long)slot, 1, 64);
    const bool cont = lane > 0 && slot > 0 && (slot & (bs - 1)) != 0 && slot == before + 1;
    const uint32_t conts = (uint32_t)(__ballot(cont) >> 1);
    const uint32_t starts = (uint32_t)(__ballot(slot >= 0 && !cont) >> 1);
    if (lane > 0 && lane < 33) sh_slot[32 * wv + lane - 1] = slot;
    if (lane == 0) {
      sh_start[wv] = starts;
      sh_cont[wv] = conts;
    }
  }
  __syncthreads();
  const size_t tstride = (size_t)H * D;
  // (bs is 32 at least, so the bs tokens whose runs are this workgroup's are whole words)
  for (int ww = 0; ww < bs >> 5; ++ww) {
    uint32_t starts = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh_start[ww]);
    while (starts) {
      const int j0 = 32 * ww + __builtin_ctz(starts);  // the run's first token, from g0
      starts &= starts - 1;
      const int64_t slot0 = lane_i64(sh_slot[j0], 0);
      const int o_min = (int)(slot0 & (bs - 1));
      int run = 1;  // (it ends with its block at the latest: fewer than bs tokens follow)
      for (int next = j0 + 1; next < 2 * bs;) {
        const uint32_t word = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh_cont[next >> 5]) >> (next & 31);
        const int room = 32 - (next & 31), n = word == ~0u ? 32 : __builtin_ctz(~word);
        run += min(n, room);
        next += room;
        if (n < room) break;
      }
      const int64_t blk = slot0 >> __builtin_ctz(bs);
      float* sp[2] = {scales + ((size_t)blk * 2 + 0) * H + h, scales + ((size_t)blk * 2 + 1) * H + h};
      // this wavefront's sub-block of the run: its valid rows, where its first valid row's
      // token lies
      const int nsb = ((o_min + run + 15) >> 4) - (o_min >> 4);
      const bool mine = wv < nsb;
      const int base = (o_min & ~15) + 16 * wv;
      const int r_lo = max(o_min - base, 0), r_hi = min(o_min + run - base, 16);
      Piece<D> k_rows[4], v_rows[4];
      uint32_t amax[2] = {0, 0};
      // (a run from offset 0 starts the block afresh)
      const float s_prev[2] = {o_min > 0 ? *sp[0] : 0.0f, o_min > 0 ? *sp[1] : 0.0f};
      const size_t row = ((size_t)(g0 + j0 + (base + r_lo - o_min)) * H + h) * D;
      if (mine) {
        load_subblock<D>(k + row, tstride, 0, lane, r_lo, r_hi, k_rows);
        load_subblock<D>(v + row, tstride, 1, lane, r_lo, r_hi, v_rows);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          amax[0] = max(amax[0], piece_absmax<D>(k_rows[i]));
          amax[1] = max(amax[1], piece_absmax<D>(v_rows[i]));
        }
        amax[0] = wave_max_u32(amax[0]);
        amax[1] = wave_max_u32(amax[1]);
      }
      if (lane == 0) {
        sh_amax[0][wv] = amax[0];
        sh_amax[1][wv] = amax[1];
      }
      __syncthreads();
      // (wavefront 0 stores the scales behind this barrier, when every wavefront has read the old ones)
      float s_new[2];
      bool grew = false;  // over older codes: they have to be re-expressed
#pragma unroll
      for (int kv = 0; kv < 2; ++kv) {
        const uint32_t all = row_max_u32<16>((lane & 15) < nw ? sh_amax[kv][lane & 15] : 0u);
        s_new[kv] = grown_scale(s_prev[kv], lane_u32(all, 0));
        grew |= o_min > 0 && s_new[kv] > s_prev[kv] && s_prev[kv] > 0.0f;
      }
      if (!grew) {
        if (mine) {
          fp8_subblock<D, false>(k_rows, k + row, tstride, 0, cache + tile_offset(blk, 0, h, H, bs, D), base, r_lo, r_hi,
                                 s_new[0], bs, lane);
          __builtin_amdgcn_sched_barrier(0);
          fp8_subblock<D, false>(v_rows, v + row, tstride, 1, cache + tile_offset(blk, 1, h, H, bs, D), base, r_lo, r_hi,
                                 s_new[1], bs, lane);
        }
        if (wv == 0 && lane == 0) {
          *sp[0] = s_new[0];
          *sp[1] = s_new[1];
        }
      } else if (wv == 0) {
#pragma unroll 1
        for (int kv = 0; kv < 2; ++kv)
          fp8_run<D>(k, v, cache, scales, H, bs, kv, h, g0 + j0, slot0, run, lane, table);
      }
      __syncthreads();  // (the absmax words are written again for the next run)
    }
  }
}

}  // namespace

hipError_t launch_write(const void* k, const void* v, const int64_t* slot_mapping,
                        int32_t num_tokens, void* cache, float* scales,
                        const kvq_cache_desc_t& desc, hipStream_t stream) {
  const uint16_t* kk = (const uint16_t*)k;
  const uint16_t* vv = (const uint16_t*)v;
  uint8_t* c = (uint8_t*)cache;
  const int32_t H = desc.num_kv_heads, bs = desc.block_size;
  // many tokens (a prompt): a wavefront per window of 16 tokens; few (a decode step): a
  // wavefront per token, so that runs are handled in parallel rather than one after another (a chunk of
  // 512 tokens takes 11 us a call either way, of which 10 are the caller's; token after token it took 31)
  const bool bulk = num_tokens >= kBulkTokens;
#define KVQ_LAUNCH_WRITE(KERNEL, GRID, BLOCK)                                                       \
  hipLaunchKernelGGL(KERNEL, dim3((unsigned)(GRID)), dim3(BLOCK), 0, stream, kk, vv, slot_mapping,   \
                     num_tokens, c, scales, H, bs)
  if (bulk && desc.mode == KVQ_FP8E4M3_BLOCK_HEAD && bs > 16) {
    // a workgroup per (block_size consecutive tokens, head), a wavefront per sub-block
    const int64_t groups = ((int64_t)num_tokens + bs - 1) / bs;
    if (desc.head_dim == 128) KVQ_LAUNCH_WRITE(write_fp8_block_kernel<128>, groups * H, bs / 16 * 64);
    else KVQ_LAUNCH_WRITE(write_fp8_block_kernel<64>, groups * H, bs / 16 * 64);
    return hipGetLastError();
  }
  const int64_t units = bulk ? ((int64_t)num_tokens + 15) / 16 * H : (int64_t)num_tokens * H * 2;
  const int64_t grid = (units + kWaves - 1) / kWaves;
#define KVQ_LAUNCH_MODE(MODE, DD)                                                                   \
  if (bulk) KVQ_LAUNCH_WRITE((write_window_kernel<MODE, DD>), grid, kWaves * 64);                    \
  else KVQ_LAUNCH_WRITE((write_run_kernel<MODE, DD>), grid, kWaves * 64)
#define KVQ_LAUNCH_DIMS(MODE)                                                                       \
  if (desc.head_dim == 128) {                                                                       \
    KVQ_LAUNCH_MODE(MODE, 128);                                                                     \
  } else {                                                                                          \
    KVQ_LAUNCH_MODE(MODE, 64);                                                                      \
  }
  switch (desc.mode) {
    case KVQ_INT8_TOKEN_HEAD: KVQ_LAUNCH_DIMS(KVQ_INT8_TOKEN_HEAD) break;
    case KVQ_FP8E4M3_BLOCK_HEAD: KVQ_LAUNCH_DIMS(KVQ_FP8E4M3_BLOCK_HEAD) break;
    case KVQ_FP8E4M3_TENSOR: KVQ_LAUNCH_DIMS(KVQ_FP8E4M3_TENSOR) break;
    case KVQ_BF16_PLAIN: KVQ_LAUNCH_DIMS(KVQ_BF16_PLAIN) break;
    // (int4 comes with head_dim 128 only)
    case KVQ_INT4_TOKEN_HEAD: KVQ_LAUNCH_MODE(KVQ_INT4_TOKEN_HEAD, 128); break;
    default: KVQ_LAUNCH_MODE(KVQ_INT4_GROUP32, 128); break;
  }
#undef KVQ_LAUNCH_DIMS
#undef KVQ_LAUNCH_MODE
#undef KVQ_LAUNCH_WRITE
  return hipGetLastError();
}

}  // namespace kvq
