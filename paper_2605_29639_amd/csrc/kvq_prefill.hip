// paged_decode_attn for many query rows per kv head (a chunk of a prompt attending over its
// quantized prefix and itself, Section 2's prefill phase fed from the Section 7.2.2 cache).
//
// With many query rows per kv head (128 and more; from 33 on where the plan finds it faster)
// the work is arithmetic, not memory traffic, and what has to be shared is the dequantization:
// the streaming kernel converts a group's codes once per 32 rows, these kernels once per 128 or 256.  A
// workgroup of four wavefronts (attn_rows_kernel) owns 128 query rows of one (sequence, kv head) and walks
// the context from position 0 to the last position any of its rows may see, or a piece of it where the call
// has too few such workgroups to fill the chip or some contexts are far longer than others (see
// context_piece and merge_kernel below).  Per 64-token group each wavefront loads a quarter of the K and V
// codes, converts them to f16 and puts them in LDS in the order the matrix instruction wants its A operand
// (one 16-byte read per lane and instruction, no bank conflicts); after a barrier every wavefront runs
// QK^T, the online softmax and P.V for its own 32 rows against the shared operands.  LDS holds two groups,
// so one barrier per group suffices: while a group is consumed, the next one's codes are in
// flight and are converted into the other half.
//
// A wavefront issues one vector instruction in 4.4 cycles, whatever its neighbour does, and a matrix
// instruction keeps the matrix unit busy for 16: what a wavefront can do under its own matrix instructions
// is free.  So the conversions of the next group's codes are dealt out under P.V and the logits of the first
// tokens under the contraction of the last ones (sched_group_barrier; the conversions are pinned by an
// empty asm, and the loop has no branch around a matrix phase: code that two branches share is moved ahead
// of both, and the wait for its loads with it).  Against a kernel that did one after the other, 32 / 8 heads:
// 3 x 1000 tokens over 3000 int8 183 -> 170 us, e4m3 163 -> 154, bf16 212 -> 197, int4 183 -> 175; 16 x 33 over
// 2000 61.8 -> 55.5, 56.2 -> 52.2, 69.2 -> 63.1, 62.9 -> 58.5; one workgroup alone with the last, long context of a batch,
// 398 x 64 tokens, one over 9807 and the rest over 180: 273 -> 249, 248 -> 235, 309 -> 281, 277 -> 257.
//
// The arithmetic (logits in base 2 with the K scale applied after the contraction, V scale
// folded into the probability, f16 probabilities scaled by 2^10, masks) is the streaming
// kernel's, and so is the treatment of an unquantized cache: its bf16 rows are the operands
// as they are (copied to LDS, no conversion) and a probability enters P.V as two bf16 terms.
#include "kvq_attn_common.h"

namespace kvq {
namespace {

constexpr int kWavesPerGroup = 4;  // (the kernels for 128 rows)
static_assert(kRowsPerWorkgroup == kWavesPerGroup * 32, "a wavefront owns two 16-row tiles");
static_assert(kWideRows == 2 * kRowsPerWorkgroup, "twice the wavefronts");

// minimum over the wavefront (by shuffles: with a result the compiler knows to be uniform it makes two
// copies of the PREFIX kernel's loop and spills)
__device__ inline int wave_min_int(int v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v = min(v, __shfl_xor(v, d, 64));
  return v;
}

// A workgroup's place among the pieces the contexts are cut into.
struct Piece {
  int b, chunk, pieces;  // chunk of `pieces` of sequence b's context
  int extra;             // pieces beyond the first ones of their sequences that come before this one
};

// The f-th piece of the batch.  Decided here, from the lengths themselves, because the host has only an
// upper bound on them: sequences are cut into pieces of k groups, the smallest k (p.piece_min,
// p.piece_share of all groups at least) that makes no more than p.extra_pieces cuts.  So a batch of equal
// contexts is cut evenly, one long context among short ones is cut alone, and short ones are left
// whole however large the declared bound.  Every wavefront works it out for itself, a round trip
// ahead of its first code.  `leave` (wave-uniform): also store the extra pieces before every
// sequence, for the merge.  Returns false for a piece that does not exist.
__device__ inline bool context_piece(const AttnArgs& p, int f, bool leave, Piece& piece) {
  const int lane = threadIdx.x & 63, B = p.batch, E = p.extra_pieces;
  const int32_t* __restrict__ seq_lens = p.seq_lens;
  if (B == 1) {  // (the rule below, on scalars)
    const int g = (seq_lens[0] + 63) >> 6;
    const int k = max(max(p.piece_min, (int)((float)g * p.piece_share)), (g + E) / (E + 1));
    piece = Piece{0, f, g > 0 ? (g - 1) / k + 1 : 1, max(f - 1, 0)};
    if (leave && lane < 2) p.ws_prefix[lane] = lane == 0 ? 0 : piece.pieces - 1;
    return f < piece.pieces;
  }
  auto groups = [&](int i) { return i < B ? (seq_lens[i] + 63) >> 6 : 0; };
  const int own = groups(lane);  // (up to 64 sequences: a lane each, and no further loads)
  int total = own, top = own;
  for (int i = lane + 64; i < B; i += 256) {
    const int g[4] = {groups(i), groups(i + 64), groups(i + 128), groups(i + 192)};
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      total += g[n];
      top = max(top, g[n]);
    }
  }
  total = wave_sum(total);
  top = -wave_min(-top);
  int k = max(p.piece_min, (int)((float)total * p.piece_share));
  if (B > 64) {
    k = max(k, (total + E - 1) / E);  // (a sequence of g groups is cut (g - 1) / k times)
  } else {
    k = max(k, (total + E + B - 1) / (E + B));  // (no smaller one can do)
    while (k < top && wave_sum(own > 0 ? (own - 1) / k : 0) > E) k += max(1, k >> 3);
  }
  if (k >= top) {  // nothing to cut
    if (leave)
      for (int i = lane; i <= B; i += 64) p.ws_prefix[i] = 0;
    piece = Piece{f, 0, 1, 0};
    return f < B;
  }
  int base = 0;
  bool found = false;
  for (int i0 = 0; i0 < B; i0 += 64) {
    const int g = i0 == 0 ? own : groups(i0 + lane), cuts = g > 0 ? (g - 1) / k : 0;
    const int incl = wave_incl_scan(cuts);  // cuts up to and including the lane's sequence
    if (leave) {
      if (i0 + lane < B) p.ws_prefix[i0 + lane + 1] = base + incl;
      if (i0 == 0 && lane == 0) p.ws_prefix[0] = 0;
    }
    if (!found) {
      // the sequences here whose pieces all lie before piece f
      const int n = __popcll(__ballot(i0 + lane < B && base + incl + i0 + lane + 1 <= f));
      if (n < 64 && i0 + n < B) {
        found = true;
        const int before = base + (n > 0 ? lane_value(incl, n - 1) : 0);
        piece.b = i0 + n;
        piece.chunk = f - before - piece.b;
        piece.pieces = lane_value(cuts, n) + 1;
        piece.extra = before + max(piece.chunk - 1, 0);
      }
    }
    base += lane_value(incl, 63);
    if (found && !leave) break;
  }
  return found;
}

// What a wavefront of either many-row kernel works on: 32 query rows from r0 on of `all_rows` that kv head
// h has here (one sequence's, or under PREFIX all sequences' stacked), over groups [g0, ng) of sequence
// b's context.
struct Place {
  int all_rows, h, r0, b, L, g0, ng, n_min, chunk;  // n_min: the shortest causal length of the rows
  bool wave_live;
  Piece piece;
};
// Where the plan launches both kernels, which of them the lengths give the call to: the wide one where all
// contexts together have p.wide_groups groups and the shortest p.wide_least.
__device__ inline bool whole_wide(const AttnArgs& p, int lane) {
  int total = 0, least = 0x7FFFFFFF;
  for (int i = lane; i < p.batch; i += 64) {
    const int groups = (p.seq_lens[i] + 63) >> 6;
    total += groups;
    least = min(least, groups);
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) total += __shfl_xor(total, d, 64);  // (shuffles: as in wave_min_int)
  return total >= p.wide_groups && wave_min_int(least) >= p.wide_least;
}
// Returns false for a workgroup that has nothing to do (the same in all its wavefronts).
// CHOICE: the plan launches both kernels.
template <bool PREFIX, int ROWS, bool CHOICE>
__device__ inline bool place_rows(const AttnArgs& p, int lane, int wv, Place& o) {
  const int H = p.num_kv_heads, G = p.group;
  // rows a (kv head) has in this kernel: one sequence's, or all sequences' stacked
  o.all_rows = PREFIX ? p.batch * p.rows : p.rows;
  const int row_blocks = (o.all_rows + ROWS - 1) / ROWS;
  int P = 0;  // PREFIX: the shared groups, if every sequence has that many full ones
  if constexpr (PREFIX) {
    int min_full = 0x7FFFFFFF;
    for (int i = lane; i < p.batch; i += 64) min_full = min(min_full, p.seq_lens[i] >> 6);
    if (p.shared_groups > wave_min_int(min_full)) return false;  // the streaming kernel does it all
    P = p.shared_groups;
  } else if constexpr (CHOICE) {
    if (whole_wide(p, lane) != (ROWS == kWideRows)) return false;  // the other kernel's
  }
  // Workgroup -> (sequence, kv head, row block).  The hardware hands consecutive workgroups to
  // the eight XCDs in turn, each with an L2 of its own, and the row blocks of one (sequence,
  // kv head) read the same codes: they are placed on one XCD (workgroups x, x + 8, x + 16, ...)
  // so that the codes leave HBM once, not once per XCD.
  int pair, rb;  // pair = (piece of the contexts, kv head); PREFIX: (piece of the prefix, kv head)
  {
    const int pairs = (PREFIX ? p.prefix_chunks : p.batch + p.extra_pieces) * H, id = blockIdx.x;
    if (pairs % 8 == 0) {
      const int x = id & 7, k = id >> 3;
      pair = x + 8 * (k / row_blocks);
      rb = k % row_blocks;
    } else {
      pair = id / row_blocks;
      rb = id - pair * row_blocks;
    }
    rb = row_blocks - 1 - rb;  // the later a chunk's rows, the longer their walk: the longest start first
  }
  o.h = pair % H;
  // this wavefront's rows, and the groups [g0, ng) the workgroup has to walk
  o.r0 = rb * ROWS + wv * 32;
  o.wave_live = o.r0 < o.all_rows;
  o.chunk = 0;
  o.piece = Piece{0, 0, 1, 0};
  if constexpr (PREFIX) {
    o.chunk = pair / H;
    o.b = rb * ROWS / p.rows;  // whose block table: the first row's sequence (all agree)
    o.L = P << 6;                           // every position below it exists in every sequence
    o.g0 = (int)((long long)o.chunk * P / p.prefix_chunks);
    o.ng = (int)((long long)(o.chunk + 1) * P / p.prefix_chunks);
    o.n_min = 0;  // (set below, from the rows' own causal lengths)
  } else {
    o.piece.b = pair / H;
    const int leave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x == 0 && wv == 0));
    if (p.extra_pieces > 0) {
      if (!context_piece(p, o.piece.b, leave, o.piece)) return false;
    } else if (CHOICE && p.merge && leave) {  // (a merge is launched for the other kernel's cuts)
      for (int i = lane; i <= p.batch; i += 64) p.ws_prefix[i] = 0;
    }
    o.b = o.piece.b;
    o.L = p.seq_lens[o.b];
    const int r_last = min(p.rows, (rb + 1) * ROWS) - 1;
    const int n_max = o.L - p.q_len + r_last / G + 1;
    const int all = (n_max + 63) >> 6;
    o.g0 = (int)((long long)o.piece.chunk * all / o.piece.pieces);
    o.ng = (int)((long long)(o.piece.chunk + 1) * all / o.piece.pieces);
    o.n_min = o.wave_live ? o.L - p.q_len + o.r0 / G + 1 : o.L;  // shortest causal length here
  }
  return true;
}

// q of a wavefront's rows as the B operand of QK^T, the rows' causal lengths, an empty running state.
template <int MODE, int D, bool PREFIX, class Operand>
__device__ inline void load_queries(const AttnArgs& p, int lane, Place& o, Operand (&qb)[2][D / 32], int (&nrow)[2],
                                    floatx4 (&acc)[2][D / 16], float (&m_run)[2], float (&l_run)[2]) {
  constexpr bool PLAIN = MODE == KVQ_BF16_PLAIN, INT4 = MODE == KVQ_INT4_TOKEN_HEAD;
  constexpr int NT = 2, KS = D / 32, DT = D / 16;
  const int m16 = lane & 15, g4 = lane >> 4, G = p.group;
  const uint32_t q_sign = PLAIN && p.scale_log2 < 0.0f ? 0x80008000u : 0u;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int rs = o.r0 + nt * 16 + m16;  // PREFIX: stacked row = sequence * rows + row
    const bool live = rs < o.all_rows;
    const int br = PREFIX ? (live ? rs / p.rows : 0) : o.b;
    const int r = PREFIX ? rs - br * p.rows : rs;
    const int j = live ? r / G : 0;
    const int gi = live ? r - j * G : 0;
    nrow[nt] = live ? (PREFIX ? p.seq_lens[br] : o.L) - p.q_len + j + 1 : o.L;
    const uint16_t* qrow =
        p.q + (((size_t)br * p.q_len + j) * p.num_q_heads + (size_t)o.h * G + gi) * D;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int d0 = PLAIN || INT4 ? 32 * s + 8 * g4 : 64 * (s >> 1) + 16 * g4 + 8 * (s & 1);
      const uintx4 raw = *(const uintx4*)(qrow + d0);
      if constexpr (PLAIN) {
        qb[nt][s] = __builtin_bit_cast(bf16x8, live ? raw ^ q_sign : uintx4{0u, 0u, 0u, 0u});
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const _Float16 lo = (_Float16)__uint_as_float(raw[e] << 16);
          const _Float16 hi = (_Float16)__uint_as_float(raw[e] & 0xFFFF0000u);
          qb[nt][s][2 * e] = live ? lo : (_Float16)0.0f;
          qb[nt][s][2 * e + 1] = live ? hi : (_Float16)0.0f;
        }
      }
    }
    m_run[nt] = -INFINITY;
    l_run[nt] = 0.0f;
#pragma unroll
    for (int tt = 0; tt < DT; ++tt) acc[nt][tt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  if constexpr (PREFIX) o.n_min = wave_min_int(min(nrow[0], nrow[1]));
}

// Where a wavefront's rows go at the end.
template <int D, bool PREFIX>
__device__ inline void store_rows(const AttnArgs& p, int lane, const Place& o, const floatx4 (&acc)[2][D / 16],
                                  const float (&m_run)[2], const float (&l_run)[2]) {
  constexpr int NT = 2, DT = D / 16;
  const int m16 = lane & 15, g4 = lane >> 4, G = p.group;
  if constexpr (PREFIX) {
    // ---- partials: slot = wavefronts + (1 + piece) * pairs + the row's pair, as the reduce
    // expects them ----
    const int rt = 16 * p.row_tiles;
    const size_t slot0 = (size_t)p.num_waves + (size_t)(o.chunk + 1) * p.batch * p.pairs_per_seq;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const float l = xor16_sum(l_run[nt]);
      const int rs = o.r0 + nt * 16 + m16;
      if (rs >= o.all_rows) continue;
      const int br = rs / p.rows, r = rs - br * p.rows;
      const int rg = r / rt, rl = r - rg * rt;
      const size_t row =
          (slot0 + (size_t)br * p.pairs_per_seq + o.h * p.num_row_groups + rg) * rt + rl;
      float* arow = p.ws_acc + row * D;
#pragma unroll
      for (int tt = 0; tt < DT; ++tt) *(floatx4*)(arow + 16 * tt + 4 * g4) = acc[nt][tt];
      if (g4 == 0) {
        p.ws_ml[row * 2] = m_run[nt];
        p.ws_ml[row * 2 + 1] = l;
      }
    }
    return;
  }
  // ---- normalised rows: those of a sequence's first piece (mostly the only one) go to `out`, the
  // others' to the workspace, a piece's rows in the order its sequence's have in `out`; the logarithms
  // of the denominators likewise, those of first pieces ahead ----
  const size_t seq_rows = (size_t)p.q_len * p.num_q_heads;
  const size_t to = (size_t)(o.piece.chunk == 0 ? o.b : o.piece.extra) * seq_rows;
  float* dst = (o.piece.chunk == 0 ? p.out : p.ws_acc) + to * D;
  float* lse = p.ws_ml + ((o.piece.chunk == 0 ? 0 : (size_t)p.batch * seq_rows) + to);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float l = xor16_sum(l_run[nt]);
    const int r = o.r0 + nt * 16 + m16;
    if (r >= p.rows) continue;
    const int j = r / G, gi = r - j * G;
    const size_t row = (size_t)j * p.num_q_heads + (size_t)o.h * G + gi;
    float* orow = dst + row * D;
    float inv = 1.0f / l;
    if (o.piece.pieces > 1) {  // a row may see nothing of a piece
      inv = l > 0.0f ? inv : 0.0f;
      if (g4 == 0) lse[row] = l > 0.0f ? m_run[nt] + __builtin_amdgcn_logf(l) : -INFINITY;
    }
#pragma unroll
    for (int tt = 0; tt < DT; ++tt) *(floatx4*)(orow + 16 * tt + 4 * g4) = acc[nt][tt] * inv;
  }
}

// PREFIX = true is the kernel for a prefix that every sequence of a decode or verification
// batch shares (the same physical blocks at the head of every block table; Section 1 and
// Section 5.2.3: prompt prefixes served from the prefix cache).  The query rows of all
// sequences are stacked, 128 to a workgroup, so a group of the prefix is read and converted
// once per 128 rows (four sequences of a 4-token verification step with 8 query heads per kv
// head) instead of once per sequence.  The prefix is cut into p.prefix_chunks pieces to get
// enough workgroups; a workgroup walks one piece and leaves, per row, an unnormalised partial
// (max, sum, accumulator) in the workspace, in the slots behind the streaming kernel's, which
// the reduce merges with the streaming kernel's partials over the rest of each sequence.
template <int MODE, int D, bool PREFIX, bool CHOICE>
__global__ __launch_bounds__(64 * kWavesPerGroup, 2) void attn_rows_kernel(const AttnArgs p) {
  constexpr bool PLAIN = MODE == KVQ_BF16_PLAIN;  // unquantized cache: the operands are its bytes
  constexpr bool FP8 = MODE == KVQ_FP8E4M3_BLOCK_HEAD || MODE == KVQ_FP8E4M3_TENSOR;
  constexpr bool INT4 = MODE == KVQ_INT4_TOKEN_HEAD;  // two codes per byte (head_dim 128)
  constexpr bool TOKEN_SCALE = MODE == KVQ_INT8_TOKEN_HEAD || INT4;
  static_assert(!INT4 || D == 128, "int4 codes come with head_dim 128 only");
  constexpr int NT = 2;
  constexpr int EB = PLAIN ? 2 : 1;  // bytes per cache element
  constexpr int RB = INT4 ? D / 2 : D * EB;  // bytes per token row in a tile
  constexpr int DT = D / 16;       // 16-channel tiles of V / of the output
  constexpr int KJ = RB / 64;      // 16-byte K pieces per lane and quad
  constexpr int KS = D / 32;       // matrix-instruction steps over the channels
  constexpr int NP = RB / 16;      // 16-byte pieces per lane that K (and V) of a group consist of
  constexpr int WP = NP / kWavesPerGroup;  // and those that a wavefront converts
  constexpr int kPace = INT4 ? 5 : 2;  // vector instructions behind a matrix instruction
  // matrix-instruction operand of 8 values: f16 (from codes) or the cache's own bf16
  using Operand = std::conditional_t<PLAIN, bf16x8, half8>;
  __shared__ half8 k_ops[2][4][KS][64];    // [half][quad of the sub-block][step][lane]
  __shared__ half8 v_ops[2][DT][2][64];    // [half][channel tile][tokens 0-7 | 8-15][lane]
  // [half]: K scale * log2e / sqrt(D), log2 and reciprocal of the V scale of the 64 tokens
  __shared__ __align__(16) float s_ops[2][3][64];

  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int m16 = lane & 15, g4 = lane >> 4;
  const int H = p.num_kv_heads, bs = p.block_size, bs_shift = p.bs_shift;
  Place at;
  if (!place_rows<PREFIX, kRowsPerWorkgroup, CHOICE>(p, lane, wv, at)) return;
  const int h = at.h, b = at.b, L = at.L, g0 = at.g0, ng = at.ng;

  const uint8_t* __restrict__ cache = p.cache;
  const float* __restrict__ scales = p.scales;
  const int32_t* __restrict__ table = p.block_tables + (size_t)b * p.max_blocks_per_seq;
  const uint32_t tile_bytes = (uint32_t)bs * RB;
  const uint32_t block_stride = 2u * (uint32_t)H * tile_bytes;
  const int sbk = m16 >> 2;  // sub-block this lane reads K from
  const uint32_t s_block_stride = TOKEN_SCALE ? 2u * H * bs : (MODE == KVQ_FP8E4M3_TENSOR ? 0u : 2u * H);
  const uint32_t s_kv = TOKEN_SCALE ? (uint32_t)H * bs : (MODE == KVQ_FP8E4M3_TENSOR ? 1u : (uint32_t)H);
  const int last_sb = ((L - 1) >> 4) << 4;

  // ---- q as the B operand of QK^T, causal lengths, running state ----
  Operand qb[NT][KS];
  int nrow[NT];
  floatx4 acc[NT][DT];
  float m_run[NT], l_run[NT];
  load_queries<MODE, D, PREFIX>(p, lane, at, qb, nrow, acc, m_run, l_run);
  const int n_min = at.n_min;

  // ---- producer side: this wavefront's quarter of a group's codes ----
  const int first = wv * WP;  // its pieces of K, and of V
  const uint32_t k_fixed = (uint32_t)h * tile_bytes + 64u * g4 + 16u * (m16 & 3);
  const uint32_t v_fixed = (uint32_t)(H + h) * tile_bytes + 16u * m16;
  // Table entries are requested ahead of the codes of the group before, so that waiting for them is not
  // waiting for those.  (indices past the end repeat the last group)
  uint32_t entry_k, entry_v;
  auto positions = [&](int g, uint32_t& tk, uint32_t& tv) {
    g = min(g, ng - 1);
    tk = (uint32_t)min((g << 6) + 16 * sbk, last_sb);
    tv = (uint32_t)min((g << 6) + 16 * g4, last_sb);
  };
  auto fetch_entries = [&](int g) {
    uint32_t tk, tv;
    positions(g, tk, tv);
    entry_k = (uint32_t)table[tk >> bs_shift];
    entry_v = (uint32_t)table[tv >> bs_shift];
  };
  uint64_t k_from = 0, v_from = 0;  // byte offsets in the cache
  uintx4 rk[WP], rv[WP];
  float sk_next = 0.0f, sv_next = 0.0f;
  auto locate = [&](int g) {  // whose entries have been fetched
    uint32_t tk, tv;
    positions(g, tk, tv);
    k_from = (uint64_t)entry_k * block_stride + ((tk & (uint32_t)(bs - 1)) * RB + k_fixed);
    v_from = (uint64_t)entry_v * block_stride + ((tv & (uint32_t)(bs - 1)) * RB + v_fixed);
    asm volatile("" : "+v"(k_from), "+v"(v_from));  // (here, not where they are used)
  };
  auto request_scales = [&](int g, float& sk, float& sv) {  // the same; lane = token
    uint32_t tk, tv;
    positions(g, tk, tv);
    const float* from = scales + ((uint64_t)entry_v * s_block_stride + (TOKEN_SCALE ? (uint32_t)(h * bs + m16) + (tv & (uint32_t)(bs - 1)) : (MODE == KVQ_FP8E4M3_TENSOR ? 0u : (uint32_t)h)));
    sk = from[0];
    sv = from[s_kv];
  };
  auto request = [&](uintx4 (&rk)[WP], uintx4 (&rv)[WP]) {
#pragma unroll
    for (int x = 0; x < WP; ++x) {
      const int pc = first + x;
      rk[x] = *(const uintx4*)(cache + k_from + (pc / KJ) * (4 * RB) + 256 * (pc % KJ));
    }
    // (unquantized: piece 2 t + hf is channel tile t, tokens 8 hf .. 8 hf + 7)
#pragma unroll
    for (int x = 0; x < WP; ++x) {
      const int pc = first + x;
      rv[x] = *(const uintx4*)(cache + v_from + (PLAIN ? (pc & 1) * (16 * D) + 256 * (pc >> 1) : 256 * pc));
    }
  };
  auto publish_k = [&](uintx4& codes, int x, int buf) {
    asm volatile("" : "+v"(codes));  // (converted here, not earlier)
    const int pc = first + x, u = pc / KJ, at = pc % KJ;
    if constexpr (PLAIN) {  // bf16 rows are operands as they are; the LDS arrays hold their bits
      k_ops[buf][u][at][lane] = __builtin_bit_cast(half8, codes);
    } else if constexpr (INT4) {  // word st of the lane's piece holds the 8 channels of step st
#pragma unroll
      for (int st = 0; st < 4; ++st) k_ops[buf][u][st][lane] = cvt_int4(codes[st]);
    } else {
      k_ops[buf][u][2 * at][lane] = cvt8<MODE>(codes[0], codes[1]);
      k_ops[buf][u][2 * at + 1][lane] = cvt8<MODE>(codes[2], codes[3]);
    }
  };
  auto publish_v = [&](uintx4& codes, int x, int half) {
    asm volatile("" : "+v"(codes));
    const int pc = first + x;
    if constexpr (PLAIN) {
      v_ops[half][pc >> 1][pc & 1][lane] = __builtin_bit_cast(half8, codes);
    } else if constexpr (INT4) {
#pragma unroll
      for (int w4 = 0; w4 < 4; ++w4) v_ops[half][2 * pc + (w4 >> 1)][w4 & 1][lane] = cvt_int4(codes[w4]);
    } else {
      v_ops[half][pc][0][lane] = cvt8<MODE>(codes[0], codes[1]);
      v_ops[half][pc][1][lane] = cvt8<MODE>(codes[2], codes[3]);
    }
  };
  // V bits of tokens past the last position are cleared first: a NaN times 0 is NaN
  auto clear_missing = [&](int g, uintx4 (&rv)[WP]) {
    if (!(PLAIN || FP8) || (g << 6) + 64 <= L) return;
    const int live = L - ((g << 6) + 16 * g4);  // tokens of this lane's sub-block below L
#pragma unroll
    for (int x = 0; x < WP; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (PLAIN) {
          const int n = live - (8 * ((first + x) & 1) + 2 * e);
          rv[x][e] &= n >= 2 ? ~0u : n == 1 ? 0xFFFFu : 0u;
        } else {
          const int n = min(max(live - 4 * e, 0), 4);
          rv[x][e] &= n == 4 ? ~0u : (1u << (8 * n)) - 1u;
        }
      }
  };
  auto publish_scales = [&](int j, float sk, float sv) {  // of group g0 + j
    const int g = min(g0 + j, ng - 1), buf = j & 1;
    float skp = sk * p.scale_log2;
    float lsv = __builtin_amdgcn_logf(fmaxf(sv, kMinVScale));
    float rsv = __builtin_amdgcn_exp2f(-lsv);
    if (TOKEN_SCALE && (g << 6) + lane >= L) {
      skp = 0.0f;  // a slot that was never written: its scales are not data
      lsv = 0.0f;
      rsv = 0.0f;
    }
    s_ops[buf][0][lane] = skp;
    s_ops[buf][1][lane] = lsv;
    s_ops[buf][2][lane] = rsv;
  };

  // ---- consumer side ----
  floatx4 S[NT][4];
  Operand pb[NT][2 * EB];  // unquantized: a probability goes in as two bf16 terms (hi, lo)
  auto load_op = [&](const half8& bits) {
    if constexpr (PLAIN) return __builtin_bit_cast(bf16x8, bits);
    else return bits;
  };
  auto mma = [&](const Operand& a, const Operand& b, const floatx4& c) {
    if constexpr (PLAIN) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  };
  float scales_here[3] = {};  // e4m3: the lane's scales of the group in hand
  float mx[NT];
  constexpr float skp = 0.0f, lsv = 0.0f;  // (the maxima of formats without token scales are those of S)
  Operand op[2][4];  // operands of two chunks of eight matrix instructions
  floatx4 k4[2] = {}, l4[2] = {};
  constexpr int HS = KS / 2, QC = 2 * HS, PC = DT / 2;  // chunks of QK^T (two quads, two steps) and of P.V (two tiles)
  auto read_k = [&](int c, int buf) {
#pragma unroll
    for (int x = 0; x < 4; ++x) op[c & 1][x] = load_op(k_ops[buf][2 * (c / HS) + (x & 1)][2 * (c % HS) + (x >> 1)][lane]);
  };
  auto read_v = [&](int c, int half) {
#pragma unroll
    for (int x = 0; x < 4; ++x) op[(QC + c) & 1][x] = load_op(v_ops[half][2 * c + (x & 1)][x >> 1][lane]);
  };
  auto read_scales = [&](int pair, int buf) {
    const floatx4* sc = (const floatx4*)&s_ops[buf][0][16 * g4];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      k4[x] = sc[2 * pair + x];
      l4[x] = sc[kScalePitch + 2 * pair + x];
    }
  };
  auto mm_k = [&](int c) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int u = 2 * (c / HS) + (x & 1);
        S[nt][u] = mma(op[c & 1][x], qb[nt][2 * (c % HS) + (x >> 1)], S[nt][u]);
      }
  };
  auto mm_v = [&](int c) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        floatx4& d = acc[nt][2 * c + (x & 1)];
        d = mma(op[(QC + c) & 1][x], pb[nt][x >> 1], d);
        if constexpr (PLAIN) d = mma(op[(QC + c) & 1][x], pb[nt][2 + (x >> 1)], d);
      }
  };
  // N matrix instructions, an LDS read behind each of the first READS and VALU vector ones behind all.  (The reads
  // dealt out over all N came too late for the next chunk where a workgroup has its compute unit to itself:
  // 3 x 1000 tokens over 3000 int8 173.5 -> 171 us, int4 180 -> 177.)
  auto pace = [&](auto N, auto READS, auto VALU) {
    static_for<decltype(N)::value>([&](auto X) {
      constexpr int x = decltype(X)::value, r = decltype(READS)::value;
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      if constexpr (x < r) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if constexpr (decltype(VALU)::value > 0) __builtin_amdgcn_sched_group_barrier(0x2, decltype(VALU)::value, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  using Whole = SoftmaxForm<MODE, false>;
  // TAIL: some row's causal length ends inside the group: positions past it are masked, and the
  // maxima taken again.
  auto vector_phase = [&](auto TAILC, int g, int sbuf) {
    constexpr bool TAIL = decltype(TAILC)::value;
    using F = SoftmaxForm<MODE, TAIL>;
    const floatx4* sc = (const floatx4*)&s_ops[sbuf][0][16 * g4];
    floatx4 r4[4] = {};
    if constexpr (F::TOKEN_SCALE) {
#pragma unroll
      for (int u = 0; u < 4; ++u) r4[u] = sc[2 * kScalePitch + u];
    }
    float skp = fabsf(p.scale_log2), lsv = 0.0f, rsv = 1.0f;
    if constexpr (FP8) {
      skp = scales_here[0];
      lsv = scales_here[1];
      rsv = scales_here[2];
    }
    if constexpr (TAIL) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        mx[nt] = -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float z = S[nt][u][i];
            if constexpr (!F::kLogits) z = __builtin_fmaf(z, skp, lsv);
            z = (g << 6) + 16 * g4 + 4 * u + i < nrow[nt] ? z : -INFINITY;
            S[nt][u][i] = z;
            mx[nt] = fmaxf(mx[nt], z);
          }
      }
    } else if constexpr (FP8) {
      if (__any(skp < 0.0f)) {  // (a negative softmax scale, or static scale)
        const float sign = skp < 0.0f ? -1.0f : 1.0f;
        skp *= sign;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          mx[nt] = -INFINITY;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            S[nt][u] *= sign;
            softmax_logits<MODE, NT, TAIL>(S, u, k4[0], l4[0], skp, lsv, 0, nrow, mx);
          }
        }
      }
    }
    float alpha[NT], msub[NT];
    softmax_maxima<MODE, NT, TAIL>(mx, skp, lsv, m_run, alpha, msub);
    softmax_probabilities<MODE, NT, TAIL, true>(S, sc, r4, skp, rsv, alpha, msub, l_run, pb);
    softmax_rescale<NT, DT>(alpha, acc);
  };

  // The matrix instructions: QK^T of group g0 + j from half j % 2, the logits of the first tokens and their
  // maxima (unmasked) worked out while the last ones' are contracted; and P.V, the next group's codes
  // converted into the other half under it.
  auto contract_k = [&](int half) {
    if constexpr (FP8) {
#pragma unroll
      for (int x = 0; x < 3; ++x) scales_here[x] = s_ops[half][x][lane];
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      mx[nt] = -INFINITY;
#pragma unroll
      for (int u = 0; u < 4; ++u) S[nt][u] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    read_k(0, half);
    __builtin_amdgcn_sched_barrier(0);
    static_for<QC>([&](auto C) {
      constexpr int c = decltype(C)::value;
      constexpr bool sc = Whole::kLogits && (c + 1) % HS == 0;
      mm_k(c);
      if constexpr (c + 1 < QC) read_k(c + 1, half);
      if constexpr (c == HS) {
        softmax_logits<MODE, NT, false>(S, 0, k4[0], l4[0], skp, lsv, 0, nrow, mx);
        softmax_logits<MODE, NT, false>(S, 1, k4[1], l4[1], skp, lsv, 0, nrow, mx);
      }
      if constexpr (sc) read_scales(c / HS, half);
      pace(std::integral_constant<int, 8>{}, std::integral_constant<int, (c + 1 < QC ? 4 : 0) + (sc ? 4 : 0)>{}, std::integral_constant<int, c == HS ? kPace : 0>{});
    });
    softmax_logits<MODE, NT, false>(S, 2, k4[0], l4[0], skp, lsv, 0, nrow, mx);
    softmax_logits<MODE, NT, false>(S, 3, k4[1], l4[1], skp, lsv, 0, nrow, mx);
  };
  constexpr int PIECES = 2 * WP;
  auto publish = [&](uintx4 (&rk)[WP], uintx4 (&rv)[WP], int x, int half) {
    if (x < WP) publish_k(rk[x], x, half);
    else publish_v(rv[x - WP], x - WP, half);
  };
  auto contract_v = [&](int half) {
    static_for<PC>([&](auto C) {
      constexpr int c = decltype(C)::value;
      mm_v(c);
      if constexpr (c + 1 < PC) read_v(c + 1, half);
#pragma unroll
      for (int x = c * PIECES / PC; x < (c + 1) * PIECES / PC; ++x) publish(rk, rv, x, half ^ 1);
      pace(std::integral_constant<int, PLAIN ? 16 : 8>{}, std::integral_constant<int, c + 1 < PC ? 4 : 0>{}, std::integral_constant<int, PLAIN ? 0 : kPace>{});
    });
  };
  // ---- the walk: group g is consumed from half g % 2 while group g + 1 is converted into the
  // other half and group g + 2 is requested ----
  const bool live = __builtin_amdgcn_readfirstlane((int)at.wave_live) != 0;
  const int n = ng - g0;
  if (n > 0) {  // (a chunk's first rows see fewer groups than there may be pieces)
    // (start: the entries of three groups, then the codes of two, a round trip each.  Asked for group by group
    // they took contexts of one group two round trips more: 113 x 64 tokens over 64, 64 / 8 heads, int8 102 -> 90 us,
    // e4m3 100 -> 90.)
    const bool scale_wave = !PLAIN && wv == 0;
    uintx4 first_k[WP], first_v[WP];
    float sk = 0.0f, sv = 0.0f;
    fetch_entries(g0);
    const uint32_t k0 = entry_k, v0 = entry_v;
    fetch_entries(g0 + 1);
    const uint32_t k1 = entry_k, v1 = entry_v;
    fetch_entries(g0 + 2);
    const uint32_t k2 = entry_k, v2 = entry_v;
    entry_k = k0, entry_v = v0;
    locate(g0);
    request(first_k, first_v);
    if (scale_wave) request_scales(g0, sk, sv);
    entry_k = k1, entry_v = v1;
    locate(g0 + 1);
    request(rk, rv);
    if (scale_wave) {
      request_scales(g0 + 1, sk_next, sv_next);
      publish_scales(0, sk, sv);
    }
    entry_k = k2, entry_v = v2;
    clear_missing(g0, first_v);
#pragma unroll
    for (int x = 0; x < PIECES; ++x) publish(first_k, first_v, x, 0);
    __syncthreads();
    // codes of group i + 2 located, scales of i + 1 published, of i + 2 requested.  (Behind the matrix instructions: both
    // wait for loads that were requested at the end of the last iteration.  Ahead of the softmax, a lone workgroup
    // waited there for every group: 398 x 64 tokens, one over 9807 and the rest over 180, int8 285 -> 249 us, e4m3
    // 267 -> 233, bf16 317 -> 282, int4 284 -> 258.)
    auto prepare = [&](int i) {
      locate(g0 + i + 2);
      if (scale_wave) {
        publish_scales(i + 1, sk_next, sv_next);
        request_scales(g0 + i + 2, sk_next, sv_next);
      }
    };
    auto advance = [&](int i) {
      fetch_entries(g0 + i + 3);
      request(rk, rv);
      __syncthreads();
    };
    if (live) {
      for (int i = 0; i < n; ++i) {
        const int g = g0 + i, half = i & 1;
        contract_k(half);
        if ((g << 6) + 64 > n_min) vector_phase(std::true_type{}, g, half);
        else vector_phase(std::false_type{}, g, half);
        read_v(0, half);
        clear_missing(min(g + 1, ng - 1), rv);
        contract_v(half);
        prepare(i);
        advance(i);
      }
    } else {
      for (int i = 0; i < n; ++i) {
        prepare(i);
        clear_missing(min(g0 + i + 1, ng - 1), rv);
#pragma unroll
        for (int x = 0; x < PIECES; ++x) publish(rk, rv, x, ~i & 1);
        advance(i);
      }
    }
  }

  store_rows<D, PREFIX>(p, lane, at, acc, m_run, l_run);
}

// The same at head_dim 64 for the int8 and the unquantized cache, a phase after the other: in 164 registers,
// so that three wavefronts run on a SIMD, which is worth more there than logits and conversions under the
// matrix instructions unless there are few workgroups.  Here and above, int8 (175 registers): 3 x 1000 tokens over 3000
// 119 and 125 us, 40 x 64 over 300 21.9 and 24.0, 16 x 33 over 2000 45.8 and 41.7; bf16 (167, but 188 for a shared
// prefix) 128.6 and 127.8, 23.2 and 22.8, 46.7 and 43.9, 60 sequences of 1451 tokens that share 704, 28 rows, 45.3 and 47.8.  The e4m3
// formats fit either way and are faster above (105.9 -> 104.8).
template <int MODE, bool PREFIX>
__global__ __launch_bounds__(64 * kWavesPerGroup, 2) void attn_rows64_kernel(const AttnArgs p) {
  constexpr bool PLAIN = MODE == KVQ_BF16_PLAIN;  // unquantized cache: the operands are its bytes
  static_assert(PLAIN || MODE == KVQ_INT8_TOKEN_HEAD, "the other formats take attn_rows_kernel");
  constexpr int NT = 2, D = 64;
  constexpr int EB = PLAIN ? 2 : 1;  // bytes per cache element
  constexpr int RB = D * EB;         // bytes per token row in a tile
  constexpr int DT = D / 16;       // 16-channel tiles of V / of the output
  constexpr int KJ = RB / 64;      // 16-byte K pieces per lane and quad
  constexpr int KS = D / 32;       // matrix-instruction steps over the channels
  constexpr int VT = DT / kWavesPerGroup;  // V tiles a wavefront converts
  constexpr int VP = VT * EB;      // 16-byte V pieces per lane
  // matrix-instruction operand of 8 values: f16 (from codes) or the cache's own bf16
  using Operand = std::conditional_t<PLAIN, bf16x8, half8>;
  __shared__ half8 k_ops[2][4][KS][64];    // [half][quad of the sub-block][step][lane]
  __shared__ half8 v_ops[2][DT][2][64];    // [half][channel tile][tokens 0-7 | 8-15][lane]
  // [half]: K scale * log2e / sqrt(D), log2 and reciprocal of the V scale of the 64 tokens
  __shared__ __align__(16) float s_ops[2][3][64];

  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int m16 = lane & 15, g4 = lane >> 4;
  const int H = p.num_kv_heads, bs = p.block_size, bs_shift = p.bs_shift;
  Place at;
  if (!place_rows<PREFIX, kRowsPerWorkgroup, false>(p, lane, wv, at)) return;
  const int h = at.h, b = at.b, L = at.L, g0 = at.g0, ng = at.ng;
  const bool wave_live = at.wave_live;

  const uint8_t* __restrict__ cache = p.cache;
  const float* __restrict__ scales = p.scales;
  const int32_t* __restrict__ table = p.block_tables + (size_t)b * p.max_blocks_per_seq;
  const uint32_t tile_bytes = (uint32_t)bs * RB;
  const uint32_t block_stride = 2u * (uint32_t)H * tile_bytes;
  const int sbk = m16 >> 2;  // sub-block this lane reads K from
  const uint32_t k_lane = 64u * g4 + 16u * (m16 & 3) + (uint32_t)wv * (4 * RB);  // quad wv
  const uint32_t v_lane = (uint32_t)H * tile_bytes + 16u * m16 + 256u * (wv * VT);
  const uint32_t s_block_stride = 2u * H * bs;
  const uint32_t s_kv = (uint32_t)H * bs;
  const int last_sb = ((L - 1) >> 4) << 4;

  // ---- q as the B operand of QK^T, causal lengths, running state ----
  Operand qb[NT][KS];
  int nrow[NT];
  floatx4 acc[NT][DT];
  float m_run[NT], l_run[NT];
  load_queries<MODE, D, PREFIX>(p, lane, at, qb, nrow, acc, m_run, l_run);
  const int n_min = at.n_min;

  // ---- producer side: this wavefront's quarter of a group's codes ----
  // (a group's table entries come with the lane's offsets inside their blocks: the position that
  // gives the one gives the other)
  struct Entries {
    uint32_t k, v, k_at, v_at;
  };
  const uint32_t k_fixed = (uint32_t)h * tile_bytes + k_lane, v_fixed = (uint32_t)h * tile_bytes + v_lane;
  auto fetch_entries = [&](int g, Entries& e) {  // g is clamped by the caller
    const uint32_t tk = (uint32_t)min((g << 6) + 16 * sbk, last_sb), tv = (uint32_t)min((g << 6) + 16 * g4, last_sb);
    e.k = (uint32_t)table[tk >> bs_shift];
    e.v = (uint32_t)table[tv >> bs_shift];
    e.k_at = (tk & (uint32_t)(bs - 1)) * RB + k_fixed;
    e.v_at = tv & (uint32_t)(bs - 1);
  };
  uintx4 rk[KJ], rv[VP];
  float sk_next = 0.0f, sv_next = 0.0f;
  auto issue_loads = [&](const Entries& e) {
    const uint8_t* kbase = cache + ((uint64_t)e.k * block_stride + e.k_at);
    const uint8_t* vbase = cache + ((uint64_t)e.v * block_stride + (e.v_at * RB + v_fixed));
#pragma unroll
    for (int j = 0; j < KJ; ++j) rk[j] = *(const uintx4*)(kbase + 256 * j);
    // (unquantized: piece 2 t + hf is channel tile t, tokens 8 hf .. 8 hf + 7)
#pragma unroll
    for (int x = 0; x < VP; ++x)
      rv[x] = *(const uintx4*)(vbase + (PLAIN ? (x & 1) * (16 * D) + 256 * (x >> 1) : 256 * x));
    if (!PLAIN && wv == 0) {  // the scales of the group's 64 tokens, lane = token
      const uint32_t s_lane = (uint32_t)(h * bs + m16) + e.v_at;
      const float* sp = scales + ((uint64_t)e.v * s_block_stride + s_lane);
      sk_next = sp[0];
      sv_next = sp[s_kv];
    }
  };
  auto publish = [&](int g, int half) {  // convert the loaded codes and put them in LDS
    if constexpr (PLAIN) {  // bf16 rows are operands as they are; the LDS arrays hold their bits
#pragma unroll
      for (int j = 0; j < KJ; ++j) k_ops[half][wv][j][lane] = __builtin_bit_cast(half8, rk[j]);
      const int live = L - ((g << 6) + 16 * g4);  // tokens of this lane's sub-block below L
#pragma unroll
      for (int x = 0; x < VP; ++x) {
        uintx4 raw = rv[x];
        if ((g << 6) + 64 > L) {  // bf16 bit patterns of missing tokens: a NaN times 0 is NaN
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int n = live - (8 * (x & 1) + 2 * e);
            raw[e] &= n >= 2 ? ~0u : n == 1 ? 0xFFFFu : 0u;
          }
        }
        v_ops[half][wv * VT + (x >> 1)][x & 1][lane] = __builtin_bit_cast(half8, raw);
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < KJ; ++j) {
      k_ops[half][wv][2 * j][lane] = cvt8<MODE>(rk[j][0], rk[j][1]);
      k_ops[half][wv][2 * j + 1][lane] = cvt8<MODE>(rk[j][2], rk[j][3]);
    }
#pragma unroll
    for (int t = 0; t < VT; ++t) {
      v_ops[half][wv * VT + t][0][lane] = cvt8<MODE>(rv[t][0], rv[t][1]);
      v_ops[half][wv * VT + t][1][lane] = cvt8<MODE>(rv[t][2], rv[t][3]);
    }
    // The scales go the same way: held in registers from the load to the softmax two iterations
    // later, they would have to be copied at the end of the iteration that requested them, and
    // that copy waits for the whole round trip to memory.
    if (wv == 0) {
      float skp = sk_next * p.scale_log2;
      float lsv = __builtin_amdgcn_logf(fmaxf(sv_next, kMinVScale));
      float rsv = __builtin_amdgcn_exp2f(-lsv);
      if ((g << 6) + lane >= L) {
        skp = 0.0f;  // a slot that was never written: its scales are not data
        lsv = 0.0f;
        rsv = 0.0f;
      }
      s_ops[half][0][lane] = skp;
      s_ops[half][1][lane] = lsv;
      s_ops[half][2][lane] = rsv;
    }
  };

  // ---- consumer side ----
  floatx4 S[NT][4];
  Operand pb[NT][2 * EB];  // unquantized: a probability goes in as two bf16 terms (hi, lo)
  auto load_op = [&](const half8& bits) {
    if constexpr (PLAIN) return __builtin_bit_cast(bf16x8, bits);
    else return bits;
  };
  auto mma = [&](const Operand& a, const Operand& b, const floatx4& c) {
    if constexpr (PLAIN) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  };
  auto qk = [&](int half) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int u = 0; u < 4; ++u) S[nt][u] = floatx4{0.f, 0.f, 0.f, 0.f};
    // step by step over the channels: eight independent instructions (4 quads x 2 row tiles)
    // per step, the next step's four operands read from LDS while they run.  The scheduling
    // barriers keep that order; left alone, the compiler reads two operands, waits, issues
    // four instructions and so exposes the LDS latency eight times per group.
    Operand a[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[0][u] = load_op(k_ops[half][u][0][lane]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s + 1 < KS) {
#pragma unroll
        for (int u = 0; u < 4; ++u) a[(s + 1) & 1][u] = load_op(k_ops[half][u][s + 1][lane]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          S[nt][u] = mma(a[s & 1][u], qb[nt][s], S[nt][u]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto softmax_impl = [&](auto TAILC, int g, int half) {
    constexpr bool TAIL = decltype(TAILC)::value;
    const int pos0 = g << 6;
    online_softmax<MODE, NT, DT, TAIL>(S, (const floatx4*)&s_ops[half][0][16 * g4], fabsf(p.scale_log2), 0.0f, 1.0f,
                                       pos0 + 16 * g4, nrow, m_run, l_run, acc, pb);
  };
  auto pv = [&](int half) {
    // two channel tiles at a time: their four operands are read while the previous pair's
    // eight instructions run; the instructions alternate between four accumulators
    Operand a[2][2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) a[0][x][hf] = load_op(v_ops[half][x][hf][lane]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t2 = 0; t2 < DT / 2; ++t2) {
      if (t2 + 1 < DT / 2) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf)
            a[(t2 + 1) & 1][x][hf] = load_op(v_ops[half][2 * (t2 + 1) + x][hf][lane]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            acc[nt][2 * t2 + x] = mma(a[t2 & 1][x][hf], pb[nt][hf], acc[nt][2 * t2 + x]);
            if constexpr (PLAIN)
              acc[nt][2 * t2 + x] = mma(a[t2 & 1][x][hf], pb[nt][2 + hf], acc[nt][2 * t2 + x]);
          }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- the walk: group g is consumed from half g % 2 while group g + 1 is converted into the
  // other half and group g + 2 is requested (indices past the end repeat the last group) ----
  Entries e_next, e_after;
  if (g0 < ng) {  // (a chunk's first rows see fewer groups than there may be pieces)
    Entries e0;
    fetch_entries(g0, e0);
    fetch_entries(min(g0 + 1, ng - 1), e_next);
    issue_loads(e0);
    publish(g0, 0);
    issue_loads(e_next);
    fetch_entries(min(g0 + 2, ng - 1), e_after);
  }
  __syncthreads();
  for (int g = g0; g < ng; ++g) {
    const int half = (g - g0) & 1;
    if (wave_live) {
      qk(half);
      if ((g << 6) + 64 > n_min) softmax_impl(std::true_type{}, g, half);
      else softmax_impl(std::false_type{}, g, half);
      pv(half);
    }
    // group g + 1 (requested one iteration ago) into the other half; request group g + 2
    publish(min(g + 1, ng - 1), half ^ 1);
    issue_loads(e_after);
    fetch_entries(min(g + 3, ng - 1), e_after);
    __syncthreads();
  }
  store_rows<D, PREFIX>(p, lane, at, acc, m_run, l_run);
}

// The same for group-scaled int4 (head_dim 128): a phase after the other, since the scales by channel group leave no
// registers for more.  A step of QK^T contracts one group of 32 channels, and the logit is the four steps' results
// weighted by the token's four K scales in fp32, as in the streaming kernel; P.V takes the probabilities times the V
// scale of the group its channels belong to, worked out once a group for both of its channel tiles.  Scales go to LDS
// by channel group, so that four tokens' come in one read.  Vector-bound: a logit costs four multiply-adds, and four
// products and conversions behind the softmax, where the other formats have one and half of one; what it spares is
// the conversion of all codes for every 16 rows.  One path behind the mask: with two copies of the softmax, as above,
// 41 registers spilled and 8 x 512 tokens over 4608 took 630 us.  The same now 502, streaming 1204; 1 x 512 over
// 16896, in the two pieces that the workspace has room for, 256 workgroups of the 512 that fit, 309 and 534; 64
// sequences of 2000 to 4000, 128 rows, 231 and 433.
__global__ __launch_bounds__(64 * kWavesPerGroup, 2) void attn_rows_group_kernel(const AttnArgs p) {
  constexpr int NT = 2, D = 128, RB = D / 2, DT = D / 16, KS = D / 32;
  constexpr int MODE = KVQ_INT4_GROUP32;
  static_assert(kWavesPerGroup == 4, "a wavefront converts a quad of K and two channel tiles of V");
  __shared__ half8 k_ops[2][4][KS][64];    // [half][quad of the sub-block][step][lane]
  __shared__ half8 v_ops[2][DT][2][64];    // [half][channel tile][tokens 0-7 | 8-15][lane]
  __shared__ __align__(16) float k_scales[2][KS][64];  // [half][channel group][token], times log2e / sqrt(D)
  __shared__ __align__(16) float v_scales[2][KS][64];  // relative to the token's largest
  __shared__ __align__(16) float s_ops[2][3][64];      // (unused,) log2 and reciprocal of the largest V scale

  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int m16 = lane & 15, g4 = lane >> 4;
  const int H = p.num_kv_heads, bs = p.block_size, bs_shift = p.bs_shift;
  Place at;
  if (!place_rows<false, kRowsPerWorkgroup, false>(p, lane, wv, at)) return;
  const int h = at.h, b = at.b, L = at.L, g0 = at.g0, ng = at.ng;
  const bool wave_live = at.wave_live;

  const uint8_t* __restrict__ cache = p.cache;
  const float* __restrict__ scales = p.scales;
  const int32_t* __restrict__ table = p.block_tables + (size_t)b * p.max_blocks_per_seq;
  const uint32_t tile_bytes = (uint32_t)bs * RB;
  const uint32_t block_stride = 2u * (uint32_t)H * tile_bytes;
  const int sbk = m16 >> 2;  // sub-block this lane reads K from
  const int last_sb = ((L - 1) >> 4) << 4;

  half8 qb[NT][KS];
  int nrow[NT];
  floatx4 acc[NT][DT];
  float m_run[NT], l_run[NT];
  load_queries<KVQ_INT4_TOKEN_HEAD, D, false>(p, lane, at, qb, nrow, acc, m_run, l_run);  // (the same words)
  const int n_min = at.n_min;

  // ---- producer side: quad wv of K, channel tiles 2 wv and 2 wv + 1 of V, the scales of K or of V ----
  struct Entries {
    uint32_t k, v, k_at, v_at;
  };
  const uint32_t k_fixed = (uint32_t)h * tile_bytes + 64u * g4 + 16u * (m16 & 3) + (uint32_t)wv * (4 * RB);
  const uint32_t v_fixed = (uint32_t)(H + h) * tile_bytes + 16u * m16 + 256u * wv;
  auto fetch_entries = [&](int g, Entries& e) {  // g is clamped by the caller
    const uint32_t tk = (uint32_t)min((g << 6) + 16 * sbk, last_sb), tv = (uint32_t)min((g << 6) + 16 * g4, last_sb);
    e.k = (uint32_t)table[tk >> bs_shift];
    e.v = (uint32_t)table[tv >> bs_shift];
    e.k_at = (tk & (uint32_t)(bs - 1)) * RB + k_fixed;
    e.v_at = tv & (uint32_t)(bs - 1);
  };
  uintx4 rk, rv;
  floatx4 rs = {};
  auto issue_loads = [&](const Entries& e) {
    rk = *(const uintx4*)(cache + ((uint64_t)e.k * block_stride + e.k_at));
    rv = *(const uintx4*)(cache + ((uint64_t)e.v * block_stride + (e.v_at * RB + v_fixed)));
    if (wv < 2)  // lane = token: wavefront 0 the K scales, 1 the V scales
      rs = ((const floatx4*)scales)[(uint64_t)e.v * (2u * H * bs) + ((uint32_t)((wv * H + h) * bs + m16) + e.v_at)];
  };
  auto publish = [&](int g, int half) {  // convert the loaded codes and put them in LDS
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      k_ops[half][wv][st][lane] = cvt_int4(rk[st]);
      v_ops[half][2 * wv + (st >> 1)][st & 1][lane] = cvt_int4(rv[st]);
    }
    const bool dead = (g << 6) + lane >= L;  // a slot that was never written: its scales are not data
    if (wv == 0) {
#pragma unroll
      for (int s = 0; s < KS; ++s) k_scales[half][s][lane] = dead ? 0.0f : rs[s] * p.scale_log2;
    } else if (wv == 1) {
      const float top = fmaxf(fmaxf(rs[0], rs[1]), fmaxf(rs[2], rs[3]));
      const float lsv = dead ? 0.0f : __builtin_amdgcn_logf(fmaxf(top, kMinVScale));
      const float rsv = dead ? 0.0f : __builtin_amdgcn_exp2f(-lsv);
#pragma unroll
      for (int s = 0; s < KS; ++s) v_scales[half][s][lane] = dead ? 0.0f : rs[s] * rsv;
      s_ops[half][1][lane] = lsv;
      s_ops[half][2][lane] = rsv;
    }
  };

  // ---- consumer side ----
  floatx4 S[NT][4];
  auto qk = [&](int half) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      half8 a[KS];
      floatx4 k4[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) a[s] = k_ops[half][u][s][lane];
      const floatx4 l4 = *(const floatx4*)&s_ops[half][1][16 * g4 + 4 * u];
#pragma unroll
      for (int s = 0; s < KS; ++s) k4[s] = *(const floatx4*)&k_scales[half][s][16 * g4 + 4 * u];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        floatx4 part[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s)
          part[s] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s], qb[nt][s], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float z = __builtin_fmaf(part[0][i], k4[0][i], l4[i]);
#pragma unroll
          for (int s = 1; s < KS; ++s) z = __builtin_fmaf(part[s][i], k4[s][i], z);
          S[nt][u][i] = z;
        }
      }
    }
  };
  half8 none[NT][2];  // (not written: the softmax leaves group-scaled probabilities in S)
  auto softmax = [&](int g, int half) {
    // some row's causal length ends inside the group: positions past it are masked here, one path for all that follows
    if ((g << 6) + 64 > n_min) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            S[nt][u][i] = (g << 6) + 16 * g4 + 4 * u + i < nrow[nt] ? S[nt][u][i] : -INFINITY;
    }
    online_softmax<MODE, NT, DT, false>(S, (const floatx4*)&s_ops[half][0][16 * g4], 0.0f, 0.0f, 0.0f, 0, nrow, m_run,
                                        l_run, acc, none);
  };
  auto pv = [&](int half) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      half8 a[2][2];
#pragma unroll
      for (int x = 0; x < 4; ++x) a[x >> 1][x & 1] = v_ops[half][2 * s + (x >> 1)][x & 1][lane];
      half8 pb[NT][2];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const floatx4 r4 = *(const floatx4*)&v_scales[half][s][16 * g4 + 4 * u];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int i = 0; i < 4; ++i) pb[nt][u >> 1][4 * (u & 1) + i] = (_Float16)__builtin_fmaf(S[nt][u][i], r4[i], 0.0f);
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[nt][2 * s + x] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[x][hf], pb[nt][hf], acc[nt][2 * s + x], 0, 0, 0);
    }
  };

  // ---- the walk: group g is consumed from half g % 2 while group g + 1 is converted into the
  // other half and group g + 2 is requested (indices past the end repeat the last group) ----
  Entries e_next, e_after;
  if (g0 < ng) {  // (a chunk's first rows see fewer groups than there may be pieces)
    Entries e0;
    fetch_entries(g0, e0);
    fetch_entries(min(g0 + 1, ng - 1), e_next);
    fetch_entries(min(g0 + 2, ng - 1), e_after);
    issue_loads(e0);
    publish(g0, 0);
    issue_loads(e_next);
  }
  __syncthreads();
  for (int g = g0; g < ng; ++g) {
    const int half = (g - g0) & 1;
    if (wave_live) {
      qk(half);
      softmax(g, half);
      pv(half);
    }
    // group g + 1 (requested one iteration ago) into the other half; request group g + 2
    publish(min(g + 1, ng - 1), half ^ 1);
    issue_loads(e_after);
    fetch_entries(min(g + 3, ng - 1), e_after);
    __syncthreads();
  }
  store_rows<D, false>(p, lane, at, acc, m_run, l_run);
}

// The kernel for more than kRowsPerWorkgroup rows at head_dim 128: eight wavefronts own 256 rows, one such
// workgroup runs on a compute unit, two wavefronts on a SIMD.  The matrix unit and the vector unit of a SIMD
// work side by side only for different wavefronts or for independent instructions of one, and two
// workgroups of the kernel above on a compute unit drift into doing the same thing at the same time: its
// two wavefronts took 4900 cycles for a group each (int8), of which the matrix unit was busy 2050.  Here
// the two wavefronts of a SIMD belong to two teams (0-3 and 4-7), and barriers hold them half a group
// apart, one in its matrix phase while the other is in its vector phase:
//   matrix phase: QK^T of the next group and P.V of this one; under the matrix instructions the wavefront's
//     share (an eighth, half of what it is above) of the codes is converted and published, and the
//     logits of the first tokens and their maxima are worked out while the last ones' are contracted.  One
//     code path, without a branch: the compiler moves what two branches share ahead of both, which put
//     all conversions and the wait for their loads in front of the first matrix instruction;
//   vector phase: maxima across lanes, probabilities, rescaling, masks, the addresses of the next loads.
// K runs a phase ahead of V, so that a phase's first operands can be read before the barrier that opens it:
// K is held in three buffers, V in two; 83 KB of operands and scales, 64 KB of table entries.  (V phases at
// the higher priority: 318 -> 315 us int8, 295 -> 290 fp8; the matrix phases at the higher: 332 and 300.)
// 8 x 512 tokens over 4608, 32 / 8 heads, against the kernel above: int8 343 -> 330 us, fp8 309 -> 298.  (An
// unquantized and a plain int4 cache, with 192 and 72 bytes of registers spilled, gained half of that.)  What
// bounds it: a wavefront is resident about 5000 cycles for a group, of which it waits 26 % (barriers and loads)
// and 33 % to issue; its 1024 cycles of matrix and 1600 of vector instructions are 2600 of the 3000 that its SIMD
// spends on a wavefront's group, so the teams' phases follow each other more than they overlap.  Each phase lasts as
// long as the slower team's: the two barriers of a group are the next thing to take out.
template <int MODE>
__global__ __launch_bounds__(512, 2) void attn_wide_kernel(const AttnArgs p) {
  constexpr bool FP8 = MODE == KVQ_FP8E4M3_BLOCK_HEAD || MODE == KVQ_FP8E4M3_TENSOR;
  constexpr bool TOKEN_SCALE = MODE == KVQ_INT8_TOKEN_HEAD;
  static_assert(FP8 || TOKEN_SCALE, "the formats of one code per byte");
  constexpr int W = 8, D = 128, NT = 2;
  constexpr int RB = D;            // bytes per token row in a tile
  constexpr int DT = D / 16;       // 16-channel tiles of V / of the output
  constexpr int KJ = RB / 64;      // 16-byte K pieces per lane and quad
  constexpr int KS = D / 32;       // matrix-instruction steps over the channels
  static_assert(RB / 16 == W, "K (and V) of a group are eight 16-byte pieces per lane: a wavefront converts one of each");
  constexpr int kPace = 2;  // vector instructions behind a matrix instruction
  __shared__ half8 k_ops[3][4][KS][64];  // [buffer][quad of the sub-block][step][lane]
  __shared__ half8 v_ops[2][DT][2][64];  // [half][channel tile][tokens 0-7 | 8-15][lane]
  // [buffer]: K scale * log2e / sqrt(D), log2 and reciprocal of the V scale of the 64 tokens
  __shared__ __align__(16) float s_ops[3][3][64];
  __shared__ int32_t sh_table[kWideTable];  // block-table entries of the walk

  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int m16 = lane & 15, g4 = lane >> 4;
  const int H = p.num_kv_heads, bs = p.block_size, bs_shift = p.bs_shift;
  Place at;
  if (!place_rows<false, kWideRows, true>(p, lane, wv, at)) return;
  const int h = at.h, b = at.b, L = at.L, g0 = at.g0, ng = at.ng;

  const uint8_t* __restrict__ cache = p.cache;
  const float* __restrict__ scales = p.scales;
  const int32_t* __restrict__ table = p.block_tables + (size_t)b * p.max_blocks_per_seq;
  const uint32_t tile_bytes = (uint32_t)bs * RB;
  const uint32_t block_stride = 2u * (uint32_t)H * tile_bytes;
  const int sbk = m16 >> 2;  // sub-block this lane reads K from
  const uint32_t s_block_stride = TOKEN_SCALE ? 2u * H * bs : (MODE == KVQ_FP8E4M3_TENSOR ? 0u : 2u * H);
  const uint32_t s_kv = TOKEN_SCALE ? (uint32_t)H * bs : (MODE == KVQ_FP8E4M3_TENSOR ? 1u : (uint32_t)H);
  const int last_sb = ((L - 1) >> 4) << 4;

  // ---- q as the B operand of QK^T, causal lengths, running state ----
  half8 qb[NT][KS];
  int nrow[NT];
  floatx4 acc[NT][DT];
  float m_run[NT], l_run[NT];
  load_queries<MODE, D, false>(p, lane, at, qb, nrow, acc, m_run, l_run);
  const int n_min = at.n_min;

  // ---- producer side: this wavefront's share of a group's codes.  K runs a group ahead of V ----
  const uint32_t k_fixed = (uint32_t)h * tile_bytes + 64u * g4 + 16u * (m16 & 3);
  const uint32_t v_fixed = (uint32_t)(H + h) * tile_bytes + 16u * m16;
  const int blk0 = (g0 << 6) >> bs_shift;
  // (the table entries of the walk come from LDS: as loads they would have to be waited for, and every
  // load in flight behind them, before the addresses they give can be worked out)
  auto entry = [&](uint32_t pos) { return (uint64_t)(uint32_t)sh_table[min((int)(pos >> bs_shift) - blk0, kWideTable - 1)]; };
  uintx4 rk, rv;
  float sk_next = 0.0f, sv_next = 0.0f;
  uint64_t k_from = 0, v_from = 0;  // byte offsets in the cache
  // K of group g0 + jk, V of group g0 + jv: where this lane's pieces lie
  // (indices past the end repeat the last group)
  auto locate = [&](int jk, int jv) {
    const int gk = min(g0 + jk, ng - 1), gv = min(g0 + jv, ng - 1);
    const uint32_t tk = (uint32_t)min((gk << 6) + 16 * sbk, last_sb), tv = (uint32_t)min((gv << 6) + 16 * g4, last_sb);
    k_from = entry(tk) * block_stride + ((tk & (uint32_t)(bs - 1)) * RB + k_fixed);
    v_from = entry(tv) * block_stride + ((tv & (uint32_t)(bs - 1)) * RB + v_fixed);
    asm volatile("" : "+v"(k_from), "+v"(v_from));  // (here, not where they are used)
  };
  auto request_scales_at = [&](uint64_t block, uint32_t t) {
    const float* from = scales + (block * s_block_stride + (TOKEN_SCALE ? (uint32_t)(h * bs + m16) + (t & (uint32_t)(bs - 1)) : (MODE == KVQ_FP8E4M3_TENSOR ? 0u : (uint32_t)h)));
    sk_next = from[0];  // lane = token
    sv_next = from[s_kv];
  };
  auto request_scales = [&](int j) {
    const uint32_t t = (uint32_t)min((min(g0 + j, ng - 1) << 6) + 16 * g4, last_sb);
    request_scales_at(entry(t), t);
  };
  auto request_k = [&]() { rk = *(const uintx4*)(cache + k_from + (wv / KJ) * (4 * RB) + 256 * (wv % KJ)); };
  auto request_v = [&]() { rv = *(const uintx4*)(cache + v_from + 256 * wv); };
  auto request = [&]() {
    request_k();
    request_v();
  };
  auto publish_k = [&](uintx4& codes, int buf) {
    asm volatile("" : "+v"(codes));  // (converted here, not earlier)
    const int u = wv / KJ, at = wv % KJ;
    k_ops[buf][u][2 * at][lane] = cvt8<MODE>(codes[0], codes[1]);
    k_ops[buf][u][2 * at + 1][lane] = cvt8<MODE>(codes[2], codes[3]);
  };
  auto publish_v = [&](int half) {
    asm volatile("" : "+v"(rv));
    v_ops[half][wv][0][lane] = cvt8<MODE>(rv[0], rv[1]);
    v_ops[half][wv][1][lane] = cvt8<MODE>(rv[2], rv[3]);
  };
  // V bits of tokens past the last position are cleared first: a NaN times 0 is NaN
  auto clear_missing = [&](int g) {
    if (!FP8 || (g << 6) + 64 <= L) return;
    const int live = L - ((g << 6) + 16 * g4);  // tokens of this lane's sub-block below L
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = min(max(live - 4 * e, 0), 4);
      rv[e] &= n == 4 ? ~0u : (1u << (8 * n)) - 1u;
    }
  };
  auto publish_scales = [&](int j, float sk, float sv) {  // of group g0 + j
    const int g = min(g0 + j, ng - 1), buf = j % 3;
    float skp = sk * p.scale_log2;
    float lsv = __builtin_amdgcn_logf(fmaxf(sv, kMinVScale));
    float rsv = __builtin_amdgcn_exp2f(-lsv);
    if (TOKEN_SCALE && (g << 6) + lane >= L) {
      skp = 0.0f;  // a slot that was never written: its scales are not data
      lsv = 0.0f;
      rsv = 0.0f;
    }
    s_ops[buf][0][lane] = skp;
    s_ops[buf][1][lane] = lsv;
    s_ops[buf][2][lane] = rsv;
  };

  // ---- consumer side ----
  floatx4 S[NT][4];
  half8 pb[NT][2];
  auto mma = [&](const half8& a, const half8& b, const floatx4& c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); };
  float mx[NT];
  constexpr float skp = 0.0f, lsv = 0.0f;  // (the maxima of formats without token scales are those of S)
  half8 op[2][4];  // operands of two chunks of eight matrix instructions
  floatx4 k4[2] = {}, l4[2] = {};
  constexpr int HS = KS / 2, QC = 2 * HS, PC = DT / 2;  // chunks of QK^T (two quads, two steps) and of P.V (two tiles)
  auto read_k = [&](int c, int buf) {
#pragma unroll
    for (int x = 0; x < 4; ++x) op[c & 1][x] = k_ops[buf][2 * (c / HS) + (x & 1)][2 * (c % HS) + (x >> 1)][lane];
  };
  auto read_v = [&](int c, int half) {
#pragma unroll
    for (int x = 0; x < 4; ++x) op[(QC + c) & 1][x] = v_ops[half][2 * c + (x & 1)][x >> 1][lane];
  };
  auto read_scales = [&](int pair, int buf) {
    const floatx4* sc = (const floatx4*)&s_ops[buf][0][16 * g4];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      k4[x] = sc[2 * pair + x];
      l4[x] = sc[kScalePitch + 2 * pair + x];
    }
  };
  auto mm_k = [&](int c) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int u = 2 * (c / HS) + (x & 1);
        S[nt][u] = mma(op[c & 1][x], qb[nt][2 * (c % HS) + (x >> 1)], S[nt][u]);
      }
  };
  auto mm_v = [&](int c) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        floatx4& d = acc[nt][2 * c + (x & 1)];
        d = mma(op[(QC + c) & 1][x], pb[nt][x >> 1], d);
      }
  };
  // N matrix instructions, with READS LDS reads dealt out between them and VALU vector ones behind each
  auto pace = [&](auto N, auto READS, auto VALU) {
    static_for<decltype(N)::value>([&](auto X) {
      constexpr int x = decltype(X)::value, n = decltype(N)::value, r = decltype(READS)::value;
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      constexpr int now = (x + 1) * r / n - x * r / n;
      if constexpr (now > 0) __builtin_amdgcn_sched_group_barrier(0x100, now, 0);
      if constexpr (decltype(VALU)::value > 0) __builtin_amdgcn_sched_group_barrier(0x2, decltype(VALU)::value, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  using Whole = SoftmaxForm<MODE, false>;
  // The matrix phase: QK^T of group g0 + j (its first operands are already in op[0]), P.V of the group
  // before.  Under the matrix instructions: this wavefront's share of the next K and V is converted, and
  // the logits and their maxima are worked out (unmasked).
  auto matrix_phase = [&](auto PVC, int j, int kbuf, int next_kbuf) {
    constexpr bool PV = decltype(PVC)::value;
    const int vhalf = (j + 1) & 1;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      mx[nt] = -INFINITY;
#pragma unroll
      for (int u = 0; u < 4; ++u) S[nt][u] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<QC>([&](auto C) {
      constexpr int c = decltype(C)::value;
      constexpr bool sc = Whole::kLogits && (c + 1) % HS == 0;
      mm_k(c);
      if constexpr (c + 1 < QC) read_k(c + 1, kbuf);
      else if constexpr (PV) read_v(0, vhalf);
      if constexpr (c == HS) {
        softmax_logits<MODE, NT, false>(S, 0, k4[0], l4[0], skp, lsv, 0, nrow, mx);
        softmax_logits<MODE, NT, false>(S, 1, k4[1], l4[1], skp, lsv, 0, nrow, mx);
      }
      if constexpr (sc) read_scales(c / HS, kbuf);
      if constexpr (c == 0) publish_k(rk, next_kbuf);
      if constexpr (c == 1) publish_v(j & 1);
      pace(std::integral_constant<int, 8>{}, std::integral_constant<int, (c + 1 < QC || PV ? 4 : 0) + (sc ? 4 : 0)>{}, std::integral_constant<int, kPace>{});
      if constexpr (c == QC - 1) {
        request();
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    if constexpr (PV) {
      static_for<PC>([&](auto C) {
        constexpr int c = decltype(C)::value;
        mm_v(c);
        if constexpr (c + 1 < PC) read_v(c + 1, vhalf);
        if constexpr (c == 0) {
          softmax_logits<MODE, NT, false>(S, 2, k4[0], l4[0], skp, lsv, 0, nrow, mx);
          softmax_logits<MODE, NT, false>(S, 3, k4[1], l4[1], skp, lsv, 0, nrow, mx);
        }
        pace(std::integral_constant<int, 8>{}, std::integral_constant<int, c + 1 < PC ? 4 : 0>{}, std::integral_constant<int, c == 0 ? kPace : 0>{});
      });
    } else {
      softmax_logits<MODE, NT, false>(S, 2, k4[0], l4[0], skp, lsv, 0, nrow, mx);
      softmax_logits<MODE, NT, false>(S, 3, k4[1], l4[1], skp, lsv, 0, nrow, mx);
    }
  };
  // TAIL: some row's causal length ends inside the group: positions past it are masked, and the
  // maxima taken again.
  auto vector_phase = [&](auto TAILC, int g, int sbuf) {
    constexpr bool TAIL = decltype(TAILC)::value;
    using F = SoftmaxForm<MODE, TAIL>;
    const floatx4* sc = (const floatx4*)&s_ops[sbuf][0][16 * g4];
    floatx4 r4[4] = {};
    if constexpr (F::TOKEN_SCALE) {
#pragma unroll
      for (int u = 0; u < 4; ++u) r4[u] = sc[2 * kScalePitch + u];
    }
    float skp = 0.0f, lsv = 0.0f, rsv = 1.0f;
    if constexpr (FP8) {
      skp = s_ops[sbuf][0][lane];
      lsv = s_ops[sbuf][1][lane];
      rsv = s_ops[sbuf][2][lane];
    }
    if constexpr (TAIL) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        mx[nt] = -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float z = S[nt][u][i];
            if constexpr (!F::kLogits) z = __builtin_fmaf(z, skp, lsv);
            z = (g << 6) + 16 * g4 + 4 * u + i < nrow[nt] ? z : -INFINITY;
            S[nt][u][i] = z;
            mx[nt] = fmaxf(mx[nt], z);
          }
      }
    } else if constexpr (FP8) {
      if (__any(skp < 0.0f)) {  // (a negative softmax scale, or static scale)
        const float sign = skp < 0.0f ? -1.0f : 1.0f;
        skp *= sign;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          mx[nt] = -INFINITY;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            S[nt][u] *= sign;
            softmax_logits<MODE, NT, TAIL>(S, u, k4[0], l4[0], skp, lsv, 0, nrow, mx);
          }
        }
      }
    }
    float alpha[NT], msub[NT];
    softmax_maxima<MODE, NT, TAIL>(mx, skp, lsv, m_run, alpha, msub);
    softmax_probabilities<MODE, NT, TAIL, true>(S, sc, r4, skp, rsv, alpha, msub, l_run, pb);
    softmax_rescale<NT, DT>(alpha, acc);
  };

  // ---- the walk ----
  const int team = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
  const bool live = __builtin_amdgcn_readfirstlane((int)at.wave_live) != 0;
  const int n = ng - g0;
  if (n > 0) {  // (a chunk's first rows see fewer groups than there may be pieces)
    auto fence = [&]() {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    auto phase_end = [&]() {  // this wavefront's writes to LDS are done
      fence();
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      fence();
    };
    auto phase_end_reads = [&]() {  // nothing was written
      fence();
      __builtin_amdgcn_s_barrier();
      fence();
    };
    // (start: entries, then codes, then LDS, a round trip each and nothing twice; the entries of the first
    // groups do not go through LDS)
    const int blocks = min((min(last_sb, (ng << 6) - 1) >> bs_shift) - blk0 + 1, kWideTable);
    uintx4 first_k[2];  // K of groups 0 and (team 1) 1
    {
      uint32_t e[3], ev, es;
#pragma unroll
      for (int j = 0; j < 3; ++j) e[j] = table[min((min(g0 + j, ng - 1) << 6) + 16 * sbk, last_sb) >> bs_shift];
      const uint32_t tv = (uint32_t)min((g0 << 6) + 16 * g4, last_sb), ts = (uint32_t)min((min(g0 + 1, ng - 1) << 6) + 16 * g4, last_sb);
      ev = table[tv >> bs_shift];
      es = table[ts >> bs_shift];
      const int mine = (int)threadIdx.x < blocks ? table[blk0 + (int)threadIdx.x] : 0;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (j > team + 1) continue;
        const uint32_t tk = (uint32_t)min((min(g0 + j, ng - 1) << 6) + 16 * sbk, last_sb);
        k_from = (uint64_t)e[j] * block_stride + ((tk & (uint32_t)(bs - 1)) * RB + k_fixed);
        request_k();
        if (j <= team) first_k[j & 1] = rk;
      }
      v_from = (uint64_t)ev * block_stride + ((tv & (uint32_t)(bs - 1)) * RB + v_fixed);
      request_v();
      if (wv == 0) {
        request_scales_at(ev, tv);
        const float sk = sk_next, sv = sv_next;
        request_scales_at(es, ts);
        publish_scales(0, sk, sv);
      }
      if ((int)threadIdx.x < blocks) sh_table[threadIdx.x] = mine;
      for (int i = (int)threadIdx.x + 64 * W; i < blocks; i += 64 * W) sh_table[i] = table[blk0 + i];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (j <= team) publish_k(first_k[j], j);
    phase_end();
    locate(2 + team, 1);
    if (team == 1) phase_end_reads();
    int kbuf = 0, kb1 = 1, kb2 = 2;  // buffers of K of groups i, i + 1, i + 2
    auto rotate = [&]() {
      const int t = kbuf;
      kbuf = kb1;
      kb1 = kb2;
      kb2 = t;
    };
    auto vector_part = [&](int i) {
      if (((g0 + i) << 6) + 64 > n_min) vector_phase(std::true_type{}, g0 + i, kbuf);
      else vector_phase(std::false_type{}, g0 + i, kbuf);
    };
    auto scales_part = [&](int i) {
      if (wv == 0) {
        publish_scales(i + 1, sk_next, sv_next);
        request_scales(i + 2);
      }
    };
    if (live) {
      read_k(0, 0);
      clear_missing(g0);
      matrix_phase(std::false_type{}, 0, 0, team ? 2 : 1);
      phase_end();
      for (int i = 0; i + 1 < n; ++i) {
        scales_part(i);
        locate(i + 3 + team, i + 2);
        vector_part(i);
        // (in the registers or on their way: K of group i + 2 + team, V of group i + 1)
        rotate();
        read_k(0, kbuf);
        phase_end();
        clear_missing(g0 + i + 1);
        __builtin_amdgcn_s_setprio(0);
        matrix_phase(std::true_type{}, i + 1, kbuf, team ? kb2 : kb1);
        __builtin_amdgcn_s_setprio(1);
        phase_end();
      }
      vector_part(n - 1);
      phase_end_reads();
      read_v(0, (n - 1) & 1);
#pragma unroll
      for (int c = 0; c < PC; ++c) {
        if (c + 1 < PC) read_v(c + 1, (n - 1) & 1);
        mm_v(c);
      }
    } else {
      auto publish_all = [&](int j) {
        clear_missing(min(g0 + j, ng - 1));
        publish_k(rk, team ? kb2 : kb1);
        publish_v(j & 1);
        request();
      };
      publish_all(0);
      phase_end();
      for (int i = 0; i + 1 < n; ++i) {
        scales_part(i);
        locate(i + 3 + team, i + 2);
        rotate();
        phase_end();
        publish_all(i + 1);
        phase_end();
      }
      phase_end_reads();
    }
    if (team == 0) phase_end_reads();
  }
  store_rows<D, false>(p, lane, at, acc, m_run, l_run);
}

// ---- the pieces of cut contexts put together: out = sum_c w_c out_c / sum_c w_c with
// w_c = 2^(lse_c), lse_c the base-2 logarithm of piece c's softmax denominator.  A thread owns four
// channels of a row; workgroup = (sequence, 256 threads' worth of its rows), so that those of a
// sequence that was left whole end at once.  Memory-bound (every piece's rows read once, `out`
// written once), all loads of up to four pieces in flight together. ----
__global__ __launch_bounds__(256) void merge_kernel(const AttnArgs p, int quads_shift, int parts) {
  const int b = (int)(blockIdx.x / (uint32_t)parts), part = (int)(blockIdx.x - (uint32_t)b * parts);
  const int first = p.ws_prefix[b], splits = 1 + p.ws_prefix[b + 1] - first;
  if (splits == 1) return;
  const size_t seq_rows = (size_t)p.q_len * p.num_q_heads;
  const size_t i = (size_t)part * 256 + threadIdx.x, row = i >> quads_shift;  // (row, four channels)
  if (row >= seq_rows) return;
  const size_t quads = seq_rows << quads_shift;  // floatx4s per piece
  floatx4* const out = (floatx4*)p.out + (size_t)b * quads + i;
  // (piece c lies c pieces from here; the first one's rows are in `out`)
  const floatx4* __restrict__ pieces = (const floatx4*)p.ws_acc + (size_t)first * quads + i;
  const float* __restrict__ lse = p.ws_ml + ((size_t)p.batch + first) * seq_rows + row;
  floatx4 sum = *out;
  float M = p.ws_ml[(size_t)b * seq_rows + row], den = 1.0f;
  for (int c0 = 1; c0 < splits; c0 += 4) {
    floatx4 a[4];
    float e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = min(c0 + k, splits - 1);
      a[k] = pieces[(size_t)(c - 1) * quads];
      e[k] = c0 + k < splits ? lse[(size_t)(c - 1) * seq_rows] : -INFINITY;
    }
    const float top = fmaxf(fmaxf(fmaxf(e[0], e[1]), fmaxf(e[2], e[3])), M);
    const float safe = top == -INFINITY ? 0.0f : top;
    const float keep = __builtin_amdgcn_exp2f(M - safe);
    sum *= keep;
    den *= keep;
    M = top;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float w = __builtin_amdgcn_exp2f(e[k] - safe);
      sum += w * a[k];
      den += w;
    }
  }
  *out = sum * (1.0f / den);
}

}  // namespace

template <bool PREFIX>
hipError_t launch_many_rows(const AttnArgs& a, int all_rows, int walks, hipStream_t stream) {
  const int row_blocks = (all_rows + kRowsPerWorkgroup - 1) / kRowsPerWorkgroup;
  const dim3 grid((unsigned)((size_t)walks * a.num_kv_heads * row_blocks));
  const dim3 block(64 * kWavesPerGroup);
#define KVQ_LAUNCH_PREFILL(MODE, KERNEL_64)                                                   \
  if (a.head_dim == 128)                                                                      \
    hipLaunchKernelGGL((attn_rows_kernel<MODE, 128, PREFIX, false>), grid, block, 0, stream, a); \
  else                                                                                        \
    hipLaunchKernelGGL(KERNEL_64, grid, block, 0, stream, a)
  if (a.mode == KVQ_INT8_TOKEN_HEAD) {
    KVQ_LAUNCH_PREFILL(KVQ_INT8_TOKEN_HEAD, (attn_rows64_kernel<KVQ_INT8_TOKEN_HEAD, PREFIX>));
  } else if (a.mode == KVQ_FP8E4M3_BLOCK_HEAD) {
    KVQ_LAUNCH_PREFILL(KVQ_FP8E4M3_BLOCK_HEAD, (attn_rows_kernel<KVQ_FP8E4M3_BLOCK_HEAD, 64, PREFIX, false>));
  } else if (a.mode == KVQ_BF16_PLAIN) {
    KVQ_LAUNCH_PREFILL(KVQ_BF16_PLAIN, (attn_rows64_kernel<KVQ_BF16_PLAIN, PREFIX>));
  } else if (a.mode == KVQ_INT4_TOKEN_HEAD) {  // (head_dim 128 only)
    hipLaunchKernelGGL((attn_rows_kernel<KVQ_INT4_TOKEN_HEAD, 128, PREFIX, false>), grid, block, 0, stream, a);
  } else if (a.mode == KVQ_INT4_GROUP32) {  // (and never with a shared prefix)
    if constexpr (!PREFIX) hipLaunchKernelGGL(attn_rows_group_kernel, grid, block, 0, stream, a);
  } else {
    KVQ_LAUNCH_PREFILL(KVQ_FP8E4M3_TENSOR, (attn_rows_kernel<KVQ_FP8E4M3_TENSOR, 64, PREFIX, false>));
  }
#undef KVQ_LAUNCH_PREFILL
  return hipGetLastError();
}

// The kernel for 256 rows and, behind it, the one for 128: the lengths have one of them end at once.
template <int MODE>
hipError_t launch_either(const AttnArgs& a, hipStream_t stream) {
  const int blocks = (a.rows + kRowsPerWorkgroup - 1) / kRowsPerWorkgroup, wide_blocks = (a.rows + kWideRows - 1) / kWideRows;
  AttnArgs wide = a;
  wide.extra_pieces = a.wide_extra;
  hipLaunchKernelGGL((attn_wide_kernel<MODE>), dim3((unsigned)((size_t)(a.batch + a.wide_extra) * a.num_kv_heads * wide_blocks)),
                     dim3(512), 0, stream, wide);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_rows_kernel<MODE, 128, false, true>), dim3((unsigned)((size_t)(a.batch + a.extra_pieces) * a.num_kv_heads * blocks)),
                     dim3(64 * kWavesPerGroup), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_prefill(const AttnArgs& a, hipStream_t stream) {
  hipError_t e;
  if (a.wide_groups == 0) e = launch_many_rows<false>(a, a.rows, a.batch + a.extra_pieces, stream);
  else if (a.mode == KVQ_INT8_TOKEN_HEAD) e = launch_either<KVQ_INT8_TOKEN_HEAD>(a, stream);
  else if (a.mode == KVQ_FP8E4M3_BLOCK_HEAD) e = launch_either<KVQ_FP8E4M3_BLOCK_HEAD>(a, stream);
  else e = launch_either<KVQ_FP8E4M3_TENSOR>(a, stream);
  if (e != hipSuccess || !a.merge) return e;
  const int quads_shift = a.head_dim == 128 ? 5 : 4;
  const int64_t parts = ((((int64_t)a.q_len * a.num_q_heads) << quads_shift) + 255) / 256;
  hipLaunchKernelGGL(merge_kernel, dim3((unsigned)(a.batch * parts)), dim3(256), 0, stream, a, quads_shift,
                     (int)parts);
  return hipGetLastError();
}

// the shared groups of a decode or verification batch (a.shared_groups > 0), ahead of the
// streaming kernel
hipError_t launch_prefix(const AttnArgs& a, hipStream_t stream) {
  return launch_many_rows<true>(a, a.batch * a.rows, a.prefix_chunks, stream);
}

}  // namespace kvq
