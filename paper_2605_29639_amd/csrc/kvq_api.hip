// extern "C" entry points declared in include/kvq.h: host-side validation first (no HIP call
// is made for a bad argument), then the kernel launches on the caller's stream.
#include <math.h>
#include <stdlib.h>

#include <mutex>

#include "kvq_internal.h"
#ifdef KVQ_PROFILE
#include "../../include/kvq_prof.h"
#endif

namespace {

bool desc_ok(const kvq_cache_desc_t* d, int* err) {
  if (!d) { *err = KVQ_E_NULLPTR; return false; }
  if (d->mode != KVQ_INT8_TOKEN_HEAD && d->mode != KVQ_FP8E4M3_BLOCK_HEAD &&
      d->mode != KVQ_BF16_PLAIN && d->mode != KVQ_FP8E4M3_TENSOR &&
      d->mode != KVQ_INT4_TOKEN_HEAD && d->mode != KVQ_INT4_GROUP32) {
    *err = KVQ_E_BAD_MODE;
    return false;
  }
  const int bs = d->block_size;
  const bool bs_ok = bs >= 16 && bs <= 256 && (bs & (bs - 1)) == 0;
  if (d->num_blocks < 0 || !bs_ok || d->num_kv_heads <= 0 ||
      (d->head_dim != 64 && d->head_dim != 128) ||
      (kvq::is_int4(d->mode) && d->head_dim != 128)) {
    *err = KVQ_E_BAD_SHAPE;
    return false;
  }
  // a pool beyond 2^46 bytes (64 TiB) is not a real one, and sizes must not wrap
  const unsigned __int128 bytes = (unsigned __int128)d->num_blocks * 2 * (unsigned)d->num_kv_heads *
                                  (unsigned)bs * (unsigned)d->head_dim * 2;
  if (bytes > ((unsigned __int128)1 << 46)) {
    *err = KVQ_E_BAD_SHAPE;
    return false;
  }
  return true;
}

// Wavefronts the current GPU holds at once at two per SIMD: compute units x 4 SIMDs x 2 (2048
// on a whole MI355X; fewer under a partition mode or a CU mask).  Read once per device; where
// no device can be asked (a machine without a GPU, where only sizes and validation run) the
// whole chip's figure stands in.
constexpr int kMaxDevices = 64;
std::mutex g_device_mutex;
int g_resident_waves[kMaxDevices] = {};

int64_t auto_waves() {
  constexpr int64_t kWholeChip = 256 * 4 * 2;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return kWholeChip;
  std::lock_guard<std::mutex> lock(g_device_mutex);
  if (g_resident_waves[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0 || cus > 4096)
      return kWholeChip;
    g_resident_waves[dev] = cus * 4 * 2;
  }
  return g_resident_waves[dev];
}

// the KVQ_DEBUG checks (defined with their kernels further down)
bool debug_checks();
int debug_check_slots(const int64_t* slot_mapping, int32_t num_tokens, int64_t num_slots,
                      hipStream_t stream);

int ilog2(int x) {
  int s = 0;
  while ((1 << s) < x) ++s;
  return s;
}

// Pieces the many-row kernel should cut the contexts into where all sequences have `groups` 64-token
// groups, given how many the workspace has room for.  Without a split a call launches `walks` workgroups
// of 128 query rows, and one sequence's chunk of a prompt leaves most of the chip idle (512 tokens of
// 32 / 8 heads: 128 workgroups, where two run on each of 256 compute units).  The estimate below is in
// microseconds, from measurements at head_dim 128: 2.6 per 64-token group and workgroup with two
// of them on a compute unit, 0.6 of that with one, about 3 until a workgroup's first group is
// consumed; splitting adds the second launch and writes and reads 64 KB per workgroup.  One
// sequence's 512 tokens over 16384 cached ones (fp8, 32 / 8 heads): 427 us in one piece, 178 in
// four with the merge (159 with the present kernels); eight such chunks over 4096 (1024 workgroups, two full rounds) stay whole.
// (wide: the kernel for kWideRows, one workgroup of 256 rows on a compute unit where the other kernel has two
// of 128: 2.3 us per group, the same for the last round, 5 until a first group is consumed and 9 from one
// workgroup of a compute unit to the next, which nothing overlaps.)
int64_t equal_pieces(int64_t slots, int64_t walks, int64_t groups, int64_t room, bool wide, double* least_us) {
  int64_t best = 1;
  double best_us = 0.0;
  for (int64_t c = 1; c <= room && c <= kvq::kMaxContextSplits && (c == 1 || c * 2 <= groups); ++c) {
    const int64_t n = walks * c, rest = n % slots;
    if (c > 1 && (n > 4 * slots || walks >= 4 * slots)) break;
    const double rounds = (double)(n / slots) + (rest == 0 ? 0.0 : 2 * rest <= slots && !wide ? 0.6 : 1.0);
    const double piece = (double)((groups + c - 1) / c);
    const double us = (wide ? rounds * 2.3 * piece + 5.0 + 9.0 * (rounds > 1.0 ? rounds - 1.0 : 0.0)
                            : rounds * (3.0 + 2.6 * piece)) +
                      (c > 1 ? 6.0 + (wide ? 0.05 : 0.025) * (double)n : 0.0);
    if (c == 1 || us < best_us) {
      best = c;
      best_us = us;
    }
  }
  *least_us = best_us;
  return best;
}

// How the many-row kernel may cut the contexts: the pieces themselves are worked out on the device, from
// the lengths (max_seq_len is only a bound on them).  With few workgroups: as many cuts as equal
// contexts of max_seq_len would get, and pieces long enough to be worth the partials they leave (a
// workgroup's partials cost the chip 0.025 us, its groups 1.6 us of one slot).  With enough
// workgroups and fewer than 128 rows: one slot's worth of cuts per (kv head, row block), for contexts
// longer than 1.5 times what a slot gets on average; the streaming kernel, which such calls would
// otherwise take, splits any mixture of lengths evenly.  64 sequences, one of 65536 tokens and the rest
// of 1000, 96 rows, 64 / 8 heads, int8: streaming 211 us, many-row uncut 1629, cut 109; 300 of 40 to
// 2000 tokens: 414, 162 and 175 (the pieces are worked out, and none is needed).  A 512-token chunk
// on its own under a bound of 32768: 21 us without leave to cut, 28 cut by the bound, 23 now (the
// second launch finds nothing to do); over 4096 tokens, same bound: 117, 63 and 63.
// The kernel for kWideRows gets int8 and e4m3 calls whose walks all take long and are much alike: both kernels
// are launched then, and the lengths decide on the device which of them does the call, this one where the
// contexts hold three quarters of what the bound allows and the shortest has half of it.  In 3915 random
// calls, those the rule takes with lengths near the bound: its time by that of the kernel for 128 rows 0.924
// (int8) and 0.932 (e4m3) on average, 0.97 and 1.01 at most; with lengths as far apart as allowed 0.965, up to
// 1.05.  Below 100 us the launch that ends at once takes back what it gains (4 x 256 tokens over 3000: int8
// 80 -> 75, e4m3 71.7 -> 70.8 without that launch), with chunks of more than an eighth of the context (whose first
// rows see much less than their last) it loses up to 8 %, with a quarter of the sequences short 12 %; bf16 and
// int4 gain half as much.  The kernel for 128 rows alone -> both launched: 8 x 512 tokens over 4608 int8
// 343 -> 330 us, e4m3 309 -> 298; 1 x 512 over 16896 175 -> 164, 159 -> 148.  The launch that ends at once takes
// 2.1 us ahead of or behind the other (3 to 4 above 512 workgroups; 4.6 as a profiler sees it), also where the contexts are far
// below the bound: 8 x 512 over 520 under a bound of 32768 49.6 -> 53.0 us, 1 x 512 over 512 21.3 -> 24.0.
void cut_contexts(const kvq_cache_desc_t* d, int64_t batch, int64_t q_len, int64_t rows, int64_t seq_rows,
                  int64_t groups, int64_t slot_rows, int64_t slots, kvq::AttnPlan* plan) {
  const int64_t room = slot_rows / seq_rows;
  const int64_t per_seq = d->num_kv_heads * ((rows + kvq::kRowsPerWorkgroup - 1) / kvq::kRowsPerWorkgroup);
  double us, wide_us;
  const int64_t c = equal_pieces(slots, batch * per_seq, groups, room / batch + 1, false, &us);
  const bool codes = d->mode == KVQ_INT8_TOKEN_HEAD || d->mode == KVQ_FP8E4M3_BLOCK_HEAD || d->mode == KVQ_FP8E4M3_TENSOR;
  if (codes && d->head_dim == 128 && rows > kvq::kRowsPerWorkgroup && us >= 100.0 && 8 * q_len <= 64 * groups &&
      groups * 64 <= (int64_t)kvq::kWideTable * d->block_size) {
    const int64_t wide_per_seq = d->num_kv_heads * ((rows + kvq::kWideRows - 1) / kvq::kWideRows);
    const int64_t wide_c = equal_pieces(slots / 2, batch * wide_per_seq, groups, room / batch + 1, true, &wide_us);
    if (wide_us < 0.92 * us) {
      plan->wide_groups = (int32_t)((3 * batch * groups + 3) / 4);
      plan->wide_least = (int32_t)((groups + 1) / 2);
      // (of its own: a batch of which one context is at the bound and the others are short goes to the kernel
      // for 128 rows, whose cuts it needs.  4 x 771 tokens, one over 8963 and three over 800, int8: 201 us where
      // it has them, 229 where the other kernel's none stood for both; 14 x 115 tokens, 64 / 8 heads, one over
      // 10649: 127 and 260.)
      plan->wide_extra = (int32_t)(batch * (wide_c - 1));
    }
  }
  plan->piece_min = (int32_t)(per_seq < 32 ? 2 : per_seq / 16);
  if (c > 1) {
    plan->extra_pieces = (int32_t)(batch * (c - 1));
  } else if ((rows < kvq::kRowsPerWorkgroup || d->mode == KVQ_INT4_GROUP32) && groups > 2 * plan->piece_min) {
    // (group-scaled int4 with any number of rows, since its streaming kernel splits any mixture evenly: 5 x 266 tokens
    // over 266 to 5000, 4 kv heads, 99 us streaming, 138 with the longest context uncut, 60 with it cut)
    const int64_t extra = (slots + per_seq - 1) / per_seq;
    plan->extra_pieces = (int32_t)(extra < room ? extra : room);
    plan->piece_share = 1.5f * (float)per_seq / (float)slots;
  }
}

// Whether a call goes to the many-row kernel (a workgroup per 128 query rows of a kv head, keys and values
// dequantized once for all of them) or to the streaming kernel (32 rows at a time, the keys and values
// streamed again for each such group).  128 rows and more always do; below that the workgroup is not full,
// and what decides is how often the streaming kernel would read the cache.  Measured streaming -> many-row,
// us a call: 32 sequences of 2 k to 8 k tokens, 64 / 8 heads, head_dim 128, 96 rows: int8 213 -> 162,
// int4 180 -> 160, bf16 363 -> 194; 64 rows: int8 158 -> 158, int4 126 -> 154, bf16 246 -> 184; 40 rows:
// int8 140 -> 148, bf16 236 -> 177.  head_dim 64: int8 96 rows 125 -> 117 and, short, 43 -> 45, 120 rows
// 77 -> 41; bf16 40 rows 117 -> 118, 96 rows 180 -> 123.  With a workgroup for every slot of the chip
// and short contexts (little to lose to uneven lengths) 33 rows are enough: 200 sequences of up to 300
// tokens, 48 rows, 91 -> 49; 128 of up to 2000, 48 rows, 177 -> 138; but 60 of up to 6000, 56 rows,
// 190 -> 204.  (Group-scaled int4 has a kernel and a rule of its own: group_rows.)
bool many_rows(const kvq_cache_desc_t* d, int64_t batch, int64_t rows, int64_t max_seq_len,
               int64_t chunk_tokens, int64_t slots) {
  if (d->mode == KVQ_INT4_GROUP32) return false;
  if (rows >= kvq::kRowsPerWorkgroup) return true;
  if (chunk_tokens > 0) return false;  // (a caller's split-K granule is the streaming kernel's)
  // (the merge's launch has 32 threads for every output row, and fewer than 2^32)
  if (batch * d->num_kv_heads > 1 << 19) return false;
  const int64_t passes = (rows + 31) / 32 + (d->mode == KVQ_BF16_PLAIN ? 1 : 0);
  if (passes >= (d->head_dim == 128 ? 3 : 4)) return rows > 32;
  return rows > 32 && d->head_dim == 128 && max_seq_len <= 2048 &&
         batch * d->num_kv_heads >= slots;
}

// Whether a call goes to the many-row kernel of group-scaled int4 (one that a caller's granule does not keep on the
// streaming kernel, and whose pairs do not get a workgroup each).  The streaming kernel takes 2.2 us for a wavefront's
// group of 16 rows, two wavefronts to a SIMD's time, and 8.3 beside that; the other one 1.35 of what equal_pieces says,
// with no less for a row block of 33 rows than for one of 128.  A tenth in doubt is the streaming kernel's, whose
// ranges are even whatever the mixture of lengths, and a twentieth beside as many pieces as the workspace has room for
// (34 random calls that the second line leaves to the streaming kernel: many-row 1.00 of its time on average, up to
// 1.28, 22 of 2300 to 9300 tokens, 160 rows, 4 kv heads, 196 and 252; as strict as the first it would leave 32 more,
// of which it takes 0.96).  us a call by the estimates and measured, streaming and many-row, 8 kv heads: 64 sequences
// of 2000 to 4000 tokens, 64 rows, 285 and 225
// (bounds), 231 and 221; 20 of 500 to 1000, 96 rows, 41 and 36, 44.7 and 35.4; 2 x 128 tokens over 2500, 512 rows, 52
// and 40, 54 and 42; 1 x 512 over 16896, 2048 rows, 590 and 297, 531 and 310; not taken: 8 of 2000 to 8000, 64 rows,
// 77 and 85, 56 and 62; 1 x 441 tokens over 469, 2 kv heads, 14 and 20, 22 and 25; 32 rows, of which one wavefront in
// four is busy, 147 and 225, 126 and 153 at the first lengths.  Of 45 random calls that it takes, mixtures of long
// and short among them, 0.64 of the streaming kernel's time on average and 1.00 at most; the error against 64 bits is
// no larger (1.67e-4 and now 1.65e-4, 1.54e-4 and 1.52e-4, 1.64e-4 twice, 1.72e-4 twice).
bool group_rows(const kvq_cache_desc_t* d, int64_t batch, int64_t rows, int64_t groups, int64_t slots, int64_t room) {
  if (d->mode != KVQ_INT4_GROUP32 || rows <= 32 || batch < 1) return false;
  const int64_t blocks = (rows + kvq::kRowsPerWorkgroup - 1) / kvq::kRowsPerWorkgroup;
  // (a grid and its merge have fewer than 2^32 threads)
  if (batch * d->num_kv_heads * blocks > 1 << 19) return false;
  const double pairs = (double)(batch * d->num_kv_heads) * (double)((rows + 15) / 16);
  const double streaming = 8.3 + 2.2 * pairs * (double)groups / (double)(2 * slots);
  double us, cut_us;
  equal_pieces(slots, batch * d->num_kv_heads * blocks, groups, kvq::kMaxContextSplits, false, &us);
  equal_pieces(slots, batch * d->num_kv_heads * blocks, groups, room, false, &cut_us);
  return 1.35 * us <= 0.9 * streaming && 1.35 * cut_us <= 0.95 * streaming;
}

// Microseconds that a 64-token group takes a wavefront of the streaming kernel where all compute units have theirs
// (bound by memory, for int4 and two row tiles by arithmetic).
double crowded_us(const kvq_cache_desc_t* d, int row_tiles) {
  const bool small = d->head_dim == 64, bf16 = d->mode == KVQ_BF16_PLAIN;
  if (row_tiles == 2 && !bf16) return 2.65;
  if (d->mode == KVQ_INT4_TOKEN_HEAD) return 2.9;
  if (d->mode == KVQ_INT4_GROUP32) return 3.2;
  return small ? 2.65 : bf16 ? 4.6 : 5.0;
}

// Wavefronts of the workgroup that each (sequence, kv head, row group) pair gets in a call that does without the flat
// list and the reduce, or 0.  The wavefronts of a pair take its groups in turn and put their sums together in LDS, so
// a second launch and a round trip of partials through memory fall away; what it costs is that a compute unit's share
// is whole pairs, however few there are and however long.  All in units of microseconds and 64-token groups, fitted
// to measurements with 1 to 60 sequences of 40 to 8000 tokens, 8 kv heads, equal lengths, when a wavefront had a
// slice of adjacent groups and began behind the sequence's length (the chain is up to 1 us shorter now, the lines are
// where they were): a group takes a wavefront `alone` where few compute units have one and `crowded` where all have;
// beside that a workgroup per pair takes 3.7 and the flat list with its reduce 8.3.  us a call, flat list ->
// workgroup per pair: 4 query heads per kv head, int8, 1 x 600 tokens 8.6 -> 6.8, 12 x 1500 17.3 -> 12.8, 32 x 600
// 16.1 -> 9.3, 32 of 300 to 2500 23.6 -> 20.8; 32 query rows, 31 x 600 26.6 -> 12.3; not taken: 12 x 4000 24.2 ->
// 27.4, 1 x 2500 9.9 -> 13.6.  With more pairs than compute units a workgroup has half of the wavefronts, and two
// share one.
// A long context among short ones keeps its own workgroup for as many `rounds` as a wavefront has groups, where
// the flat list would spread it over the chip; so its walk may not take longer than the reduce and the partials
// are worth, which is more the more rows they have (a wavefront's accumulators hold 16 rows, or 32, whose halves it
// works on one after the other).  Of 16335 random calls with four to eight rounds, mixtures of long and short among
// them, measured with slices: 15281 inside these lines, 0.57 of the flat list's time on average, 15 above 1.03 of it
// and none above 1.08; 1054 beyond them, 86 above 1.03, up to 1.35 (e4m3, one row, 63 sequences of 40 to 1819
// tokens, 16.5 -> 22.2 us).  500 random calls of up to 2500 tokens with the present kernels: 0.65, 1.01 at most.
int32_t pair_waves(const kvq_cache_desc_t* d, int64_t pairs, int64_t rows, int64_t groups, int row_tiles,
                   int64_t waves) {
  const int per_simd = kvq::waves_per_simd(d->mode, d->head_dim, row_tiles);
  const int64_t cus = waves / 8;
  if (pairs < 1 || pairs > 2 * cus || groups < 1) return 0;
  const int64_t team = pairs <= cus ? 4 * per_simd : 2 * per_simd, slots = pairs <= cus ? cus : 2 * cus;
  const int64_t rounds = (groups + team - 1) / team;
  const bool small = d->head_dim == 64, bf16 = d->mode == KVQ_BF16_PLAIN;
  const double crowded = crowded_us(d, row_tiles);
  double alone = small ? 1.4 : 2.1;
  if (d->mode == KVQ_INT4_GROUP32) alone = 2.9;
  if (row_tiles == 2 && !bf16) alone = small ? 1.9 : 2.1;
  const double longest = (double)rounds * (bf16 && !small ? 2.7 : alone);
  if (rounds > 8 || longest > (rows == 1 ? 8.8 : rows < 4 ? 10.5 : rows <= 8 ? 13.5 : rows <= 16 ? 17.0 : 15.0)) return 0;
  const double here = 3.7 + (double)rounds * (alone + (crowded - alone) * (double)pairs / (double)slots);
  const double flat = 8.3 + crowded * (double)(pairs * groups) / (double)(4 * cus * per_simd);
  return here <= flat ? (int32_t)team : 0;
}

// Whether the prefix kernel is worth its launch for the plan's shared groups, and in how many pieces
// (plan->prefix_chunks at most, for which the workspace has room).  In microseconds: what the streaming kernel is
// spared, (batch - 1) times the shared groups of every pair, against a round of the many-row kernel's workgroups (3
// and 2.6 a group, see equal_pieces; 1.5 at head_dim 64, bf16 3.2), the partials of all stacked rows that it writes and
// the reduce reads (2.1 MB a microsecond) and 2 of launch.  Cost (+) or gain, predicted and measured, 8 kv heads, int8:
// 64 sequences of 2 k to 16 k tokens, 32 rows, prefix 1024 +9 and +9 of 234 us, of 8 k to 16 k with 4096 -23 and -27
// of 294; 128 of 2 k to 4 k, 8 rows, 1024 -15 and -16 of 143; 16 of them, 32 rows +8 and +11 of 35; 9 of 2 k to
// 6 k, head_dim 64, +6 and +6 of 26.
// A tenth and 5 us in doubt are the plain call's: the estimate errs towards the prefix kernel by as much where the
// call is short (int8, 37 sequences of 4 k tokens, prefix 3584, 0.3 gained by it and 6 lost of 35).  Of a
// call of 300 us and more by the bound half a percent is enough: 128 sequences of 2 k to 16 k tokens, 32 rows, prefix
// 1024, 5 by it, e4m3 445 -> 440 us, int8 462 -> 460; 10 random calls that this adds 0.95 to 1.01, 0.98 on average,
// where 19 of 140 to 300 us take 0.93 to 1.11, 1.01.  (Not int4, whose groups are cheaper than crowded_us says:
// 367 -> 372.)  600 random hinted calls took 1.15 of the plain call's time on average and up to 2.16 of it where every
// hint was followed; now 0.95, 1.15 at most.
// A call that is a many-row kernel's without a hint keeps it only where that kernel would take clearly longer than
// the prefix and the rest together: by 6 us and 15 %, with codes 40 % (whose kernel is faster than equal_pieces says
// in the short contexts where it takes so few rows).  bf16, 32 sequences of 8192 tokens, 40 rows: 203 us, 177 with
// 6144 shared; 91 of 4000, 48 rows, 4 kv heads, 154 and 120 with 3840; but 29 of 2000 to 3300, 64 rows, 71 and 99
// with 2048, 35 of 1600, 56 rows, 36 and 45 with 1536; e4m3, 132 of 1100, 44 rows, 102 and 116 with 832.  160
// random such calls: 0.91 of their time without a hint on average, 1.06 at most, and 0.77 of where every hint was
// followed, 1.10 at most.
bool prefix_pays(const kvq_cache_desc_t* d, int64_t batch, int64_t rows, int64_t max_groups, int64_t slots,
                 int64_t room, bool many, kvq::AttnPlan* plan) {
  const int64_t groups = plan->shared_groups, stacked = batch * rows;
  const int64_t walks = d->num_kv_heads * ((stacked + kvq::kRowsPerWorkgroup - 1) / kvq::kRowsPerWorkgroup);
  const double partials = (double)stacked * d->num_kv_heads * d->head_dim * 4.0 / 2.1e6;
  const double piece_us = d->mode == KVQ_BF16_PLAIN ? 3.2 : d->head_dim == 64 ? 1.5 : 2.6;
  double least = 0.0;
  for (int64_t c = 1, most = plan->prefix_chunks; c <= most; ++c) {
    const int64_t n = walks * c, rest = n % slots;
    const double rounds = (double)(n / slots) + (rest == 0 ? 0.0 : 2 * rest <= slots ? 0.6 : 1.0);
    const double us = rounds * (3.0 + piece_us * (double)((groups + c - 1) / c)) + (double)c * partials + 2.0;
    if (c == 1 || us < least) {
      least = us;
      plan->prefix_chunks = (int32_t)c;
    }
  }
  const int per_simd = kvq::waves_per_simd(d->mode, d->head_dim, plan->row_tiles);
  const double group_us = crowded_us(d, plan->row_tiles) / (double)(2 * slots * per_simd);
  const double list = (double)batch * (double)plan->pairs_per_seq * group_us;  // (for one group of every context)
  if (many) {
    if (d->head_dim != 128) return false;
    double alone;
    equal_pieces(slots, batch * d->num_kv_heads, max_groups, room, false, &alone);
    return least + 8.3 + list * (double)(max_groups - groups) + 6.0 <
           (d->mode == KVQ_BF16_PLAIN ? 0.85 : 0.6) * alone;
  }
  const double whole = list * (double)max_groups;
  const double doubt = whole >= 300.0 && d->mode != KVQ_INT4_TOKEN_HEAD ? 0.005 * whole : 0.1 * least + 5.0;
  return list * (double)groups * (double)(batch - 1) / (double)batch >= least + doubt;
}

// Everything the launch needs that depends only on host-side arguments.
bool make_plan(const kvq_cache_desc_t* d, int32_t batch, int32_t q_len, int32_t num_q_heads,
               int32_t max_seq_len, int32_t chunk_tokens, int32_t shared_prefix_tokens,
               kvq::AttnPlan* plan, int* err) {
  if (!desc_ok(d, err)) return false;
  if (batch < 0 || q_len < 1 || q_len > KVQ_MAX_Q_LEN || num_q_heads <= 0 ||
      num_q_heads % d->num_kv_heads != 0 || max_seq_len < 0 || chunk_tokens < 0 ||
      chunk_tokens % 64 != 0 || shared_prefix_tokens < 0) {
    *err = KVQ_E_BAD_SHAPE;
    return false;
  }
  const int group = num_q_heads / d->num_kv_heads;
  // (every product below is taken in a type that holds it: the arguments are only known to be
  // non-negative 32-bit numbers at this point)
  const int64_t rows = (int64_t)group * q_len;
  // (the group-scaled int4 kernels hold one accumulator per channel group: one row tile)
  const int64_t row_tiles = rows <= 16 || d->mode == KVQ_INT4_GROUP32 ? 1 : 2;
  const int64_t row_groups = (rows + 16 * row_tiles - 1) / (16 * row_tiles);
  const int64_t pairs = (int64_t)d->num_kv_heads * row_groups;
  // the flat list of 64-token groups can be no longer than this
  const unsigned __int128 flat_wide =
      (unsigned __int128)batch * (uint64_t)(((int64_t)max_seq_len + 63) / 64) * (uint64_t)pairs;
  if (rows > 0x7FFFFFFF || pairs > 0x7FFFFFFF || flat_wide > 0x7FFFFFFF) {
    *err = KVQ_E_BAD_SHAPE;
    return false;
  }
  const int64_t flat_max = (int64_t)flat_wide;
  const int64_t waves = auto_waves(), slots_128 = waves / 4;  // (workgroups of the many-row kernel)
  plan->rows = (int32_t)rows;
  plan->row_tiles = (int32_t)row_tiles;
  plan->num_row_groups = (int32_t)row_groups;
  plan->pairs_per_seq = (int32_t)pairs;
  if (chunk_tokens == 0) {
    // even split over as many wavefronts as an MI355X keeps resident at this kernel's
    // register footprint: 256 CUs x 4 SIMDs x 2 (one 16-row tile, or two at head_dim 64) or
    // x 1 (two tiles at head_dim 128)
    // (an unquantized cache needs twice the registers per group: one wavefront per SIMD; so
    // does the group-scaled int4 cache, for its four accumulators per logit, in the workspace; see
    // below for its launch)
    const bool two_per_simd = kvq::waves_per_simd(d->mode, d->head_dim, plan->row_tiles) == 2 &&
                              d->mode != KVQ_INT4_GROUP32;
    const int64_t resident = two_per_simd ? waves : waves / 2;
    plan->range_groups = 0;
    plan->num_waves = (int32_t)(flat_max < resident ? flat_max : resident);
  } else {
    plan->range_groups = chunk_tokens / 64;
    plan->num_waves = (int32_t)((flat_max + plan->range_groups - 1) / plan->range_groups);
  }
  if (plan->num_waves < 1) plan->num_waves = 1;
  // A shared prefix goes to the many-row kernel with all sequences' rows stacked, where that
  // kernel exists for the format, the call is not already its own (128 rows and more per kv
  // head), there is a second sequence to share with and the prefix fits the declared lengths.
  // It is cut into pieces so that about two workgroups per compute unit come about.
  plan->shared_groups = 0;
  plan->prefix_chunks = 1;
  const int64_t stacked = (int64_t)batch * rows;
  if (shared_prefix_tokens >= 64 && shared_prefix_tokens <= max_seq_len && batch >= 2 &&
      rows < 128 && d->mode != KVQ_INT4_GROUP32 && stacked <= (1 << 30)) {
    plan->shared_groups = shared_prefix_tokens / 64;
    const int64_t walks = d->num_kv_heads * ((stacked + 127) / 128);
    int64_t chunks = (slots_128 + walks - 1) / walks;
    if (chunks > kvq::kMaxPrefixChunks) chunks = kvq::kMaxPrefixChunks;
    if (chunks > plan->shared_groups) chunks = plan->shared_groups;
    plan->prefix_chunks = (int32_t)chunks;
  }
  // one partial per (wavefront range, pair) crossing, numbered wave + pair index; behind them
  // one per (piece of the shared prefix, pair)
  const size_t slots =
      (size_t)plan->num_waves +
      (size_t)batch * plan->pairs_per_seq * (plan->shared_groups > 0 ? 1 + plan->prefix_chunks : 1);
  const size_t slot_rows = slots * 16 * plan->row_tiles;
  plan->slot_rows = (int32_t)(16 * plan->row_tiles);
  plan->acc_floats = slot_rows * d->head_dim;
  plan->ml_floats = slot_rows * 2;
  plan->prefix_ints = ((size_t)batch + 2 + 3) & ~(size_t)3;  // prefix sums, prefix length
  // pieces of a context that a many-row kernel has room for in the workspace of a call without a hint
  const int64_t room = batch == 0 ? 1
                                  : (plan->num_waves + batch * pairs) * 16 * row_tiles /
                                            ((int64_t)q_len * num_q_heads) / batch + 1;
  // The group-scaled int4 kernel runs two wavefronts per SIMD as well.  Its workspace is that of one, so
  // twice the wavefronts have room for their partials where a slot needs only eight rows; with
  // more the call keeps to one.  So do lists of less than four groups for each of the 2048, where a
  // wavefront has little to stream and leaves as many partials (one against two wavefronts per SIMD, 8
  // rows of 8 kv heads, 1600 tokens: 21 sequences 20.2 and 22.9 us, 40 27.4 and 27.3, 100 54.5 and 47.9).
  if (d->mode == KVQ_INT4_GROUP32 && chunk_tokens == 0 && rows <= 8 && flat_max >= 4 * waves) {
    plan->slot_rows = 8;
    plan->num_waves = (int32_t)waves;
  }
  plan->few_waves = plan->num_waves <= waves / 2;
  // A many-row call has the same workspace as if it went through the streaming kernel; the pieces
  // of a cut context beyond the first (whose rows go to `out`) use it, a sequence's rows each.
  plan->extra_pieces = plan->wide_extra = 0;
  plan->piece_min = 1;
  plan->piece_share = 0.0f;
  plan->many_rows = batch > 0 && many_rows(d, batch, rows, max_seq_len, chunk_tokens, slots_128);
  // What follows a shared prefix is the streaming kernel's, so such a call does without the prefix where
  // that costs more than the stacked rows save: with more than 64 rows they are little denser than the
  // many-row kernel's own; up to 64 a prefix of half the context is worth it.  (The workspace keeps
  // its size.)  32 sequences of 8192 tokens, 64 / 8 heads, hints of 64, 4096 and 6144 tokens, us with the
  // prefix kernel and without: 96 rows int8 300, 262, 234 and 184, 166, 164; bf16 520, 385, 309 and 214,
  // 192, 184; 40 rows bf16 342, 240, 177 and 203, 188 (at 2048), 203.
  plan->promised_groups = plan->shared_groups;
  if (plan->many_rows && (rows > 64 || 2 * (int64_t)plan->shared_groups < ((int64_t)max_seq_len + 63) / 64))
    plan->shared_groups = 0;
  // (a caller's split-K granule keeps the prefix in as many pieces as there is room for)
  plan->prefix_pays = plan->shared_groups > 0 &&
                      (chunk_tokens > 0 || prefix_pays(d, batch, rows, ((int64_t)max_seq_len + 63) / 64, slots_128,
                                                       room, plan->many_rows, plan));
  if (plan->shared_groups > 0) plan->many_rows = 0;
  // (A call whose pairs get a workgroup each needs no prefix kernel either, and the same whether it has a
  // hint or not.)
  plan->pair_waves = plan->many_rows || chunk_tokens > 0
                         ? 0 : pair_waves(d, batch * pairs, rows, ((int64_t)max_seq_len + 63) / 64, plan->row_tiles, waves);
  plan->group_rows = chunk_tokens == 0 && plan->pair_waves == 0 &&
                     group_rows(d, batch, rows, ((int64_t)max_seq_len + 63) / 64, slots_128, room);
  if (plan->pair_waves > 0) plan->shared_groups = 0;
  plan->wide_groups = plan->wide_least = 0;
  if (plan->many_rows || plan->group_rows)
    cut_contexts(d, batch, q_len, rows, (int64_t)q_len * num_q_heads, ((int64_t)max_seq_len + 63) / 64,
                 (int64_t)slot_rows, slots_128, plan);
  return true;
}

size_t workspace_bytes(const kvq::AttnPlan& plan) {
  return (plan.acc_floats + plan.ml_floats + plan.prefix_ints) * sizeof(float);
}

// The plan that a call launches, and the workspace it asks for.  A prefix that is not worth its kernel leaves the call
// paged_decode_attn's, in a workspace of the hint's size; the promise stays, for the checks.
bool call_plan(const kvq_cache_desc_t* d, int32_t batch, int32_t q_len, int32_t num_q_heads, int32_t max_seq_len,
               int32_t chunk_tokens, int32_t shared_prefix_tokens, kvq::AttnPlan* plan, size_t* need, int* err) {
  if (!make_plan(d, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, shared_prefix_tokens, plan, err))
    return false;
  *need = workspace_bytes(*plan);
  if (plan->shared_groups == 0 || plan->prefix_pays) return true;
  const int32_t promised = plan->promised_groups;
  if (!make_plan(d, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, 0, plan, err)) return false;
  plan->promised_groups = promised;
  return true;
}

}  // namespace

extern "C" {

size_t kvq_cache_bytes(const kvq_cache_desc_t* desc) {
  int err;
  if (!desc_ok(desc, &err)) return 0;
  return (size_t)desc->num_blocks * 2 * desc->num_kv_heads * desc->block_size *
         kvq::row_bytes(desc->mode, desc->head_dim);
}

size_t kvq_scales_bytes(const kvq_cache_desc_t* desc) {
  int err;
  if (!desc_ok(desc, &err) || desc->mode == KVQ_BF16_PLAIN) return 0;
  if (desc->mode == KVQ_FP8E4M3_TENSOR) return 2 * sizeof(float);
  return (size_t)desc->num_blocks * sizeof(float) *
         kvq::block_scale_floats(desc->mode, desc->num_kv_heads, desc->block_size, desc->head_dim);
}

int kv_quant_write(const void* k, const void* v, const int64_t* slot_mapping,
                   int32_t num_tokens, void* cache, float* scales,
                   const kvq_cache_desc_t* desc, void* stream) {
  int err;
  if (!desc_ok(desc, &err)) return err;
  // one wavefront per (token, kv head, K|V) at most, four to a workgroup: the grid must fit
  if (num_tokens < 0 || (int64_t)num_tokens * desc->num_kv_heads * 2 / 4 > 0x7FFFFFFF)
    return KVQ_E_BAD_SHAPE;
  if (num_tokens == 0) return KVQ_OK;
  if (!k || !v || !slot_mapping || !cache) return KVQ_E_NULLPTR;
  if (!scales && desc->mode != KVQ_BF16_PLAIN) return KVQ_E_NULLPTR;
  if ((((uintptr_t)k | (uintptr_t)v | (uintptr_t)cache) & 15) != 0) return KVQ_E_BAD_SHAPE;
  if (debug_checks()) {
    const int rc = debug_check_slots(slot_mapping, num_tokens,
                                     (int64_t)desc->num_blocks * desc->block_size,
                                     (hipStream_t)stream);
    if (rc != KVQ_OK) return rc;
  }
  const hipError_t e = kvq::launch_write(k, v, slot_mapping, num_tokens, cache, scales, *desc,
                                         (hipStream_t)stream);
  return e == hipSuccess ? KVQ_OK : KVQ_E_HIP;
}

size_t paged_decode_attn_workspace_bytes(const kvq_cache_desc_t* desc, int32_t batch,
                                         int32_t q_len, int32_t num_q_heads,
                                         int32_t max_seq_len, int32_t chunk_tokens) {
  kvq::AttnPlan plan;
  int err;
  if (!make_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, 0, &plan, &err))
    return 0;
  return workspace_bytes(plan);
}

size_t paged_decode_attn_prefix_workspace_bytes(const kvq_cache_desc_t* desc, int32_t batch,
                                                int32_t q_len, int32_t num_q_heads,
                                                int32_t max_seq_len, int32_t chunk_tokens,
                                                int32_t shared_prefix_tokens) {
  kvq::AttnPlan plan;
  int err;
  if (!make_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, shared_prefix_tokens,
                 &plan, &err))
    return 0;
  return workspace_bytes(plan);
}

}  // extern "C"

// The scratch buffer of paged_decode_attn_static: device memory of the library's own, so that
// the call needs no workspace from a caller who cannot allocate one.  In host code this name is
// only a handle for hipGetSymbolAddress; the address kernels may use is looked up once per
// device (each device has its own copy at its own address).
static __device__ __align__(256) unsigned char scratch[KVQ_STATIC_WORKSPACE_BYTES];

namespace {

void* g_scratch_ptr[kMaxDevices] = {};  // per device, filled on the first call made there

// Device address of `scratch` on the current device (nullptr if the lookup fails).
void* scratch_on_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_device_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

// ---- KVQ_DEBUG=1 in the environment: the indices the kernels would follow blindly are checked
// on the device first.  A checking kernel runs ahead of the real one, the call waits for it
// (so a debug call synchronises with its stream and must not be made under graph capture), and
// an index out of range becomes KVQ_E_BAD_INDEX instead of a memory fault: nothing is trapped
// and the real kernel is not launched. ----
bool debug_checks() {
  const char* e = getenv("KVQ_DEBUG");
  return e && e[0] != '\0' && !(e[0] == '0' && e[1] == '\0');
}

__global__ void check_slots_kernel(const int64_t* __restrict__ slot_mapping, int32_t num_tokens,
                                   int64_t num_slots, int* __restrict__ word) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= num_tokens) return;
  if (slot_mapping[t] >= num_slots) {  // (negative = skip the token)
    atomicOr(&word[0], 1);
    atomicMin(&word[1], (int)t);
  }
}

// entry (b, j): sequence lengths inside [q_len, max_seq_len]; the table entries of every block
// below ceil(seq_lens[b] / block_size) inside [0, num_blocks); the first shared_blocks entries
// equal to sequence 0's (where both sequences are long enough for the prefix to be used)
__global__ void check_tables_kernel(const int32_t* __restrict__ block_tables,
                                    const int32_t* __restrict__ seq_lens, int32_t batch,
                                    int32_t max_blocks_per_seq, int32_t num_blocks,
                                    int32_t block_size, int32_t q_len, int32_t max_seq_len,
                                    int32_t shared_blocks, int32_t shared_tokens,
                                    int* __restrict__ word) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)batch * max_blocks_per_seq) return;
  const int b = (int)(i / max_blocks_per_seq), j = (int)(i - (int64_t)b * max_blocks_per_seq);
  const int L = seq_lens[b];
  if (L < q_len || L > max_seq_len) {
    if (j == 0) {
      atomicOr(&word[0], 2);
      atomicMin(&word[1], b);
    }
    return;
  }
  if (j >= (L + block_size - 1) / block_size) return;
  const int e = block_tables[i];
  if (e < 0 || e >= num_blocks) {
    atomicOr(&word[0], 4);
    atomicMin(&word[1], b);
  }
  if (j < shared_blocks && L >= shared_tokens && seq_lens[0] >= shared_tokens &&
      e != block_tables[j]) {
    atomicOr(&word[0], 8);
    atomicMin(&word[1], b);
  }
}

}  // namespace

static __device__ int debug_word[2];  // [0] what was found (bit set), [1] first token / sequence

namespace {

// Runs `launch_check(word)` on the stream and waits for its verdict.
template <class F>
int debug_verdict(hipStream_t stream, F launch_check) {
  int* word = nullptr;
  if (hipGetSymbolAddress((void**)&word, HIP_SYMBOL(debug_word)) != hipSuccess) return KVQ_E_HIP;
  const int init[2] = {0, 0x7FFFFFFF};
  int found[2] = {0, 0};
  if (hipMemcpyAsync(word, init, sizeof(init), hipMemcpyHostToDevice, stream) != hipSuccess)
    return KVQ_E_HIP;
  launch_check(word);
  if (hipGetLastError() != hipSuccess) return KVQ_E_HIP;
  if (hipMemcpyAsync(found, word, sizeof(found), hipMemcpyDeviceToHost, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)
    return KVQ_E_HIP;
  return found[0] ? KVQ_E_BAD_INDEX : KVQ_OK;
}

int debug_check_slots(const int64_t* slot_mapping, int32_t num_tokens, int64_t num_slots,
                      hipStream_t stream) {
  return debug_verdict(stream, [&](int* word) {
    hipLaunchKernelGGL(check_slots_kernel, dim3((unsigned)((num_tokens + 255) / 256)), dim3(256), 0,
                       stream, slot_mapping, num_tokens, num_slots, word);
  });
}

// Validation and launch shared by paged_decode_attn and paged_decode_attn_static.  With
// own_scratch the workspace is the library's static buffer, looked up only after every other
// check has passed (so that bad arguments are rejected without any HIP call).
int attn_call(const void* q, const void* cache, const float* scales,
              const kvq_cache_desc_t* desc, const int32_t* block_tables,
              int32_t max_blocks_per_seq, const int32_t* seq_lens, int32_t batch, int32_t q_len,
              int32_t num_q_heads, int32_t max_seq_len, float sm_scale, int32_t chunk_tokens,
              int32_t shared_prefix_tokens, float* out, void* workspace, size_t workspace_bytes,
              bool own_scratch, void* stream) {
  kvq::AttnPlan plan;
  size_t need;
  int err;
  if (!call_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, shared_prefix_tokens,
                 &plan, &need, &err))
    return err;
  if (max_blocks_per_seq < 0 ||
      (int64_t)max_blocks_per_seq * desc->block_size < (int64_t)max_seq_len)
    return KVQ_E_BAD_SHAPE;
  if (batch == 0) return KVQ_OK;
  if (max_seq_len < q_len) return KVQ_E_BAD_SHAPE;
  if (!q || !cache || !block_tables || !seq_lens || !out) return KVQ_E_NULLPTR;
  if (!scales && desc->mode != KVQ_BF16_PLAIN) return KVQ_E_NULLPTR;
  // the kernels read q and the cache and write out in 16-byte pieces
  if ((((uintptr_t)q | (uintptr_t)cache | (uintptr_t)out) & 15) != 0) return KVQ_E_BAD_SHAPE;
  if (own_scratch) {
    if (need > (size_t)KVQ_STATIC_WORKSPACE_BYTES) return KVQ_E_WORKSPACE;
    workspace = scratch_on_current_device();
    if (!workspace) return KVQ_E_HIP;
  } else if (need > 0) {
    if (!workspace) return KVQ_E_NULLPTR;
    if (workspace_bytes < need) return KVQ_E_WORKSPACE;
    if (((uintptr_t)workspace & 15) != 0) return KVQ_E_BAD_SHAPE;
  }

  if (debug_checks()) {
    const int64_t entries = (int64_t)batch * max_blocks_per_seq;
    if (entries > 0) {
      const int rc = debug_verdict((hipStream_t)stream, [&](int* word) {
        hipLaunchKernelGGL(check_tables_kernel, dim3((unsigned)((entries + 255) / 256)), dim3(256),
                           0, (hipStream_t)stream, block_tables, seq_lens, batch,
                           max_blocks_per_seq, desc->num_blocks, desc->block_size, q_len,
                           max_seq_len,
                           (plan.promised_groups * 64 + desc->block_size - 1) / desc->block_size,
                           plan.promised_groups * 64, word);
      });
      if (rc != KVQ_OK) return rc;
    }
  }

  kvq::AttnArgs a;
  a.q = (const uint16_t*)q;
  a.cache = (const uint8_t*)cache;
  a.scales = scales;
  a.block_tables = block_tables;
  a.seq_lens = seq_lens;
  a.out = out;
  a.ws_acc = (float*)workspace;
  a.ws_ml = (float*)workspace + plan.acc_floats;
  a.ws_prefix = (int32_t*)((float*)workspace + plan.acc_floats + plan.ml_floats);
  a.max_blocks_per_seq = max_blocks_per_seq;
  a.batch = batch;
  a.q_len = q_len;
  a.num_q_heads = num_q_heads;
  a.num_kv_heads = desc->num_kv_heads;
  a.group = num_q_heads / desc->num_kv_heads;
  a.rows = plan.rows;
  a.block_size = desc->block_size;
  a.bs_shift = ilog2(desc->block_size);
  a.head_dim = desc->head_dim;
  a.mode = desc->mode;
  a.row_tiles = plan.row_tiles;
  a.slot_rows = plan.slot_rows;
  a.num_row_groups = plan.num_row_groups;
  a.pairs_per_seq = plan.pairs_per_seq;
  a.range_groups = plan.range_groups;
  a.num_waves = plan.num_waves;
  a.few_waves = plan.few_waves;
  a.scale_log2 = sm_scale * 1.4426950408889634f;
  a.wave_clock = nullptr;
  a.shared_groups = plan.shared_groups;
  a.prefix_chunks = plan.prefix_chunks;
  a.pair_waves = plan.pair_waves;
  a.many_rows = plan.many_rows | plan.group_rows;
  a.wide_groups = plan.wide_groups;
  a.wide_least = plan.wide_least;
  a.extra_pieces = plan.extra_pieces;
  a.wide_extra = plan.wide_extra;
  a.merge = plan.extra_pieces > 0 || plan.wide_extra > 0;
  a.piece_min = plan.piece_min;
  a.piece_share = plan.piece_share;
  const hipError_t e = kvq::launch_attn(a, (hipStream_t)stream);
  return e == hipSuccess ? KVQ_OK : KVQ_E_HIP;
}

}  // namespace

extern "C" {

int paged_decode_attn(const void* q, const void* cache, const float* scales,
                      const kvq_cache_desc_t* desc, const int32_t* block_tables,
                      int32_t max_blocks_per_seq, const int32_t* seq_lens, int32_t batch,
                      int32_t q_len, int32_t num_q_heads, int32_t max_seq_len, float sm_scale,
                      int32_t chunk_tokens, float* out, void* workspace,
                      size_t workspace_bytes, void* stream) {
  return attn_call(q, cache, scales, desc, block_tables, max_blocks_per_seq, seq_lens, batch,
                   q_len, num_q_heads, max_seq_len, sm_scale, chunk_tokens, 0, out, workspace,
                   workspace_bytes, false, stream);
}

int paged_decode_attn_prefix(const void* q, const void* cache, const float* scales,
                             const kvq_cache_desc_t* desc, const int32_t* block_tables,
                             int32_t max_blocks_per_seq, const int32_t* seq_lens, int32_t batch,
                             int32_t q_len, int32_t num_q_heads, int32_t max_seq_len,
                             float sm_scale, int32_t chunk_tokens, int32_t shared_prefix_tokens,
                             float* out, void* workspace, size_t workspace_bytes, void* stream) {
  return attn_call(q, cache, scales, desc, block_tables, max_blocks_per_seq, seq_lens, batch,
                   q_len, num_q_heads, max_seq_len, sm_scale, chunk_tokens, shared_prefix_tokens,
                   out, workspace, workspace_bytes, false, stream);
}

int paged_decode_attn_static(const void* q, const void* cache, const float* scales,
                             const kvq_cache_desc_t* desc, const int32_t* block_tables,
                             int32_t max_blocks_per_seq, const int32_t* seq_lens, int32_t batch,
                             int32_t q_len, int32_t num_q_heads, int32_t max_seq_len,
                             float sm_scale, int32_t chunk_tokens, float* out, void* stream) {
  return attn_call(q, cache, scales, desc, block_tables, max_blocks_per_seq, seq_lens, batch,
                   q_len, num_q_heads, max_seq_len, sm_scale, chunk_tokens, 0, out, nullptr, 0,
                   true, stream);
}

int kvq_cache_to_canonical(const void* cache, void* canonical, const kvq_cache_desc_t* desc,
                           void* stream) {
  int err;
  if (!desc_ok(desc, &err)) return err;
  if (kvq_cache_bytes(desc) == 0) return KVQ_OK;
  if (!cache || !canonical) return KVQ_E_NULLPTR;
  return kvq::launch_repack(cache, canonical, *desc, true, (hipStream_t)stream) == hipSuccess
             ? KVQ_OK
             : KVQ_E_HIP;
}

int kvq_cache_from_canonical(const void* canonical, void* cache, const kvq_cache_desc_t* desc,
                             void* stream) {
  int err;
  if (!desc_ok(desc, &err)) return err;
  if (kvq_cache_bytes(desc) == 0) return KVQ_OK;
  if (!cache || !canonical) return KVQ_E_NULLPTR;
  return kvq::launch_repack(canonical, cache, *desc, false, (hipStream_t)stream) == hipSuccess
             ? KVQ_OK
             : KVQ_E_HIP;
}

static int block_copy(const void* pool_cache, const float* pool_scales,
                      const kvq_cache_desc_t* desc, const int32_t* block_ids, int32_t num,
                      void* packed_cache, float* packed_scales, bool to_packed, void* stream) {
  int err;
  if (!desc_ok(desc, &err)) return err;
  // one workgroup per 4 KiB piece of a block; 32-bit byte offsets inside a block
  const int64_t block_bytes = (int64_t)2 * desc->num_kv_heads * desc->block_size *
                              kvq::row_bytes(desc->mode, desc->head_dim);
  if (num < 0 || block_bytes > 0x7FFFFFFF || (int64_t)num * ((block_bytes + 4095) / 4096) > 0x7FFFFFFF)
    return KVQ_E_BAD_SHAPE;
  if (num == 0) return KVQ_OK;
  if (!pool_cache || !block_ids || !packed_cache) return KVQ_E_NULLPTR;
  const bool block_scales = kvq::block_scale_floats(desc->mode, desc->num_kv_heads,
                                                    desc->block_size, desc->head_dim) != 0;
  if (block_scales && (!pool_scales || !packed_scales)) return KVQ_E_NULLPTR;
  if ((((uintptr_t)pool_cache | (uintptr_t)packed_cache) & 15) != 0) return KVQ_E_BAD_SHAPE;
  const hipError_t e = kvq::launch_block_copy(pool_cache, pool_scales, *desc, block_ids, num,
                                              packed_cache, packed_scales, to_packed,
                                              (hipStream_t)stream);
  return e == hipSuccess ? KVQ_OK : KVQ_E_HIP;
}

int kvq_blocks_export(const void* cache, const float* scales, const kvq_cache_desc_t* desc,
                      const int32_t* block_ids, int32_t num, void* packed_cache,
                      float* packed_scales, void* stream) {
  return block_copy(cache, scales, desc, block_ids, num, packed_cache, packed_scales, true, stream);
}

int kvq_blocks_import(const void* packed_cache, const float* packed_scales,
                      const kvq_cache_desc_t* desc, const int32_t* block_ids, int32_t num,
                      void* cache, float* scales, void* stream) {
  return block_copy(cache, scales, desc, block_ids, num, (void*)packed_cache,
                    (float*)packed_scales, false, stream);
}

#ifdef KVQ_PROFILE  // exported by the measurement build only (include/kvq_prof.h)
int kvq_profile_plan(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                     int32_t max_seq_len, int32_t chunk_tokens, int32_t shared_prefix_tokens,
                     int64_t plan_out[8]) {
  kvq::AttnPlan p;
  size_t need;
  int err;
  if (!call_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, shared_prefix_tokens, &p, &need, &err))
    return err;
  if (batch == 0) return KVQ_E_BAD_SHAPE;
  const kvq::ReduceLaunch r =
      kvq::reduce_launch(batch, p.pairs_per_seq, p.num_waves, p.rows, p.row_tiles, desc->head_dim);
  const int64_t values[8] = {p.many_rows + (p.wide_groups > 0), p.extra_pieces, p.num_waves, p.shared_groups,
                             16 * p.row_tiles, r.pairs, r.parts, r.threads};
  for (int i = 0; i < 8; ++i) plan_out[i] = values[i];
  return KVQ_OK;
}

int kvq_profile_wide(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                     int32_t max_seq_len, int64_t wide_out[3]) {
  kvq::AttnPlan p;
  int err;
  if (!make_plan(desc, batch, q_len, num_q_heads, max_seq_len, 0, 0, &p, &err)) return err;
  wide_out[0] = p.wide_groups;
  wide_out[1] = p.wide_extra;
  wide_out[2] = p.wide_least;
  return KVQ_OK;
}

int kvq_profile_pair_waves(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                           int32_t max_seq_len, int32_t chunk_tokens) {
  kvq::AttnPlan p;
  int err;
  if (!make_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, 0, &p, &err)) return err;
  return p.pair_waves;
}

int kvq_profile_prefix_pieces(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                              int32_t max_seq_len, int32_t chunk_tokens, int32_t shared_prefix_tokens) {
  kvq::AttnPlan p;
  size_t need;
  int err;
  if (!call_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, shared_prefix_tokens, &p, &need, &err))
    return err;
  return p.shared_groups > 0 ? p.prefix_chunks : 0;
}

int kvq_profile_group_rows(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                           int32_t max_seq_len, int32_t chunk_tokens) {
  kvq::AttnPlan p;
  int err;
  if (!make_plan(desc, batch, q_len, num_q_heads, max_seq_len, chunk_tokens, 0, &p, &err)) return err;
  return p.group_rows;
}

void kvq_profile_split_events(void* before, void* after) {
  kvq::set_profile_events((hipEvent_t)before, (hipEvent_t)after);
}

void kvq_profile_read_ceiling(int on) { kvq::set_read_ceiling(on != 0); }

void kvq_profile_skip_reduce(int on) { kvq::set_skip_reduce(on != 0); }
void kvq_profile_prefill_kernel(int on) { kvq::set_prefill_kernel(on != 0); }

void kvq_profile_wave_clock(void* buf) { kvq::set_wave_clock((unsigned long long*)buf); }
#endif

const char* kvq_strerror(int code) {
  switch (code) {
    case KVQ_OK: return "ok";
    case KVQ_E_NULLPTR: return "a required pointer is NULL";
    case KVQ_E_BAD_MODE: return "unknown quantization mode";
    case KVQ_E_BAD_SHAPE: return "unsupported shape or size argument";
    case KVQ_E_WORKSPACE: return "workspace too small";
    case KVQ_E_HIP: return "kernel launch failed";
    case KVQ_E_BAD_INDEX: return "slot, block-table entry or sequence length out of range (KVQ_DEBUG)";
    default: return "unknown error code";
  }
}

}  // extern "C"
