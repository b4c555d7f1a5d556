// Conversions between the library's physical cache (K in 4-token quads, V channel-major per
// 16-token sub-block, int8 codes in offset-binary form) and the canonical
// [block][K|V][head][token][channel] array of plain codes.  Not on the hot
// path: used to hand a cache to, or take one from, code that expects the canonical order.
#include "kvq_internal.h"

namespace kvq {
namespace {

typedef uint32_t uintx4v __attribute__((ext_vector_type(4)));

constexpr uint32_t kHostUnits = 256;        // 4 KiB pieces in flight from or to host memory, where they are bounded:
constexpr uint32_t kHostReadAll = 320;      // in a move from it of more pieces than this
constexpr uint32_t kHostWriteAll = 2048;    // and in one to it

__global__ __launch_bounds__(256) void repack_kernel(const uint8_t* __restrict__ src,
                                                     uint8_t* __restrict__ dst, size_t total,
                                                     int H, int bs, int D, int mode,
                                                     bool to_canonical) {
  const size_t tile_bytes = (size_t)bs * D;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    // i indexes the canonical array
    const size_t tile = i / tile_bytes;
    const int within = (int)(i - tile * tile_bytes);
    const int off = within / D, d = within - off * D;
    const int kv = (int)((tile / H) & 1);
    const size_t phys = tile * tile_bytes + (kv ? v_elem(off, d, bs, D) : k_elem(off, d, bs, D));
    // stored_byte is its own inverse
    if (to_canonical) dst[i] = stored_byte(src[phys], mode);
    else dst[phys] = stored_byte(src[i], mode);
  }
}

// int4 (head_dim 128): canonical byte j of a token = channels 2j (low nibble) and 2j+1 (high),
// 4-bit two's complement; physical nibble = code + 8 in the word / nibble given by
// int4_k_word / int4_v_word / int4_nibble.  One thread per canonical byte when converting to
// the canonical form (it gathers two nibbles), one per physical 32-bit word the other way (it
// gathers eight), so every output location has exactly one writer.
__global__ __launch_bounds__(256) void repack_int4_kernel(const uint8_t* __restrict__ src,
                                                          uint8_t* __restrict__ dst, size_t total,
                                                          int H, int bs, bool to_canonical) {
  constexpr int D = 128;
  const size_t tile_bytes = (size_t)bs * (D / 2);
  if (to_canonical) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
      const size_t tile = i / tile_bytes;
      const int within = (int)(i - tile * tile_bytes);
      const int off = within / (D / 2), j = within - off * (D / 2);
      const int kv = (int)((tile / H) & 1);
      uint32_t byte = 0;
      for (int half = 0; half < 2; ++half) {
        const int d = 2 * j + half;
        const int word = kv ? int4_v_word(off, d) : int4_k_word(off, d);
        const int nib = int4_nibble(kv ? (off & 7) : (d & 7));
        const uint32_t w = *(const uint32_t*)(src + tile * tile_bytes + word);
        const uint32_t code = (((w >> (4 * nib)) & 15u) - 8u) & 15u;
        byte |= code << (4 * half);
      }
      dst[i] = (uint8_t)byte;
    }
  } else {
    const size_t words = total / 4;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (size_t)gridDim.x * blockDim.x) {
      const size_t tile = (i * 4) / tile_bytes;
      const int word = (int)(i * 4 - tile * tile_bytes);
      const int kv = (int)((tile / H) & 1);
      uint32_t w = 0;
      for (int e = 0; e < 8; ++e) {
        int off, d;
        if (kv == 0) {  // invert int4_k_word: the word's token and its 8 channels
          off = (word >> 8) * 4 + ((word >> 4) & 3);
          d = ((word >> 2) & 3) * 32 + ((word >> 6) & 3) * 8 + e;
        } else {        // invert int4_v_word: the word's channel and its 8 tokens
          off = (word >> 10) * 16 + ((word >> 2) & 1) * 8 + e;
          d = ((word >> 8) & 3) * 32 + ((word >> 3) & 1) * 16 + ((word >> 4) & 15);
        }
        const uint32_t byte = src[tile * tile_bytes + (size_t)off * (D / 2) + d / 2];
        const uint32_t code = (d & 1) ? (byte >> 4) : (byte & 15u);
        w |= ((code + 8u) & 15u) << (4 * int4_nibble(e));
      }
      *(uint32_t*)(dst + tile * tile_bytes + word) = w;
    }
  }
}

__global__ __launch_bounds__(256) void repack16_kernel(const uint16_t* __restrict__ src,
                                                       uint16_t* __restrict__ dst, size_t total,
                                                       int H, int bs, int D, bool to_canonical) {
  const size_t tile_elems = (size_t)bs * D;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const size_t tile = i / tile_elems;
    const int within = (int)(i - tile * tile_elems);
    const int off = within / D, d = within - off * D;
    const int kv = (int)((tile / H) & 1);
    const size_t phys = tile * tile_elems + (kv ? v_elem16(off, d, D) : k_elem16(off, d, D));
    if (to_canonical) dst[i] = src[phys];
    else dst[phys] = src[i];
  }
}

// Whole blocks between the pool and a packed staging area.  A unit is one 4 KiB piece of one block's codes (16 bytes
// per lane) and, as far as there are any, 256 of the block's scales (one a lane: no format has more than four bytes
// of scales to 16 of codes), both requested before either is stored.  Non-temporal on both sides: every byte is
// touched once.  (With a block's scales in a loop of its first workgroup, 47 blocks of 128 tokens under group-scaled
// int4, 4096 scales each, took 8.0 us, now 3.6.)
// STRIDED: fewer workgroups than units.
template <bool TO_PACKED, bool STRIDED>
__global__ __launch_bounds__(256) void block_copy_kernel(
    uint8_t* __restrict__ pool_cache, float* __restrict__ pool_scales,
    uint8_t* __restrict__ packed_cache, float* __restrict__ packed_scales,
    const int32_t* __restrict__ block_ids, uint32_t block_bytes, uint32_t scale_floats,
    uint32_t pieces, uint32_t units) {
  uint32_t u = blockIdx.x;
  do {
    const uint32_t i = u / pieces, piece = u - i * pieces;
    const size_t blk = (size_t)block_ids[i];
    const uint32_t at = piece * 4096u + threadIdx.x * 16u, k = piece * 256u + threadIdx.x;
    uintx4v* in_pool = (uintx4v*)(pool_cache + blk * block_bytes + at);
    uintx4v* in_packed = (uintx4v*)(packed_cache + (size_t)i * block_bytes + at);
    float* s_pool = pool_scales + (blk * scale_floats + k);
    float* s_packed = packed_scales + ((size_t)i * scale_floats + k);
    uintx4v x;
    float s;
    if (at < block_bytes) x = __builtin_nontemporal_load(TO_PACKED ? in_pool : in_packed);
    if (k < scale_floats) s = *(TO_PACKED ? s_pool : s_packed);
    if (at < block_bytes) __builtin_nontemporal_store(x, TO_PACKED ? in_packed : in_pool);
    if (k < scale_floats) *(TO_PACKED ? s_packed : s_pool) = s;
    u += gridDim.x;
  } while (STRIDED && u < units);
}

}  // namespace

hipError_t launch_block_copy(const void* pool_cache, const float* pool_scales,
                             const kvq_cache_desc_t& desc, const int32_t* block_ids, int32_t num,
                             void* packed_cache, float* packed_scales, bool to_packed,
                             hipStream_t stream) {
  const uint32_t block_bytes =
      2u * desc.num_kv_heads * desc.block_size * row_bytes(desc.mode, desc.head_dim);
  const uint32_t scale_floats = (uint32_t)block_scale_floats(desc.mode, desc.num_kv_heads,
                                                             desc.block_size, desc.head_dim);
  const uint32_t pieces = (block_bytes + 4095u) / 4096u, units = (uint32_t)num * pieces;
  uint32_t grid = units;
  // Read from host memory, more than about 1 MiB of requests at once slows the link down: 8.65 MB with a workgroup
  // for every unit (2112) 198 us, 1024 workgroups 181, 256 158, 64 with four requests a lane 161; a copy engine 160.
  // (A few units more than are in flight cost a second round trip: 1.1 MB 28.1 us all at once and 29.4, 1.2 MB 30.3 and
  // 31.7, 1.3 MB 32.7 both, 1.5 MB 37.7 and 35.5.)
  // Writes to host memory: up to 8 MiB the same (256 blocks of int8, 161 us and 165), above it 327 -> 309 us
  // (500 blocks of e4m3), 314 -> 300 (60 of bf16, 64 tokens).  Device memory needs all of them in flight.
  if (units > (to_packed ? kHostWriteAll : kHostReadAll)) {
    hipPointerAttribute_t where;
    if (hipPointerGetAttributes(&where, packed_cache) != hipSuccess) (void)hipGetLastError();  // (memory HIP does not know)
    else if (where.type == hipMemoryTypeHost) grid = kHostUnits;
  }
#define KVQ_LAUNCH_COPY(TO_PACKED, STRIDED)                                                               \
  hipLaunchKernelGGL((block_copy_kernel<TO_PACKED, STRIDED>), dim3(grid), dim3(256), 0, stream,           \
                     (uint8_t*)pool_cache, (float*)pool_scales, (uint8_t*)packed_cache, packed_scales,    \
                     block_ids, block_bytes, scale_floats, pieces, units)
  if (to_packed) {
    if (grid < units) KVQ_LAUNCH_COPY(true, true);
    else KVQ_LAUNCH_COPY(true, false);
  } else {
    if (grid < units) KVQ_LAUNCH_COPY(false, true);
    else KVQ_LAUNCH_COPY(false, false);
  }
#undef KVQ_LAUNCH_COPY
  return hipGetLastError();
}

hipError_t launch_repack(const void* src, void* dst, const kvq_cache_desc_t& desc,
                         bool to_canonical, hipStream_t stream) {
  const size_t total = (size_t)desc.num_blocks * 2 * desc.num_kv_heads * desc.block_size *
                       (is_int4(desc.mode) ? desc.head_dim / 2 : desc.head_dim);
  if (total == 0) return hipSuccess;
  size_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (is_int4(desc.mode)) {
    hipLaunchKernelGGL(repack_int4_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                       (const uint8_t*)src, (uint8_t*)dst, total, desc.num_kv_heads,
                       desc.block_size, to_canonical);
    return hipGetLastError();
  }
  if (desc.mode == KVQ_BF16_PLAIN) {
    hipLaunchKernelGGL(repack16_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                       (const uint16_t*)src, (uint16_t*)dst, total, desc.num_kv_heads,
                       desc.block_size, desc.head_dim, to_canonical);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(repack_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                     (const uint8_t*)src, (uint8_t*)dst, total, desc.num_kv_heads,
                     desc.block_size, desc.head_dim, desc.mode, to_canonical);
  return hipGetLastError();
}

}  // namespace kvq
