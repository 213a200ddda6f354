// Shared by the attention kernels that keep key and value blocks in LDS.
#pragma once

#include "common.h"
#include "device.h"

namespace pipo {

// LDS slot of 16-byte chunk `chunk` of key row `key` (an involution: the
// DMA puts cache chunk kv_swz(row, s) into slot s, a read of chunk c goes
// to slot kv_swz(row, c)).  The chunk is XORed with a mask that depends on
// the row's low four bits, chosen with the LDS bank-conflict counters: over
// the K fragment reads (ds_read_b128; lane r + 16 g reads row r of a 16-row
// group, chunk 4 kk + g) and the transposed V reads (ds_read_b64_tr_b16;
// rows 4 g .. 4 g + 3 of a group, chunks 2 n and 2 n + 1), a plain XOR with
// the row leaves the K reads conflict-free but gives every V read a 2-way
// conflict, the row rotated left by one bit the reverse, and of 240 random
// masks that clear the V reads three cleared the K reads as well; the table
// below is the first of them (head_dim 128: 16 chunks per row).  For
// head_dim 64 (two rows per 256 bytes) the mask row & 6 measured no
// conflicts on either read.
template <int D>
__device__ __forceinline__ int kv_swz(int key, int chunk) {
  if constexpr (D == 128) {
    constexpr uint64_t kMask = 0x618d34ea5b2f0c97ull;  // nibble x: mask of rows with key % 16 == x
    return chunk ^ (int)((kMask >> (4 * (key & 15))) & 15);
  } else {
    return chunk ^ (key & 6);
  }
}

// the pair of values that v_permlane16/32_swap leave in a lane: its own
// and that of the lane 16 (32) apart, in either order
template <typename P>
__device__ __forceinline__ float pair_max(P p) {
  return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
template <typename P>
__device__ __forceinline__ float pair_sum(P p) {
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// decode attention with G = 2, 4 or 8 query heads per key/value head
// (attention_gqa.hip): S splits of `chunk` keys, the partials of S > 1 to `part`
void launch_decode_gqa(const uint16_t* q, const void* kc, const void* vc, uint16_t* o, int b,
                       int Hkv, int G, int head_dim, int t, bool kv4, int S, int chunk,
                       float* part, hipStream_t st);

}  // namespace pipo
