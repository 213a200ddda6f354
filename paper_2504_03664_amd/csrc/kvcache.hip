// INT4 KV cache rows (Section 2: the KV cache may be kept in 4 bits; the
// conversion belongs to the cache's loading and saving, Section 3.1.2).
// A row of d elements: d/2 code bytes, element 2i in the low nibble of byte
// i, then d/64 fp16 (scale, min) pairs, one per 64 consecutive elements.
//
//   kv_quant_k:   fp16 rows -> INT4 rows; per group, in fp32:
//                 scale = fp16((max - min) / 15), min = fp16(min),
//                 code = clamp(rint((x - min) / scale), 0, 15), half to
//                 even, 0 where scale is 0 (both divisions IEEE-rounded).
//   kv_dequant_k: INT4 rows -> fp16 rows, code * scale + min rounded once.
// Eight lanes per group of 64, 8 elements each: a lane moves 16 bytes of fp16
// and 4 of codes, so a wave's accesses are contiguous and a decode step's few
// rows spread over the chip.  (One lane per group, 128 bytes and 64 divisions
// in a row, took 6 us for 128 rows of 7168, about 2 more than a launch.)
#include "common.h"
#include "device.h"

namespace pipo {

// largest of the 8 lanes of a group, by DPP moves within a row of 16 lanes
// (swap neighbours, swap pairs, mirror within 8)
template <int CTRL>
__device__ __forceinline__ float lane_move(float v) {
  return __uint_as_float(
      __builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float group_max8(float v) {
  v = fmaxf(v, lane_move<0xB1>(v));
  v = fmaxf(v, lane_move<0x4E>(v));
  return fmaxf(v, lane_move<0x141>(v));
}
__device__ __forceinline__ float group_min8(float v) {
  v = fminf(v, lane_move<0xB1>(v));
  v = fminf(v, lane_move<0x4E>(v));
  return fminf(v, lane_move<0x141>(v));
}

// row and 8-element piece of this thread; false past the end.  A row has a
// multiple of 32 pieces, so the 8 lanes of a group are all in or all out.
// The division is 32-bit where the pieces allow (64-bit took a third of the
// quantizer's time).
__device__ __forceinline__ bool piece_of(int64_t rows, int64_t d, int64_t& r, int& c) {
  const int64_t per_row = d / 8;
  const int64_t e = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
  if (e >= rows * per_row) return false;
  if (rows * per_row < ((int64_t)1 << 32)) {
    const uint32_t row = (uint32_t)e / (uint32_t)per_row;
    r = row;
    c = (int)((uint32_t)e - row * (uint32_t)per_row);
  } else {
    r = e / per_row;
    c = (int)(e - r * per_row);
  }
  return true;
}

__global__ __launch_bounds__(256) void kv_quant_k(const uint16_t* __restrict__ x,
                                                  uint8_t* __restrict__ out, int64_t rows,
                                                  int64_t d) {
  int64_t r;
  int c;  // 8-element piece of row r
  if (!piece_of(rows, d, r, c)) return;
  const h8 h = load_h8(x + r * d + 8 * c);
  float v[8], mn, mx;
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = (float)h[j];
  mn = mx = v[0];
#pragma unroll
  for (int j = 1; j < 8; ++j) {
    mn = fminf(mn, v[j]);
    mx = fmaxf(mx, v[j]);
  }
  mn = group_min8(mn);
  mx = group_max8(mx);
  const _Float16 s16 = (_Float16)((mx - mn) / 15.f);
  const _Float16 m16 = (_Float16)mn;
  const float s = (float)s16, m = (float)m16;
  // (x - min) / scale, correctly rounded from the correctly rounded reciprocal
  // and one residual step (Markstein, IBM J. Res. Dev. 34, 1990): an eighth of
  // a division per element.  Infinite inputs give NaN and code 0, as the
  // division would.
  const float inv = s != 0.f ? 1.f / s : 0.f;
  uint32_t word = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float x = v[j] - m, q0 = x * inv;
    const float q = __builtin_fmaf(__builtin_fmaf(-q0, s, x), inv, q0);
    word |= (uint32_t)(s != 0.f ? fminf(fmaxf(__builtin_rintf(q), 0.f), 15.f) : 0.f) << (4 * j);
  }
  uint8_t* row = out + r * (d / 2 + d / 16);
  *reinterpret_cast<uint32_t*>(row + 4 * c) = word;
  if (c % 8 == 0)
    *reinterpret_cast<uint32_t*>(row + d / 2 + c / 8 * 4) =
        (uint32_t)__builtin_bit_cast(uint16_t, s16) |
        ((uint32_t)__builtin_bit_cast(uint16_t, m16) << 16);
}

__global__ __launch_bounds__(256) void kv_dequant_k(const uint8_t* __restrict__ in,
                                                    uint16_t* __restrict__ y, int64_t rows,
                                                    int64_t d) {
  int64_t r;
  int c;
  if (!piece_of(rows, d, r, c)) return;
  const uint8_t* row = in + r * (d / 2 + d / 16);
  const uint32_t codes = *reinterpret_cast<const uint32_t*>(row + 4 * c);
  h2 s2, m2;
  scale_min_pairs(*reinterpret_cast<const uint32_t*>(row + d / 2 + c / 8 * 4), s2, m2);
  *reinterpret_cast<h8*>(y + r * d + 8 * c) = dequant8_fp8(codes, s2, m2);
}

// a thread per 8 elements, up to 2^30 threads (a launch takes under 2^32 in a
// dimension) in each row of the grid; piece_of drops the excess
static dim3 piece_grid(int64_t pieces) {
  const int64_t blocks = (pieces + 255) / 256, row = (int64_t)1 << 22;
  return blocks <= row ? dim3((unsigned)blocks)
                       : dim3((unsigned)row, (unsigned)((blocks + row - 1) / row));
}

pipo_status launch_kv_quant(const uint16_t* x, uint8_t* out, int64_t rows, int64_t d,
                            hipStream_t st) {
  if (rows < 0 || d <= 0 || d % 256 != 0) {
    set_error("kv_quant: rows %lld, d %lld (d must be a multiple of 256)", (long long)rows,
              (long long)d);
    return PIPO_ERR_UNSUPPORTED;
  }
  const int64_t n = rows * (d / 8);
  if (n == 0) return PIPO_OK;
  launch(kv_quant_k, piece_grid(n), dim3(256), 0, st, x, out, rows, d);
  PIPO_HIP_TRY(hipGetLastError());
  return PIPO_OK;
}

pipo_status launch_kv_dequant(const uint8_t* in, uint16_t* y, int64_t rows, int64_t d,
                              hipStream_t st) {
  if (rows < 0 || d <= 0 || d % 256 != 0) {
    set_error("kv_dequant: rows %lld, d %lld (d must be a multiple of 256)", (long long)rows,
              (long long)d);
    return PIPO_ERR_UNSUPPORTED;
  }
  const int64_t n = rows * (d / 8);
  if (n == 0) return PIPO_OK;
  launch(kv_dequant_k, piece_grid(n), dim3(256), 0, st, in, y, rows, d);
  PIPO_HIP_TRY(hipGetLastError());
  return PIPO_OK;
}

}  // namespace pipo
