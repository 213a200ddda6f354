// Shared by the GEMM sources: epilogues, the split-K merge and the slab
// kernels' launchers.
#pragma once

#include "common.h"
#include "device.h"

namespace pipo {

constexpr int kXcds = 8;  // accelerator complex dies of an MI355X, each with its own L2

// Epilogue, split into what depends on the output row only (its offsets,
// computed once per row by kernels that own many columns of it) and the
// per-element part.  EPI_QKV: row m is sequence m / rows_per_seq at
// position pos0 + m % rows_per_seq, whose k and v go to cache row
// position * batch + sequence.
struct EpiRow {
  int64_t m;      // output row (>= M: none)
  int64_t off;    // m * ldo, or m * d for q (EPI_QKV)
  int64_t kvoff;  // EPI_QKV: cache row * dkv
};

template <int EPI>
__device__ __forceinline__ EpiRow epilogue_row(const GemmArgs& a, int64_t m) {
  EpiRow r{m, 0, 0};
  if (m >= a.M) return r;
  if constexpr (EPI == EPI_QKV) {
    // launch_gemm keeps M below 2^31, so 32-bit division is exact
    const uint32_t mm = (uint32_t)m, rps = (uint32_t)a.rows_per_seq;
    const uint32_t seq = mm / rps;
    const int64_t pos = a.pos0 + (int64_t)(mm - seq * rps);
    r.off = m * a.d;
    r.kvoff = (pos * a.batch + seq) * a.dkv;
  } else {
    r.off = m * a.ldo;
  }
  return r;
}

// bias of column n (0 past N or without bias)
__device__ __forceinline__ float epilogue_bias(const GemmArgs& a, int64_t n) {
  return (a.bias && n < a.N) ? h2f(a.bias[n]) : 0.f;
}

// v: the sum with the column's bias added
template <int EPI>
__device__ __forceinline__ void epilogue_store(const GemmArgs& a, const EpiRow& r, int64_t n,
                                               float v) {
  if (r.m >= a.M || n >= a.N) return;
  if constexpr (EPI == EPI_F16) {
    a.out16[r.off + n] = f2h(v);
  } else if constexpr (EPI == EPI_RELU_F16) {
    a.out16[r.off + n] = f2h(v > 0.f ? v : 0.f);
  } else if constexpr (EPI == EPI_ADD_F32) {
    a.out32[r.off + n] += v;
  } else if constexpr (EPI == EPI_F32) {
    a.out32[r.off + n] = v;
  } else {  // EPI_QKV
    if (n < a.d)
      a.q_out[r.off + n] = f2h(v * a.q_scale);
    else if (n < a.d + a.dkv)
      a.k_out[r.kvoff + (n - a.d)] = f2h(v);
    else
      a.v_out[r.kvoff + (n - a.d - a.dkv)] = f2h(v);
  }
}

template <int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& a, int64_t m, int64_t n, float acc) {
  epilogue_store<EPI>(a, epilogue_row<EPI>(a, m), n, acc + epilogue_bias(a, n));
}

// whether four consecutive columns n (n % 4 == 0) of a row can be stored at
// once: they stay in one output matrix and its rows are aligned for it
template <int EPI>
__device__ __forceinline__ bool epilogue_vec4(const GemmArgs& a) {
  if (a.N % 4 != 0) return false;
  if constexpr (EPI == EPI_QKV) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a.q_out) | reinterpret_cast<uintptr_t>(a.k_out) |
                        reinterpret_cast<uintptr_t>(a.v_out);
    return p % 8 == 0 && a.d % 4 == 0 && a.dkv % 4 == 0;
  } else if constexpr (EPI == EPI_ADD_F32 || EPI == EPI_F32) {
    return a.ldo % 4 == 0 && reinterpret_cast<uintptr_t>(a.out32) % 16 == 0;
  } else {
    return a.ldo % 4 == 0 && reinterpret_cast<uintptr_t>(a.out16) % 8 == 0;
  }
}

// columns n .. n + 3 (n < N) of a row m < M; v: the sums with the bias added
template <int EPI>
__device__ __forceinline__ void epilogue_store4(const GemmArgs& a, const EpiRow& r, int64_t n,
                                                f4 v) {
  if constexpr (EPI == EPI_ADD_F32 || EPI == EPI_F32) {
    f4* p = reinterpret_cast<f4*>(a.out32 + r.off + n);
    *p = EPI == EPI_ADD_F32 ? *p + v : v;
  } else {
    uint16_t* p;
    if constexpr (EPI == EPI_QKV) {
      if (n < a.d) {
        v *= a.q_scale;
        p = a.q_out + r.off + n;
      } else {
        p = n < a.d + a.dkv ? a.k_out + r.kvoff + (n - a.d) : a.v_out + r.kvoff + (n - a.d - a.dkv);
      }
    } else {
      p = a.out16 + r.off + n;
      if constexpr (EPI == EPI_RELU_F16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = v[j] > 0.f ? v[j] : 0.f;
      }
    }
    u32x2 w;
    w[0] = (uint32_t)f2h(v[0]) | ((uint32_t)f2h(v[1]) << 16);
    w[1] = (uint32_t)f2h(v[2]) | ((uint32_t)f2h(v[3]) << 16);
    *reinterpret_cast<u32x2*>(p) = w;
  }
}

// out = sum over z = 0 .. S-1 of the partials ws[z][M][N], then the epilogue
// (gemm.hip); S is 2, 4 or 8 and M * N < 2^31
void launch_combine(const GemmArgs& a, int epi, const float* ws, int S, hipStream_t st);

// Slab kernels (gemm_slab.h) by index into the tables below, PIPO_SLAB_F16
// in gemm_slab_f16.hip and PIPO_SLAB_W4 in gemm_slab_w4.hip; S K ranges
// (S > 1: partials to ws, without the merge), K % (64 S) == 0.  direct: X and
// the weights are 16-byte aligned, the (scale, min) pairs 4-byte aligned; it
// must be so for MF = 1 and for 256 columns.
//      index, MF, NF, WN, KS, PD   (tile 16 MF x 16 NF WN, WN KS waves)
#define PIPO_SLAB_F16(X)                                                                \
  X(0, 1, 1, 1, 8, 3) X(1, 1, 2, 1, 8, 2)                                               \
  X(2, 2, 1, 2, 4, 3) X(3, 2, 3, 2, 2, 3) X(4, 2, 2, 4, 2, 2)                           \
  X(5, 4, 1, 4, 2, 3) X(6, 4, 3, 2, 2, 2) X(7, 4, 1, 8, 1, 3)                           \
  X(8, 8, 1, 4, 2, 2) X(9, 8, 1, 8, 1, 3)                                               \
  X(10, 1, 2, 2, 4, 2)
#define PIPO_SLAB_W4(X)                                                                 \
  X(0, 1, 2, 1, 8, 4)                                                                   \
  X(1, 2, 2, 2, 4, 3) X(2, 2, 2, 4, 4, 2)                                               \
  X(3, 4, 2, 2, 4, 2) X(4, 4, 4, 2, 4, 2)                                               \
  X(5, 8, 2, 2, 4, 1) X(6, 8, 2, 4, 2, 2) X(7, 8, 4, 4, 2, 2) X(8, 8, 2, 8, 1, 3)
void launch_slab_f16(const GemmArgs& a, int epi, int idx, bool direct, int S, float* ws,
                     hipStream_t st);
void launch_slab_w4(const GemmArgs& a, int epi, int idx, bool direct, int S, float* ws,
                    hipStream_t st);

}  // namespace pipo
