// Causal softmax attention over a position-major KV cache: row p * b + i
// of K (or V) holds sequence i's key (value) at position p, all key/value
// heads side by side.  With grouped-query attention, query head h reads
// key/value head h / (H / Hkv).  This is the layout the copy engine streams when the cache lives
// in host memory: a layer's prefix 0..t-1 is one contiguous range.
//
//   attn_decode:  one new query per (sequence, head) against keys 0..t
//                 (with grouped-query attention: attention_gqa.hip).
//   attn_prefill: P queries per (sequence, head), causal, flash-style with
//                 v_mfma_f32_16x16x32_f16 for Q K^T and P V.
// Softmax is max-subtracted in fp32; every reduction has a fixed order.
#include <algorithm>
#include <cfloat>
#include <mutex>

#include "attention_common.h"

namespace pipo {

// Sum over aligned groups of N <= 16 lanes with DPP moves inside a row of 16
// lanes (swap neighbours, swap pairs, mirror within 8, mirror within 16):
// ALU operations instead of the LDS round trips of lane shuffles.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __uint_as_float(
      __builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xF, 0xF, false));
}
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(N == 1 || N == 2 || N == 4 || N == 8 || N == 16, "groups of up to 16 lanes");
  if constexpr (N >= 2) v += dpp_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  if constexpr (N >= 4) v += dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  if constexpr (N >= 8) v += dpp_move<0x141>(v);  // row_half_mirror
  if constexpr (N >= 16) v += dpp_move<0x140>(v); // row_mirror
  return v;
}

// ---------------------------------------------------------------------------
// decode without grouping: grid (head groups, b, splits), 256 threads.  A
// workgroup serves HP adjacent heads of one sequence, so each cached row is
// read from HBM once per step and a key's HP heads are one contiguous HP * D
// * 2-byte read.  Split z of a (sequence, head group) covers keys
// [z * chunk, min(T, (z + 1) * chunk)).  A key's head is handled by D/8 lanes
// (8 dims each; fp16 rows are read with non-temporal loads, as every row is
// read once); every lane group keeps its own online softmax state (running
// max m, sum l, 8 accumulators) over the keys it visits, two keys at a time
// so that K and V of both are in flight together (the second one's index is
// clamped, so the loads are unconditional).  Groups are merged by a butterfly
// inside the wave, waves in order through LDS.  With one split the result is
// final; otherwise (m, l, acc[D]) of each head goes to `part` and
// attn_decode_combine merges the splits in split order.
__device__ __forceinline__ void online_merge(float& m, float& l, float (&acc)[8], float m2,
                                             float l2, const float (&acc2)[8]) {
  const float M = fmaxf(m, m2);
  const float a1 = m == -INFINITY ? 0.f : expf(m - M);
  const float a2 = m2 == -INFINITY ? 0.f : expf(m2 - M);
  l = l * a1 + l2 * a2;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = acc[i] * a1 + acc2[i] * a2;
  m = M;
}

template <int D, int HP>
__global__ __launch_bounds__(256) void attn_decode_k(const uint16_t* __restrict__ q,
                                                     const uint16_t* __restrict__ kc,
                                                     const uint16_t* __restrict__ vc,
                                                     uint16_t* __restrict__ o,
                                                     float* __restrict__ part, int b, int H,
                                                     int t, int chunk) {
  constexpr int LPP = D / 8;      // lanes per head of a key
  constexpr int LPK = HP * LPP;   // lanes per key
  constexpr int PPW = 64 / LPK;   // keys per wave per pass
  __shared__ float wm[4][HP], wl[4][HP];
  __shared__ float wacc[4][HP * D];
  const int kb = blockIdx.x, bi = blockIdx.y, sp = blockIdx.z, S = gridDim.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane / LPK, cl = lane % LPK, hl = cl / LPP, cd = (cl % LPP) * 8;
  const int64_t d = (int64_t)H * D;
  const int T = t + 1;
  const int p0 = sp * chunk, p1 = min(T, p0 + chunk);
  const int64_t col = (int64_t)(kb * HP + hl) * D + cd;

  float qf[8];
  const h8 qv = load_h8(q + (int64_t)bi * d + col);
#pragma unroll
  for (int i = 0; i < 8; ++i) qf[i] = (float)qv[i];
  float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;

  const int64_t lane_off = (int64_t)bi * d + col;
  const auto load_kv = [&](const uint16_t* base, int p) -> h8 {
    return load_h8_stream(base + (int64_t)p * b * d + lane_off);
  };
  const auto visit = [&](h8 kv, h8 vv) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += qf[i] * (float)kv[i];
    // (bound by HBM: DPP sums measured no faster)
#pragma unroll
    for (int off = LPP / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    const float mn = fmaxf(m, s);
    const float alpha = expf(m - mn);
    const float e = expf(s - mn);
    l = l * alpha + e;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = acc[i] * alpha + e * (float)vv[i];
    m = mn;
  };
  for (int p = p0 + wave * PPW + sub; p < p1; p += 8 * PPW) {
    const int p2 = min(p + 4 * PPW, p1 - 1);
    const h8 ka = load_kv(kc, p);
    const h8 va = load_kv(vc, p);
    const h8 kb2 = load_kv(kc, p2);
    const h8 vb2 = load_kv(vc, p2);
    visit(ka, va);
    if (p + 4 * PPW < p1) visit(kb2, vb2);
  }
  // merge the lane groups of the wave (butterfly over the group index)
#pragma unroll
  for (int off = LPK; off < 64; off <<= 1) {
    float acc2[8];
    const float m2 = __shfl_xor(m, off, 64);
    const float l2 = __shfl_xor(l, off, 64);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc2[i] = __shfl_xor(acc[i], off, 64);
    online_merge(m, l, acc, m2, l2, acc2);
  }
  if (sub == 0) {
    if (cd == 0) {
      wm[wave][hl] = m;
      wl[wave][hl] = l;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) wacc[wave][hl * D + cd + i] = acc[i];
  }
  __syncthreads();
  for (int c = tid; c < HP * D; c += 256) {
    const int j = c / D, cc = c % D, h = kb * HP + j;
    float M = wm[0][j], L = wl[0][j], A = wacc[0][c];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float m2 = wm[w][j];
      const float Mn = fmaxf(M, m2);
      const float a1 = M == -INFINITY ? 0.f : expf(M - Mn);
      const float a2 = m2 == -INFINITY ? 0.f : expf(m2 - Mn);
      L = L * a1 + wl[w][j] * a2;
      A = A * a1 + wacc[w][c] * a2;
      M = Mn;
    }
    if (S == 1) {
      o[(int64_t)bi * d + (int64_t)h * D + cc] = f2h(A / L);
    } else {
      float* pp = part + (((int64_t)bi * H + h) * S + sp) * (D + 2);
      pp[cc] = A;
      if (cc == 0) {
        pp[D] = M;
        pp[D + 1] = L;
      }
    }
  }
}

// decode over an INT4 cache without grouping: the same structure as
// attn_decode_k, but a lane holds 32 elements of a key's head (one 16-byte
// load of codes and one (scale, min) pair), D/32 lanes per head of a key.
// The kernel is bound by its arithmetic.  A word's eight codes become fp16 by
// the fp8 converter (a byte c is the fp8 number c 2^-9; the low and the high
// nibbles of the word's bytes, two codes per conversion: elements (0, 2),
// (4, 6), (1, 3), (5, 7)), and scale and min leave the inner loops: with one
// pair per lane and key,
//   q . k = scale (q . codes) + min sum(q)      (two-element dot products)
//   O += p v = (p scale) codes + p min          (p min: one sum for the lane)
// all in fp32 from exact codes, so no expanded value is rounded to fp16 (the
// error against 64 bits falls with it: 4.9e-4 -> 2.1e-4 at b 128, 544 keys).
// The softmax uses the hardware exp2 and the accumulators are rescaled only
// when some lane's running maximum grew.  26 instructions for a word of key
// and a word of value codes, where expanding both to fp16 took 48.  us at b
// 128, 56 heads of 128, 544 keys, with the quantization of the step's rows:
// 149.7 -> 145.8, and 127.7 with the workgroups of a sequence on one XCD
// (about 115 for this kernel, of which the instructions issue for 82; the
// cache alone is 88 at 6.4 TB/s).
template <int D, int HP>
__global__ __launch_bounds__(256) void attn_decode_kv4_k(const uint16_t* __restrict__ q,
                                                         const void* __restrict__ kc,
                                                         const void* __restrict__ vc,
                                                         uint16_t* __restrict__ o,
                                                         float* __restrict__ part, int b, int H,
                                                         int t, int chunk) {
  constexpr int EPL = 32;            // elements per lane
  constexpr int LPP = D / EPL;       // lanes per head of a key
  constexpr int LPK = HP * LPP;      // lanes per key
  constexpr int PPW = 64 / LPK;      // keys per wave per pass
  __shared__ float wm[4][HP], wl[4][HP];
  __shared__ float wacc[4][HP * D];
  // XCD x (workgroups x, x + 8, ..) takes a contiguous range of (sequence,
  // head group) pairs: the head groups of a sequence share the lines at their
  // borders and those of the (scale, min) pairs, which then meet in one L2
  const int groups = H / HP;
  const int64_t id = blockIdx.x + (int64_t)gridDim.x * blockIdx.z;
  const int64_t pair = id % 8 * ((int64_t)gridDim.x / 8 * gridDim.z) + id / 8;
  if (pair >= (int64_t)groups * b) return;
  const int bi = (int)(pair / groups), kb = (int)(pair - (int64_t)bi * groups);
  const int sp = blockIdx.y, S = gridDim.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane / LPK, cl = lane % LPK, hl = cl / LPP, cd = (cl % LPP) * EPL;
  const int64_t d = (int64_t)H * D;
  const int T = t + 1;
  const int p0 = sp * chunk, p1 = min(T, p0 + chunk);
  const int64_t col = (int64_t)(kb * HP + hl) * D + cd;

  constexpr float kLog2e = 1.4426950408889634f;
  // qh[4 j + u]: elements 8 j + kElem[2 u], 8 j + kElem[2 u + 1]; acc the same
  // order
  constexpr int kElem[8] = {0, 2, 4, 6, 1, 3, 5, 7};
  h2 qh[EPL / 2];
  float qsum = 0.f;
#pragma unroll
  for (int j = 0; j < EPL / 8; ++j) {
    const h8 qv = load_h8(q + (int64_t)bi * d + col + 8 * j);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      qh[4 * j + u] = h2{qv[kElem[2 * u]], qv[kElem[2 * u + 1]]};
      qsum += (float)qv[kElem[2 * u]] + (float)qv[kElem[2 * u + 1]];
    }
  }
  // the output is acc[i] + accm
  float m = -INFINITY, l = 0.f, acc[EPL], accm = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) acc[i] = 0.f;

  const int64_t row_bytes = d / 2 + d / 16;
  const int64_t code_off = (int64_t)bi * row_bytes + col / 2;            // 16-byte aligned
  const int64_t sm_off = (int64_t)bi * row_bytes + d / 2 + (col / 64) * 4;
  struct Row {
    u32x4 codes;
    uint32_t sm;
  };
  const auto load_row = [&](const void* base, int p) -> Row {
    const char* row = static_cast<const char*>(base) + (int64_t)p * b * row_bytes;
    return Row{*reinterpret_cast<const u32x4*>(row + code_off),
               *reinterpret_cast<const uint32_t*>(row + sm_off)};
  };
  // pair u (0..3) of a word's codes as fp16
  const auto codes2 = [](uint32_t w, int u) -> h2 {
    const uint32_t n = (u < 2 ? w : w >> 4) & 0x0F0F0F0Fu;
    return u & 1 ? __builtin_bit_cast(h2, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(n, 512.f, true))
                 : __builtin_bit_cast(h2, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(n, 512.f, false));
  };
  const auto visit = [&](const Row& kr, const Row& vr) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        s = __builtin_amdgcn_fdot2(qh[4 * j + u], codes2(kr.codes[j], u), s, false);
    s = group_sum<LPP>(s * h2f((uint16_t)kr.sm) + h2f((uint16_t)(kr.sm >> 16)) * qsum);
    const float mn = fmaxf(m, s);
    // m = -inf on the first key: exp2(-inf) = 0
    const float alpha = __builtin_amdgcn_exp2f((m - mn) * kLog2e);
    const float e = __builtin_amdgcn_exp2f((s - mn) * kLog2e);
    l = l * alpha + e;
    // the running maxima rarely grow after the first keys: rescale only
    // when some lane's did (alpha = 1 exactly otherwise)
    if (__any(alpha != 1.f)) {
      accm *= alpha;
#pragma unroll
      for (int i = 0; i < EPL; ++i) acc[i] *= alpha;
    }
    const float es = e * h2f((uint16_t)vr.sm);
    accm += e * h2f((uint16_t)(vr.sm >> 16));
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const h2 c = codes2(vr.codes[j], u);
        acc[8 * j + 2 * u] += es * (float)c[0];
        acc[8 * j + 2 * u + 1] += es * (float)c[1];
      }
    m = mn;
  };
  for (int p = p0 + wave * PPW + sub; p < p1; p += 8 * PPW) {
    const int p2 = min(p + 4 * PPW, p1 - 1);
    const Row ka = load_row(kc, p), va = load_row(vc, p);
    const Row kb2 = load_row(kc, p2), vb2 = load_row(vc, p2);
    visit(ka, va);
    if (p + 4 * PPW < p1) visit(kb2, vb2);
  }
#pragma unroll
  for (int i = 0; i < EPL; ++i) acc[i] += accm;
  // merge the key slots of the wave, then the waves through LDS
#pragma unroll
  for (int off = LPK; off < 64; off <<= 1) {
    const float m2 = __shfl_xor(m, off, 64);
    const float l2 = __shfl_xor(l, off, 64);
    const float M = fmaxf(m, m2);
    const float a1 = m == -INFINITY ? 0.f : expf(m - M);
    const float a2 = m2 == -INFINITY ? 0.f : expf(m2 - M);
    l = l * a1 + l2 * a2;
#pragma unroll
    for (int i = 0; i < EPL; ++i) acc[i] = acc[i] * a1 + __shfl_xor(acc[i], off, 64) * a2;
    m = M;
  }
  if (sub == 0) {
    if (cd == 0) {
      wm[wave][hl] = m;
      wl[wave][hl] = l;
    }
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      wacc[wave][hl * D + cd + 8 * (i / 8) + kElem[i % 8]] = acc[i];
  }
  __syncthreads();
  for (int c = tid; c < HP * D; c += 256) {
    const int j = c / D, cc = c % D, h = kb * HP + j;
    float M = wm[0][j], L = wl[0][j], A = wacc[0][c];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float m2 = wm[w][j];
      const float Mn = fmaxf(M, m2);
      const float a1 = M == -INFINITY ? 0.f : expf(M - Mn);
      const float a2 = m2 == -INFINITY ? 0.f : expf(m2 - Mn);
      L = L * a1 + wl[w][j] * a2;
      A = A * a1 + wacc[w][c] * a2;
      M = Mn;
    }
    if (S == 1) {
      o[(int64_t)bi * d + (int64_t)h * D + cc] = f2h(A / L);
    } else {
      float* pp = part + (((int64_t)bi * H + h) * S + sp) * (D + 2);
      pp[cc] = A;
      if (cc == 0) {
        pp[D] = M;
        pp[D + 1] = L;
      }
    }
  }
}

// merge the splits of each (sequence, head) in split order
template <int D>
__global__ __launch_bounds__(D) void attn_decode_combine(const float* __restrict__ part,
                                                         uint16_t* __restrict__ o, int H,
                                                         int S) {
  const int h = blockIdx.x, bi = blockIdx.y, c = threadIdx.x;
  const float* pp = part + ((int64_t)bi * H + h) * S * (D + 2);
  float M = pp[D], L = pp[D + 1], A = pp[c];
  for (int z = 1; z < S; ++z) {
    const float* pz = pp + (int64_t)z * (D + 2);
    const float m2 = pz[D];
    const float Mn = fmaxf(M, m2);
    const float a1 = M == -INFINITY ? 0.f : expf(M - Mn);
    const float a2 = m2 == -INFINITY ? 0.f : expf(m2 - Mn);
    L = L * a1 + pz[D + 1] * a2;
    A = A * a1 + pz[c] * a2;
    M = Mn;
  }
  o[((int64_t)bi * H + h) * D + c] = f2h(A / L);
}

// ---------------------------------------------------------------------------
// prefill (flash-style): a workgroup owns 32 NW queries of one head and
// sequence, NW waves x 32 queries (two sub-blocks of 16).  Keys come in
// blocks of kPK, K and V moved from the cache straight into LDS by the load
// unit (NS buffers), rows stored with their 16-byte chunks permuted by
// row (kv_swz) so that the K fragment reads and the transposed V reads hit
// distinct banks.  The wave
// computes S^T = K Q^T (keys on the MFMA rows, its queries on the columns,
// so each lane holds scores of one query), an online softmax per query in
// fp32, and O^T += V^T P^T: the probabilities stay in the registers they
// were computed in (a lane's 8 keys per MFMA are the ones its S^T fragment
// gave it; V^T is read with the same key order through transposed LDS
// reads).
//
// Which workgroup takes what, with several query blocks per head: workgroups
// go to the XCDs in turn, and within one to its shader engines and CUs in
// turn, so an order in which the blocks of a head follow each other (1, 2, ..
// n key blocks of work) gives the same class of work to the same CUs again
// and again (with 4 or 8 query blocks the heaviest to one XCD).  XCD x takes
// 1/8 of the (sequence, head) pairs, in groups of 32 (its CUs), and of a group
// first every pair's last query block, then the one before, and so on; the
// pairs % 8 left over are dealt to all XCDs in the same order, first.  us
// before and after: b 32, 512 tokens, 40 heads of 128 251 -> 200; 64 heads over
// 8 376 -> 314; 40 heads of 64 131 -> 104; 8 x 1024, 40 heads of 128 220 -> 157.
// With
// many pairs of few blocks the reads of K and V count more than the balance:
// groups of 5 (no divisor of the CUs) while the XCD has more than 32 pairs of
// at most 6 blocks.  us with the grid's order, groups of 32, groups of 5: b 32,
// 384 tokens, 40 heads of 128 142, 145, 133; 16 x 600 142, 142, 134; 8 x 700 96,
// 92, 84; 16 x 250 45, 47, 41; but 8 x 640, 32 heads over 8 62, 54, 60; 1 x
// 1500, 56 heads 77, 50, 57.  Grid's order and groups of 32 further up: b 2,
// 2048 tokens, 40 heads 189, 117; 1 x 4096 347, 203.  With one query block the
// order of the grid is 4 % the faster (39 against 41 at b 32, 128 tokens).
// What is left is the softmax between the two products: 1024 cycles of MFMA
// and about as many of vector and of LDS work for a wave and 64-key block.
//
// Up to 32 tokens one wave has all the queries: two waves and one block of 32
// keys (the other keys of 64 are masked, so the bits are the same) let more
// workgroups share a CU: b 64, 32 tokens, 56 heads of 128 33 -> 24 us, b 128,
// 32 heads over 8 37 -> 22.
constexpr int kPQ = 128;     // queries per workgroup
constexpr int kPK = 64;      // keys per block
constexpr int kPShort = 32;  // prompts that take the short form
// pairs whose query blocks are interleaved
constexpr uint32_t kPGroup = 32, kPGroupSmall = 5;
constexpr int kPrefillStages = 2;

template <int NS, int DMA>
__device__ __forceinline__ void wait_blocks_landed(int pending) {
  // at most `pending` later blocks (2 DMA loads per wave each) outstanding
  if constexpr (NS >= 4) {
    if (pending >= 3) {
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(3 * 2 * DMA, false));
      return;
    }
  }
  if constexpr (NS >= 3) {
    if (pending >= 2) {
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * 2 * DMA, false));
      return;
    }
  }
  if (pending >= 1) {
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * DMA, false));
    return;
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));
}

template <int D, int NS, int PK, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void attn_prefill_k(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc,
    const uint16_t* __restrict__ vc, uint16_t* __restrict__ o, int b, int P, int H, int Hkv) {
  constexpr int PQ = 32 * NW;              // queries per workgroup
  constexpr int ROWB = 2 * D;               // bytes per key row in LDS
  constexpr int BLK = PK * ROWB;            // bytes of K (or V) per block
  constexpr int DMA = BLK / 1024 / NW;      // DMA instructions per wave for K (and for V)
  constexpr int KK = D / 32;                // MFMA k steps over the head dimension
  constexpr int NF = D / 16;                // head-dimension fragments of O^T
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ __attribute__((aligned(1024))) uint8_t kv[NS][2][BLK];  // [stage][K, V]

  // (32-bit: every workgroup has at least 128 bytes of q to itself)
  const uint32_t nqb = gridDim.x;
  const uint32_t id = blockIdx.x + nqb * (blockIdx.y + (uint32_t)H * blockIdx.z);
  uint32_t pair = id, qi = 0;
  if (nqb > 1) {
    const uint32_t xcd = id % 8, pairs = (uint32_t)H * b, own = pairs / 8, rest = pairs % 8;
    const uint32_t shared = (nqb * rest + 7 - xcd) / 8;  // of the pairs % 8 last pairs
    uint32_t i = id / 8;
    if (i < shared) {
      const uint32_t t = 8 * i + xcd;
      qi = t / rest;
      pair = 8 * own + (t - qi * rest);
    } else {
      i -= shared;
      const uint32_t group = nqb <= 6 && own > kPGroup ? kPGroupSmall : kPGroup;
      const uint32_t first = i / (group * nqb) * group, n = min(group, own - first);
      i -= first * nqb;
      qi = i / n;
      pair = xcd * own + first + (i - qi * n);
    }
  }
  const int qb = (int)(nqb - 1 - qi);  // most key blocks first
  const int bi = (int)(pair / (uint32_t)H), h = (int)(pair - (uint32_t)bi * H);
  const int64_t d = (int64_t)H * D, dkv = (int64_t)Hkv * D;
  const int kh = h / (H / Hkv);
  // the wave index in a scalar register, so that everything derived from
  // it (the wave's queries, which blocks it masks) is wave-uniform
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int qw = qb * PQ + wave * 32;        // this wave's first query
  const int nkb = (min(qb * PQ + PQ, P) + PK - 1) / PK;

  // Q^T fragments (B operand): lane (r, g) holds query qw + 16 u + r, dims 32 kk + 8 g ..
  h8 qf[2][KK];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int qp = qw + 16 * u + r;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      qf[u][kk] = qp < P ? load_h8(q + ((int64_t)bi * P + qp) * d + (int64_t)h * D + 32 * kk + 8 * g)
                         : zero_h8();
  }

  // DMA of key block kb into buffer buf: LDS byte p of a block holds row
  // p / ROWB, chunk slot (p % ROWB) / 16, i.e. cache chunk kv_swz(row, slot).
  // The block's first row is a wave-uniform address and a lane's offsets
  // from it do not depend on the block (32-bit: the host checks that a
  // block of rows spans less than 2^31 elements), so they are computed
  // once; only a block that reaches past P clamps its rows.
  const int row_elems = b * (int)dkv;  // elements between positions
  const uint16_t* kbase = kc + (int64_t)bi * dkv + (int64_t)kh * D;
  const uint16_t* vbase = vc + (int64_t)bi * dkv + (int64_t)kh * D;
  int doff[DMA];
#pragma unroll
  for (int i = 0; i < DMA; ++i) {
    const int p = (wave * DMA + i) * 1024 + lane * 16;
    doff[i] = (p / ROWB) * row_elems + 8 * kv_swz<D>(p / ROWB, (p % ROWB) / 16);
  }
  const auto issue = [&](int kb, int buf) {
    const int k0 = kb * PK;
    const uint16_t* kblk = kbase + (int64_t)k0 * row_elems;
    const uint16_t* vblk = vbase + (int64_t)k0 * row_elems;
    const bool clamp = k0 + PK > P;
#pragma unroll
    for (int i = 0; i < DMA; ++i) {
      int off = doff[i];
      if (clamp) {
        const int p = (wave * DMA + i) * 1024 + lane * 16, row = p / ROWB;
        off += (min(k0 + row, P - 1) - (k0 + row)) * row_elems;
      }
      lds_dma16(kblk + off, &kv[buf][0][(wave * DMA + i) * 1024]);
      lds_dma16(vblk + off, &kv[buf][1][(wave * DMA + i) * 1024]);
    }
  };

  f4 oacc[2][NF];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int n = 0; n < NF; ++n) oacc[u][n] = f4{0.f, 0.f, 0.f, 0.f};
  float mrow[2] = {-INFINITY, -INFINITY}, lrow[2] = {0.f, 0.f};

#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i < nkb) issue(i, i);
  for (int kb = 0; kb < nkb; ++kb) {
    const int buf = kb % NS;
    // block kb landed (blocks kb + 1 .. kb + NS - 1 may still be in flight)
    wait_blocks_landed<NS, DMA>(min(NS - 1, nkb - 1 - kb));
    wg_barrier();
    const int k0 = kb * PK;
    if (k0 <= qw + 31) {  // some key of the block is visible to this wave
      const uint8_t* Kl = kv[buf][0];
      const uint8_t* Vl = kv[buf][1];
      // S^T: s[u][j][e] = score of key k0 + 16 j + 4 g + e for query qw + 16 u + r
      f4 s[2][PK / 16];
#pragma unroll
      for (int j = 0; j < PK / 16; ++j) {
        s[0][j] = f4{0.f, 0.f, 0.f, 0.f};
        s[1][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const int row = 16 * j + r;
          const h8 kf = *reinterpret_cast<const h8*>(Kl + row * ROWB + 16 * kv_swz<D>(row, 4 * kk + g));
          s[0][j] = mfma16(kf, qf[0][kk], s[0][j]);
          s[1][j] = mfma16(kf, qf[1][kk], s[1][j]);
        }
      }
      // the block needs masking (a wave-uniform test)
      const bool edge = k0 + PK - 1 > qw || k0 + PK > P;
      if (edge) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int qp = qw + 16 * u + r;
#pragma unroll
          for (int j = 0; j < PK / 16; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int key = k0 + 16 * j + 4 * g + e;
              s[u][j][e] = key > qp || key >= P ? -INFINITY : s[u][j][e];
            }
        }
      }
      h8 pf[2][PK / 32];  // P^T fragments (B operand) per sub-block and 32 keys
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float bm = -INFINITY;
#pragma unroll
        for (int j = 0; j < PK / 16; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) bm = fmaxf(bm, s[u][j][e]);
        bm = pair_max(__builtin_amdgcn_permlane16_swap(__float_as_uint(bm), __float_as_uint(bm), false, false));
        bm = pair_max(__builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false));
        const float mnew = fmaxf(mrow[u], bm);
        // every query row has a visible key in its first block, so mnew is finite
        const float alpha = exp2f((mrow[u] - mnew) * kLog2e);
        const float mb = mnew * kLog2e;
        mrow[u] = mnew;
        float rs = 0.f;
#pragma unroll
        for (int j = 0; j < PK / 16; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // v_exp_f32 without denormal scaling: p below 2^-126 becomes 0
            const float p = __builtin_amdgcn_exp2f(s[u][j][e] * kLog2e - mb);
            s[u][j][e] = p;
            rs += p;
          }
        rs = pair_sum(__builtin_amdgcn_permlane16_swap(__float_as_uint(rs), __float_as_uint(rs), false, false));
        rs = pair_sum(__builtin_amdgcn_permlane32_swap(__float_as_uint(rs), __float_as_uint(rs), false, false));
        lrow[u] = lrow[u] * alpha + rs;
        // after the first blocks the running maxima rarely grow: rescale
        // only when some lane's did (alpha is exactly 1 otherwise)
        if (__any(alpha != 1.f)) {
#pragma unroll
          for (int n = 0; n < NF; ++n) oacc[u][n] *= alpha;
        }
#pragma unroll
        for (int hk = 0; hk < PK / 32; ++hk)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            pf[u][hk][e] = (_Float16)s[u][2 * hk][e];
            pf[u][hk][4 + e] = (_Float16)s[u][2 * hk + 1][e];
          }
      }
      // O^T += V^T P^T over the runs of 32 keys: lane (r, g) needs V rows
      // 32 hk + 4 g + (0..3) and 32 hk + 16 + 4 g + (0..3), dim 16 n + r;
      // lane i' of its group addresses row base + i' / 4, dims 16 n + 4 (i' % 4)
#pragma unroll
      for (int hk = 0; hk < PK / 32; ++hk)
#pragma unroll
        for (int n = 0; n < NF; ++n) {
          h8 vf;
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int row = 32 * hk + 16 * half + 4 * g + (r >> 2);
            const int dim = 16 * n + 4 * (r & 3);
            const h4 t = lds_read_tr16(Vl + row * ROWB + 16 * kv_swz<D>(row, dim / 8) + 2 * (dim % 8));
#pragma unroll
            for (int e = 0; e < 4; ++e) vf[4 * half + e] = t[e];
          }
          oacc[0][n] = mfma16(vf, pf[0][hk], oacc[0][n]);
          oacc[1][n] = mfma16(vf, pf[1][hk], oacc[1][n]);
        }
    }
    // every wave is done with this buffer
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
    wg_barrier();
    if (kb + NS < nkb) issue(kb + NS, buf);
  }

  // oacc[u][n][e]: dim 16 n + 4 g + e of query qw + 16 u + r
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int qp = qw + 16 * u + r;
    if (qp >= P) continue;
    const float inv = 1.f / lrow[u];
    uint16_t* orow = o + ((int64_t)bi * P + qp) * d + (int64_t)h * D;
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      u32x2 w;
      w[0] = (uint32_t)f2h(oacc[u][n][0] * inv) | ((uint32_t)f2h(oacc[u][n][1] * inv) << 16);
      w[1] = (uint32_t)f2h(oacc[u][n][2] * inv) | ((uint32_t)f2h(oacc[u][n][3] * inv) << 16);
      *reinterpret_cast<u32x2*>(orow + 16 * n + 4 * g) = w;
    }
  }
}

// ---------------------------------------------------------------------------
int attn_decode_heads_per_wg(int b, int n_heads, int n_kv_heads, bool kv4) {
  if (n_heads != n_kv_heads) return 1;
  int hp = n_heads % 4 == 0 ? 4 : (n_heads % 2 == 0 ? 2 : 1);
  // fp16 rows are bound by HBM: fewer heads per workgroup while that leaves
  // fewer than kAttnDecodeWideWGs workgroups (six per CU keep more loads in
  // flight than a longer key loop per wave).  INT4 rows are bound by the
  // expansion arithmetic, which the wide rows amortise better.
  if (!kv4)
    while (hp > 1 && (int64_t)b * (n_heads / hp) < kAttnDecodeWideWGs) hp /= 2;
  return hp;
}

int attn_decode_splits(int b, int n_heads, int n_kv_heads, int t, bool kv4) {
  // at least kAttnDecodeMinWGs workgroups (three per CU: fewer leave HBM
  // idle, more only add merge traffic), at least 64 keys per split
  const int T = t + 1;
  if (n_heads != n_kv_heads) {
    // grouped: a workgroup's eight waves already share its keys, so splits
    // only where they fill the chip and keep 512 keys each, up to 8 (2048 each
    // beyond: merging more costs more than it gains; b 1, 8000 keys: 14.8 us
    // with 8, 15.9 with 16).  Between one workgroup per CU and one and a half the
    // unsplit grid gives a few CUs two and leaves the others waiting for
    // them: four splits (32/8 heads, us: b 33, 2048 keys 63 -> 55, 8000 keys
    // 240 -> 187, b 48, 8000 keys 276 -> 248; but b 56, 448 workgroups, 2048
    // keys 80.0 -> 81.4, and b 33, 544 keys, too few for a range, 19 -> 25).
    // With ranges of 2000 keys they pay up to two and a half (b 64 342 -> 332,
    // heads of 64 193 -> 180; b 80 430 -> 414; b 90 456 -> 482).
    const int64_t wgs = (int64_t)b * n_kv_heads;
    const bool even = wgs > kAttnGqaWGs && 2 * wgs <= (T >= 8000 ? 5 : 3) * kAttnGqaWGs;
    const int fill = even ? 4 : (int)std::max<int64_t>(1, kAttnGqaWGs / wgs);
    const int keys = std::max(std::min(T / 512, 8), std::min(T / 2048, kAttnDecodeMaxSplits));
    const int S = std::max(1, std::min(fill, keys));
    const int chunk = (T + S - 1) / S;
    return (T + chunk - 1) / chunk;
  }
  const int wgs = b * (n_kv_heads / attn_decode_heads_per_wg(b, n_heads, n_kv_heads, kv4));
  int S = (kAttnDecodeMinWGs + wgs - 1) / wgs;
  S = std::min(S, std::max(1, T / 64));
  S = std::min(S, kAttnDecodeMaxSplits);
  const int chunk = (T + S - 1) / S;
  return (T + chunk - 1) / chunk;
}

int64_t attn_decode_workspace_bytes(int b, int n_heads, int head_dim, int splits) {
  return splits > 1 ? (int64_t)b * n_heads * splits * (head_dim + 2) * 4 : 0;
}

template <int D>
static void launch_decode_combine(const float* workspace, uint16_t* o, int b, int H, int S,
                                  hipStream_t st) {
  if (S > 1)
    launch(attn_decode_combine<D>, dim3((unsigned)H, (unsigned)b), dim3(D), 0, st, workspace, o, H,
           S);
}

template <int D, int HP>
static void launch_decode_mha(const uint16_t* q, const void* kc, const void* vc, uint16_t* o,
                              int b, int H, int t, bool kv4, int S, int chunk, float* workspace,
                              hipStream_t st) {
  const dim3 grid((unsigned)(H / HP), (unsigned)b, (unsigned)S);
  // INT4: the pairs in one dimension, with rows of 2^22 workgroups beyond that (a
  // launch takes under 2^32 threads in a dimension)
  const int64_t pairs = ((int64_t)(H / HP) * b + 7) / 8 * 8;
  const int64_t row = std::min(pairs, (int64_t)1 << 22);
  const dim3 grid4((unsigned)row, (unsigned)S, (unsigned)((pairs + row - 1) / row));
  if (kv4)
    launch(attn_decode_kv4_k<D, HP>, grid4, dim3(256), 0, st, q, kc, vc, o, workspace, b, H, t,
           chunk);
  else
    launch(attn_decode_k<D, HP>, grid, dim3(256), 0, st, q, static_cast<const uint16_t*>(kc),
           static_cast<const uint16_t*>(vc), o, workspace, b, H, t, chunk);
}

template <int D>
static void launch_decode_d(const uint16_t* q, const void* kc, const void* vc, uint16_t* o, int b,
                            int Hkv, int G, int HP, int t, bool kv4, int S, int chunk,
                            float* workspace, hipStream_t st) {
  if (G > 1)
    launch_decode_gqa(q, kc, vc, o, b, Hkv, G, D, t, kv4, S, chunk, workspace, st);
  else if (HP == 4)
    launch_decode_mha<D, 4>(q, kc, vc, o, b, Hkv, t, kv4, S, chunk, workspace, st);
  else if (HP == 2)
    launch_decode_mha<D, 2>(q, kc, vc, o, b, Hkv, t, kv4, S, chunk, workspace, st);
  else
    launch_decode_mha<D, 1>(q, kc, vc, o, b, Hkv, t, kv4, S, chunk, workspace, st);
  launch_decode_combine<D>(workspace, o, b, Hkv * G, S, st);
}

static pipo_status check_heads(const char* what, int n_heads, int n_kv_heads, int head_dim) {
  if (head_dim != 64 && head_dim != 128) {
    set_error("%s: head_dim %d not supported (64 or 128)", what, head_dim);
    return PIPO_ERR_UNSUPPORTED;
  }
  if (n_kv_heads < 1 || n_heads % n_kv_heads != 0) {
    set_error("%s: %d query heads are not a multiple of %d key/value heads", what, n_heads,
              n_kv_heads);
    return PIPO_ERR_ARG;
  }
  const int G = n_heads / n_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8) {
    set_error("%s: %d query heads per key/value head not supported (1, 2, 4, 8)", what, G);
    return PIPO_ERR_UNSUPPORTED;
  }
  return PIPO_OK;
}

pipo_status launch_attn_decode(const uint16_t* q, const void* kc, const void* vc, uint16_t* o,
                               int b, int n_heads, int n_kv_heads, int head_dim, int t, bool kv4,
                               float* workspace, int64_t workspace_bytes, hipStream_t st) {
  if (b < 1 || n_heads < 1 || t < 0) {
    set_error("attn_decode: bad shape b=%d heads=%d t=%d", b, n_heads, t);
    return PIPO_ERR_ARG;
  }
  if (t >= kAttnDecodeMaxT) {
    set_error("attn_decode: %d keys, above the %d this kernel takes", t + 1, kAttnDecodeMaxT);
    return PIPO_ERR_UNSUPPORTED;
  }
  PIPO_TRY(check_heads("attn_decode", n_heads, n_kv_heads, head_dim));
  if (kv4 && ((int64_t)n_kv_heads * head_dim) % 256 != 0) {
    set_error("attn_decode: INT4 KV rows need a width %% 256 == 0 (%d)", n_kv_heads * head_dim);
    return PIPO_ERR_UNSUPPORTED;
  }
  const int G = n_heads / n_kv_heads;
  const int HP = attn_decode_heads_per_wg(b, n_heads, n_kv_heads, kv4);
  const int T = t + 1;
  int S = attn_decode_splits(b, n_heads, n_kv_heads, t, kv4);
  if (!workspace || workspace_bytes < attn_decode_workspace_bytes(b, n_heads, head_dim, S)) S = 1;
  const int chunk = (T + S - 1) / S;
  S = (T + chunk - 1) / chunk;
  (head_dim == 128 ? launch_decode_d<128> : launch_decode_d<64>)(
      q, kc, vc, o, b, n_kv_heads, G, HP, t, kv4, S, chunk, workspace, st);
  PIPO_HIP_TRY(hipGetLastError());
  return PIPO_OK;
}

pipo_status launch_attn_prefill(const uint16_t* q, const uint16_t* kc, const uint16_t* vc,
                                uint16_t* o, int b, int P, int n_heads, int n_kv_heads,
                                int head_dim, hipStream_t st) {
  if (b < 1 || n_heads < 1 || P < 1) {
    set_error("attn_prefill: bad shape b=%d P=%d heads=%d", b, P, n_heads);
    return PIPO_ERR_ARG;
  }
  PIPO_TRY(check_heads("attn_prefill", n_heads, n_kv_heads, head_dim));
  if ((int64_t)b * n_kv_heads * head_dim * kPK >= ((int64_t)1 << 31)) {
    set_error("attn_prefill: %d sequences of %d key/value heads of %d: a key block spans 2^31 "
              "elements or more", b, n_kv_heads, head_dim);
    return PIPO_ERR_UNSUPPORTED;
  }
  const dim3 grid((unsigned)((P + kPQ - 1) / kPQ), (unsigned)n_heads, (unsigned)b);
  const auto go = [&](auto kernel, int threads) {
    launch(kernel, grid, dim3(threads), 0, st, q, kc, vc, o, b, P, n_heads, n_kv_heads);
  };
  if (P <= kPShort) {
    if (head_dim == 128) go(attn_prefill_k<128, 1, kPShort, 2>, 128);
    else go(attn_prefill_k<64, 1, kPShort, 2>, 128);
  } else {
    if (head_dim == 128) go(attn_prefill_k<128, kPrefillStages, kPK, 4>, 256);
    else go(attn_prefill_k<64, kPrefillStages, kPK, 4>, 256);
  }
  PIPO_HIP_TRY(hipGetLastError());
  return PIPO_OK;
}

}  // namespace pipo

// ---------------------------------------------------------------------------
// Decode attention for callers that cannot allocate (pipo_ops.h,
// pipo_op_attn_decode_noalloc): the split partials go to a fixed device
// array instead of a caller workspace.  In host code `scratch` names a
// host-side stand-in, so the array's device address is taken once per
// device with hipGetSymbolAddress and only that address is used.
namespace {

constexpr int64_t kScratchBytes = 4 << 20;
__device__ __align__(256) char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

pipo_status scratch_address(void** out) {
  int dev = 0;
  PIPO_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    pipo::set_error("attn_decode_noalloc: device %d beyond %d", dev, kMaxDevices);
    return PIPO_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      pipo::set_error("attn_decode_noalloc: hipGetSymbolAddress failed (%s)",
                      hipGetErrorString(e));
      return PIPO_ERR_HIP;
    }
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return PIPO_OK;
}

}  // namespace

extern "C" pipo_status pipo_op_attn_decode_noalloc(const uint16_t* q, const uint16_t* kc,
                                                   const uint16_t* vc, uint16_t* o, int32_t b,
                                                   int32_t n_heads, int32_t head_dim, int32_t t,
                                                   void* stream) {
  pipo::clear_error();
  if (!q || !kc || !vc || !o) {
    pipo::set_error("attn_decode_noalloc: NULL pointer");
    return PIPO_ERR_ARG;
  }
  if (b < 1 || n_heads < 1 || t < 0 || head_dim < 1) {
    pipo::set_error("attn_decode_noalloc: bad shape b=%d heads=%d t=%d", b, n_heads, t);
    return PIPO_ERR_ARG;
  }
  const int64_t need = pipo::attn_decode_workspace_bytes(
      b, n_heads, head_dim, pipo::attn_decode_splits(b, n_heads, n_heads, t, false));
  if (need > kScratchBytes) {
    pipo::set_error("attn_decode_noalloc: the split partials need %lld bytes, above the %lld "
                    "bytes of the library's scratch array",
                    (long long)need, (long long)kScratchBytes);
    return PIPO_ERR_UNSUPPORTED;
  }
  void* ws = nullptr;
  if (need > 0) PIPO_TRY(scratch_address(&ws));
  return pipo::launch_attn_decode(q, kc, vc, o, b, n_heads, n_heads, head_dim, t, false,
                                  static_cast<float*>(ws), need,
                                  static_cast<hipStream_t>(stream));
}
