// Grouped-query decode attention on the matrix cores: one new query per
// (sequence, head) against keys 0..t, the G query heads of a key/value head
// as columns of 16 x 16 products.
//
// A workgroup is W waves on one (sequence, key/value head, split) that take
// the split's keys by turns, 32 at a time, through LDS of their own (no
// barrier in the key loop).  fp16 rows come straight from the
// cache by the load unit, INT4 rows through registers, where they are
// expanded; both are laid out as in attn_prefill_k (kv_swz), so the two cache
// formats run the same arithmetic.  The wave computes S^T = K Q^T (keys on
// the rows, heads on the columns, so a lane holds scores of one head), an
// online softmax per head in fp32, and O^T += V^T P^T with V^T read by
// transposed LDS reads in the key order that S^T left P in.  P goes to the
// product in two fp16 parts of y = 2^15 p: hi = fp16(y) and lo = fp16(2^11 (y
// - hi)), each with a sum of its own, put together as hi + 2^-11 lo at the
// end.  That keeps 22 bits of every p down to 2^-29 of the largest one so far
// (20 below its score) and 11, those of the output, down to 2^-40; what it
// drops of smaller ones is under 2^-51 each.  Waves are merged in
// pairs through LDS, splits in order by attn_decode_combine.
//
// Bound by HBM and the fixed cost of a launch.  The kernel it replaced did
// the G dot products and accumulator updates on the vector units, about 150
// instructions for 4 keys, where 32 keys now take about 170; and it needed
// more, smaller workgroups, so more splits to merge.  us with the merge, fp16
// (INT4): b 16, 32/8 heads of 128, 544 keys 18.0 -> 10.4 (19.5 -> 10.5); b 128,
// 64/8 heads 105 -> 50 (5.7 TB/s); b 16, 64/8 heads, 2000 keys 61 -> 28.5 (65 ->
// 26); b 1, 32/8 heads, 8000 keys 30 -> 19.
#include "attention_common.h"

namespace pipo {

constexpr int kGqaKeys = 32;  // keys of a block
constexpr float kPScale = 32768.f, kLoScale = 2048.f;  // of P's two parts
constexpr _Float16 kPMin = 5.9604644775390625e-8f16;    // 2^-24, the smallest fp16

// Eight waves (128 KiB of LDS at head_dim 128, one workgroup per CU) while
// that gives every workgroup a CU, else four, two workgroups per CU, so that
// one's loads run beside the other's products (b 64, 8 key/value heads, 544
// keys: 32.9 us with eight, 30.8 with four; b 16: 9.9 and 11.9).  Above two
// workgroups per CU, one or two waves where there are no more blocks: idle
// waves hold LDS that other workgroups need (b 256, 32/8 heads, 9 keys: 14.8
// us with four, 6.9 with one; 64 keys: 21.7 and 16.3 with two).
constexpr int kGqaWideWGs = kAttnGqaWGs;

// DIRECT: fp16 rows by global -> LDS loads (16-byte aligned cache); INT4 rows
// and others through registers.  Two waves per SIMD are what LDS leaves room for; told
// so, the compiler keeps the sums in plain registers (those of four waves
// went to accumulation registers, with 400 moves between the two).
template <int D, int W, bool KV4, bool DIRECT>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(2))) void attn_decode_gqa_k(
    const uint16_t* __restrict__ q, const void* __restrict__ kc, const void* __restrict__ vc,
    uint16_t* __restrict__ o, float* __restrict__ part, int b, int Hkv, int G, int t, int chunk) {
  constexpr int ROWB = 2 * D, BLK = kGqaKeys * ROWB;  // bytes of a key row, of K (or V) per block
  constexpr int DMA = BLK / 1024, RPD = 1024 / ROWB;  // loads of a block, rows per load
  constexpr int KK = D / 32, NF = D / 16;
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[W * 2 * BLK];
  __shared__ float wm[W][8], wl[W][8];
  const int kh = blockIdx.x, bi = blockIdx.y, sp = blockIdx.z, S = gridDim.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int H = Hkv * G, T = t + 1;
  const int64_t d = (int64_t)H * D, dkv = (int64_t)Hkv * D;
  // the split's keys end at p1, and this wave takes every W-th block of them
  // from p0 on: all workgroups then read the same range of positions at a time
  // (contiguous shares touch W times the pages; b 128, 2048 keys 190 -> 184 us)
  const int p1 = min(T, (sp + 1) * chunk), p0 = sp * chunk + wave * kGqaKeys;
  uint8_t* const kl = lds + wave * (2 * BLK);
  uint8_t* const vl = kl + BLK;

  // Q^T (B operand): lane (r, g) holds head r, dims 32 kk + 8 g ..; the
  // columns past G are zero and never stored
  h8 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qf[kk] = r < G ? load_h8(q + (int64_t)bi * d + (int64_t)(kh * G + r) * D + 32 * kk + 8 * g)
                   : zero_h8();

  const int64_t row_bytes = KV4 ? dkv / 2 + dkv / 16 : 2 * dkv;
  const int64_t pos_bytes = (int64_t)b * row_bytes;  // between positions
  const char* const kbase = static_cast<const char*>(kc) + (int64_t)bi * row_bytes;
  const char* const vbase = static_cast<const char*>(vc) + (int64_t)bi * row_bytes;

  // fp16: the 16 bytes of load i of the block at position p; rows past the
  // split repeat its last
  const int drow = lane / (ROWB / 16);
  const auto source = [&](const char* base, int p, int i) {
    const int row = i * RPD + drow;
    const int c = kv_swz<D>(row, lane % (ROWB / 16));
    return base + (int64_t)min(p + row, p1 - 1) * pos_bytes + (int64_t)kh * ROWB + 16 * c;
  };
  // (read once per step, so non-temporal: b 128, 32/8 heads, 2048 keys 184 ->
  // 170 us, 6.3 TB/s)
  const auto issue = [&](const char* base, uint8_t* dst, int p) {
#pragma unroll
    for (int i = 0; i < DMA; ++i) lds_dma16_w<true>(source(base, p, i), dst + i * 1024);
  };
  // through registers: INT4, 32 elements (one 16-byte word of codes, one
  // pair) per lane and pass, or fp16 as `issue` moves it
  constexpr int LPR = D / 32, PASS = kGqaKeys * LPR / 64;  // lanes per row, passes
  constexpr int WORDS = KV4 ? PASS : DMA;
  struct Block {
    u32x4 c[WORDS];
    uint32_t sm[WORDS];
  };
  const auto load = [&](const char* base, int p) {
    Block x;
#pragma unroll
    for (int i = 0; i < WORDS; ++i) {
      if constexpr (KV4) {
        const int row = i * (64 / LPR) + lane / LPR, e = 32 * (lane % LPR);
        const char* src = base + (int64_t)min(p + row, p1 - 1) * pos_bytes;
        x.c[i] = *reinterpret_cast<const u32x4*>(src + ((int64_t)kh * D + e) / 2);
        x.sm[i] =
            *reinterpret_cast<const uint32_t*>(src + dkv / 2 + ((int64_t)kh * D + e) / 64 * 4);
      } else {
        x.c[i] = load_u32x4_stream(source(base, p, i));
      }
    }
    return x;
  };
  const auto store = [&](const Block& x, uint8_t* dst) {
#pragma unroll
    for (int i = 0; i < WORDS; ++i) {
      if constexpr (KV4) {
        const int row = i * (64 / LPR) + lane / LPR;
        h2 s2, m2;
        scale_min_pairs(x.sm[i], s2, m2);
#pragma unroll
        for (int w = 0; w < 4; ++w)
          *reinterpret_cast<h8*>(dst + row * ROWB + 16 * kv_swz<D>(row, 4 * (lane % LPR) + w)) =
              dequant8_fp8(x.c[i][w], s2, m2);
      } else {
        *reinterpret_cast<u32x4*>(dst + i * 1024 + lane * 16) = x.c[i];
      }
    }
  };

  f4 ohi[NF], olo[NF];
#pragma unroll
  for (int n = 0; n < NF; ++n) ohi[n] = olo[n] = f4{0.f, 0.f, 0.f, 0.f};
  float mrow = -INFINITY, lrow = 0.f;
  Block ck, cv;
  if constexpr (!DIRECT) {
    if (p0 < p1) {
      ck = load(kbase, p0);
      cv = load(vbase, p0);
    }
  }
  for (int p = p0; p < p1; p += W * kGqaKeys) {
    if constexpr (DIRECT) {
      issue(kbase, kl, p);
      issue(vbase, vl, p);
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(DMA, false));  // K landed
    } else {
      store(ck, kl);
      store(cv, vl);
      if (p + W * kGqaKeys < p1) {  // the next block travels beside this block's products
        ck = load(kbase, p + W * kGqaKeys);
        cv = load(vbase, p + W * kGqaKeys);
      }
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
    }
    __builtin_amdgcn_sched_barrier(0);
    // s[j][e]: score of key p + 16 j + 4 g + e for head r
    f4 s[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      s[j] = f4{0.f, 0.f, 0.f, 0.f};
      const int row = 16 * j + r;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        s[j] = mfma16(*reinterpret_cast<const h8*>(kl + row * ROWB + 16 * kv_swz<D>(row, 4 * kk + g)),
                      qf[kk], s[j]);
    }
    if (p + kGqaKeys > p1) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (p + 16 * j + 4 * g + e >= p1) s[j][e] = -INFINITY;
    }
    float bm = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                     fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    bm = pair_max(__builtin_amdgcn_permlane16_swap(__float_as_uint(bm), __float_as_uint(bm), false, false));
    bm = pair_max(__builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false));
    const float mnew = fmaxf(mrow, bm);  // finite: every block has a key
    const float alpha = __builtin_amdgcn_exp2f((mrow - mnew) * kLog2e);
    mrow = mnew;
    float rs = 0.f;
    h8 hi, lo;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = __builtin_amdgcn_exp2f((s[j][e] - mnew) * kLog2e);
        rs += x;
        s[j][e] = x;
        // (fused, so that it is one instruction with the rounding)
        hi[4 * j + e] = (_Float16)__builtin_fmaf(x, kPScale, 0.f);
      }
    // never zero (lo takes it off again), so that an infinity in V comes out as
    // one: under keys past the split, which repeat its last, and tiny p
    hi = __builtin_elementwise_max(hi, h8(kPMin));
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        lo[4 * j + e] = (_Float16)__builtin_fmaf(s[j][e], kPScale * kLoScale,
                                                 (float)hi[4 * j + e] * -kLoScale);
    rs = pair_sum(__builtin_amdgcn_permlane16_swap(__float_as_uint(rs), __float_as_uint(rs), false, false));
    rs = pair_sum(__builtin_amdgcn_permlane32_swap(__float_as_uint(rs), __float_as_uint(rs), false, false));
    lrow = lrow * alpha + rs;
    if (__any(alpha != 1.f)) {  // the running maxima rarely grow after the first blocks
#pragma unroll
      for (int n = 0; n < NF; ++n) {
        ohi[n] *= alpha;
        olo[n] *= alpha;
      }
    }
    if constexpr (DIRECT) __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));  // V landed
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      h8 vf;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int row = 16 * half + 4 * g + (r >> 2), dim = 16 * n + 4 * (r & 3);
        const h4 x = lds_read_tr16(vl + row * ROWB + 16 * kv_swz<D>(row, dim / 8) + 2 * (dim % 8));
#pragma unroll
        for (int e = 0; e < 4; ++e) vf[4 * half + e] = x[e];
      }
      ohi[n] = mfma16(vf, hi, ohi[n]);
      olo[n] = mfma16(vf, lo, olo[n]);
    }
    // this block's LDS is read
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
    __builtin_amdgcn_sched_barrier(0);
  }

  // merge the waves: element e of ohi[n] and olo[n] is dim 16 n + 4 g + e of
  // head r.  An infinity in V may make the low parts' sum NaN (some are zero
  // or negative); the high parts' sum is the result then.
  float* const wacc = reinterpret_cast<float*>(lds + wave * (2 * BLK));  // [G][D]
  if (r < G) {
    if (g == 0) {
      wm[wave][r] = mrow;
      wl[wave][r] = lrow;
    }
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      f4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float sum = __builtin_fmaf(olo[n][e], 1.f / kLoScale, ohi[n][e]);
        v[e] = sum == sum ? sum : ohi[n][e];
      }
      *reinterpret_cast<f4*>(wacc + r * D + 16 * n + 4 * g) = v;
    }
  }
  __syncthreads();
  for (int c = tid; c < G * D; c += W * 64) {
    const int j = c / D, cc = c % D, h = kh * G + j;
    float M = wm[0][j];
#pragma unroll
    for (int w = 1; w < W; ++w) M = fmaxf(M, wm[w][j]);
    float l[W], acc[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {  // a wave may have no key (its maximum -inf)
      const float a = __builtin_amdgcn_exp2f((wm[w][j] - M) * kLog2e);
      l[w] = wl[w][j] * a;
      acc[w] = reinterpret_cast<const float*>(lds + w * (2 * BLK))[c] * a;
    }
#pragma unroll
    for (int n = W / 2; n >= 1; n /= 2)  // in pairs: log2(W) roundings of a sum
#pragma unroll
      for (int w = 0; w < n; ++w) {
        l[w] += l[w + n];
        acc[w] += acc[w + n];
      }
    const float L = l[0];
    float A = acc[0];
    A *= 1.f / kPScale;
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

template <int D, bool KV4, bool DIRECT>
static void launch_gqa_d(const uint16_t* q, const void* kc, const void* vc, uint16_t* o, int b,
                         int Hkv, int G, int t, int S, int chunk, float* part, hipStream_t st) {
  const dim3 grid((unsigned)Hkv, (unsigned)b, (unsigned)S);
  const int64_t wgs = (int64_t)b * Hkv * S;
  const auto go = [&](auto kernel, int waves) {
    launch(kernel, grid, dim3(waves * 64), 0, st, q, kc, vc, o, part, b, Hkv, G, t, chunk);
  };
  if (wgs <= kGqaWideWGs)
    go(attn_decode_gqa_k<D, 8, KV4, DIRECT>, 8);
  else if (wgs > 2 * kGqaWideWGs && chunk <= kGqaKeys)
    go(attn_decode_gqa_k<D, 1, KV4, DIRECT>, 1);
  else if (wgs > 2 * kGqaWideWGs && chunk <= 2 * kGqaKeys)
    go(attn_decode_gqa_k<D, 2, KV4, DIRECT>, 2);
  else
    go(attn_decode_gqa_k<D, 4, KV4, DIRECT>, 4);
}

void launch_decode_gqa(const uint16_t* q, const void* kc, const void* vc, uint16_t* o, int b,
                       int Hkv, int G, int head_dim, int t, bool kv4, int S, int chunk,
                       float* part, hipStream_t st) {
  const bool direct = (reinterpret_cast<uintptr_t>(kc) | reinterpret_cast<uintptr_t>(vc)) % 16 == 0;
  const auto go = [&](auto kernel) { kernel(q, kc, vc, o, b, Hkv, G, t, S, chunk, part, st); };
  if (head_dim == 128)
    go(kv4 ? launch_gqa_d<128, true, false>
           : (direct ? launch_gqa_d<128, false, true> : launch_gqa_d<128, false, false>));
  else
    go(kv4 ? launch_gqa_d<64, true, false>
           : (direct ? launch_gqa_d<64, false, true> : launch_gqa_d<64, false, false>));
}

}  // namespace pipo
