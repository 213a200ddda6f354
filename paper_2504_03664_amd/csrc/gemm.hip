// Projection GEMMs of the decoder layer and the output head:
//   Y[M][N] = X[M][K] . W[N][K]^T  (+ bias, fused epilogue)
// with W in fp16 or group-wise INT4 (codes expanded to fp16 in registers,
// the paper's "compute directly on 4-bit weights", Section 3.4).
//
// The kernel is chosen from the shape (gemm_plan):
//   * gemm_skinny (M <= 16, decode): every workgroup owns 16 or 64 rows of
//     W and all M rows of X; its waves split K; W streams from HBM straight
//     into MFMA operand registers (no LDS), X comes from L2.  Partial sums
//     are combined across waves in LDS in a fixed order.
//   * gemm_slab (gemm_slab.h; M <= 128, and prefill with few tiles): X shared
//     through LDS, every W row owned by one wave, all moved by global -> LDS
//     loads several stages ahead; K split over waves, and over workgroups
//     whose fp32 partial sums go to a workspace that gemm_combine adds up in
//     a fixed order.
//   * gemm_stream_w4 (16 < M <= 32, row-major INT4 W with N above 4096 and K from
//     2048 or 4096 on, or of 14336).
//   * gemm_big_f16 / gemm_big_w4 (prefill with 256 x 256 tiles): 8 waves of
//     128 x 64 fed by global -> LDS loads through rings of LDS stages; INT4
//     codes reach LDS the same way and are expanded there, once per tile;
//     fp16 may split K like gemm_slab.
//   * gemm_tiled (prefill with operands that are not 16-byte aligned, and fp16
//     with one to two tiles of 128 x 128 per CU and little K or row-major W):
//     128 x 128 output tiles, K staged through registers into double-buffered
//     LDS in steps of 64, 4 waves of 64 x 64; tiles ordered per XCD so that each
//     XCD's L2 serves a compact block.
// The decode kernels read each weight once per pass and do so with
// non-temporal loads.
// All accumulate in fp32 with v_mfma_f32_16x16x32_f16, and INT4 codes
// become the same fp16 values (code * scale + min, rounded once) in every
// kernel.  The kernel, its configuration and the K ranges depend only on
// (M, N, K), the weight format and layout and the workspace, so a given call
// always sums in the same order; no workgroup reads another workgroup's
// results within a launch.
#include <algorithm>

#include "gemm_common.h"

namespace pipo {

// ---------------------------------------------------------------------------
// skinny GEMM (decode)
//
// Workgroup = KW waves; it owns 16 NF rows of W (NF fragments) and all M
// (<= 16 MF) rows of X.  K is walked in 128-wide steps; wave w takes steps
// w, w + KW, ... UNR at a time so that UNR steps of W are in flight per
// lane.  In a step, lane (r, g) feeds four MFMAs (8 k each) with W row
// 16 f + r and X row 16 mf + r at the same k: fp16 W is read so that load i
// of the 16 lanes of a row covers 64 contiguous bytes (k = 32 i + 8 g), INT4
// codes as 32 consecutive k per lane (k = 32 g + 8 i).  Wave partials are
// added in LDS in wave order, then the epilogue runs.
template <int NF, int MF, int KW, int UNR, bool W4, bool PK>
struct SkinnyStep {
  u32x4 w[NF][4];  // fp16: four 8-half chunks; int4: w[f][0] holds 32 codes
  uint32_t sm[NF];
  h8 x[MF][4];

  __device__ __forceinline__ static int koff(int i, int g) { return W4 ? 32 * g + 8 * i : 32 * i + 8 * g; }

  // nb[f]: the first W row of fragment f
  __device__ __forceinline__ void load(const GemmArgs& a, const int64_t (&nb)[NF], int64_t s,
                                       int r, int g) {
    const int64_t K = a.K;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int64_t n = nb[f] + r;
      const bool ok = n < a.N;
      if constexpr (W4) {
        const int64_t kb = s * 128 + 32 * g;
        w[f][0] = ok ? load_u32x4_stream(a.Wq + w4_byte<PK>(n, kb, K))
                     : u32x4{0, 0, 0, 0};
        sm[f] = ok ? *reinterpret_cast<const uint32_t*>(a.Wsm + w4_sm<PK>(n, kb, K) * 2) : 0u;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          w[f][i] = ok ? load_u32x4_stream(a.W + w16_index<PK>(n, s * 128 + koff(i, g), K))
                       : u32x4{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) {
      const int64_t m = 16 * mf + r;
      const uint16_t* p = a.X + m * K + s * 128;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[mf][i] = m < a.M ? load_h8(p + koff(i, g)) : zero_h8();
    }
  }

  __device__ __forceinline__ void mma(f4 (&acc)[NF][MF]) const {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      h2 s2, m2;
      if constexpr (W4) scale_min_pairs(sm[f], s2, m2);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const h8 wv = W4 ? dequant8_fp8(w[f][0][i], s2, m2) : __builtin_bit_cast(h8, w[f][i]);
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) acc[f][mf] = mfma16(wv, x[mf][i], acc[f][mf]);
      }
    }
  }
};

template <int NF, int MF, int KW, int UNR, bool W4, int EPI, bool PK>
__global__ __launch_bounds__(KW * 64) void gemm_skinny(GemmArgs a) {
  __shared__ f4 red[KW][NF][MF][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  static_assert(EPI != EPI_SWIGLU || NF % 2 == 0, "SwiGLU pairs gate and up fragments");
  const int64_t n0 = (int64_t)blockIdx.x * (16 * NF);
  const int64_t nsteps = a.K / 128;
  // fragment f's first W row: 16 NF consecutive rows, or with EPI_SWIGLU the
  // gate rows h0 .. h0 + 8 NF - 1 and the up rows F + h0 .. (F = N / 2)
  const int64_t h0 = (int64_t)blockIdx.x * (8 * NF);
  int64_t nb[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    if constexpr (EPI == EPI_SWIGLU)
      nb[f] = f < NF / 2 ? h0 + 16 * f : a.N / 2 + h0 + 16 * (f - NF / 2);
    else
      nb[f] = n0 + 16 * f;
  }

  f4 acc[NF][MF];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) acc[f][mf] = f4{0.f, 0.f, 0.f, 0.f};

  for (int64_t s = wave; s < nsteps; s += UNR * KW) {
    SkinnyStep<NF, MF, KW, UNR, W4, PK> st[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (s + u * KW < nsteps) st[u].load(a, nb, s + u * KW, r, g);
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (s + u * KW < nsteps) st[u].mma(acc);
  }

#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) red[wave][f][mf][lane] = acc[f][mf];
  __syncthreads();

  if constexpr (EPI == EPI_SWIGLU) {
    // element (f < NF / 2, mf, lane', j): output column h0 + 16 f + 4 (lane' / 16) + j
    // from the gate sum of fragment f and the up sum of fragment f + NF / 2,
    // each rounded to fp16 as a separate GEMM output would be
    constexpr int kElems = NF / 2 * MF * 64 * 4;
    const int64_t F = a.N / 2;
    for (int e = threadIdx.x; e < kElems; e += KW * 64) {
      const int j = e & 3, ln = (e >> 2) & 63, fm = e >> 8;
      const int f = fm / MF, mf = fm % MF;
      float gs = 0.f, us = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) {
        gs += red[w][f][mf][ln][j];
        us += red[w][f + NF / 2][mf][ln][j];
      }
      const int64_t m = 16 * mf + (ln & 15), i = h0 + 16 * f + 4 * (ln >> 4) + j;
      if (m < a.M && i < F) {
        const float gv = h2f(f2h(gs + 0.f)), uv = h2f(f2h(us + 0.f));
        a.out16[m * a.ldo + i] = f2h(gv / (1.f + expf(-gv)) * uv);
      }
    }
  } else {
    // element (f, mf, lane', j): W row n0 + 16 f + 4 (lane' / 16) + j, X row 16 mf + lane' % 16
    constexpr int kElems = NF * MF * 64 * 4;
    for (int e = threadIdx.x; e < kElems; e += KW * 64) {
      const int j = e & 3, ln = (e >> 2) & 63, fm = e >> 8;
      const int f = fm / MF, mf = fm % MF;
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) sum += red[w][f][mf][ln][j];
      epilogue<EPI>(a, 16 * mf + (ln & 15), n0 + 16 * f + 4 * (ln >> 4) + j, sum);
    }
  }
}

// ---------------------------------------------------------------------------
// streaming GEMM (row-major INT4 W, 16 < M <= 32)
//
// Workgroup = 8 waves: KS = 1, wave w owns W rows n0 + 16 w .. + 15; KS = 2, the
// waves w and w + 4 share rows n0 + 16 w .. + 15, one for each half of a
// chunk.  The workgroup covers k in [z kper, (z + 1) kper), z = blockIdx.y.  K
// is walked in chunks of KC: the X chunk (32 rows x KC) is loaded once per
// workgroup, PD chunks ahead into registers and then into one of two LDS
// buffers, one barrier per chunk; each wave holds PD chunks of its W rows in
// registers, refilling a chunk's registers as soon as its MFMAs are issued.
// Every load is unconditional (row and chunk indexes are clamped: rows past M
// or N are computed and never stored, a clamped chunk is loaded again and not
// used), which keeps the compiler's wait counts exact so that the prefetch
// really stays in flight.  Lane (r, g) reads 32 consecutive codes of 128 (64 or
// 128 bytes of a row at a time, where the slab kernel reads 32), then the lanes
// of a row exchange them (two swaps a word) so that each has 16 consecutive
// codes of each 64, as a slab lane does, and every fourth 64 go to a sum of
// their own: the products and sums of the slab kernel in its order, so W in
// either layout gives the same bits.  us at M = 32, with its register-staged
// predecessor of one sum / the slab kernel / now: 16384 x 4096 22.0 / 20.5 / 18.2,
// 21504 x 7168 46.9 / 59 / 45.9, 7168 x 28672 51 / 62 / 52.
constexpr int kStreamWaves = 8;

__device__ __forceinline__ int64_t clamp_hi(int64_t v, int64_t hi) { return v < hi ? v : hi; }

template <int PD, int KC, int KS, int EPI>
__global__ __launch_bounds__(kStreamWaves * 64) void gemm_stream_w4(GemmArgs a, float* part,
                                                                    int64_t kper) {
  constexpr int MF = 2, KW = kStreamWaves / KS, kThreads = kStreamWaves * 64;
  constexpr int T = KC / 128 / KS;  // runs of 128 k of a chunk that a wave takes
  constexpr int kSums = 4 / KS;     // of a wave
  static_assert(T >= 1 && (T * 2 >= kSums || PD % 2 == 0), "a run's sums are known");
  constexpr int kXLd = KC + 8;  // halves per LDS row (padding against bank conflicts)
  constexpr int kXPerThread = 16 * MF * KC / 8 / kThreads;  // 8-half pieces of an X chunk
  static_assert(kXPerThread * kThreads * 8 == 16 * MF * KC, "X pieces split evenly");
  __shared__ __attribute__((aligned(16))) uint16_t Xs[2][16 * MF * kXLd];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = KS == 1 ? 0 : wave / KW, kw = wave - ks * KW;
  const int r = lane & 15, g = lane >> 4;
  const int64_t nw0 = ((int64_t)blockIdx.x * KW + kw) * 16;
  const int64_t kbeg = (int64_t)blockIdx.y * kper;
  const int64_t nch = kper / KC;
  const int64_t K = a.K;
  const int64_t wrow = clamp_hi(nw0 + r, a.N - 1);

  struct WChunk {
    u32x4 w[T];
    u32x2 sm[T];  // (scale, min) of both 64
  };
  const auto load_w = [&](WChunk& F, int64_t c) {
    const int64_t k0 = kbeg + clamp_hi(c, nch - 1) * KC + 128 * T * ks;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      F.w[t] = load_u32x4_stream(a.Wq + w4_byte<false>(wrow, k0 + 128 * t + 32 * g, K));
      F.sm[t] = *reinterpret_cast<const u32x2*>(a.Wsm + w4_sm<false>(wrow, k0 + 128 * t, K) * 2);
    }
  };
  // X chunks travel through registers PD chunks ahead of their use, like W:
  // chunk c sits in ring slot c % PD from its load (iteration c - 1 - PD)
  // until it is stored to LDS (end of iteration c - 1)
  h8 xr[PD][kXPerThread];
  const auto load_x = [&](int slot, int64_t c) {
    const int64_t k0 = kbeg + clamp_hi(c, nch - 1) * KC;
#pragma unroll
    for (int j = 0; j < kXPerThread; ++j) {
      const int e = tid + j * kThreads;
      const int row = e / (KC / 8), col = (e % (KC / 8)) * 8;
      xr[slot][j] = load_h8(a.X + clamp_hi(row, a.M - 1) * K + k0 + col);
    }
  };
  const auto store_x = [&](int b, int slot) {
#pragma unroll
    for (int j = 0; j < kXPerThread; ++j) {
      const int e = tid + j * kThreads;
      const int row = e / (KC / 8), col = (e % (KC / 8)) * 8;
      *reinterpret_cast<h8*>(&Xs[b][row * kXLd + col]) = xr[slot][j];
    }
  };
  f4 acc[kSums][MF];
#pragma unroll
  for (int u = 0; u < kSums; ++u)
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) acc[u][mf] = f4{0.f, 0.f, 0.f, 0.f};
  // odd: whether the chunk's number is
  const auto compute = [&](const WChunk& F, int b, int odd) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      // (all reads of the run first: left to the compiler, each waits right
      // before its product, 46 us where it takes 42 so at M = 17, 21504 x 7168)
      h8 xv[4][MF];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
          xv[i][mf] = *reinterpret_cast<const h8*>(
              &Xs[b][(16 * mf + r) * kXLd + 128 * (T * ks + t) + 64 * (i >> 1) + 16 * g + 8 * (i & 1)]);
      uint32_t w[4];  // 64 i / 2, word i % 2
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const auto p = __builtin_amdgcn_permlane16_swap(F.w[t][i], F.w[t][2 + i], false, false);
        const auto q = __builtin_amdgcn_permlane32_swap(p[0], p[1], false, false);
        w[i] = q[0];
        w[2 + i] = q[1];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h2 s2, m2;
        scale_min_pairs(F.sm[t][i >> 1], s2, m2);
        const h8 wv = dequant8_fp8(w[i], s2, m2);
        const int u = (2 * (T * odd + t) + (i >> 1)) % kSums;
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) acc[u][mf] = mfma16(wv, xv[i][mf], acc[u][mf]);
      }
    }
  };

  WChunk F[PD];
  load_x(0, 0);
  store_x(0, 0);
#pragma unroll
  for (int p = 1; p <= PD; ++p) load_x(p % PD, p);
#pragma unroll
  for (int p = 0; p < PD; ++p) {
    load_w(F[p], p);
    __builtin_amdgcn_sched_barrier(0);  // keep the chunks' loads in chunk order
  }
  __syncthreads();
  for (int64_t c0 = 0; c0 < nch; c0 += PD) {
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      const int64_t c = c0 + p;
      if (c < nch) compute(F[p], (int)(c & 1), p & 1);
      load_w(F[p], c + PD);
      __builtin_amdgcn_sched_barrier(0);
      // buffer (c + 1) & 1 was last read in chunk c - 1, before the barrier
      store_x((int)((c + 1) & 1), (p + 1) % PD);
      load_x((p + 1) % PD, c + 1 + PD);
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
    }
  }

  // the sums in order; those of the second halves through LDS
  f4 sum[MF];
#pragma unroll
  for (int mf = 0; mf < MF; ++mf) {
    sum[mf] = acc[0][mf];
    if constexpr (KS == 1) {
#pragma unroll
      for (int u = 1; u < kSums; ++u) sum[mf] += acc[u][mf];
    }
  }
  if constexpr (KS == 2) {
    static_assert(KW * 64 * kSums * MF * 16 <= sizeof(Xs), "the second halves' sums fit");
    f4* red = reinterpret_cast<f4*>(&Xs[0][0]);
    if (ks == 1) {
#pragma unroll
      for (int u = 0; u < kSums; ++u)
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) red[((u * MF + mf) * KW + kw) * 64 + lane] = acc[u][mf];
    }
    __syncthreads();
    if (ks == 1) return;
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) {
      sum[mf] += acc[1][mf];
#pragma unroll
      for (int u = 0; u < kSums; ++u) sum[mf] += red[((u * MF + mf) * KW + kw) * 64 + lane];
    }
  }
  // sum[mf] element j: W row nw0 + 4 g + j, X row 16 mf + r
#pragma unroll
  for (int mf = 0; mf < MF; ++mf)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t m = 16 * mf + r, n = nw0 + 4 * g + j;
      if (gridDim.y == 1) {
        epilogue<EPI>(a, m, n, sum[mf][j]);
      } else if (m < a.M && n < a.N) {
        part[((int64_t)blockIdx.y * a.M + m) * a.N + n] = sum[mf][j];
      }
    }
}

// out = sum over z = 0 .. S-1 (in that order, from 0) of part[z], then the
// epilogue.  A thread takes V adjacent columns of one row (V = 4 when N is a
// multiple of 4 and the partials are 16-byte aligned) and issues the loads
// of all S partials before the first add; M * N < 2^31 (checked by the host).
template <int EPI, int S, int V>
__global__ __launch_bounds__(256) void gemm_combine(GemmArgs a, const float* __restrict__ part) {
  const int NV = (int)(a.N / V);
  const int q = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (q >= (int)a.M * NV) return;
  const int m = q / NV, n = (q - m * NV) * V;
  const int64_t MN = a.M * a.N;
  const float* p = part + (int64_t)m * a.N + n;
  float v[S][V];
#pragma unroll
  for (int z = 0; z < S; ++z) {
    if constexpr (V == 4) {
      const f4 t = *reinterpret_cast<const f4*>(p + z * MN);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[z][j] = t[j];
    } else {
      v[z][0] = p[z * MN];
    }
  }
  const EpiRow row = epilogue_row<EPI>(a, m);
#pragma unroll
  for (int j = 0; j < V; ++j) {
    float sum = 0.f;
#pragma unroll
    for (int z = 0; z < S; ++z) sum += v[z][j];
    epilogue_store<EPI>(a, row, n + j, sum + epilogue_bias(a, n + j));
  }
}

template <int EPI, int V>
static void launch_combine_v(const GemmArgs& a, const float* ws, int S, hipStream_t st) {
  const dim3 grid((unsigned)((a.M * (a.N / V) + 255) / 256));
  switch (S) {
    case 2: launch((gemm_combine<EPI, 2, V>), grid, dim3(256), 0, st, a, ws); break;
    case 4: launch((gemm_combine<EPI, 4, V>), grid, dim3(256), 0, st, a, ws); break;
    default: launch((gemm_combine<EPI, 8, V>), grid, dim3(256), 0, st, a, ws); break;
  }
}

template <int EPI>
static void launch_combine_epi(const GemmArgs& a, const float* ws, int S, hipStream_t st) {
  if (a.N % 4 == 0 && reinterpret_cast<uintptr_t>(ws) % 16 == 0)
    launch_combine_v<EPI, 4>(a, ws, S, st);
  else
    launch_combine_v<EPI, 1>(a, ws, S, st);
}

void launch_combine(const GemmArgs& a, int epi, const float* ws, int S, hipStream_t st) {
  switch (epi) {
    case EPI_F16: return launch_combine_epi<EPI_F16>(a, ws, S, st);
    case EPI_RELU_F16: return launch_combine_epi<EPI_RELU_F16>(a, ws, S, st);
    case EPI_ADD_F32: return launch_combine_epi<EPI_ADD_F32>(a, ws, S, st);
    case EPI_F32: return launch_combine_epi<EPI_F32>(a, ws, S, st);
    default: return launch_combine_epi<EPI_QKV>(a, ws, S, st);
  }
}

// ---------------------------------------------------------------------------
// tiled GEMM (prefill with operands off 16-byte alignment, and fp16 prefill
// with one to two of its tiles per CU: see plan_prefill)
constexpr int kTBM = 128, kTBN = 128, kTBK = 64, kTPad = 8;
constexpr int kTThreads = 256;  // 2 x 2 waves of 64 x 64
constexpr int kTGroupM = 4;

template <bool W4, int EPI, bool PK>
__global__ __launch_bounds__(kTThreads) void gemm_tiled(GemmArgs a) {
  constexpr int LDS_ROW = kTBK + kTPad;  // halves
  __shared__ __attribute__((aligned(16))) uint16_t As[2][kTBM * LDS_ROW];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kTBN * LDS_ROW];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  // Tile order.  Workgroups are dealt to the 8 XCDs round-robin, and each
  // XCD has its own L2: give XCD x a contiguous range of tiles, and walk
  // that range in groups of kTGroupM row tiles (row tile fastest), so that
  // the workgroups an XCD runs at once share A rows and B columns in L2.
  const int64_t tiles_m = (a.M + kTBM - 1) / kTBM, tiles_n = (a.N + kTBN - 1) / kTBN;
  const int64_t total = tiles_m * tiles_n;
  const int64_t per_xcd = (total + kXcds - 1) / kXcds;
  const int64_t tile = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (tile >= total) return;
  const int64_t group = tile / (kTGroupM * tiles_n);
  const int64_t first_m = group * kTGroupM;
  const int64_t gm = tiles_m - first_m < kTGroupM ? tiles_m - first_m : kTGroupM;
  const int64_t in_group = tile - group * kTGroupM * tiles_n;
  const int64_t m0 = (first_m + in_group % gm) * kTBM;
  const int64_t n0 = (in_group / gm) * kTBN;
  const int64_t K = a.K;
  const int64_t KT = K / kTBK;

  // global -> register staging: A and fp16 B take 4 chunks of 8 halves per
  // thread (row = c / 8, col = 8 (c % 8)); INT4 B takes one 32-code chunk.
  // With B in fragment order a wave's 64 chunks are one 16-row x 32-k
  // block (1 KiB contiguous; INT4: 32 threads read a 512-byte half block).
  const auto b_row = [](int c) { return PK ? ((c >> 7) << 4) + (c & 15) : c >> 3; };
  const auto b_col = [](int c) { return PK ? ((c >> 6) & 1) * 32 + ((c >> 4) & 3) * 8 : (c & 7) * 8; };
  const auto b_row_w4 = [](int t, int64_t) { return PK ? ((t >> 5) << 4) + (t & 15) : t >> 1; };
  const auto b_half_w4 = [](int t, int64_t) { return PK ? (t >> 4) & 1 : t & 1; };
  h8 ra[4], rb[4];
  const auto load_tile = [&](int64_t kt) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = tid + i * kTThreads;
      const int row = c >> 3, col = (c & 7) * 8;
      const int64_t m = m0 + row;
      ra[i] = m < a.M ? load_h8(a.X + m * K + kt * kTBK + col) : zero_h8();
    }
    if constexpr (W4) {
      const int row = b_row_w4(tid, kt), half = b_half_w4(tid, kt);
      const int64_t n = n0 + row;
      if (n < a.N) {
        const int64_t kc = kt * kTBK + half * 32;
        const u32x4 codes = *reinterpret_cast<const u32x4*>(a.Wq + w4_byte<PK>(n, kc, K));
        const uint32_t smw = *reinterpret_cast<const uint32_t*>(a.Wsm + w4_sm<PK>(n, kc, K) * 2);
        h2 s2, m2;
        scale_min_pairs(smw, s2, m2);
#pragma unroll
        for (int i = 0; i < 4; ++i) rb[i] = dequant8_fp8(codes[i], s2, m2);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) rb[i] = zero_h8();
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = tid + i * kTThreads;
        const int row = b_row(c), col = b_col(c);
        const int64_t n = n0 + row;
        rb[i] = n < a.N ? load_h8(a.W + w16_index<PK>(n, kt * kTBK + col, K)) : zero_h8();
      }
    }
  };
  const auto store_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = tid + i * kTThreads;
      const int row = c >> 3, col = (c & 7) * 8;
      *reinterpret_cast<h8*>(&As[buf][row * LDS_ROW + col]) = ra[i];
    }
    if constexpr (W4) {
      const int row = b_row_w4(tid, 0), half = b_half_w4(tid, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<h8*>(&Bs[buf][row * LDS_ROW + half * 32 + 8 * i]) = rb[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = tid + i * kTThreads;
        *reinterpret_cast<h8*>(&Bs[buf][b_row(c) * LDS_ROW + b_col(c)]) = rb[i];
      }
    }
  };

  f4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  load_tile(0);
  store_tile(0);
  __syncthreads();
  for (int64_t kt = 0; kt < KT; ++kt) {
    const int buf = (int)(kt & 1);
    if (kt + 1 < KT) load_tile(kt + 1);
#pragma unroll
    for (int ks = 0; ks < kTBK / 32; ++ks) {
      h8 af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        af[i] = *reinterpret_cast<const h8*>(
            &As[buf][(wm * 64 + i * 16 + r) * LDS_ROW + ks * 32 + g * 8]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        bf[j] = *reinterpret_cast<const h8*>(
            &Bs[buf][(wn * 64 + j * 16 + r) * LDS_ROW + ks * 32 + g * 8]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma16(af[i], bf[j], acc[i][j]);
    }
    if (kt + 1 < KT) store_tile(buf ^ 1);
    __syncthreads();
  }

  // acc[i][j] element e: row m0 + 64 wm + 16 i + 4 g + e, col n0 + 64 wn + 16 j + r;
  // biases once per column, row offsets once per row
  float bias[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) bias[j] = epilogue_bias(a, n0 + wn * 64 + j * 16 + r);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const EpiRow row = epilogue_row<EPI>(a, m0 + wm * 64 + i * 16 + 4 * g + e);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        epilogue_store<EPI>(a, row, n0 + wn * 64 + j * 16 + r, acc[i][j][e] + bias[j]);
    }
}

// ---------------------------------------------------------------------------
// big-tile GEMMs (prefill): each W element read into LDS feeds 256 rows of X
// instead of 128, and each LDS operand read feeds more MFMAs.  Same tile
// order as gemm_tiled; the same MFMA per 32-wide k block in the same k order,
// so over one K range every kernel with one K group gives the same bits.
// ---------------------------------------------------------------------------
constexpr int kBM = 256, kBN = 256;

// fp16 W (fragment order, or row-major: PK): 8 waves (two per SIMD) of 128 x 64 (8 x 4
// accumulator fragments), K in stages of 32.  Everything moves from global
// memory straight into LDS by the load unit (global_load_lds_dwordx4: lane
// l of a wave writes bytes 16 l .. 16 l + 15 of its destination).  A W
// stage is 16 row blocks of 16 rows x 32 k = 1 KiB in MFMA operand order
// (lane slot r + 16 g holds row r, k = 8 g .. 8 g + 7), in a ring of four
// stages; fragment reads are one contiguous KiB per wave.  X moves 64 k at
// a time: each load covers 8 rows x 128 bytes, whole cache lines of the
// row-major activations (loads of 16 rows x 64 bytes fetched every line
// twice, once per 32-k stage), into a ring of three 32 KiB slots where row
// r of a 16-row block keeps its 16-byte chunk c at position c ^ ((r / 2) %
// 8), which leaves the fragment reads free of bank conflicts (160 KiB of
// LDS in all).  Stage t is read while the next two are in flight and the
// loads of stage t + 3 (W) and of half a 64-k X stage are issued into
// buffers already read.  Fragment registers are double-buffered: the reads
// of stage t are spread over the MFMAs of stage t - 1.  Rows past M (and
// row blocks past N) are loaded from the last valid row and their results
// dropped.
constexpr int kFThreads = 512;
constexpr int kFStages = 4;              // LDS stages of the INT4 kernel's ring

template <int EPI, bool PK>
__global__ __launch_bounds__(kFThreads) void gemm_big_f16(GemmArgs a, float* part,
                                                          int64_t kper) {
  constexpr int FM = 8, FN = 4;  // fragments per wave
  constexpr int BPW = 2;         // W row blocks each wave moves per stage
  constexpr int PER_STAGE = 2 * BPW;
  constexpr int XSLOT = 32 * 1024, XSLOTS = 3, WSLOT = 16 * 1024, WSLOTS = 4;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[XSLOTS * XSLOT + WSLOTS * WSLOT];
  uint8_t* const xring = lds;
  uint8_t* const wring = lds + XSLOTS * XSLOT;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int64_t tiles_m = (a.M + kBM - 1) / kBM, tiles_n = (a.N + kBN - 1) / kBN;
  const int64_t total = tiles_m * tiles_n;
  const int64_t per_xcd = (total + kXcds - 1) / kXcds;
  const int64_t tile = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (tile >= total) return;
  const int64_t group = tile / (kTGroupM * tiles_n);
  const int64_t first_m = group * kTGroupM;
  const int64_t gm = tiles_m - first_m < kTGroupM ? tiles_m - first_m : kTGroupM;
  const int64_t in_group = tile - group * kTGroupM * tiles_n;
  const int64_t m0 = (first_m + in_group % gm) * kBM;
  const int64_t n0 = (in_group / gm) * kBN;
  const int64_t K = a.K;
  const int64_t kbeg = (int64_t)blockIdx.y * kper;
  const int KT = (int)(kper / 32);
  const int KS = KT / 2;         // 64-wide X stages

  const int r = lane & 15, g = lane >> 4;
  // X: wave w moves row blocks 2w and 2w + 1, half q (rows 8q .. 8q + 7)
  // of a 64-k stage per step; lane l takes row 8q + l / 8 and chunk
  // (l % 8) ^ ((row >> 1) & 7) of the row's 128 bytes
  const uint16_t* xsrc[2][2];
#pragma unroll
  for (int bb = 0; bb < 2; ++bb)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = 8 * q + (lane >> 3);
      const int c = (lane & 7) ^ ((row >> 1) & 7);
      int64_t m = m0 + 16 * (2 * wave + bb) + row;
      m = m < a.M ? m : a.M - 1;
      xsrc[bb][q] = a.X + m * K + kbeg + 8 * c;
    }
  const uint16_t* bsrc[BPW];
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    if constexpr (PK) {
      int64_t nb = (n0 >> 4) + BPW * wave + i;
      nb = nb < (a.N >> 4) ? nb : (a.N >> 4) - 1;
      bsrc[i] = a.W + (nb * (K >> 5) + (kbeg >> 5)) * 512 + lane * 8;
    } else {
      int64_t n = n0 + 16 * (BPW * wave + i) + r;
      n = n < a.N ? n : a.N - 1;
      bsrc[i] = a.W + n * K + kbeg + 8 * g;
    }
  }
  constexpr int kBStep = PK ? 512 : 32;
  // step u issues W stage u + 3 and half u & 1 of X stage (u >> 1) + 2
  // (arithmetic shift: u = -4 .. -1 are the prologue)
  const auto issue = [&](int u) {
    if (u >= -3) {
      const int ws = u + 3 < KT ? u + 3 : KT - 1;
      uint8_t* st = wring + ((u + 3) % WSLOTS) * WSLOT;
#pragma unroll
      for (int i = 0; i < BPW; ++i)
        lds_dma16(bsrc[i] + ws * kBStep, st + (BPW * wave + i) * 1024);
    }
    const int s = (u >> 1) + 2, q = u & 1;
    const int sc = s < KS ? s : KS - 1;
    uint8_t* xs = xring + (s % XSLOTS) * XSLOT;
#pragma unroll
    for (int bb = 0; bb < 2; ++bb)
      lds_dma16(xsrc[bb][q] + sc * 64, xs + (2 * wave + bb) * 2048 + q * 1024);
  };
  const auto read = [&](int t, h8 (&fa)[FM], h8 (&fb)[FN]) {
    const uint8_t* ws = wring + (t % WSLOTS) * WSLOT;
#pragma unroll
    for (int j = 0; j < FN; ++j)
      fb[j] = *reinterpret_cast<const h8*>(ws + (FN * wn + j) * 1024 + lane * 16);
    const uint8_t* xs = xring + ((t >> 1) % XSLOTS) * XSLOT;
    const int c = (g + 4 * (t & 1)) ^ ((r >> 1) & 7);
    const int off = (r >> 3) * 1024 + (r & 7) * 128 + 16 * c;
#pragma unroll
    for (int i = 0; i < FM; ++i)
      fa[i] = *reinterpret_cast<const h8*>(xs + (FM * wm + i) * 2048 + off);
  };
  f4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  const auto mma = [&](const h8 (&fa)[FM], const h8 (&fb)[FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = mfma16(fa[i], fb[j], acc[i][j]);
  };
  h8 fa0[FM], fb0[FN], fa1[FM], fb1[FN];
  const auto step = [&](int t, h8 (&ra)[FM], h8 (&rb)[FN], h8 (&ca)[FM], h8 (&cb)[FN]) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * PER_STAGE, true));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    issue(t);
    read(t, ra, rb);
    mma(ca, cb);
#pragma unroll
    for (int k = 0; k < PER_STAGE; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global -> LDS load
    }
#pragma unroll
    for (int k = 0; k < FM + FN; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
    }
    __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - 2 * PER_STAGE - 2 * (FM + FN), 0);
  };
  issue(-4);  // X stage 0, rows 0-7 of each block (no W)
  issue(-3);
  issue(-2);
  issue(-1);
  // W stage 0 and both halves of X stage 0 landed (steps -2, -1 may be in flight)
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * PER_STAGE, true));
  __builtin_amdgcn_s_barrier();
  issue(0);
  read(0, fa0, fb0);
  int t = 1;
  for (; t < KT - 1; t += 2) {
    step(t, fa1, fb1, fa0, fb0);
    step(t + 1, fa0, fb0, fa1, fb1);
  }
  step(t, fa1, fb1, fa0, fb0);
  // every load landed (none may write LDS after the workgroup ends)
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
  mma(fa1, fb1);

  // acc[i][j] element e: row m0 + 128 wm + 16 i + 4 g + e, col n0 + 64 wn + 16 j + r
  if (gridDim.y > 1) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t m = m0 + wm * 128 + i * 16 + 4 * g + e;
        float* p = part + ((int64_t)blockIdx.y * a.M + m) * a.N;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int64_t n = n0 + wn * 64 + j * 16 + r;
          if (m < a.M && n < a.N) p[n] = acc[i][j][e];
        }
      }
    return;
  }
  float bias[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) bias[j] = epilogue_bias(a, n0 + wn * 64 + j * 16 + r);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const EpiRow row = epilogue_row<EPI>(a, m0 + wm * 128 + i * 16 + 4 * g + e);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        epilogue_store<EPI>(a, row, n0 + wn * 64 + j * 16 + r, acc[i][j][e] + bias[j]);
    }
}

// INT4 W (fragment order or row-major): as gemm_big_f16, with the W area of
// a stage filled by the threads.  The codes (16 bytes per W row and stage)
// and (scale, min) pairs of a stage reach LDS through the load unit one
// stage ahead of X; at step t every thread expands 16 codes of stage t + 1
// (W row tid / 2, k 16 (tid & 1) .. + 15) into two 16-byte fragment slots,
// (through the fp8 converter) so each code is expanded once per 256 rows of X.  A stage is X 16 KiB,
// expanded W 16 KiB, codes 4 KiB, pairs 1 KiB; four stages, 148 KiB.
template <int EPI, bool PK>
__global__ __launch_bounds__(kFThreads) void gemm_big_w4(GemmArgs a) {
  constexpr int FM = 8, FN = 4;
  constexpr int BPW = 2;
  constexpr int PER_STEP = BPW + 1;               // X blocks + one code or pair load
  constexpr int STAGE = 32 * 1024 + 4096 + 1024;  // bytes per LDS stage
  constexpr int WOFF = 16 * 1024, COFF = 32 * 1024, SOFF = 36 * 1024;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kFStages * STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int64_t tiles_m = (a.M + kBM - 1) / kBM, tiles_n = (a.N + kBN - 1) / kBN;
  const int64_t total = tiles_m * tiles_n;
  const int64_t per_xcd = (total + kXcds - 1) / kXcds;
  const int64_t tile = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (tile >= total) return;
  const int64_t group = tile / (kTGroupM * tiles_n);
  const int64_t first_m = group * kTGroupM;
  const int64_t gm = tiles_m - first_m < kTGroupM ? tiles_m - first_m : kTGroupM;
  const int64_t in_group = tile - group * kTGroupM * tiles_n;
  const int64_t m0 = (first_m + in_group % gm) * kBM;
  const int64_t n0 = (in_group / gm) * kBN;
  const int64_t K = a.K;
  const int KT = (int)(K / 32);

  const int r = lane & 15, g = lane >> 4;
  const uint16_t* asrc[BPW];
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    int64_t m = m0 + 16 * (BPW * wave + i) + r;
    m = m < a.M ? m : a.M - 1;
    asrc[i] = a.X + m * K + 8 * g;
  }
  // waves 0-3: the codes of W rows 64 w + lane; waves 4-7: their pairs
  int64_t wn_row = n0 + 64 * (wave & 3) + lane;
  wn_row = wn_row < a.N ? wn_row : a.N - 1;
  const auto issue_x = [&](int src, int buf) {
    uint8_t* st = lds + (buf % kFStages) * STAGE;
#pragma unroll
    for (int i = 0; i < BPW; ++i) lds_dma16(asrc[i] + src * 32, st + (BPW * wave + i) * 1024);
  };
  const auto issue_w = [&](int src, int buf) {
    uint8_t* st = lds + (buf % kFStages) * STAGE;
    if (wave < 4)
      lds_dma16(a.Wq + w4_byte<PK>(wn_row, 32 * src, K), st + COFF + 64 * wave * 16);
    else
      __builtin_amdgcn_global_load_lds(a.Wsm + w4_sm<PK>(wn_row, 32 * src, K) * 2,
                                       (__attribute__((address_space(3))) void*)(st + SOFF + 64 * (wave - 4) * 4),
                                       4, 0, 0);
  };
  // thread: W row tid / 2 of the tile, k 16 (tid & 1) .. + 15 of the stage
  const auto expand = [&](int buf) {
    uint8_t* st = lds + (buf % kFStages) * STAGE;
    const int row = tid >> 1, half = tid & 1;
    const u32x2 c = *reinterpret_cast<const u32x2*>(st + COFF + row * 16 + half * 8);
    const uint32_t sm = *reinterpret_cast<const uint32_t*>(st + SOFF + row * 4);
    h2 s2, m2;
    scale_min_pairs(sm, s2, m2);
    uint8_t* wb = st + WOFF + (row >> 4) * 1024 + ((row & 15) + 32 * half) * 16;
    *reinterpret_cast<h8*>(wb) = dequant8_fp8(c[0], s2, m2);
    *reinterpret_cast<h8*>(wb + 256) = dequant8_fp8(c[1], s2, m2);
  };
  const auto read = [&](int t, h8 (&fa)[FM], h8 (&fb)[FN]) {
    const uint8_t* st = lds + (t % kFStages) * STAGE;
#pragma unroll
    for (int j = 0; j < FN; ++j)
      fb[j] = *reinterpret_cast<const h8*>(st + WOFF + (FN * wn + j) * 1024 + lane * 16);
#pragma unroll
    for (int i = 0; i < FM; ++i)
      fa[i] = *reinterpret_cast<const h8*>(st + (FM * wm + i) * 1024 + lane * 16);
  };
  f4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  const auto mma = [&](const h8 (&fa)[FM], const h8 (&fb)[FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = mfma16(fa[i], fb[j], acc[i][j]);
  };
  const auto clampk = [&](int s) { return s < KT ? s : KT - 1; };
  // step t: codes of stage t + 1 and X of stage t landed; codes of t + 4
  // and X of t + 3 issued; codes of t + 1 expanded; stage t read while the
  // MFMAs of t - 1 run
  h8 fa0[FM], fb0[FN], fa1[FM], fb1[FN];
  const auto step = [&](int t, h8 (&ra)[FM], h8 (&rb)[FN], h8 (&ca)[FM], h8 (&cb)[FN], bool mm) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * PER_STEP, true));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    issue_w(clampk(t + 4), t + 4);
    issue_x(clampk(t + 3), t + 3);
    expand(t + 1);
    read(t, ra, rb);
    if (mm) mma(ca, cb);
    // two MFMAs before the loads, so that the MFMA pipe restarts right
    // after the barrier; then one fragment read and two MFMAs, in turn
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, PER_STEP, 0);
#pragma unroll
    for (int k = 0; k < FM + FN; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - 2 - 2 * (FM + FN), 0);
  };
  issue_w(0, 0);
  issue_w(1, 1);
  issue_x(0, 0);
  issue_w(2, 2);
  issue_x(1, 1);
  issue_w(3, 3);
  issue_x(2, 2);
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * PER_STEP + 2, true));  // codes of stage 0
  __builtin_amdgcn_s_barrier();
  expand(0);
  step(0, fa0, fb0, fa1, fb1, false);
  int t = 1;
  for (; t < KT - 1; t += 2) {
    step(t, fa1, fb1, fa0, fb0, true);
    step(t + 1, fa0, fb0, fa1, fb1, true);
  }
  step(t, fa1, fb1, fa0, fb0, true);
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
  mma(fa1, fb1);

  float bias[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) bias[j] = epilogue_bias(a, n0 + wn * 64 + j * 16 + r);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const EpiRow row = epilogue_row<EPI>(a, m0 + wm * 128 + i * 16 + 4 * g + e);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        epilogue_store<EPI>(a, row, n0 + wn * 64 + j * 16 + r, acc[i][j][e] + bias[j]);
    }
}

// ---------------------------------------------------------------------------
// The kernel of a shape, from (M, N, K) and the weight format (and for two
// cases the layout and alignment).  Times are us of one launch with its
// merge over rotating weights (fragment order unless stated).
// ---------------------------------------------------------------------------
constexpr int64_t kSkinnyMaxM = 16;
constexpr int kMaxSplits = 8;
// About one workgroup per CU measured best: a slab workgroup takes most of a
// CU's LDS, so more of them only queue.
constexpr int64_t kMaxWGs = 256;

enum GemmKernel { kSkinny, kSlab, kStreamW4, kBig, kTiled };
struct GemmPlan {
  GemmKernel kernel;
  int slab = 0;    // row of the slab tables
  int splits = 1;  // K ranges
};

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// K ranges: the largest power of two up to the cap (and the `fit` the workspace
// holds) that keeps the grid within kMaxWGs workgroups and every range at
// least kper_min long
static int split_k(int64_t wgs, int64_t K, int64_t kper_min, int fit = kMaxSplits) {
  int S = 1;
  while (2 * S <= fit && wgs * 2 * S <= kMaxWGs && K % (2ll * S * 128) == 0 &&
         K / (2 * S) >= kper_min)
    S *= 2;
  return S;
}

// rows of the slab tables (gemm_common.h) by what they are for
enum { kF16M16n16 = 0, kF16M16n32, kF16M32n32, kF16M32n96, kF16M32n128, kF16M64n64, kF16M64n96,
       kF16M64n128, kF16M128n64, kF16M128n128, kF16M16n64 };
enum { kW4M16n32 = 0, kW4M32n64, kW4M32n128, kW4M64n64, kW4M64n128, kW4M128n64, kW4M128n128,
       kW4M128n256, kW4M128n256k1 };

// M <= 16.  The skinny kernel has no LDS staging and no barrier, and its 16
// or 64 rows per workgroup fill the chip at many N; what it lacks is the
// balance at N of 4096 to 8192, where 257 to 512 workgroups of 16 rows leave
// a second round half empty and X is read by each: there 32-row slab
// workgroups (at most 256) take over, K split over their waves, once the K
// range of a wave outlasts its first loads (M = 16: fp16 7168 x 28672 82.9 ->
// 61.8, 6144 x 4096 14.4 -> 11.1; M = 12, 8192 x 2048 8.0 and 8.6; INT4 63.2 ->
// 35.7 and 11.4 -> 8.5, but M = 12, 6912 x 2304 6.7 and 7.0); at M <= 8 the two
// are equal (17.6 against 17.9) but for fp16 and long K (M = 1, 5120 x 20480:
// 41.0 -> 34.6).  Up to N = 4096, 16-row slab workgroups for fp16 (M = 16, 4096 x
// 14336: 23.3 -> 22.0, x 3072 7.6 -> 7.2, but x 2048 5.7 and 6.1; at N = 4608, a
// second round of them, x 1536 6.9 and 8.6; INT4 fragments come in pairs, 32
// rows, which would leave half the CUs idle).
// With fp16 W both kernels give the same bits; with INT4 W an EPI_F16 output
// stays with the skinny kernel: EPI_SWIGLU, which only that kernel has, gives
// the values of EPI_F16 and the SwiGLU kernel bit for bit.
// Row-major fp16 W: the skinny kernel's loads take 64 bytes of each of 16
// rows, half of every 128-byte line, the slab kernel's whole lines, so it is
// the faster one at every M and N (M = 16: 128256 x 4096 224 -> 188, 50272 x
// 7168 182 -> 126; M = 1: 5120 x 5120 19.2 -> 11.9, 4096 x 14336 26 -> 21), with
// 64 columns above N = 8192, 32 above 4096 (M = 16, 4608 x 1024 5.3, with 16
// 7.0); but where there is little to read (N up to 4096, K up to 1536: M = 1,
// 4096 x 1536 5.0 and 5.3).
static GemmPlan plan_m16(int64_t M, int64_t N, int64_t K, bool w4, int epi, bool packed) {
  if (w4 && epi == EPI_F16) return {kSkinny};
  if (!w4 && !packed) {
    if (N <= 4096) return K <= 1536 ? GemmPlan{kSkinny} : GemmPlan{kSlab, kF16M16n16};
    return {kSlab, N <= 8192 ? kF16M16n32 : kF16M16n64};
  }
  const bool rows16 = M > 8;
  if (w4)
    return rows16 && N >= 5120 && N <= 8192 && K >= 3072 ? GemmPlan{kSlab, kW4M16n32}
                                                         : GemmPlan{kSkinny};
  if (N > 4096 && N <= 8192 && (rows16 ? K >= 2560 : K >= 16384)) return {kSlab, kF16M16n32};
  if (N <= 4096 && rows16 && K >= 3072) return {kSlab, kF16M16n16};
  return {kSkinny};
}

// 16 < M <= 128: the slab kernel with 64 columns per workgroup while that
// fills the chip (N up to 16384), else 128.  Long K goes to the wide
// workgroups too: each reads all of X, and K ranges give the workgroups
// (fp16 M = 64, 7168 x 28672: 81.5 with 64 columns and 2 ranges, 70.6 with
// 128 and 4; at 8192 x 8192 29.4 against 32.4).  fp16 grids of 128-column
// workgroups that leave a quarter of the CUs idle (N of 16384 to 24576; at
// M <= 32 from 8192) take 96 columns (M = 64, 21504 x 7168: 62.5 -> 51.9); at
// M <= 32 and N <= 8192 32 columns and no split measured best (8192 x 8192:
// 29.3 -> 24.0).  Splitting K pays only for its second launch (about 2.5 us)
// when a range is long enough: not below K = 1536.  Where the workspace does
// not hold the ranges that wide workgroups need, the narrow ones take over
// (4096 x 14336, one range: fp16 M = 32 82 -> 35, M = 64 97 -> 65, INT4 M = 128
// 120 -> 79).
// Where long K begins, by format and 32, 64 or 128 rows, lies between the two
// sides of what was measured, later at N = 4096 (one round either way) than at
// 5120 to 14336 (64 columns / 128, with their ranges; fragment order): INT4 M = 32,
// 4096 x 13312 14.8 / 15.4, x 16384 16.6 / 16.6, 14336 x 8192 22.9 / 23.6, x 14336
// 36.8 / 33.3; M = 64, 8192 x 12288 26.7 / 27.4, x 16384 32.6 / 31.7; M = 128, 4096 x
// 8192 21.3 / 22.6, x 11264 25.9 / 25.8, 8192 x 4096 21.8 / 22.9, x 9216 36.3 / 33.3;
// fp16 M = 64, 4096 x 16384 29.0 / 30.5, 14336 x 8192 43.2 / 44.2, x 16384 81.3 /
// 76.9; M = 128, 4096 x 6144 20.9 / 21.9, 8192 x 7168 35.7 / 33.7.
//
// Row-major INT4 W at M <= 32: the streaming kernel in place of the 128-column
// slab kernel, and in its 64-column form of the 64-column one where K is long
// enough for its start (M = 32, us with the slab kernel: 16384 x 2048 12.6 -> 12.0,
// x 13312 61 -> 48, 5120 x 4096 14.6 -> 14.2, 8192 x 8192 23.7 -> 21.7; but 8192 x
// 3072 14.1 and 14.3) and it is not one round with many ranges (4096 x 4096 11.5
// and 12.1).  Above M = 32 the slab kernel is the faster one throughout (M = 33 to
// 128, the streaming kernel it replaced: 4096 x 4096 31 -> 12, 28672 x 7168 75 ->
// 63, 7168 x 28672 101 -> 83).
static GemmPlan plan_decode(int64_t M, int64_t N, int64_t K, bool w4, bool packed, int fit) {
  const int mf = M <= 32 ? 2 : (M <= 64 ? 4 : 8);
  GemmPlan p{kSlab};
  int cols;
  if (w4) {
    const bool narrow = N <= 16384 && K < (mf == 8 ? 8193 : (mf == 4 ? 16384 : 14336));
    p.slab = (mf == 2 ? kW4M32n64 : (mf == 4 ? kW4M64n64 : kW4M128n64)) + (narrow ? 0 : 1);
    cols = narrow ? 64 : 128;
  } else if (mf == 2) {
    if (N <= 8192 && K <= 8192) {
      p.slab = kF16M32n32;
      cols = 32;
    } else if (N > 8192 && N <= 24576) {
      p.slab = kF16M32n96;
      cols = 96;
    } else {
      p.slab = kF16M32n128;
      cols = 128;
    }
  } else if (mf == 4 && N > 16384 && N <= 24576) {
    p.slab = kF16M64n96;
    cols = 96;
  } else {
    const bool narrow = N <= 16384 && K < (mf == 8 ? 6145 : 16384);
    p.slab = mf == 4 ? (narrow ? kF16M64n64 : kF16M64n128) : (narrow ? kF16M128n64 : kF16M128n128);
    cols = narrow ? 64 : 128;
  }
  if (K >= 1536) p.splits = split_k(ceil_div(N, cols), K, 256);
  if (p.splits > fit) {
    const int64_t narrow = ceil_div(N, !w4 && mf == 2 ? 32 : 64);
    if (narrow <= kMaxWGs) {
      p.slab = w4 ? (mf == 2 ? kW4M32n64 : (mf == 4 ? kW4M64n64 : kW4M128n64))
                  : (mf == 2 ? kF16M32n32 : (mf == 4 ? kF16M64n64 : kF16M128n64));
      p.splits = split_k(narrow, K, 256, fit);
    } else {
      p.splits = fit;
    }
  }
  if (w4 && !packed &&
      (p.slab == kW4M32n128 || (p.slab == kW4M32n64 && N > 4096 &&
                                K >= (N > 8192 ? 2048 : 4096) && K % (256 * p.splits) == 0)))
    p.kernel = kStreamW4;
  return p;
}

// M > 128 (prefill): 256 x 256 tiles while they fill the chip, else smaller
// tiles and K ranges.  INT4: the 128-row slab kernels below 192 big tiles
// (us at M = 512: 4096 x 14336 301 with 128 x 128 tiles -> 72, 28672 x 4096,
// 224 big tiles, 227 -> 129; M = 2048, 4096 x 4096, 128 big tiles: 104 big,
// 70 slab); 128 columns while one K range gives at most kMaxWGs workgroups,
// else 256 while those do; beyond, big tiles are one round where these are two
// (M = 2048, 5120 x 4096: 99 against 128; row-major, M = 4096, 2304 x 768, 44 and
// 30, with 128 x 128 tiles through registers 40).  Their two K groups sum in another order than the big tiles; K
// under 512 (four chunks a group) stays with one group.  fp16: big tiles with
// K ranges (M = 512, 4096 x 14336: 202 -> 71; 28672 x 4096 202 -> 104), and
// 128 x 128 slab tiles where even 8 ranges give few workgroups (M = 200,
// 768 x 3072: 46 -> 15).
//
// fp16 K ranges pay while the products saved outlast the partial sums' traffic
// (8 S M N bytes) and the merge, that is from K = 14 per workgroup on (S = 2: 72
// big tiles, K = 1536 33.5 against 35.1 unsplit, 2048 37.9, 43.4; 96, 2048 43.0,
// 43.7; 128, 2048 52.5, 45.7, 3072 65, 62 and 4096 77, 80; S = 4 against 2: 64
// tiles, 2048 40.8, 37.2, 4096 52, 55; with row-major W two or three us later).
// Below that, 128 x 128 slab tiles unsplit while they are half a chip to one
// (K = 2048: M = 1024, 4096 columns 27 against 42 with four ranges; 3072 38, 48;
// 4096 47, 54, but 6144 69, 69), and between one tile of 128 x 128 per CU and
// two, gemm_tiled, which keeps two workgroups on a CU, where the start counts
// (M = 1500, 3072 x 768 20.6 against 22.3, x 1024 25.1, 26.3, x 2048 43.4, 43.4) and
// where W is row-major, 64 bytes of a row per load of the big tiles (M = 384,
// 20480 x 5120 108 against 137; M = 1500, 3072 x 2048 43, 52).
//
// The ranges are those that fit the workspace, and the same for W in either
// layout (one range gives the same bits in all of these kernels, so both do).
// Where the ones that a wide tile needs do not fit, 128 x 128 slab tiles take its
// place while they are at most kMaxWGs (4096 x 14336, one range: fp16 M = 509
// 254 -> 141, INT4 194 -> 121; gemm_tiled takes 229 and 326).
// Outputs of fewer than 512 columns stay unsplit: the workspace query answers
// 0 for them, as callers that size their buffers by it have seen (M = 150,
// 384 x 1536: 19 us where four ranges would take 11; 26 with gemm_tiled).
static GemmPlan plan_prefill(int64_t M, int64_t N, int64_t K, bool w4, bool packed, int fit) {
  const int64_t big = ceil_div(M, 256) * ceil_div(N, 256), mt = ceil_div(M, 128);
  const int64_t t128 = mt * ceil_div(N, 128), t256 = mt * ceil_div(N, 256);
  const int64_t kper = N < 512 ? K : 512;
  if (w4) {
    if (big >= 192 || t256 > kMaxWGs) return {kBig};
    if (K < 512) return {kSlab, kW4M128n256k1};
    if (t128 <= kMaxWGs && (K < 8192 || split_k(t256, K, kper) > fit))
      return {kSlab, kW4M128n128, split_k(t128, K, kper, fit)};
    return {kSlab, kW4M128n256, split_k(t256, K, kper, fit)};
  }
  int S = split_k(big, K, kper);
  while (S > 1 && K < 14 * big * S) S /= 2;
  const int s = S < fit ? S : fit;
  if (t128 > kMaxWGs) {
    const bool tiled = t128 <= 2 * kMaxWGs && (packed ? K <= 1024 : s == 1);
    return tiled ? GemmPlan{kTiled} : GemmPlan{kBig, 0, s};
  }
  if (big * S > 64 && s > 1 && s == S && K > (2 * t128 > kMaxWGs ? 3072 : 2048))
    return {kBig, 0, s};
  int n = split_k(t128, K, kper, fit);
  while (n > 1 && K < 8 * t128 * n) n /= 2;
  return {kSlab, kF16M128n128, n};
}

// fit: the most K ranges the workspace has room for
static GemmPlan gemm_plan(int64_t M, int64_t N, int64_t K, bool w4, int epi, bool packed,
                          int fit = kMaxSplits) {
  if (M <= kSkinnyMaxM) return plan_m16(M, N, K, w4, epi, packed);
  return M <= kDecodeMaxM ? plan_decode(M, N, K, w4, packed, fit)
                          : plan_prefill(M, N, K, w4, packed, fit);
}

int64_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K, bool w4) {
  if (M <= kSkinnyMaxM || N <= 0 || K <= 0 || K % 128 != 0) return 0;
  const GemmPlan p = gemm_plan(M, N, K, w4, EPI_F32, true);  // as many as any call's
  return p.splits > 1 ? (int64_t)p.splits * M * N * 4 : 0;
}

// The plan is the same for every M of (16, 32], (32, 64], (64, 128] and of each
// 128 rows beyond, and at most two ranges of kMaxWGs / 2 of the widest tiles
// split: at most 64 MiB in all.
int64_t gemm_workspace_bytes_upto(int64_t M_max, int64_t N, int64_t K, bool w4) {
  int64_t best = 0;
  for (int64_t M = 32;; M += M < kDecodeMaxM ? M : 128) {
    const int64_t m = std::min(M, M_max);
    best = std::max(best, gemm_workspace_bytes(m, N, K, w4));
    if (m == M_max || ceil_div(m, kBM) * ceil_div(N, kBN) > kMaxWGs / 2) return best;
  }
}

template <int NF, bool W4, int EPI, bool PK>
static void launch_skinny(const GemmArgs& a, hipStream_t st) {
  constexpr int KW = 8, UNR = 2;  // waves, steps in flight per wave
  const dim3 grid((unsigned)((a.N + 16 * NF - 1) / (16 * NF)));
  launch((gemm_skinny<NF, 1, KW, UNR, W4, EPI, PK>), grid, dim3(KW * 64), 0, st, a);
}

template <int KS, int EPI>
static void launch_stream_w4(const GemmArgs& a, int S, float* ws, hipStream_t st) {
  constexpr int cols = 16 * kStreamWaves / KS;
  const dim3 grid((unsigned)ceil_div(a.N, cols), (unsigned)S), block(kStreamWaves * 64);
  if constexpr (KS == 2)
    launch((gemm_stream_w4<4, 256, 2, EPI>), grid, block, 0, st, a, ws, a.K / S);
  else if (a.K % (256 * S) == 0)
    launch((gemm_stream_w4<2, 256, 1, EPI>), grid, block, 0, st, a, ws, a.K / S);
  else
    launch((gemm_stream_w4<4, 128, 1, EPI>), grid, block, 0, st, a, ws, a.K / S);
}

template <bool W4, int EPI, bool PK>
static pipo_status launch_epi(const GemmArgs& a, float* ws, int64_t ws_bytes, hipStream_t st) {
  if constexpr (EPI == EPI_SWIGLU) {
    (void)ws;
    (void)ws_bytes;
    if (a.M > kSkinnyMaxM) {
      set_error("gemm: the SwiGLU epilogue needs M <= 16 (M=%lld)", (long long)a.M);
      return PIPO_ERR_UNSUPPORTED;
    }
    launch_skinny<4, W4, EPI, PK>(a, st);
    PIPO_HIP_TRY(hipGetLastError());
    return PIPO_OK;
  } else {
    int fit = ws == nullptr || a.M * a.N >= ((int64_t)1 << 31) ? 1 : kMaxSplits;
    while (fit > 1 && ws_bytes < (int64_t)fit * a.M * a.N * 4) fit /= 2;
    GemmPlan p = gemm_plan(a.M, a.N, a.K, W4, EPI, PK, fit);
    // loads straight into LDS take 16 bytes at a time: operands off that
    // alignment go through registers, in decode by the same plan
    const uintptr_t at = reinterpret_cast<uintptr_t>(a.X) |
                         (W4 ? reinterpret_cast<uintptr_t>(a.Wq) : reinterpret_cast<uintptr_t>(a.W));
    const bool direct =
        at % 16 == 0 && (!W4 || reinterpret_cast<uintptr_t>(a.Wsm) % 4 == 0);
    if (!direct && a.M <= kSkinnyMaxM) p = GemmPlan{kSkinny};
    if (!direct && a.M > kDecodeMaxM) p = GemmPlan{kTiled};
    switch (p.kernel) {
      case kSkinny:
        // 64 W rows per workgroup (less X traffic per W byte) once that still
        // gives enough workgroups to fill the chip, else 16
        if (a.N >= 64 * 192)
          launch_skinny<4, W4, EPI, PK>(a, st);
        else
          launch_skinny<1, W4, EPI, PK>(a, st);
        break;
      case kSlab:
        (W4 ? launch_slab_w4 : launch_slab_f16)(a, EPI, p.slab, direct, p.splits, ws, st);
        break;
      case kStreamW4:
        if constexpr (W4 && !PK) {
          if (p.slab == kW4M32n128)
            launch_stream_w4<1, EPI>(a, p.splits, ws, st);
          else
            launch_stream_w4<2, EPI>(a, p.splits, ws, st);
        }
        break;
      case kBig: {
        const int64_t per_xcd = ceil_div(ceil_div(a.M, kBM) * ceil_div(a.N, kBN), kXcds);
        const dim3 grid((unsigned)(per_xcd * kXcds), (unsigned)p.splits);
        if constexpr (W4)
          launch((gemm_big_w4<EPI, PK>), grid, dim3(kFThreads), 0, st, a);
        else
          launch((gemm_big_f16<EPI, PK>), grid, dim3(kFThreads), 0, st, a, ws, a.K / p.splits);
        break;
      }
      case kTiled: {
        const int64_t per_xcd = ceil_div(ceil_div(a.M, kTBM) * ceil_div(a.N, kTBN), kXcds);
        launch((gemm_tiled<W4, EPI, PK>), dim3((unsigned)(per_xcd * kXcds)), dim3(kTThreads), 0, st,
               a);
        break;
      }
    }
    if (p.splits > 1) launch_combine(a, EPI, ws, p.splits, st);
    PIPO_HIP_TRY(hipGetLastError());
    return PIPO_OK;
  }
}

template <bool W4, bool PK>
static pipo_status launch_fmt(const GemmArgs& a, int epi, float* ws, int64_t ws_bytes,
                              hipStream_t st) {
  switch (epi) {
    case EPI_F16: return launch_epi<W4, EPI_F16, PK>(a, ws, ws_bytes, st);
    case EPI_RELU_F16: return launch_epi<W4, EPI_RELU_F16, PK>(a, ws, ws_bytes, st);
    case EPI_ADD_F32: return launch_epi<W4, EPI_ADD_F32, PK>(a, ws, ws_bytes, st);
    case EPI_F32: return launch_epi<W4, EPI_F32, PK>(a, ws, ws_bytes, st);
    case EPI_QKV: return launch_epi<W4, EPI_QKV, PK>(a, ws, ws_bytes, st);
    case EPI_SWIGLU: return launch_epi<W4, EPI_SWIGLU, PK>(a, ws, ws_bytes, st);
    default: set_error("gemm: unknown epilogue %d", epi); return PIPO_ERR_ARG;
  }
}

pipo_status launch_gemm(const GemmArgs& a, bool w4, int epi, float* workspace,
                        int64_t workspace_bytes, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) {
    set_error("gemm: empty shape M=%lld N=%lld K=%lld", (long long)a.M, (long long)a.N,
              (long long)a.K);
    return PIPO_ERR_ARG;
  }
  if (a.K % 128 != 0) {
    set_error("gemm: K=%lld is not a multiple of 128", (long long)a.K);
    return PIPO_ERR_UNSUPPORTED;
  }
  if (a.X == nullptr || (w4 ? (a.Wq == nullptr || a.Wsm == nullptr) : a.W == nullptr)) {
    set_error("gemm: null operand");
    return PIPO_ERR_ARG;
  }
  if (a.M >= (int64_t(1) << 31)) {
    set_error("gemm: M=%lld rows exceeds 2^31 - 1", (long long)a.M);
    return PIPO_ERR_UNSUPPORTED;
  }
  if (epi == EPI_QKV && a.rows_per_seq < 1) {
    set_error("gemm: QKV output with rows_per_seq=%lld", (long long)a.rows_per_seq);
    return PIPO_ERR_ARG;
  }
  if (epi == EPI_QKV && (a.dkv <= 0 || a.N != a.d + 2 * a.dkv)) {
    set_error("gemm: QKV output of %lld columns for d=%lld dkv=%lld", (long long)a.N,
              (long long)a.d, (long long)a.dkv);
    return PIPO_ERR_ARG;
  }
  if (epi == EPI_SWIGLU && (a.N % 2 != 0 || a.bias != nullptr || a.out16 == nullptr ||
                            a.ldo < a.N / 2)) {
    set_error("gemm: the SwiGLU epilogue needs an even N (gate over up rows), no bias and an "
              "fp16 output of N / 2 columns (N=%lld ldo=%lld)", (long long)a.N, (long long)a.ldo);
    return PIPO_ERR_ARG;
  }
  if (a.packed && a.N % 16 != 0) {
    set_error("gemm: fragment-ordered W needs N %% 16 == 0 (N=%lld)", (long long)a.N);
    return PIPO_ERR_UNSUPPORTED;
  }
  if (a.packed)
    return w4 ? launch_fmt<true, true>(a, epi, workspace, workspace_bytes, st)
              : launch_fmt<false, true>(a, epi, workspace, workspace_bytes, st);
  return w4 ? launch_fmt<true, false>(a, epi, workspace, workspace_bytes, st)
            : launch_fmt<false, false>(a, epi, workspace, workspace_bytes, st);
}

}  // namespace pipo
