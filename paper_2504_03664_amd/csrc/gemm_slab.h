// GEMM kernel of decode (M <= 128) and of prefill with few tiles.
#pragma once

#include <type_traits>

#include "gemm_common.h"

namespace pipo {

// ---------------------------------------------------------------------------
// slab GEMM: X shared through LDS, every W row owned by one wave
//
// Workgroup = WN x KS waves on 16 MF rows of X and 16 NF WN rows of W; wave
// (wn, ks) owns 16 NF rows of W and every KS-th 64-wide chunk of K.  K is
// walked in slabs of KS KC (KC = 64): a stage is the slab of X and each wave's W
// chunk, moved from global memory straight into LDS by the load unit, PD
// stages ahead in a ring of PD + 1, so the bytes in flight cost no registers
// and the waits are exact counts (one barrier per slab).  A wave reads an X
// fragment from LDS for NF products and expands each INT4 code once, with
// no other wave repeating it.  X keeps whole 128-byte lines per load, row r
// of a 16-row block holding its 16-byte chunk c at position c ^ ((r / 2) %
// 8), which leaves the fragment reads free of bank conflicts.  A chunk's
// INT4 codes are 512 bytes per 16 rows (slot r + 16 i: row r, k = 32 i ..
// + 31), its (scale, min) pairs one word per row; fp16 W in row-major order
// is loaded and kept like X (whole lines; 16 rows x 64 bytes per load
// fetched every line twice).  For MF = 8 every product covers 32 consecutive
// k in k order, as in the other prefill kernels, so for KS = 1 and one K
// range the sums are the same bits; for MF < 8 an INT4 lane takes 16
// consecutive k of a chunk with one 8-byte read of its codes.
//
// Measured against the kernels it replaced (register-staged X and W; rotating
// weights, us, S K ranges with their merge): fp16 M = 64, N x K = 28672 x
// 7168: 73.3 -> 66.5 (6.2 TB/s of weights; loads alone take 65.7), 4096 x
// 4096: 18.8 -> 14.0; M = 128, 28672 x 4096: 74.1 -> 50.7; INT4 M = 64, 28672
// x 4096: 42.8 -> 25.9, M = 128, 4096 x 14336: 51.0 -> 29.3.  What bounds
// fp16 decode is HBM; INT4 decode the expansion (without it M = 32, 28672 x
// 16384 takes 56 instead of 76 us, loads alone 44); MF = 8 the MFMAs and
// the expansion.
template <int MF, int NF, int WN, int KS, int PD, bool W4>
struct SlabCfg {
  static_assert(!W4 || NF % 2 == 0, "INT4 fragments are loaded in pairs");
  static constexpr int KC = 64;  // k per chunk: one 128-byte line of a row of X
  static constexpr int kWaves = WN * KS, kThreads = kWaves * 64;
  static constexpr int kXBytes = 16 * MF * KS * KC * 2;           // of a stage
  static constexpr int kWBlocks = W4 ? NF / 2 : 2 * NF;           // 1 KiB loads of a wave
  static constexpr int kSmLoads = W4 ? (NF + 3) / 4 : 0;          // 256-byte loads of a wave
  static constexpr int kWBytes = kWBlocks * 1024 + kSmLoads * 256;
  static constexpr int kStage = kXBytes + kWaves * kWBytes;
  static constexpr int kRing = PD + 1;
  static constexpr int kXLoads = kXBytes / 1024 / kWaves;         // of a wave
  static constexpr int kOps = kXLoads + kWBlocks + kSmLoads;
  static_assert(kRing * kStage <= 160 * 1024, "LDS");
  static_assert(kXBytes / 1024 % kWaves == 0, "X loads split evenly");
  static_assert((PD - 1) * kOps <= 63, "vmcnt counts up to 63");
  static constexpr int kRows = 16 * MF, kCols = 16 * NF * WN;     // of the output tile
};

// wait until at most min(left, N) later stages of OPS loads are in flight
template <int OPS, int N>
__device__ __forceinline__ void wait_stages(int left) {
  if constexpr (N == 0) {
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
  } else {
    if (left >= N)
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(N * OPS, true));
    else
      wait_stages<OPS, N - 1>(left);
  }
}

// DIRECT: operands aligned as loads into LDS need (16 bytes, a (scale, min)
// pair 4); others come through registers, one slab ahead (fp16 row-major M = 64,
// 4096 x 14336: 36 us, with DIRECT 28; through 128 x 128 tiles without K ranges
// 264; INT4 58 with the register-staged kernel before this one, 34 here)
template <int MF, int NF, int WN, int KS, int PD, bool W4, int EPI, bool PK, bool DIRECT>
__global__ __launch_bounds__(WN * KS * 64) void gemm_slab(GemmArgs a, float* part, int64_t kper) {
  using C = SlabCfg<MF, NF, WN, KS, PD, W4>;
  constexpr int KC = C::KC;
  constexpr bool NT = MF < 8;  // decode: W is read once per pass
  __shared__ __attribute__((aligned(1024))) uint8_t lds[C::kRing * C::kStage];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WN, ks = wave / WN;
  const int r = lane & 15, g = lane >> 4;
  const int64_t K = a.K;
  // tile order: XCD x takes a contiguous range of tiles, row tiles fastest,
  // so that the workgroups that share W rows run on one L2 at the same time
  const int64_t tiles_m = (a.M + C::kRows - 1) / C::kRows;
  const int64_t tiles_n = (a.N + C::kCols - 1) / C::kCols;
  const int64_t per_xcd = gridDim.x / kXcds;
  const int64_t tile = tiles_m == 1 ? (int64_t)blockIdx.x
                                    : (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  const int64_t tn = tile / tiles_m;
  if (tn >= tiles_n) return;
  const int64_t m0 = (tile - tn * tiles_m) * C::kRows;
  const int64_t nwg = tn * C::kCols, nw0 = nwg + wn * (16 * NF);
  const int64_t kbeg = (int64_t)blockIdx.y * kper;
  // chunk of K group j in round t.  MF = 1 deals the chunks in pairs, 128 k
  // at a time, as gemm_skinny deals its steps to its 8 waves, and keeps 8
  // partial sums (kSums of them in a wave), so with fp16 W the two kernels
  // sum in the same order (K, and so the chunk count, is even)
  constexpr int kSums = MF == 1 ? 8 / KS : 1;
  const auto chunk_of = [&](int t, int j) {
    return MF == 1 ? 2 * (KS * (t >> 1) + j) + (t & 1) : KS * t + j;
  };
  const int nch = (int)(kper / KC);
  const int nr = MF == 1 ? 2 * ((nch / 2 + KS - 1) / KS) : (nch + KS - 1) / KS;

  // X: a load covers 8 rows x 64 k; rows past M repeat the last one, k past
  // the range the last 64 (loaded, never used)
  const uint16_t* xsrc[C::kXLoads];
#pragma unroll
  for (int i = 0; i < C::kXLoads; ++i) {
    const int q = (wave * C::kXLoads + i) % (2 * MF);
    const int row = 8 * (q & 1) + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    int64_t m = m0 + 16 * (q >> 1) + row;
    m = m < a.M ? m : a.M - 1;
    xsrc[i] = a.X + m * K + kbeg + 8 * c;
  }
  // W: rows past N repeat the last (fragment order: the last 16)
  constexpr int WSRC = W4 ? NF / 2 : (PK ? NF : 2 * NF);
  const uint8_t* wsrc[WSRC];
  const uint8_t* ssrc[W4 ? C::kSmLoads : 1];
#pragma unroll
  for (int f = 0; f < WSRC; ++f) {
    int64_t n = nw0 + 16 * (W4 ? 2 * f + (lane >> 5) : f);  // INT4: a fragment per half wave
    if constexpr (!W4 && !PK) {  // load f: rows 8 (f % 2) .. + 7 of fragment f / 2
      const int row = 8 * (f & 1) + (lane >> 3);
      n = nw0 + 16 * (f >> 1) + row;
      n = n < a.N ? n : a.N - 1;
      wsrc[f] = reinterpret_cast<const uint8_t*>(a.W + n * K + 8 * ((lane & 7) ^ ((row >> 1) & 7)));
    } else if constexpr (PK) {
      n = n < a.N ? n : a.N - 16;
      wsrc[f] = W4 ? a.Wq + (n >> 4) * (K >> 7) * 1024 + (lane & 31) * 16
                   : reinterpret_cast<const uint8_t*>(a.W) + (n >> 4) * (K >> 5) * 1024 + lane * 16;
    } else {
      n += r;
      n = n < a.N ? n : a.N - 1;
      wsrc[f] = a.Wq + n * (K / 2) + 16 * (g & 1);
    }
  }
  if constexpr (W4) {
#pragma unroll
    for (int i = 0; i < C::kSmLoads; ++i) {
      const int f = 4 * i + g;
      int64_t n = nw0 + 16 * (f < NF ? f : NF - 1) + r;
      n = n < a.N ? n : a.N - 1;
      ssrc[i] = reinterpret_cast<const uint8_t*>(a.Wsm) + w4_sm<PK>(n, 0, K) * 4;
    }
  }
  // the loads of stage t, each with its number and its place in slot `slot`:
  // x(number, source, place) and w(..) of 16 bytes a lane, s(..) of 4
  const auto stage = [&](int t, int slot, auto x, auto w, auto s) {
    uint8_t* st = lds + slot * C::kStage;
    const int klast = (int)kper - 64;
#pragma unroll
    for (int i = 0; i < C::kXLoads; ++i) {
      const int p = wave * C::kXLoads + i;
      const int k = chunk_of(t, p / (2 * MF)) * KC;
      x(i, xsrc[i] + (k < klast ? k : klast), st + p * 1024);
    }
    const int c = chunk_of(t, ks);
    const int64_t k = kbeg + (int64_t)(c < nch ? c : nch - 1) * KC;
    uint8_t* wb = st + C::kXBytes + wave * C::kWBytes;
    if constexpr (W4) {
      const int64_t off = PK ? (k >> 7) * 1024 + ((k >> 6) & 1) * 512 : k / 2;
#pragma unroll
      for (int f = 0; f < WSRC; ++f) w(f, wsrc[f] + off, wb + f * 1024);
      const int64_t soff = PK ? (k >> 7) * 128 + ((k >> 6) & 1) * 4 : k / 64 * 4;
#pragma unroll
      for (int i = 0; i < C::kSmLoads; ++i)
        s(i, ssrc[i] + soff, wb + C::kWBlocks * 1024 + i * 256);
    } else if constexpr (PK) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          w(2 * f + i, wsrc[f] + ((k >> 5) + i) * 1024, wb + (2 * f + i) * 1024);
    } else {
#pragma unroll
      for (int f = 0; f < 2 * NF; ++f) w(f, wsrc[f] + k * 2, wb + f * 1024);
    }
  };
  const auto issue = [&](int t, int slot) {
    stage(
        t, slot, [](int, const void* g, uint8_t* to) { lds_dma16(g, to); },
        [](int, const void* g, uint8_t* to) { lds_dma16_w<NT>(g, to); },
        [](int, const void* g, uint8_t* to) { lds_dma4(g, to); });
  };
  // !DIRECT: a stage from memory into registers, and from there into a slot
  u32x4 xreg[C::kXLoads], wreg[C::kWBlocks];
  uint32_t sreg[C::kSmLoads + 1];
  const auto fetch = [&](int t) {
    stage(
        t, 0, [&](int i, const void* g, uint8_t*) { xreg[i] = *static_cast<const u32x4*>(g); },
        [&](int i, const void* g, uint8_t*) {
          wreg[i] = NT ? load_u32x4_stream(g) : *static_cast<const u32x4*>(g);
        },
        [&](int i, const void* g, uint8_t*) { sreg[i] = *static_cast<const uint32_t*>(g); });
  };
  const auto put = [&](int slot) {
    stage(
        0, slot,
        [&](int i, const void*, uint8_t* to) {
          *reinterpret_cast<u32x4*>(to + lane * 16) = xreg[i];
        },
        [&](int i, const void*, uint8_t* to) {
          *reinterpret_cast<u32x4*>(to + lane * 16) = wreg[i];
        },
        [&](int i, const void*, uint8_t* to) {
          *reinterpret_cast<uint32_t*>(to + lane * 4) = sreg[i];
        });
  };
  f4 sums[kSums][NF][MF];
#pragma unroll
  for (int u = 0; u < kSums; ++u)
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int mf = 0; mf < MF; ++mf) sums[u][f][mf] = f4{0.f, 0.f, 0.f, 0.f};
  constexpr bool kPairs = W4 && MF < 8;
  const auto compute = [&](int slot, auto sum) {
    constexpr int u = decltype(sum)::value;
    // row r of a 16-row block of X (or row-major W), and where its chunk c is
    const int row_off = (r >> 3) * 1024 + (r & 7) * 128;
    const auto chunk = [&](int c) { return row_off + 16 * (c ^ ((r >> 1) & 7)); };
    const uint8_t* xb = lds + slot * C::kStage + ks * (MF * 2048);
    const uint8_t* wb = lds + slot * C::kStage + C::kXBytes + wave * C::kWBytes;
    uint32_t codes[NF][2];
    h2 s2[NF], m2[NF];
    if constexpr (W4) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        if constexpr (kPairs) {
          const u32x2 q = *reinterpret_cast<const u32x2*>(wb + f * 512 + (r + 16 * (g >> 1)) * 16 +
                                                          8 * (g & 1));
          codes[f][0] = q[0];
          codes[f][1] = q[1];
        } else {
#pragma unroll
          for (int i = 0; i < 2; ++i)
            codes[f][i] =
                *reinterpret_cast<const uint32_t*>(wb + f * 512 + (r + 16 * i) * 16 + 4 * g);
        }
        scale_min_pairs(
            *reinterpret_cast<const uint32_t*>(wb + C::kWBlocks * 1024 + (16 * f + r) * 4), s2[f],
            m2[f]);
      }
    }
#pragma unroll
    for (int i = 0; i < KC / 32; ++i) {
      h8 xv[MF];
#pragma unroll
      for (int mf = 0; mf < MF; ++mf)
        xv[mf] = *reinterpret_cast<const h8*>(xb + mf * 2048 +
                                              chunk(kPairs ? 2 * g + i : 4 * i + g));
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const h8 wv =
            W4 ? dequant8_fp8(codes[f][i], s2[f], m2[f])
               : *reinterpret_cast<const h8*>(
                     wb + f * 2048 + (PK ? i * 1024 + lane * 16 : chunk(4 * i + g)));
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) sums[u][f][mf] = mfma16(wv, xv[mf], sums[u][f][mf]);
      }
    }
  };

  const auto round = [&](int t, int slot) {
    if (chunk_of(t, ks) >= nch) return;
    if constexpr (kSums == 2) {
      if ((t >> 1) & 1)
        compute(slot, std::integral_constant<int, kSums - 1>{});
      else
        compute(slot, std::integral_constant<int, 0>{});
    } else {
      compute(slot, std::integral_constant<int, 0>{});
    }
  };
  if constexpr (DIRECT) {
#pragma unroll
    for (int p = 0; p < PD; ++p)
      if (p < nr) issue(p, p);
    int slot = 0;
    for (int t = 0; t < nr; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      wait_stages<C::kOps, PD - 1>(nr - 1 - t);  // this wave's loads of stage t landed
      __builtin_amdgcn_s_barrier();              // everyone's did, and stage t - 1 is read
      __builtin_amdgcn_sched_barrier(0);
      if (t + PD < nr) issue(t + PD, slot == 0 ? PD : slot - 1);
      round(t, slot);
      slot = slot == PD ? 0 : slot + 1;
    }
  } else {
    fetch(0);
    put(0);
    if (nr > 1) fetch(1);
    for (int t = 0; t < nr; ++t) {
      __syncthreads();  // stage t is in its slot, and stage t - 1 is read
      if (t + 1 < nr) put((t + 1) & 1);
      if (t + 2 < nr) fetch(t + 2);
      round(t, t & 1);
    }
  }

  // element j of fragment (f, mf): W row 16 f + 4 g + j, X row 16 mf + r
  const bool vec = epilogue_vec4<EPI>(a);
  const bool pvec = a.N % 4 == 0 && reinterpret_cast<uintptr_t>(part) % 16 == 0;
  const auto finish = [&](int64_t n0, int mf, f4 v) {
    const int64_t m = m0 + 16 * mf + r, n = n0 + 4 * g;
    if (m >= a.M || n >= a.N) return;
    if (gridDim.y > 1) {
      float* p = part + ((int64_t)blockIdx.y * a.M + m) * a.N + n;
      if (pvec) {
        *reinterpret_cast<f4*>(p) = v;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (n + j < a.N) p[j] = v[j];
      }
      return;
    }
    const EpiRow row = epilogue_row<EPI>(a, m);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += epilogue_bias(a, n + j);
    if (vec) {
      epilogue_store4<EPI>(a, row, n, v);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) epilogue_store<EPI>(a, row, n + j, v[j]);
    }
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
      for (int f = 0; f < NF; ++f) finish(nw0 + 16 * f, mf, sums[0][f][mf]);
  } else {
    // the K groups' sums meet in LDS, kPer fragments of every wave at a
    // time, and are added in group order, the fragments spread over the waves
    constexpr int kFrags = NF * MF, kFit = C::kRing * C::kStage / 1024 / C::kWaves / kSums;
    constexpr int kPer = kFit >= kFrags ? kFrags : (kFit >= kFrags / 2 ? kFrags / 2 : kFrags / 4);
    static_assert(kSums <= 2, "MF = 1 needs KS of 4 or 8");
    static_assert(kPer >= 1 && kFrags % kPer == 0 && kPer <= kFit, "fragments fit LDS");
    f4* red = reinterpret_cast<f4*>(lds);  // [group][wn][kPer][lane], group kSums-major
#pragma unroll
    for (int p0 = 0; p0 < kFrags; p0 += kPer) {
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kSums; ++u)
#pragma unroll
        for (int e = 0; e < kPer; ++e)
          red[((u * C::kWaves + wave) * kPer + e) * 64 + lane] =
              sums[u][(p0 + e) / MF][(p0 + e) % MF];
      __syncthreads();
      for (int e = wave; e < WN * kPer; e += C::kWaves) {
        const int w = e / kPer, fr = e % kPer;
        f4 v = red[(w * kPer + fr) * 64 + lane];
#pragma unroll
        for (int k = 1; k < KS * kSums; ++k) v += red[((k * WN + w) * kPer + fr) * 64 + lane];
        finish(nwg + w * (16 * NF) + 16 * ((p0 + fr) / MF), (p0 + fr) % MF, v);
      }
    }
  }
}

template <int MF, int NF, int WN, int KS, int PD, bool W4, int EPI>
static void launch_slab_epi(const GemmArgs& a, bool direct, int S, float* ws, hipStream_t st) {
  using C = SlabCfg<MF, NF, WN, KS, PD, W4>;
  const int64_t tm = (a.M + C::kRows - 1) / C::kRows, tn = (a.N + C::kCols - 1) / C::kCols;
  // several row tiles: whole rounds over the XCDs (the kernel drops the excess)
  const int64_t wgs = tm == 1 ? tn : (tm * tn + kXcds - 1) / kXcds * kXcds;
  const dim3 grid((unsigned)wgs, (unsigned)S);
  const auto go = [&](auto kernel) {
    launch(kernel, grid, dim3(C::kThreads), 0, st, a, ws, a.K / S);
  };
  // (M <= 16 and the widest tiles are for aligned operands only)
  if constexpr (MF > 1 && C::kCols < 256) {
    if (!direct)
      return a.packed ? go(gemm_slab<MF, NF, WN, KS, PD, W4, EPI, true, false>)
                      : go(gemm_slab<MF, NF, WN, KS, PD, W4, EPI, false, false>);
  }
  if (a.packed)
    go(gemm_slab<MF, NF, WN, KS, PD, W4, EPI, true, true>);
  else
    go(gemm_slab<MF, NF, WN, KS, PD, W4, EPI, false, true>);
}

template <int MF, int NF, int WN, int KS, int PD, bool W4>
static void launch_slab(const GemmArgs& a, int epi, bool direct, int S, float* ws,
                        hipStream_t st) {
  const auto go = [&](auto e) {
    launch_slab_epi<MF, NF, WN, KS, PD, W4, decltype(e)::value>(a, direct, S, ws, st);
  };
  switch (epi) {
    case EPI_F16: return go(std::integral_constant<int, EPI_F16>{});
    case EPI_RELU_F16: return go(std::integral_constant<int, EPI_RELU_F16>{});
    case EPI_ADD_F32: return go(std::integral_constant<int, EPI_ADD_F32>{});
    case EPI_F32: return go(std::integral_constant<int, EPI_F32>{});
    default: return go(std::integral_constant<int, EPI_QKV>{});
  }
}

}  // namespace pipo
