// bf16 GEMMs of few tiles: C[M,N] = sum_k A(m,k) B(n,k) for micro-batches of one or a few
// images, where the large tiles of gemm_big.hip leave most of the chip idle.
//
// A block of four waves (2x2) owns a 64x64, 64x128 or 128x128 tile, each wave a 1x1, 1x2 or
// 2x2 grid of v_mfma_f32_32x32x16_bf16 accumulators in the same K order as the large
// kernels, so an output element has bitwise the same value from any of them, whatever tile
// a product's size selects.  All three layouts read their operands as they lie: NT takes a
// Linear's [out][in] weight itself (with rotary columns, its rows in pair-interleaved order,
// GemmArgs::rope_rows), so that a small micro-batch transposes no weight.
//
// K tiles are 64 deep in a ring of NST stages filled by 16-byte global->LDS DMA: whole
// 128-byte lines of a K-contiguous operand's rows, 128- or 256-byte k-rows of a K-major one.
// While tile t is multiplied from registers, tile t + 1's fragments are read and tiles
// t + 2 .. t + NST are in flight; one barrier per tile.  What bounds it is LDS bandwidth (a
// 64x64 tile reads each fragment for one MFMA: 32 KB of reads and 16 KB of DMA writes per
// K tile, about 400 cycles of which 128 are MFMA), which the larger tiles halve; rings deeper
// than these did not help back to back (64x64, 8 stages: 20.3 us against 18.7 at
// 256x1280x5120).
// Measured on MI355X, us back to back, the former kernel on a transposed weight -> this one,
// NT: 256x1280x1280 27 -> 8.7, 256x5120x1280 27 -> 10.3, 256x1280x5120 89 -> 18.5 (64x64);
// 648x2048x2048 15.3 (64x128, 64x64 14.1); 2700x1280x5120 57 -> 43 (128x128).  TN
// 1280x1280x1408 34 -> 13.  In a 32-layer pass, whose weights and activations are not in
// cache, the first three take 10, 16 and 27.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_bf16.h"
#include "internal.h"
#include "plan.h"

namespace mpipe {
namespace {

constexpr int NTHR = 256, GROUP_M = 8;

// K-major tile of C columns (C = 64, 128): logical 16-byte chunk c of k-row k is stored at
// c ^ sx<C>(k), so that the four k-rows that 16 lanes of a transposing read touch (64 bytes
// of each) lie on distinct banks.
template <int C>
__device__ __forceinline__ int sx(int k) {
  return C == 64 ? 4 * ((k >> 1) & 1) : 4 * (k & 3);
}
// source of DMA instruction q of a K-major tile: 8 (C = 64) or 4 k-rows an instruction
template <int C>
__device__ __forceinline__ const bf16* src_kmajor(const bf16* X, int64_t ld, int cols, int c0,
                                                  int k0, int kend, int q) {
  constexpr int CH = C / 8;
  const int l = threadIdx.x & 63;
  const int kr = q * (64 / CH) + l / CH;
  int col = c0 + 8 * ((l % CH) ^ sx<C>(kr));
  col = col < cols ? col : cols - 8;
  int k = k0 + kr;
  k = k < kend ? k : kend - 1;
  return X + (int64_t)k * ld + col;
}
// instruction q of an NT product's weight tile (GemmArgs::rope_rows: rows in stored order)
__device__ __forceinline__ const bf16* src_weight(const GemmArgs& p, int n0, int k0, int kend,
                                                  int q) {
  const int l = threadIdx.x & 63;
  const int row = 8 * q + (l >> 3);
  int k = k0 + 8 * ((l & 7) ^ f8(row));
  k = k < kend ? k : kend - 8;
  int n = min(n0 + row, p.N - 1);
  if (p.rope_rows) n = rope_weight_row(n, p.rope_d, p.rope_cols);
  return reinterpret_cast<const bf16*>(p.B) + (int64_t)n * p.ldb + k;
}

template <int N, int I = 0, class F>
__device__ __forceinline__ void unroll_period(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll_period<N, I + 1>(f);
  }
}
// Wait until at most `later` (<= N) tiles of IPT DMAs each are pending.
template <int IPT, int N>
__device__ __forceinline__ void wait_tiles(int later) {
  if constexpr (N > 0) {
    if (later < N) return wait_tiles<IPT, N - 1>(later);
  }
  wait_vm<N * IPT>();
}

template <bool AK, bool BKM, int MI, int NI, int NST, int EPI>
__global__ __launch_bounds__(NTHR, 2) void gemm_small_kernel(GemmArgs p) {
  constexpr int BM = 64 * MI, BN = 64 * NI;
  constexpr int A_U4 = BM * 8, B_U4 = BN * 8, ST_U4 = A_U4 + B_U4;   // 16-byte slots
  constexpr int IA = BM / 32, IB = BN / 32, IPT = IA + IB;   // DMA instructions per wave
  constexpr int SP = 32 * NI + 8;                            // epilogue staging pitch (floats)
  static_assert(NST >= 2 && (NST - 1) * IPT < 64, "ring depth");
  static_assert(4 * 16 * SP * 4 <= NST * ST_U4 * 16, "epilogue staging must fit in the ring");
  __shared__ uint4 smem[NST * ST_U4];

  // XCD-aware tile order, as in the other kernels
  const int ntiles = p.tiles_m * p.tiles_n;
  const int nb = gridDim.x;
  const int pid = (blockIdx.x % 8) * (nb / 8) + (blockIdx.x / 8);
  if (pid >= ntiles) return;
  const int group = pid / (GROUP_M * p.tiles_n);
  const int first_m = group * GROUP_M;
  const int gsize = min(p.tiles_m - first_m, GROUP_M);
  const int m0 = (first_m + (pid % gsize)) * BM;
  const int n0 = ((pid % (GROUP_M * p.tiles_n)) / gsize) * BN;
  const int split = blockIdx.y;
  const int kbeg = split * p.kps;
  const int kend = min(p.K, kbeg + p.kps);
  const int nk = kend > kbeg ? (kend - kbeg + BK64 - 1) / BK64 : 0;
  const int nfull = kend > kbeg ? (kend - kbeg) / BK64 : 0;
  const bf16* A = reinterpret_cast<const bf16*>(p.A);
  const bf16* B = reinterpret_cast<const bf16*>(p.B);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int wm = w >> 1, wn = w & 1;

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  auto src_a = [&](int k0, int i) __attribute__((always_inline)) {
    return AK ? src_kmajor<BM>(A, p.lda, p.M, m0, k0, kend, IA * w + i)
              : src_kc64(A, p.lda, p.M, m0, k0, kend, IA * w + i);
  };
  auto src_b = [&](int k0, int i) __attribute__((always_inline)) {
    return BKM ? src_kmajor<BN>(B, p.ldb, p.N, n0, k0, kend, IB * w + i)
               : src_weight(p, n0, k0, kend, IB * w + i);
  };
  const bf16* sA[IA];
  const bf16* sB[IB];
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < IA; ++i) sA[i] = src_a(kbeg, i);
#pragma unroll
    for (int i = 0; i < IB; ++i) sB[i] = src_b(kbeg, i);
  }
  const int64_t stepA = AK ? (int64_t)BK64 * p.lda : BK64;
  const int64_t stepB = BKM ? (int64_t)BK64 * p.ldb : BK64;
  auto dma_full = [&](int s, int t) __attribute__((always_inline)) {
    const uint4* sa = smem + s * ST_U4;
    const uint4* sb = sa + A_U4;
#pragma unroll
    for (int i = 0; i < IA; ++i) dma16(sA[i] + t * stepA, sa, IA * w + i);
#pragma unroll
    for (int i = 0; i < IB; ++i) dma16(sB[i] + t * stepB, sb, IB * w + i);
  };
  auto dma_tile = [&](int s, int t) __attribute__((always_inline)) {
    const uint4* sa = smem + s * ST_U4;
    const uint4* sb = sa + A_U4;
    if (t < nfull) {
      dma_full(s, t);
    } else {   // ragged last tile: clamped sources
      const int k0 = kbeg + t * BK64;
#pragma unroll
      for (int i = 0; i < IA; ++i) dma16(src_a(k0, i), sa, IA * w + i);
#pragma unroll
      for (int i = 0; i < IB; ++i) dma16(src_b(k0, i), sb, IB * w + i);
    }
  };

  // fragment addresses: K-contiguous as in the 64-deep kernel of gemm_big.hip; K-major as in
  // its K-major tiles, with this file's swizzle
  const int kc = 128 * (l & 31) + 16 * ((l >> 5) ^ f8(l & 31));
  const int kmk = 8 * (l >> 5) + ((l & 15) >> 2);                       // k-row of the lane
  const int kml = 16 * (2 * ((l >> 4) & 1) + ((l & 3) >> 1)) + 8 * (l & 1);
  auto frag = [&](auto KM, auto CC, const char* tile, int cb, int h)
      __attribute__((always_inline)) -> bf16x8 {
    constexpr int C = decltype(CC)::value;
    bf16x8 v;
    if constexpr (decltype(KM)::value) {
      const char* a = tile + (kmk + 16 * h) * (2 * C) + 16 * ((cb >> 3) ^ sx<C>(kmk)) + kml;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(a));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(a + 4 * 2 * C));
      const bf16* pl = reinterpret_cast<const bf16*>(&lo);
      const bf16* ph = reinterpret_cast<const bf16*>(&hi);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = pl[e];
        v[4 + e] = ph[e];
      }
    } else {
      const uint4 x = *reinterpret_cast<const uint4*>(tile + cb * 128 + (kc ^ (32 * h)));
      v = *reinterpret_cast<const bf16x8*>(&x);
    }
    return v;
  };
  using KA = std::integral_constant<bool, AK>;
  using KB = std::integral_constant<bool, BKM>;
  using CA = std::integral_constant<int, BM>;
  using CB = std::integral_constant<int, BN>;
  struct Frags {
    bf16x8 a[4][MI], b[4][NI];
  };
  Frags f0, f1;
  auto read_frags = [&](int s, Frags& f) __attribute__((always_inline)) {
    const char* ta = reinterpret_cast<const char*>(smem + s * ST_U4);
    const char* tb = ta + A_U4 * 16;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
#pragma unroll
      for (int i = 0; i < MI; ++i) f.a[h][i] = frag(KA{}, CA{}, ta, wm * 32 * MI + 32 * i, h);
#pragma unroll
      for (int j = 0; j < NI; ++j) f.b[h][j] = frag(KB{}, CB{}, tb, wn * 32 * NI + 32 * j, h);
    }
  };
  // ragged tile t: nothing past kend counts
  auto mask = [&](int t, Frags& f) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int kr = kend - (kbeg + t * BK64) - 16 * h - 8 * (l >> 5);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e >= kr) {
#pragma unroll
          for (int i = 0; i < MI; ++i) f.a[h][i][e] = (bf16)0.f;
#pragma unroll
          for (int j = 0; j < NI; ++j) f.b[h][j][e] = (bf16)0.f;
        }
    }
  };
  auto mma = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] =
              __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[h][i], f.b[h][j], acc[i][j], 0, 0, 0);
  };
  // wait until all but the last `later` tiles' DMAs of this wave have landed
  auto wait_later = [&](int later) __attribute__((always_inline)) {
    wait_tiles<IPT, NST - 1>(later);
  };
  // Barrier after this wave's LDS reads: the wait as a builtin, so that the compiler knows
  // that `cur` has arrived and does not wait for `nxt` before the MFMAs.
  auto reads_done_barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
    asm volatile("s_barrier" ::: "memory");
  };
  // K tile t (in stage s): its fragments are in `cur`; on exit tile t + 1's are in `nxt`.
  // At the wait the tiles issued are those below min(nk, t + NST); past the barrier every
  // wave has tile t in registers, so its stage takes tile t + NST.
  auto body = [&](int t, int s, const Frags& cur, Frags& nxt) __attribute__((always_inline)) {
    if (t + 1 < nk) wait_later(min(nk, t + NST) - (t + 2));
    reads_done_barrier();
    if (t + 1 < nk) {
      read_frags(s + 1 == NST ? 0 : s + 1, nxt);
      if (t + 1 >= nfull) mask(t + 1, nxt);
    }
    if (t + NST < nk) dma_tile(s, t + NST);
    mma(cur);
  };
  // the same with every tile up to t + NST whole, in stage S = t % NST
  auto body_full = [&](auto S, int t, const Frags& cur, Frags& nxt)
      __attribute__((always_inline)) {
    constexpr int s_ = decltype(S)::value;
    wait_vm<(NST - 2) * IPT>();
    reads_done_barrier();
    read_frags((s_ + 1) % NST, nxt);
    dma_full(s_, t + NST);
    mma(cur);
  };
  if (nk > 0) {
#pragma unroll
    for (int t = 0; t < NST; ++t)
      if (t < nk) dma_tile(t, t);
    wait_later(min(nk, NST) - 1);
    lds_barrier();
    read_frags(0, f0);
    if (nfull == 0) mask(0, f0);
    // steady state, a whole period of stages (and an even number of tiles) at a time: the
    // last tile that a pass fetches, t + PERIOD - 1 + NST, is whole
    constexpr int PERIOD = NST % 2 ? 2 * NST : NST;
    int t = 0;
    for (; t + PERIOD + NST <= nfull; t += PERIOD) unroll_period<PERIOD>([&](auto I) {
      constexpr int i = decltype(I)::value;
      using S = std::integral_constant<int, i % NST>;
      if constexpr (i % 2 == 0) body_full(S{}, t + i, f0, f1);
      else body_full(S{}, t + i, f1, f0);
    });
    int s = 0;
    for (; t < nk; t += 2) {   // the last tiles, guarded
      body(t, s, f0, f1);
      s = s + 1 == NST ? 0 : s + 1;
      if (t + 1 < nk) {
        body(t + 1, s, f1, f0);
        s = s + 1 == NST ? 0 : s + 1;
      }
    }
  }
  wait_vm<0>();

  // epilogue: each wave stages 16 rows of its accumulators at a time in its own LDS region;
  // lane (row, cg) of pass u takes row l / LR + RP u, columns 8 cg .. 8 cg + 7
  __syncthreads();
  constexpr int LR = 4 * NI, RP = 64 / LR, U = 16 / RP;
  float* stage = reinterpret_cast<float*>(smem) + w * 16 * SP;
  const int cg = l % LR;
  const int n = n0 + wn * 32 * NI + 8 * cg;   // N % 8 == 0: all eight columns or none
  const bool vec = n < p.N;
  float bias8[8];
  load_bias8(p, vec && split == 0, n, bias8);
  auto row_of = [&](int pi, int u) { return m0 + wm * 32 * MI + 16 * pi + l / LR + RP * u; };
  constexpr bool kAux = EPI == EPI_GELU_BWD || EPI == EPI_RESID || EPI == EPI_F32 ||
                        EPI == EPI_STORE_ROPE;
  AuxV ax[2 * MI][U];
  if constexpr (kAux) {
#pragma unroll
    for (int pi = 0; pi < 2 * MI; ++pi)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int m = row_of(pi, u);
        if (vec && m < p.M) aux_fetch<EPI>(p, split, m, n, ax[pi][u]);
      }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int pi = 2 * i + hh;
      lds_wave_fence();   // the previous pass's staging reads are done
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int e = 8 * hh; e < 8 * hh + 8; ++e) {
          const int rr = 8 * ((e >> 2) & 1) + 4 * (l >> 5) + (e & 3);
          stage[rr * SP + 32 * j + (l & 31)] = acc[i][j][e];
        }
      lds_wave_fence();   // this pass's staging writes are visible to the whole wave
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int m = row_of(pi, u);
        if (m < p.M && vec) {
          const float* q = stage + (l / LR + RP * u) * SP + 8 * cg;
          float v[8];
          const float4 x0 = *reinterpret_cast<const float4*>(q);
          const float4 x1 = *reinterpret_cast<const float4*>(q + 4);
          v[0] = x0.x; v[1] = x0.y; v[2] = x0.z; v[3] = x0.w;
          v[4] = x1.x; v[5] = x1.y; v[6] = x1.z; v[7] = x1.w;
          epi8_vec<EPI>(p, split, m, n, v, bias8, ax[pi][u]);
        }
      }
    }
  }
}

template <bool AK, bool BKM, int MI, int NI, int NST, int EPI>
hipError_t launch(const GemmArgs& a0, hipStream_t s) {
  constexpr int BM = 64 * MI, BN = 64 * NI;
  GemmArgs a = a0;
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + BN - 1) / BN;
  const int nb = (a.tiles_m * a.tiles_n + 7) / 8 * 8;
  const int splits = a.kps > 0 ? std::max(1, (a.K + a.kps - 1) / a.kps) : 1;
  if (a.kps <= 0) a.kps = a.K;
  hipLaunchKernelGGL((gemm_small_kernel<AK, BKM, MI, NI, NST, EPI>), dim3(nb, splits),
                     dim3(NTHR), 0, s, a);
  return hipGetLastError();
}

template <bool AK, bool BKM, int EPI>
hipError_t by_tile(const GemmArgs& a, int tile, hipStream_t s) {
  switch (tile) {
    case TILE_64x64: return launch<AK, BKM, 1, 1, 4, EPI>(a, s);
    case TILE_64x128:   // (choose_tile never takes it for a weight gradient)
      if constexpr (!AK) return launch<AK, BKM, 1, 2, 6, EPI>(a, s);
      break;
    case TILE_128x128: return launch<AK, BKM, 2, 2, 4, EPI>(a, s);
  }
  return hipErrorInvalidValue;
}
template <bool BKM>
hipError_t by_epi(const GemmArgs& a, int epi, int tile, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return by_tile<false, BKM, EPI_STORE>(a, tile, s);
    case EPI_STORE_ROPE: return by_tile<false, BKM, EPI_STORE_ROPE>(a, tile, s);
    case EPI_GELU: return by_tile<false, BKM, EPI_GELU>(a, tile, s);
    case EPI_RESID: return by_tile<false, BKM, EPI_RESID>(a, tile, s);
    case EPI_GELU_BWD: return by_tile<false, BKM, EPI_GELU_BWD>(a, tile, s);
    case EPI_F32: return by_tile<false, BKM, EPI_F32>(a, tile, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t gemm_small(int layout, int epi, int tile, const GemmArgs& a, hipStream_t s) {
  switch (layout) {
    case GEMM_NT: return by_epi<false>(a, epi, tile, s);
    case GEMM_NN: return by_epi<true>(a, epi, tile, s);
    case GEMM_TN:
      if (epi == EPI_F32) return by_tile<true, true, EPI_F32>(a, tile, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace mpipe
