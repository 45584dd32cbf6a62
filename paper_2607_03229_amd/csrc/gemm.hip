// GEMM family for the encoder: C[M,N] = sum_k A(m,k) B(n,k), with fused epilogues.
//
// One kernel template covers the three operand layouts the encoder needs:
//   forward Linear      Y  = X W^T       A [M][K],  B [N][K]   (both K-contiguous)
//   input gradient      dX = dY W        A [M][K],  B [K][N]   (B K-major)
//   weight gradient     dW = dY^T X      A [K][M],  B [K][N]   (both K-major)
// K-major tiles are transposed in registers on their way into LDS, so the
// MFMA fragment reads are always 16-byte, K-contiguous and bank-conflict free.
//
// Tiling (gfx950): 256 threads = 4 wave64 in a 2x2 grid, block tile 128x128,
// K step 64 (bf16) / 32 (fp32), each wave owns a 64x64 tile of 4x4 16x16
// accumulators.  bf16 uses v_mfma_f32_16x16x32_bf16; fp32 uses
// v_mfma_f32_16x16x4_f32 (eight per 32-wide K step, in the K order of gemm_f32.hip, whose
// kernel takes products of few tiles).  LDS is double-buffered
// (64 KB); the next tile's global loads are in flight during the MFMAs.
// Blocks are remapped so that consecutive tiles land on the same XCD and walk
// the output in groups of 8 tile-rows (L2 reuse of A rows and B columns).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "plan.h"

namespace mpipe {
namespace {

constexpr int BM = 128, BN = 128, NTHR = 256, GROUP_M = 8;

template <class T> struct KStep;
template <> struct KStep<bf16> { static constexpr int BK = 64; static constexpr int VEC = 8; };
template <> struct KStep<float> { static constexpr int BK = 32; static constexpr int VEC = 4; };

struct Regs4 { uint4 v[4]; };

// ---- global -> registers ----------------------------------------------------

// K-contiguous operand X[rows][ld]: tile rows r0..r0+127, k in [k0, k0+BK).
// Thread t loads chunk (t & 7) of rows (t >> 3) + 32 i.
template <class T>
__device__ __forceinline__ void load_kcontig(Regs4& R, const T* X, int64_t ld, int rows, int r0,
                                             int k0, int kend) {
  constexpr int VEC = KStep<T>::VEC;
  const int t = threadIdx.x;
  const int c = t & 7;
  const int k = k0 + c * VEC;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int row = r0 + (t >> 3) + 32 * i;
    row = row < rows ? row : rows - 1;
    if (k < kend)
      R.v[i] = *reinterpret_cast<const uint4*>(X + (int64_t)row * ld + k);
    else
      R.v[i] = make_uint4(0, 0, 0, 0);
  }
}

// K-major operand X[k][ld] (columns contiguous): tile cols c0..c0+127, k in
// [k0, k0+BK).  bf16: thread t loads 4 k-rows x 8 cols (cb = t & 15, kq = t >> 4);
// fp32: 4 k-rows x 4 cols (cb = t & 31, kq = t >> 5).
template <class T>
__device__ __forceinline__ void load_kmajor(Regs4& R, const T* X, int64_t ld, int cols, int c0,
                                            int k0, int kend) {
  constexpr int VEC = KStep<T>::VEC;
  constexpr int NCB = 128 / VEC;
  const int t = threadIdx.x;
  const int cb = t % NCB, kq = t / NCB;
  const int col = c0 + cb * VEC;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = k0 + 4 * kq + j;
    if (k < kend && col < cols)
      R.v[j] = *reinterpret_cast<const uint4*>(X + (int64_t)k * ld + col);
    else
      R.v[j] = make_uint4(0, 0, 0, 0);
  }
}

// ---- registers -> LDS ([row][BK] tiles, 128-byte rows, swizzled chunks) -------

__device__ __forceinline__ void store_kcontig(uint4* lds, const Regs4& R) {
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; ++i) lds[swz((t >> 3) + 32 * i, t & 7)] = R.v[i];
}

template <class T> __device__ __forceinline__ void store_kmajor(uint4* lds, const Regs4& R);

template <> __device__ __forceinline__ void store_kmajor<bf16>(uint4* lds, const Regs4& R) {
  // 4 k-rows x 8 cols -> 8 rows (one per col) of 4 k values (8 bytes each)
  const int t = threadIdx.x;
  const int cb = t & 15, kq = t >> 4;
  uint2* l2 = reinterpret_cast<uint2*>(lds);
  const uint32_t* r0 = reinterpret_cast<const uint32_t*>(&R.v[0]);
  const uint32_t* r1 = reinterpret_cast<const uint32_t*>(&R.v[1]);
  const uint32_t* r2 = reinterpret_cast<const uint32_t*>(&R.v[2]);
  const uint32_t* r3 = reinterpret_cast<const uint32_t*>(&R.v[3]);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int p = i >> 1;
    uint2 v;
    if (i & 1) {
      v.x = pack_hi(r0[p], r1[p]);
      v.y = pack_hi(r2[p], r3[p]);
    } else {
      v.x = pack_lo(r0[p], r1[p]);
      v.y = pack_lo(r2[p], r3[p]);
    }
    const int row = cb * 8 + i;
    l2[swz(row, kq >> 1) * 2 + (kq & 1)] = v;
  }
}

template <> __device__ __forceinline__ void store_kmajor<float>(uint4* lds, const Regs4& R) {
  // 4 k-rows x 4 cols -> 4 rows (one per col) of 4 k values (one 16-byte chunk)
  const int t = threadIdx.x;
  const int cb = t & 31, kq = t >> 5;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint4 v;
    v.x = (&R.v[0].x)[i];
    v.y = (&R.v[1].x)[i];
    v.z = (&R.v[2].x)[i];
    v.w = (&R.v[3].x)[i];
    lds[swz(cb * 4 + i, kq)] = v;
  }
}

// ---- MFMA on one LDS stage -------------------------------------------------------

template <class T> struct Mma;

template <> struct Mma<bf16> {
  // two 32-wide K steps per 64-wide stage
  static __device__ __forceinline__ void run(const uint4* As, const uint4* Bs, int wm, int wn,
                                             f32x4 (&acc)[4][4]) {
    const int l = threadIdx.x & 63;
    const int g = l >> 4, r = l & 15;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      bf16x8 a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint4 va = As[swz(wm * 64 + 16 * i + r, kk * 4 + g)];
        uint4 vb = Bs[swz(wn * 64 + 16 * i + r, kk * 4 + g)];
        a[i] = *reinterpret_cast<bf16x8*>(&va);
        b[i] = *reinterpret_cast<bf16x8*>(&vb);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
};

template <> struct Mma<float> {
  // 16-deep half `kk` of a 32-deep stage: lane group g holds k = 4g .. 4g + 3 of it (one
  // chunk), the operands of four successive 16x16x4 MFMAs (same mapping for A and B).
  static __device__ __forceinline__ void run(const uint4* As, const uint4* Bs, int wm, int wn,
                                             int kk, f32x4 (&acc)[4][4]) {
    const int l = threadIdx.x & 63;
    const int g = l >> 4, r = l & 15;
    float a[4][4], b[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint4 va = As[swz(wm * 64 + 16 * i + r, kk * 4 + g)];
      const uint4 vb = Bs[swz(wn * 64 + 16 * i + r, kk * 4 + g)];
      const float* pa = reinterpret_cast<const float*>(&va);
      const float* pb = reinterpret_cast<const float*>(&vb);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        a[i][s] = pa[s];
        b[i][s] = pb[s];
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
  }
};

// ---- epilogues -------------------------------------------------------------------

template <class T, int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& p, int split, int m0, int n0,
                                         f32x4 (&acc)[4][4]) {
  const int l = threadIdx.x & 63;
  const int g = l >> 4, r = l & 15;
  const T* bias = reinterpret_cast<const T*>(p.bias);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = n0 + 16 * j + r;
    if (n >= p.N) continue;
    // rotary columns (q, k) are stored pair-interleaved: bias of the original column
    const bool rot = EPI == EPI_STORE_ROPE && n < p.rope_cols;
    const int nb = rot ? n - n % p.rope_d + rope_component(n % p.rope_d, p.rope_d) : n;
    const float bv = (bias != nullptr && split == 0) ? to_f(bias[nb]) : 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + 16 * i + 4 * g + v;
        if (m >= p.M) continue;
        float x = acc[i][j][v] + bv;
        if constexpr (EPI == EPI_STORE || EPI == EPI_STORE_ROPE) {
          if (rot) {   // the pair partner (column n ^ 1, same row) is in lane l ^ 1
            const float y = __shfl_xor(x, 1);
            const float2 cs = rope_cs(p.rope_pos, p.rope_tab, p.rope_d, m, (n % p.rope_d) >> 1);
            x = (n & 1) ? rope_second(y, x, cs, false) : rope_first(x, y, cs, false);
          }
          reinterpret_cast<T*>(p.C)[(int64_t)m * p.ldc + n] = from_f<T>(x);
        } else if constexpr (EPI == EPI_GELU) {
          // GELU and GELU' at the rounded pre-activation u; the backward multiplies by
          // the stored GELU'(u)
          const float u = to_f(from_f<T>(x));
          const bool fast = std::is_same<T, bf16>::value;
          const float gv = fast ? gelu_fast(u) : gelu_f(u);
          if (p.C2)
            reinterpret_cast<T*>(p.C2)[(int64_t)m * p.ldc2 + n] =
                from_f<T>(fast ? gelu_grad_fast(u) : gelu_grad_f(u));
          reinterpret_cast<T*>(p.C)[(int64_t)m * p.ldc + n] = from_f<T>(gv);
        } else if constexpr (EPI == EPI_RESID) {
          const float* R = reinterpret_cast<const float*>(p.aux);
          const float base = R ? R[(int64_t)m * p.ld_aux + n] : 0.0f;
          reinterpret_cast<float*>(p.C)[(int64_t)m * p.ldc + n] = base + x;
        } else if constexpr (EPI == EPI_GELU_BWD) {
          const float gg = to_f(reinterpret_cast<const T*>(p.aux)[(int64_t)m * p.ld_aux + n]);
          reinterpret_cast<T*>(p.C)[(int64_t)m * p.ldc + n] = from_f<T>(x * gg);
        } else {  // EPI_F32: fp32 output (split-K partial slice, or accumulate)
          float* C = reinterpret_cast<float*>(p.C) + (int64_t)split * p.split_stride;
          const int64_t o = (int64_t)m * p.ldc + n;
          C[o] = p.beta ? C[o] + x : x;
        }
      }
    }
  }
}

// ---- the kernel ------------------------------------------------------------------

template <class T, bool AK, bool BKM, int EPI>
__global__ __launch_bounds__(NTHR, 2) void gemm_kernel(GemmArgs p) {
  constexpr int BK = KStep<T>::BK;
  __shared__ uint4 lds_a[2][BM * 8];
  __shared__ uint4 lds_b[2][BN * 8];

  // XCD-aware block order: the hardware deals consecutive block ids round-robin
  // to the 8 XCDs; undo that so each XCD works on a contiguous run of tiles.
  const int ntiles = p.tiles_m * p.tiles_n;
  const int nb = gridDim.x;  // multiple of 8
  const int b = blockIdx.x;
  const int pid = (b % 8) * (nb / 8) + (b / 8);
  if (pid >= ntiles) return;
  const int group = pid / (GROUP_M * p.tiles_n);
  const int first_m = group * GROUP_M;
  const int gsize = min(p.tiles_m - first_m, GROUP_M);
  const int tm = first_m + (pid % gsize);
  const int tn = (pid % (GROUP_M * p.tiles_n)) / gsize;
  const int split = blockIdx.y;

  const int m0 = tm * BM, n0 = tn * BN;
  const int kbeg = split * p.kps;
  const int kend = min(p.K, kbeg + p.kps);
  const int nk = (kend - kbeg + BK - 1) / BK;

  const T* A = reinterpret_cast<const T*>(p.A);
  const T* B = reinterpret_cast<const T*>(p.B);
  const int w = threadIdx.x >> 6;
  const int wm = w >> 1, wn = w & 1;

  f32x4 acc[4][4];
  auto clear = [](f32x4 (&x)[4][4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) x[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear(acc);
  // fp32 products of rows (NT, NN) sum K in the order of the 32x32 kernel of gemm_f32.hip: a
  // chain for each of four quarters (whole 16-deep steps), the quarters in order, so that a
  // row has the same bits from either kernel, whatever else its product holds.  (Costs the 64
  // registers of `total` and 1 to 2.4 % against one chain: 2048x2048x2048 NN 171 -> 173 us,
  // 4096x1536x384 85.6 -> 87.6.)
  constexpr bool QUARTERS = std::is_same<T, float>::value && !AK;
  [[maybe_unused]] f32x4 total[4][4];
  [[maybe_unused]] const int quarter = ((kend - kbeg + 15) / 16 + 3) / 4;
  [[maybe_unused]] int left = quarter;
  if constexpr (QUARTERS) clear(total);

  Regs4 ra, rb;
  auto gload = [&](int k0) {
    if constexpr (AK) load_kmajor<T>(ra, A, p.lda, p.M, m0, k0, kend);
    else load_kcontig<T>(ra, A, p.lda, p.M, m0, k0, kend);
    if constexpr (BKM) load_kmajor<T>(rb, B, p.ldb, p.N, n0, k0, kend);
    else load_kcontig<T>(rb, B, p.ldb, p.N, n0, k0, kend);
  };
  auto lstore = [&](int buf) {
    if constexpr (AK) store_kmajor<T>(lds_a[buf], ra);
    else store_kcontig(lds_a[buf], ra);
    if constexpr (BKM) store_kmajor<T>(lds_b[buf], rb);
    else store_kcontig(lds_b[buf], rb);
  };

  if (nk > 0) {
    gload(kbeg);
    lstore(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      const int cur = kt & 1;
      if (kt + 1 < nk) gload(kbeg + (kt + 1) * BK);
      if constexpr (std::is_same<T, float>::value) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          Mma<T>::run(lds_a[cur], lds_b[cur], wm, wn, kk, acc);
          if constexpr (QUARTERS) {
            if (--left == 0) {
#pragma unroll
              for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) total[i][j] += acc[i][j];
              clear(acc);
              left = quarter;
            }
          }
        }
      } else {
        Mma<T>::run(lds_a[cur], lds_b[cur], wm, wn, acc);
      }
      if (kt + 1 < nk) lstore(cur ^ 1);
      __syncthreads();
    }
  }
  if constexpr (QUARTERS) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = total[i][j] + acc[i][j];
  }
  epilogue<T, EPI>(p, split, m0 + wm * 64, n0 + wn * 64, acc);
}


template <class T, bool AK, bool BKM, int EPI>
hipError_t launch(const GemmArgs& a0, hipStream_t s) {
  GemmArgs a = a0;
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + BN - 1) / BN;
  int nt = a.tiles_m * a.tiles_n;
  int nb = (nt + 7) / 8 * 8;
  int splits = a.kps > 0 ? (a.K + a.kps - 1) / a.kps : 1;
  if (a.kps <= 0) a.kps = a.K;
  if (splits < 1) splits = 1;
  hipLaunchKernelGGL((gemm_kernel<T, AK, BKM, EPI>), dim3(nb, splits), dim3(NTHR), 0, s, a);
  return hipGetLastError();
}

template <class T, bool AK, bool BKM>
hipError_t dispatch_epi(const GemmArgs& a, int epi, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return launch<T, AK, BKM, EPI_STORE>(a, s);
    case EPI_STORE_ROPE: return launch<T, AK, BKM, EPI_STORE_ROPE>(a, s);
    case EPI_GELU: return launch<T, AK, BKM, EPI_GELU>(a, s);
    case EPI_RESID: return launch<T, AK, BKM, EPI_RESID>(a, s);
    case EPI_GELU_BWD: return launch<T, AK, BKM, EPI_GELU_BWD>(a, s);
    case EPI_F32: return launch<T, AK, BKM, EPI_F32>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Host entry: layout = NT (fwd), NN (dX) or TN (dW); requirements checked by the caller:
// K-contiguous operands need K % VEC == 0 and ld % VEC == 0; K-major operands need
// their column count and ld to be multiples of VEC; all pointers 16-byte aligned.
namespace {
// The kernels of gemm_big.hip and gemm_small.hip fetch operands by 16-byte DMA and have
// 16-byte vector epilogues only: every pointer and row stride must keep 16-byte alignment,
// else the general kernel takes the problem.
bool takes_tiled(int dtype, int epi, const GemmArgs& a) {
  if (!(dtype == DT_BF16 && a.N % 8 == 0 && a.K > 0 && a.lda % 8 == 0 && a.ldb % 8 == 0))
    return false;
  auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const bool f32out = epi == EPI_RESID || epi == EPI_F32;
  const int64_t vq = f32out ? 4 : 8;
  return al16(a.A) && al16(a.B) && al16(a.C) && a.ldc % vq == 0 && (a.bias == nullptr || al16(a.bias)) &&
         (a.aux == nullptr || (al16(a.aux) && a.ld_aux % (epi == EPI_RESID ? 4 : 8) == 0)) &&
         (a.C2 == nullptr || (al16(a.C2) && a.ldc2 % 8 == 0)) &&
         (epi != EPI_F32 || a.split_stride % 4 == 0);
}
}  // namespace

namespace {
// fp32: up to half a round of 128x128 tiles (256 CUs) goes to the 32x32 kernel, which has
// sixteen times the blocks and four waves to a tile's K; with more tiles the larger tile's
// reuse wins.  Measured on MI355X, us, 128x128 / 32x32 (M x N x K, tiles): 1040x1536x384
// (108) 42 / 26, 4096x384x1536 (96) 129 / 84, 2048x1152x384 (144) 43 / 35, 1536x1536x4096
// (144) 328 / 343, 2048x1536x384 (192) 44 / 44, 2048x2048x2048 (256) 170 / 288.  In NT
// and NN both kernels add the K terms in the same order: an item's rows must not change with
// what shares its micro-batch.
constexpr int64_t F32_SMALL_TILES = 128;
bool f32_small_tiles(int64_t M, int64_t N, int64_t splits) {
  return (M + BM - 1) / BM * ((N + BN - 1) / BN) * splits <= F32_SMALL_TILES;
}
}  // namespace

namespace {
int splits_of(const GemmArgs& a) { return a.kps > 0 ? std::max(1, (a.K + a.kps - 1) / a.kps) : 1; }
// The tile gemm() runs a takes_tiled problem on.  (gemm_small.hip has the weight-gradient
// layout with the fp32 epilogue only.)
int tile_of(int layout, int epi, const GemmArgs& a) {
  if (a.tile >= 0) return a.tile;
  if (layout == GEMM_TN && epi != EPI_F32) return TILE_BIG;
  return choose_tile(layout, a.M, a.N, a.K, splits_of(a));
}
}  // namespace

int gemm_kernel_of(int dtype, int layout, int epi, const GemmArgs& a) {
  if (takes_tiled(dtype, epi, a)) {
    const int t = tile_of(layout, epi, a);
    if (t != TILE_BIG) return GEMM_K_TILES + t;
    if (a.M >= 512 && a.N >= 256) return GEMM_K_TILES + TILE_BIG;
  }
  if (dtype == DT_F32 && f32_small_tiles(a.M, a.N, splits_of(a))) return GEMM_K_F32_SMALL;
  return GEMM_K_GENERAL;
}

bool gemm_fused_colsum(int dtype, int layout, int epi, const GemmArgs& a) {
  return layout == GEMM_NN && epi == EPI_GELU_BWD && a.kps <= 0 &&
         gemm_kernel_of(dtype, layout, epi, a) == GEMM_K_TILES + TILE_BIG;
}

int gemm_direct_tile(int dtype, int64_t M, int64_t N, int64_t K, const void* W, int64_t ldw) {
  const int vec = dtype == DT_BF16 ? 8 : 4;
  if ((reinterpret_cast<uintptr_t>(W) & 15) != 0 || ldw % vec || K % vec || N % 8) return -1;
  // fp32: the 32x32 kernel reads a K-contiguous weight as fast as a K-major one, so its
  // transposed copy (4 to 9 us a layer of the small encoders) buys nothing
  if (dtype == DT_F32) return f32_small_tiles(M, N, 1) ? 0 : -1;
  // a transposed copy costs its launch and one read and write of the weight at 4 TB/s
  // (1280x1280 to 5120x5120 weights: 4 to 35 us); the large NN kernel then multiplies it
  const int t = choose_tile(GEMM_NN, M, N, K, 1, 2000.0 + 4.0 * N * K / 4000.0);
  return t == TILE_BIG ? -1 : t;
}

hipError_t gemm(int dtype, int layout, int epi, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.colsum && !gemm_fused_colsum(dtype, layout, epi, a)) return hipErrorInvalidValue;
  if (a.rope_rows && (layout != GEMM_NT || epi != EPI_STORE_ROPE || a.tile < 0))
    return hipErrorInvalidValue;
  const int kernel = gemm_kernel_of(dtype, layout, epi, a);
  if (kernel == GEMM_K_TILES + TILE_BIG) return gemm_big(layout, epi, a, s);
  if (kernel >= GEMM_K_TILES) return gemm_small(layout, epi, kernel - GEMM_K_TILES, a, s);
  if (kernel == GEMM_K_F32_SMALL) return gemm_f32_small(layout, epi, a, s);
  if (a.rope_rows) return hipErrorInvalidValue;   // the general kernel takes B as it lies
  if (dtype == DT_BF16) {
    switch (layout) {
      case GEMM_NT: return dispatch_epi<bf16, false, false>(a, epi, s);
      case GEMM_NN: return dispatch_epi<bf16, false, true>(a, epi, s);
      case GEMM_TN: return dispatch_epi<bf16, true, true>(a, epi, s);
    }
  } else {
    switch (layout) {
      case GEMM_NT: return dispatch_epi<float, false, false>(a, epi, s);
      case GEMM_NN: return dispatch_epi<float, false, true>(a, epi, s);
      case GEMM_TN: return dispatch_epi<float, true, true>(a, epi, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace mpipe
