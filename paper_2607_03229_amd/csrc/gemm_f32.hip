// fp32 GEMMs of few tiles: C[M,N] = sum_k A(m,k) B(n,k) for the small fp32 encoders.
//
// An fp32 encoder of a few hundred rows gives the general kernel's 128x128 tiles to a
// handful of CUs, each then walking all of K alone (1,040 x 384 x 384: 27 tiles, 41 us for
// 0.3 GFLOP).  Here a block owns a 32x32 tile and its four waves a quarter of K each, so
// that product has 396 blocks of 1,584 waves and a quarter of the serial chain; the four
// partial tiles are added in wave order through LDS, which also lays the output out for
// four consecutive columns per thread.
//
// Every wave holds a 2x2 grid of v_mfma_f32_16x16x4_f32 accumulators and loads its own
// operands from L2 to registers, four 16-deep K steps ahead (no LDS or barrier in the
// loop): of a K step lane (g, r) = (l / 16, l % 16) holds reduction indices 4g .. 4g + 3,
// which are the operands of four successive MFMAs.
//   K-contiguous operand ([rows][ld]): one 16-byte load per 16 rows; sub-tile i holds rows
//     16 i + r
//   K-major operand ([k][ld]): one 8-byte load per k, columns 2r and 2r + 1; sub-tile i
//     holds columns 2 r + i, so a load covers whole 128-byte lines
// Measured on MI355X, us, general kernel -> this one: 1040x384x384 NN 41 -> 9.4,
// 1040x384x1536 NN 128 -> 27, 384x1536x1040 TN 92 -> 30, 41x512x512 NN 48 -> 8.9; the
// largest run at 55 to 60 TFLOP/s, bound by the L2-to-register loads (8 bytes per cycle and
// wave at the full MFMA rate).
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace mpipe {
namespace {

constexpr int T = 32, NTHR = 256, GROUP_M = 8, BK = 16, AHEAD = 4, PITCH = 36;

// 2 sub-tiles x 4 reduction indices of one operand's K step
struct Frag {
  float v[2][4];
};

// rows (columns, when KM) r0.. of an operand at K step k0: zero past kend, clamped rows
// (row_of: the row to read for tile row `row`)
template <bool KM, class RowOf>
__device__ __forceinline__ void load_frag(Frag& F, const float* X, int64_t ld, int rows, int r0,
                                          int k0, int kend, int g, int r, RowOf row_of) {
  const int k = k0 + 4 * g;
  if constexpr (KM) {
    int c = r0 + 2 * r;
    c = c < rows ? c : 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float2 x = make_float2(0.f, 0.f);
      if (k + s < kend) x = *reinterpret_cast<const float2*>(X + (int64_t)(k + s) * ld + c);
      F.v[0][s] = x.x;
      F.v[1][s] = x.y;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int row = r0 + 16 * i + r;
      row = row_of(row < rows ? row : rows - 1);
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < kend) x = *reinterpret_cast<const float4*>(X + (int64_t)row * ld + k);
      F.v[i][0] = x.x;
      F.v[i][1] = x.y;
      F.v[i][2] = x.z;
      F.v[i][3] = x.w;
    }
  }
}

// Epilogue of outputs (m, n .. n + 3), of which the first `cnt` are in range; `vec`: all
// rows involved are 16-byte aligned.
template <int EPI>
__device__ __forceinline__ void epilogue4(const GemmArgs& p, int split, int m, int n, int cnt,
                                          bool vec, float (&x)[4]) {
  const float* bias = reinterpret_cast<const float*>(p.bias);
  const bool rot = EPI == EPI_STORE_ROPE && n < p.rope_cols;   // four columns of one head
  if (bias != nullptr && split == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < cnt)
        x[e] += bias[rot ? n - n % p.rope_d + rope_component(n % p.rope_d + e, p.rope_d) : n + e];
  }
  if (rot) {
    const int j = (n % p.rope_d) >> 1;
    rope_rotate(x[0], x[1], rope_cs(p.rope_pos, p.rope_tab, p.rope_d, m, j));
    rope_rotate(x[2], x[3], rope_cs(p.rope_pos, p.rope_tab, p.rope_d, m, j + 1));
  }
  auto load4 = [&](const float* q, float (&v)[4]) {
    if (vec) {
      const float4 t = *reinterpret_cast<const float4*>(q);
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = e < cnt ? q[e] : 0.f;
    }
  };
  auto store4 = [&](float* q, const float (&v)[4]) {
    if (vec) {
      *reinterpret_cast<float4*>(q) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < cnt) q[e] = v[e];
    }
  };
  float* C = reinterpret_cast<float*>(p.C) + (int64_t)m * p.ldc + n;
  float y[4];
  if constexpr (EPI == EPI_GELU) {
    if (p.C2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = gelu_grad_f(x[e]);
      store4(reinterpret_cast<float*>(p.C2) + (int64_t)m * p.ldc2 + n, y);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = gelu_f(x[e]);
  } else if constexpr (EPI == EPI_RESID) {
    if (p.aux) {
      load4(reinterpret_cast<const float*>(p.aux) + (int64_t)m * p.ld_aux + n, y);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = y[e] + x[e];
    }
  } else if constexpr (EPI == EPI_GELU_BWD) {
    load4(reinterpret_cast<const float*>(p.aux) + (int64_t)m * p.ld_aux + n, y);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] *= y[e];
  } else if constexpr (EPI == EPI_F32) {
    C += (int64_t)split * p.split_stride;
    if (p.beta) {
      load4(C, y);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = y[e] + x[e];
    }
  }
  store4(C, x);
}

template <bool AK, bool BKM, int EPI>
__global__ __launch_bounds__(NTHR) void gemm_f32_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) float red[4][T][PITCH];
  // XCD-aware tile order, as in the general kernel
  const int ntiles = p.tiles_m * p.tiles_n;
  const int nb = gridDim.x;   // multiple of 8
  const int pid = (blockIdx.x % 8) * (nb / 8) + (blockIdx.x / 8);
  if (pid >= ntiles) return;
  const int group = pid / (GROUP_M * p.tiles_n);
  const int first_m = group * GROUP_M;
  const int gsize = min(p.tiles_m - first_m, GROUP_M);
  const int m0 = (first_m + (pid % gsize)) * T;
  const int n0 = ((pid % (GROUP_M * p.tiles_n)) / gsize) * T;
  const int split = blockIdx.y;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, g = l >> 4, r = l & 15;
  // this wave's quarter of the split's K steps
  const int ke = min(p.K, (split + 1) * p.kps);
  const int steps = max(0, (ke - split * p.kps + BK - 1) / BK);
  const int per = (steps + 3) / 4;
  const int kbeg = split * p.kps + w * per * BK;
  const int kend = min(ke, kbeg + per * BK);
  const int nt = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  const float* A = reinterpret_cast<const float*>(p.A);
  const float* B = reinterpret_cast<const float*>(p.B);

  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto a_row = [](int row) { return row; };
  // B's row behind output column n (GemmArgs::rope_rows)
  auto b_row = [&](int n) {
    return EPI == EPI_STORE_ROPE && p.rope_rows ? rope_weight_row(n, p.rope_d, p.rope_cols) : n;
  };
  Frag a[AHEAD], b[AHEAD];
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (u < nt) {
      load_frag<AK>(a[u], A, p.lda, p.M, m0, kbeg + u * BK, kend, g, r, a_row);
      load_frag<BKM>(b[u], B, p.ldb, p.N, n0, kbeg + u * BK, kend, g, r, b_row);
    }
  for (int t = 0; t < nt; t += AHEAD)
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (t + u < nt) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].v[i][s], b[u].v[j][s],
                                                               acc[i][j], 0, 0, 0);
        if (t + u + AHEAD < nt) {
          const int k0 = kbeg + (t + u + AHEAD) * BK;
          load_frag<AK>(a[u], A, p.lda, p.M, m0, k0, kend, g, r, a_row);
          load_frag<BKM>(b[u], B, p.ldb, p.N, n0, k0, kend, g, r, b_row);
        }
      }
  // sub-tile (i, j), element (4g + v, r): tile row and column by operand form
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        red[w][AK ? 2 * (4 * g + v) + i : 16 * i + 4 * g + v][BKM ? 2 * r + j : 16 * j + r] =
            acc[i][j][v];
  __syncthreads();
  const int tr = threadIdx.x >> 3, tc = 4 * (threadIdx.x & 7);
  const int m = m0 + tr, n = n0 + tc;
  if (m >= p.M || n >= p.N) return;
  float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float4 t = *reinterpret_cast<const float4*>(&red[k][tr][tc]);
    x[0] += t.x; x[1] += t.y; x[2] += t.z; x[3] += t.w;
  }
  const int cnt = min(4, p.N - n);
  const bool vec = cnt == 4 && p.ldc % 4 == 0 && p.ld_aux % 4 == 0 && p.ldc2 % 4 == 0 &&
                   p.split_stride % 4 == 0 &&
                   ((reinterpret_cast<uintptr_t>(p.C) | reinterpret_cast<uintptr_t>(p.aux) |
                     reinterpret_cast<uintptr_t>(p.C2)) & 15) == 0;
  epilogue4<EPI>(p, split, m, n, cnt, vec, x);
}

template <bool AK, bool BKM, int EPI>
hipError_t launch(const GemmArgs& a0, hipStream_t s) {
  GemmArgs a = a0;
  a.tiles_m = (a.M + T - 1) / T;
  a.tiles_n = (a.N + T - 1) / T;
  const int nb = (a.tiles_m * a.tiles_n + 7) / 8 * 8;
  const int splits = a.kps > 0 ? std::max(1, (a.K + a.kps - 1) / a.kps) : 1;
  if (a.kps <= 0) a.kps = a.K;
  hipLaunchKernelGGL((gemm_f32_kernel<AK, BKM, EPI>), dim3(nb, splits), dim3(NTHR), 0, s, a);
  return hipGetLastError();
}

template <bool AK, bool BKM>
hipError_t dispatch(const GemmArgs& a, int epi, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return launch<AK, BKM, EPI_STORE>(a, s);
    case EPI_STORE_ROPE: return launch<AK, BKM, EPI_STORE_ROPE>(a, s);
    case EPI_GELU: return launch<AK, BKM, EPI_GELU>(a, s);
    case EPI_RESID: return launch<AK, BKM, EPI_RESID>(a, s);
    case EPI_GELU_BWD: return launch<AK, BKM, EPI_GELU_BWD>(a, s);
    case EPI_F32: return launch<AK, BKM, EPI_F32>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t gemm_f32_small(int layout, int epi, const GemmArgs& a, hipStream_t s) {
  switch (layout) {
    case GEMM_NT: return dispatch<false, false>(a, epi, s);
    case GEMM_NN: return dispatch<false, true>(a, epi, s);
    case GEMM_TN: return dispatch<true, true>(a, epi, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace mpipe
