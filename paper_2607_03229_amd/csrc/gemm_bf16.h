// Pieces shared by the bf16 GEMM kernels (gemm_big.hip, gemm_small.hip): the global->LDS
// DMA and its waits, the source addressing of 64-deep K-contiguous tiles, and the
// eight-column vector epilogue.
#pragma once
#include "common.h"
#include "internal.h"

// (the DMA assembly declares the reserved register M0 clobbered, which clang reports)
#pragma clang diagnostic ignored "-Winline-asm"

namespace mpipe {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// The DMAs, and the waits for them, are issued as inline assembly that the compiler
// does not track: it then inserts no waits of its own for them (its conservative
// vmcnt(0) before fragment reads would drain the ring once per pass of the loop).
// This is safe because the main loop has no other vector-memory instructions and
// every DMA is waited for (wait_vm<0>) before the epilogue's loads.
template <int n>
__device__ __forceinline__ void wait_vm() {
  static_assert(n >= 0 && n < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory");
}
// Barrier after this wave's LDS reads have completed; no fence for the DMAs in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// Orders this wave's LDS writes before its later LDS reads (a wave's LDS operations
// execute in issue order; the clobber keeps the compiler from moving accesses across).
__device__ __forceinline__ void lds_wave_fence() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(lds_void*)p;
}

// 16-byte global->LDS DMA of instruction q: lane l writes LDS byte tile + 1024 q + 16 l
// (M0 holds the wave-uniform base).
// M0 is declared clobbered; nothing else in these kernels keeps a value in it.
__device__ __forceinline__ void dma16(const bf16* src, const uint4* tile, int q) {
  const uint32_t base = lds_addr(tile) + 1024u * q;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               ::"v"(src), "s"(__builtin_amdgcn_readfirstlane(base)) : "memory", "m0");
}

// ---- 64-deep K-contiguous tiles --------------------------------------------------------
// Row r's logical 16-byte chunk c (of 8) is stored at c ^ f8(r).
constexpr int BK64 = 64;
__device__ __forceinline__ int f8(int r) { return (r >> 1) & 7; }
// source of instruction q of a 256-row, 64-deep K-contiguous tile (rows r0.., k from k0)
__device__ __forceinline__ const bf16* src_kc64(const bf16* X, int64_t ld, int rows, int r0,
                                                int k0, int kend, int q) {
  const int l = threadIdx.x & 63;
  const int row = 8 * q + (l >> 3);
  int k = k0 + 8 * ((l & 7) ^ f8(row));
  k = k < kend ? k : kend - 8;
  int gr = r0 + row;
  gr = gr < rows ? gr : rows - 1;
  return X + (int64_t)gr * ld + k;
}

// ---- epilogue ------------------------------------------------------------------------

// The vector epilogue works on 8 consecutive outputs (m, n..n+7) of a lane.  Its global
// operands (GELU' factor, residual, accumulate target) are fetched one staging pass
// ahead, so their latency overlaps the previous pass instead of stalling each store.
struct AuxV { uint4 v[2]; };

template <int EPI>
__device__ __forceinline__ void aux_fetch(const GemmArgs& p, int split, int m, int n, AuxV& a) {
  if constexpr (EPI == EPI_GELU_BWD) {
    a.v[0] = *reinterpret_cast<const uint4*>(reinterpret_cast<const bf16*>(p.aux) +
                                             (int64_t)m * p.ld_aux + n);
  } else if constexpr (EPI == EPI_RESID) {
    if (p.aux) {
      const float* R = reinterpret_cast<const float*>(p.aux) + (int64_t)m * p.ld_aux + n;
      a.v[0] = *reinterpret_cast<const uint4*>(R);
      a.v[1] = *reinterpret_cast<const uint4*>(R + 4);
    }
  } else if constexpr (EPI == EPI_F32) {
    if (p.beta) {
      const float* C = reinterpret_cast<const float*>(p.C) + (int64_t)split * p.split_stride +
                       (int64_t)m * p.ldc + n;
      a.v[0] = *reinterpret_cast<const uint4*>(C);
      a.v[1] = *reinterpret_cast<const uint4*>(C + 4);
    }
  } else if constexpr (EPI == EPI_STORE_ROPE) {
    // (cos, sin) of the four rotary pairs of columns n..n+7 at row m: consecutive table
    // entries (a head's d/4 pairs per axis are a multiple of 4, so they share an axis)
    if (n < p.rope_cols) {
      const int q4 = p.rope_d >> 2, j0 = (n % p.rope_d) >> 1;
      const uint32_t pp = (uint32_t)p.rope_pos[m];
      const int coord = (int)(j0 < q4 ? (pp >> 16) : (pp & 0xFFFFu));
      const float2* t = p.rope_tab + coord * q4 + (j0 < q4 ? j0 : j0 - q4);
      a.v[0] = *reinterpret_cast<const uint4*>(t);
      a.v[1] = *reinterpret_cast<const uint4*>(t + 2);
    }
  }
}

// The bias of a lane's eight columns n..n+7 (zeros when `take` is false).  Columns that
// get the fused rotary position are stored pair-interleaved, so their bias entries come
// from the original columns.
__device__ __forceinline__ void load_bias8(const GemmArgs& p, bool take, int n, float* bias8) {
#pragma unroll
  for (int e = 0; e < 8; ++e) bias8[e] = 0.f;
  if (!take || p.bias == nullptr) return;
  const bf16* bias = reinterpret_cast<const bf16*>(p.bias);
  if (p.rope_pos != nullptr && n < p.rope_cols) {   // EPI_STORE_ROPE's q, k columns
    const int base = n - n % p.rope_d, s0 = n % p.rope_d;   // eight columns of one head
#pragma unroll
    for (int e = 0; e < 8; ++e) bias8[e] = (float)bias[base + rope_component(s0 + e, p.rope_d)];
    return;
  }
  const uint4 bb = *reinterpret_cast<const uint4*>(bias + n);
  const bf16* b8 = reinterpret_cast<const bf16*>(&bb);
#pragma unroll
  for (int e = 0; e < 8; ++e) bias8[e] = (float)b8[e];
}

template <int EPI>
__device__ __forceinline__ void epi8_vec(const GemmArgs& p, int split, int m, int n, float* v,
                                         const float* bias8, const AuxV& ax,
                                         float* sum8 = nullptr) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] += bias8[e];
  if constexpr (EPI == EPI_STORE || EPI == EPI_STORE_ROPE || EPI == EPI_GELU ||
                EPI == EPI_GELU_BWD) {
    bf16 o[8];
    if constexpr (EPI == EPI_STORE || EPI == EPI_STORE_ROPE) {
      if constexpr (EPI == EPI_STORE_ROPE) {
        if (n < p.rope_cols) {   // q, k: rotate the four pairs by the prefetched angles
          const float2* cs = reinterpret_cast<const float2*>(&ax.v[0]);
#pragma unroll
          for (int e = 0; e < 8; e += 2) rope_rotate(v[e], v[e + 1], cs[e / 2]);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (bf16)v[e];
    } else if constexpr (EPI == EPI_GELU) {
      // GELU and its derivative at the bf16-rounded pre-activation u, from one Phi/phi
      // evaluation; the derivative is what the backward needs of u
      bf16 gd[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float u = (float)(bf16)v[e];
        float P, dens;
        phi_pair(u, P, dens);
        o[e] = (bf16)(u * P);
        gd[e] = (bf16)fmaf(u, dens, P);
      }
      if (p.C2)
        *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(p.C2) + (int64_t)m * p.ldc2 + n) =
            *reinterpret_cast<const uint4*>(gd);
    } else {   // EPI_GELU_BWD: aux holds GELU'(u) from the forward
      const bf16* g8 = reinterpret_cast<const bf16*>(&ax.v[0]);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (bf16)(v[e] * (float)g8[e]);
      if (sum8) {   // column sums of what is stored (the next bias gradient)
#pragma unroll
        for (int e = 0; e < 8; ++e) sum8[e] += (float)o[e];
      }
    }
    *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(p.C) + (int64_t)m * p.ldc + n) =
        *reinterpret_cast<const uint4*>(o);
  } else {   // EPI_RESID, EPI_F32: fp32 out, plus the fetched residual / previous value
    float* C = reinterpret_cast<float*>(p.C) +
               (EPI == EPI_F32 ? (int64_t)split * p.split_stride : 0) + (int64_t)m * p.ldc + n;
    const bool add = EPI == EPI_RESID ? p.aux != nullptr : p.beta != 0;
    const float* r8 = reinterpret_cast<const float*>(&ax.v[0]);
    float4 a = make_float4(v[0], v[1], v[2], v[3]), b = make_float4(v[4], v[5], v[6], v[7]);
    if (add) {
      a.x += r8[0]; a.y += r8[1]; a.z += r8[2]; a.w += r8[3];
      b.x += r8[4]; b.y += r8[5]; b.z += r8[6]; b.w += r8[7];
    }
    *reinterpret_cast<float4*>(C) = a;
    *reinterpret_cast<float4*>(C + 4) = b;
  }
}

}  // namespace
}  // namespace mpipe
