// Candidate vectors with the columns of a row block spread over several workgroups: the raw
// projections u = E[id] W first, then a second kernel that scales each row to unit norm. A workgroup
// that owns whole rows (vectors.hip) has to stream a side's packed weights (6 d^2 bytes: 6.3 MB at
// d = 1024) through one compute unit whatever the number of rows; here it streams its own columns
// only, at the price of passing over u once more.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"
#include "projection.hpp"

namespace lilicorr {
namespace {

typedef __attribute__((address_space(3))) void* cols_lds_t;

struct ColsArgs {
  const int32_t* ids;
  const void* E;               // bf16 or fp32, V d elements below 2 GiB
  const unsigned char* frags;  // packed weights (projection.hpp)
  int64_t M, V;
  int d, nbp, dkp;
  float *in_vec, *out_vec;     // raw projections
};

constexpr uint32_t kColsOut = 0x80000000u;  // past every descriptor: loads return zeros

__device__ __forceinline__ __amdgpu_buffer_rsrc_t cols_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Byte offset in E of the 16-byte (bf16) or 32-byte (fp32) piece that lane l of a row block's A
// fragment takes at k-block 0: row l % 16, values (l / 16) * 8 onwards; kColsOut past M and for ids
// outside [0, V).
__device__ __forceinline__ uint32_t cols_row(const ColsArgs& p, int64_t row_block, int lane,
                                             int elem) {
  const int64_t row = row_block * 16 + (lane & 15);
  const int32_t id = row < p.M ? p.ids[row] : -1;
  return id >= 0 && id < p.V ? (uint32_t)id * (uint32_t)(p.d * elem) + (uint32_t)((lane >> 4) * 8 * elem)
                             : kColsOut;
}

// One accumulator tile (weights x embeddings): lane holds columns col .. col + 3 of row `row`.
__device__ __forceinline__ void cols_store(const ColsArgs& p, int side, const f32x4& v, int64_t row,
                                           int col) {
  if (row < p.M && col < p.d)
    *reinterpret_cast<f32x4*>((side == 0 ? p.in_vec : p.out_vec) + row * p.d + col) = v;
}

// ---- few rows: the contraction split over the waves ---------------------------------------------
// Eight waves on a (16 TM WM) x (16 TN WN) tile of one side: WM x WN blocks of TM x TN accumulator
// tiles and KS = 8 / (WM WN) waves per block that take every KS-th k-block, RING k-blocks in flight
// in registers, no barrier in the loop; the partial sums meet in LDS. fp32 embeddings are split into
// three bf16 terms in registers (eight of the nine products, as in cand_vectors_f32_kernel).
template <bool F32, int TM, int TN, int WM, int WN, int RING>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void vectors_split_kernel(ColsArgs p, int ntn) {
  constexpr int KS = 8 / (WM * WN), F = TM * TN, EPI = F32 ? 2 : 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char cols_smem[];
  f32x4* part = reinterpret_cast<f32x4*>(cols_smem);  // [KS][WM * WN][F][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / (WM * WN), blk = wave % (WM * WN), wm = blk / WN, wn = blk % WN;
  // column tiles innermost: the workgroups that share rows start together
  const int tn = (int)(blockIdx.x % (uint32_t)ntn), side = blockIdx.y;
  const int64_t tm = blockIdx.x / (uint32_t)ntn;
  const uint32_t slice = (uint32_t)p.nbp * 1024u;
  constexpr int ELEM = F32 ? 4 : 2;
  const __amdgpu_buffer_rsrc_t ra = cols_rsrc(p.E, (uint32_t)(p.V * p.d * ELEM));
  const __amdgpu_buffer_rsrc_t rb =
      cols_rsrc(p.frags + (size_t)side * p.dkp * 3 * slice, (uint32_t)p.dkp * 3u * slice);
  uint32_t offA[TM], offB[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) offA[i] = cols_row(p, (tm * WM + wm) * TM + i, lane, ELEM);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int nb = (tn * WN + wn) * TN + j;
    offB[j] = nb < p.nbp ? (uint32_t)(nb * 1024 + lane * 16) : kColsOut;
  }
  u32x4 a[RING][TM][EPI], b[RING][TN][3];
  auto load = [&](int r, int step) {
    const int kb = ks + step * KS;
    const uint32_t past = kb < p.dkp ? 0u : kColsOut;  // uniform; such steps multiply zeros
    const uint32_t k = kb < p.dkp ? (uint32_t)kb : 0u;
    // values past d (the half-empty last k-block) read zeros
    const uint32_t pastA = (int)k * 32 + (lane >> 4) * 8 < p.d ? past : kColsOut;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int e = 0; e < EPI; ++e)
        a[r][i][e] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (offA[i] + (uint32_t)e * 16u) | pastA,
                                                         (int)(k * 32u * ELEM), 0));
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int t = 0; t < 3; ++t)
        b[r][j][t] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rb, offB[j] | past,
                                                         (int)((k * 3u + (uint32_t)t) * slice), 0));
  };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < RING; ++r) load(r, r);
  __builtin_amdgcn_sched_barrier(0);
  const int nsteps = (p.dkp + KS - 1) / KS;
  for (int s = 0; s < nsteps; s += RING) {
#pragma unroll
    for (int r = 0; r < RING; ++r) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        bf16x8 x[3];
        if constexpr (F32) {
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            u32x4 w;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float lo = __uint_as_float(a[r][i][q / 2][(q & 1) * 2]);
              const float hi = __uint_as_float(a[r][i][q / 2][(q & 1) * 2 + 1]);
              w[q] = (uint32_t)split_term(lo, t) | ((uint32_t)split_term(hi, t) << 16);
            }
            x[t] = __builtin_bit_cast(bf16x8, w);
          }
        } else {
          x[0] = __builtin_bit_cast(bf16x8, a[r][i][0]);
        }
        // smallest products first
#pragma unroll
        for (int o = F32 ? 3 : 2; o >= 0; --o)
#pragma unroll
          for (int t = 0; t < (F32 ? 3 : 1); ++t)
            if (o - t >= 0 && o - t < 3)
#pragma unroll
              for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, b[r][j][o - t]), x[t], acc[i][j], 0, 0, 0);
      }
      load(r, s + r + RING);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  f32x4* mine = part + (size_t)(ks * WM * WN + blk) * F * 64 + lane;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) mine[(i * TN + j) * 64] = acc[i][j];
  __syncthreads();
  const int g = lane >> 4, c16 = lane & 15;
  for (int f = ks; f < F; f += KS) {
    const f32x4* q = part + ((size_t)blk * F + f) * 64 + lane;
    f32x4 v = q[0];
#pragma unroll
    for (int k = 1; k < KS; ++k) v = v + q[(size_t)k * WM * WN * F * 64];
    cols_store(p, side, v, ((tm * WM + wm) * TM + f / TN) * 16 + c16,
               ((tn * WN + wn) * TN + f % TN) * 16 + 4 * g);
  }
}

// ---- many rows, bf16: 128 x 128 tiles ------------------------------------------------------------
// Four waves (2 x 2) of 64 x 64, two workgroups per compute unit. The gathered rows reach LDS by DMA
// straight in fragment order (each lane of a copy reads its own row), in a ring of three 64-deep
// stages; the weights go to registers, a k-block (four column blocks, three terms) ahead.
constexpr int kColsStages = 3;
constexpr uint32_t kColsStageBytes = 8 * 2 * 1024;  // 8 row blocks x 2 k-blocks

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void vectors_cols_kernel(ColsArgs p, int ntn) {
  extern __shared__ __attribute__((aligned(16))) unsigned char cols_smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tn = (int)(blockIdx.x % (uint32_t)ntn), side = blockIdx.y;
  const int64_t tm = blockIdx.x / (uint32_t)ntn;
  const uint32_t slice = (uint32_t)p.nbp * 1024u;
  const __amdgpu_buffer_rsrc_t ra = cols_rsrc(p.E, (uint32_t)(p.V * p.d * 2));
  const __amdgpu_buffer_rsrc_t rb =
      cols_rsrc(p.frags + (size_t)side * p.dkp * 3 * slice, (uint32_t)p.dkp * 3u * slice);
  uint32_t offA[2], offB[4];
#pragma unroll
  for (int r = 0; r < 2; ++r) offA[r] = cols_row(p, tm * 8 + wave * 2 + r, lane, 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int nb = tn * 8 + wn * 4 + j;
    offB[j] = nb < p.nbp ? (uint32_t)(nb * 1024 + lane * 16) : kColsOut;
  }
  const int ns = p.dkp / 2;
  auto dma = [&](int s) {
    unsigned char* dst = cols_smem + (uint32_t)(s % kColsStages) * kColsStageBytes +
                         (uint32_t)wave * 2048u;
    const int k0 = s < ns ? s * 64 : 0;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const uint32_t past = s < ns && k0 + kb * 32 + (lane >> 4) * 8 < p.d ? 0u : kColsOut;
#pragma unroll
      for (int r = 0; r < 2; ++r)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (cols_lds_t)(dst + (kb * 8 + r) * 1024), 16,
                                                 offA[r] | past, (k0 + kb * 32) * 2, 0, 0);
    }
  };
  u32x4 b[2][4][3];
  auto load_b = [&](u32x4 (&dst)[4][3], int kb) {
    const uint32_t past = kb < p.dkp ? 0u : kColsOut;
    const uint32_t k = kb < p.dkp ? (uint32_t)kb * 3u * slice : 0u;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        dst[j][t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rb, offB[j] | past, (int)(k + (uint32_t)t * slice), 0));
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // in this order, which the first wait's count relies on: the copies of stage 0, then the 16 loads
  // of stage 1's copies and the first weights
  dma(0);
  __builtin_amdgcn_sched_barrier(0);
  dma(1);
  __builtin_amdgcn_sched_barrier(0);
  load_b(b[0], 0);
  __builtin_amdgcn_sched_barrier(0);
  for (int s = 0; s < ns; ++s) {
    // this wave's copies of stage s have landed once at most 16 loads (the next stage's copies and
    // the first k-block's weights) are in flight; the barrier covers every wave's, and says that all
    // are done with the slot that the next copies overwrite
    __asm__ volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");
    const unsigned char* as = cols_smem + (uint32_t)(s % kColsStages) * kColsStageBytes +
                              (uint32_t)wm * 4096u + (uint32_t)lane * 16u;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      load_b(b[ks ^ 1], 2 * s + ks + 1);
      if (ks == 0) dma(s + 2);  // behind the weights, whose wait would otherwise include it
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(as + (ks * 8 + i) * 1024));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, b[ks][j][t]), a[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // no copy into this workgroup's LDS outlives it
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      cols_store(p, side, acc[i][j], (tm * 8 + wm * 4 + i) * 16 + c16,
                 (tn * 8 + wn * 4 + j) * 16 + 4 * g);
}

// ---- rows to unit norm, in place ------------------------------------------------------------------
// One wave per row of one side.
template <int NV>  // 256-column steps: ceil(d / 256)
__global__ __launch_bounds__(256) void vectors_norm_kernel(float* __restrict__ in_vec,
                                                           float* __restrict__ out_vec, int64_t M,
                                                           int d) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  f32x4* u = reinterpret_cast<f32x4*>((blockIdx.y == 0 ? in_vec : out_vec) + row * d);
  f32x4 v[NV];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = j * 64 + lane;
    v[j] = c * 4 < d ? u[c] : f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) ss = fmaf(v[j][e], v[j][e], ss);
  ss = wave_sum(ss);
  const float inv = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = j * 64 + lane;
    if (c * 4 < d) __builtin_nontemporal_store(v[j] * inv, u + c);
  }
}

template <bool F32, int TM, int TN, int WM, int WN, int RING>
void launch_vectors_split(const ColsArgs& a, hipStream_t stream) {
  constexpr int BM = 16 * TM * WM, BN = TN * WN;
  constexpr size_t lds = (size_t)8 * TM * TN * 64 * 16;
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(vectors_split_kernel<F32, TM, TN, WM, WN, RING>),
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)attr;
  const int ntn = (a.d / 16 + BN - 1) / BN;
  hipLaunchKernelGGL((vectors_split_kernel<F32, TM, TN, WM, WN, RING>),
                     dim3((unsigned)((a.M + BM - 1) / BM * ntn), 2), dim3(512), lds, stream, a, ntn);
}

inline void launch_vectors_cols(const ColsArgs& a, hipStream_t stream) {
  constexpr size_t lds = kColsStages * kColsStageBytes;
  const int ntn = (a.d + 127) / 128;
  hipLaunchKernelGGL(vectors_cols_kernel, dim3((unsigned)((a.M + 127) / 128 * ntn), 2), dim3(256), lds,
                     stream, a, ntn);
}

inline void launch_vectors_norm(const ColsArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)((a.M + 3) / 4), 2), block(256);
  switch ((a.d + 255) / 256) {
    case 1: hipLaunchKernelGGL(vectors_norm_kernel<1>, grid, block, 0, stream, a.in_vec, a.out_vec, a.M, a.d); break;
    case 2: hipLaunchKernelGGL(vectors_norm_kernel<2>, grid, block, 0, stream, a.in_vec, a.out_vec, a.M, a.d); break;
    case 3: hipLaunchKernelGGL(vectors_norm_kernel<3>, grid, block, 0, stream, a.in_vec, a.out_vec, a.M, a.d); break;
    default: hipLaunchKernelGGL(vectors_norm_kernel<4>, grid, block, 0, stream, a.in_vec, a.out_vec, a.M, a.d); break;
  }
}

}  // namespace
}  // namespace lilicorr
