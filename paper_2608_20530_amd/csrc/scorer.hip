// Scoring-Transformer stand-in on gfx950: the encoder of the paper's speculative head
// (implementation appendix, "Architecture"; widths and depth from the hyper-parameter table), a
// stack of pre-norm bidirectional Transformer layers over each request's candidate lattice of
// S slots x K candidates, with per-head slot-distance and same-slot attention biases.
//
// One layer is seven launches (few rows: the QKV and SiLU products make their own norms, five):
//   rmsnorm -> bf16            X fp32 [M][H] -> xn bf16                       (HBM bound)
//   GEMM  xn . Wqkv            -> Q, K bf16 [M][2H] and V^T bf16 [N][H][Lv]   (matrix cores)
//   lattice attention          one workgroup per (request, head); K and V^T of the request in LDS
//   GEMM  attn . Wo, X +=      residual update in place                      (matrix cores)
//   rmsnorm -> bf16
//   GEMM  hn . W1 -> silu -> bf16 [M][F]                                     (matrix cores)
//   GEMM  a . W2, X +=                                                        (matrix cores)
// M = N * L token rows. Every matrix-core input is bf16 (round to nearest even), products
// accumulate in fp32 on v_mfma_f32_16x16x32_bf16, the residual stream stays fp32.
//
// The products are in scorer_gemm.hpp; their A operands (xn, attn, a) live in its fragment order,
// written so by the kernels that produce them, and so do the packed weights.
//
// Attention: S^T = K Q^T per 16-query chunk (keys are the MFMA rows), so each lane ends up with
// one query's logits over keys 16t + 4g + i (g = lane / 16); the softmax reduces over tiles in
// registers and over the four lane groups by shuffles, and the probabilities are already in the
// A-operand layout of P V once the k slots of a 32-key step are read as keys (4g + j, 16 + 4g + j):
// V^T is read with the same key order, so no LDS round trip is needed for P.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "common.hpp"
#include "lilicorr.h"
#include "scorer_gemm.hpp"

namespace lilicorr {
namespace {

constexpr int kHd = 128;  // head width
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kAttnThreads = 512;
constexpr int kMaxL = 256;
constexpr int kMaxH = 4096;
constexpr int kMaxF = 16384;
constexpr int64_t kMaxS = 256;
constexpr size_t kAlign = 256;

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// ---- RMSNorm -> bf16 ----------------------------------------------------------------------------
// y = bf16(x / sqrt(mean(x^2) + eps) * g) over rows of H = NV * 256 fp32 values, written in the
// matrix products' fragment order. One wave per row, WAVES rows per workgroup: the rounded rows
// meet in LDS (padded by 16 bytes, so that the rows of a fragment read fall in distinct banks) and
// leave as 16-byte lanes of their fragments.
template <int NV, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void rmsnorm_bf16_kernel(const float* __restrict__ X,
                                                                  const float* __restrict__ g,
                                                                  unsigned char* __restrict__ Y,
                                                                  int64_t M) {
  constexpr int H = NV * 256, stride = H * 2 + 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char rms_smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * WAVES;
  const int64_t row = row0 + wave < M ? row0 + wave : M - 1;
  const float4* x = reinterpret_cast<const float4*>(X + row * H);
  float4 v[NV];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    v[j] = x[j * 64 + lane];
    ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
  }
  ss = wave_sum(ss);
  const float inv = 1.0f / sqrtf(ss / (float)H + kEps);
  const float4* gg = reinterpret_cast<const float4*>(g);
  u32x2* y = reinterpret_cast<u32x2*>(rms_smem + wave * stride);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const float4 w = gg[j * 64 + lane];
    y[j * 64 + lane] = u32x2{pack_bf16x2(v[j].x * inv * w.x, v[j].y * inv * w.y),
                             pack_bf16x2(v[j].z * inv * w.z, v[j].w * inv * w.w)};
  }
  __syncthreads();
  // piece i: row i % WAVES, 16-byte chunk i / WAVES
  for (int i = tid; i < WAVES * H / 8; i += WAVES * 64) {
    const int r = i % WAVES, c = i / WAVES;
    if (row0 + r < M)
      *reinterpret_cast<u32x4*>(Y + frag_offset(row0 + r, c * 8, (M + 15) / 16)) =
          *reinterpret_cast<const u32x4*>(rms_smem + r * stride + c * 16);
  }
}

// ---- lattice attention ----------------------------------------------------------------------
struct AttnArgs {
  const uint16_t* qk;    // [N * L][2H]: Q at column h * 128, K at H + h * 128
  const uint16_t* vt;    // [N][H][Lv]
  const float* dist;     // [heads][2S - 1]
  const float* same;     // [heads]
  uint16_t* out;         // [N * L][H], fragment order
  int S, K, L, Lv, Lp, H, heads;
};

// Lattices with S * Lp <= kBiasRows keep one row of additive logit bias per query slot in LDS
// (slot-distance and same-slot terms in log2 units, -inf past the last key); larger ones look the
// bias up per element.
constexpr int kBiasRows = 4096;

inline bool attn_bias_rows(int Lp, int S) { return (int64_t)S * Lp <= kBiasRows; }

inline size_t attn_lds_bytes(int Lp, int S) {
  return (size_t)Lp * kHd * 2 + (size_t)kHd * (Lp + 4) * 2 + (size_t)((2 * S + 3) & ~3) * 4 +
         (size_t)Lp * 4 + (attn_bias_rows(Lp, S) ? (size_t)S * Lp * 4 : 0);
}

// NT = Lp / 16 key tiles (even, 2..16): the key loops are unrolled exactly.
template <bool ROWS, int NT>
__global__ __launch_bounds__(kAttnThreads) void lattice_attention_kernel(AttnArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int n = blockIdx.x / p.heads, h = blockIdx.x - n * p.heads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int Lp = 16 * NT, vstride = Lp + 4;
  const int L = p.L;
  uint16_t* sK = reinterpret_cast<uint16_t*>(smem);        // [Lp][128], chunk c of key j at c ^ (j % 8)
  uint16_t* sV = sK + Lp * kHd;                              // [128][Lp + 4]
  float* sBias = reinterpret_cast<float*>(sV + kHd * vstride);  // [2S - 1] dist, [2S - 1] same (log2 units)
  int* sSlot = reinterpret_cast<int*>(sBias + ((2 * p.S + 3) & ~3));  // [Lp] key slot, -1 past L
  float* sRow = reinterpret_cast<float*>(sSlot + Lp);  // ROWS: [S][Lp] bias of query slot x key
  const int64_t tok0 = (int64_t)n * L;
  const int64_t row_blocks = ((int64_t)(gridDim.x / p.heads) * L + 15) / 16;
  const int H2 = 2 * p.H;

  const int g = lane >> 4, c16 = lane & 15;
  const int nq = (L + 15) / 16;
  // Q fragments of this wave's first query chunk, loaded while K and V^T are staged
  bf16x8 qf[4];
  auto load_q = [&](int qc) {
    const int q = qc * 16 + c16;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      u32x4 v = u32x4{0u, 0u, 0u, 0u};
      if (q < L)
        v = *reinterpret_cast<const u32x4*>(p.qk + (tok0 + q) * H2 + h * kHd + ks * 32 + g * 8);
      qf[ks] = __builtin_bit_cast(bf16x8, v);
    }
  };
  if (wave < nq) load_q(wave);

  // K rows (16 chunks of 16 bytes each) and V^T rows (Lp / 8 = 2 NT chunks each): NT / 2 chunks
  // of each per thread, every load issued before the first LDS store
  constexpr int kPer = NT / 2;  // (Lp * 16) / 512 == (128 * Lp / 8) / 512
  constexpr int cpr = 2 * NT;
  u32x4 kv[2 * kPer];
#pragma unroll
  for (int b = 0; b < kPer; ++b) {
    const int i = tid + b * kAttnThreads;
    const int j = i >> 4, c = i & 15;
    kv[b] = u32x4{0u, 0u, 0u, 0u};
    if (j < L)
      kv[b] = *reinterpret_cast<const u32x4*>(p.qk + (tok0 + j) * H2 + p.H + h * kHd + c * 8);
  }
#pragma unroll
  for (int b = 0; b < kPer; ++b) {
    const int i = tid + b * kAttnThreads;
    const int c = i / cpr, pos = (i - c * cpr) * 8;
    kv[kPer + b] = u32x4{0u, 0u, 0u, 0u};
    if (pos < p.Lv)
      kv[kPer + b] = *reinterpret_cast<const u32x4*>(
          p.vt + ((int64_t)n * p.H + h * kHd + c) * p.Lv + pos);
  }
#pragma unroll
  for (int b = 0; b < kPer; ++b) {
    const int i = tid + b * kAttnThreads;
    const int j = i >> 4, c = i & 15;
    *reinterpret_cast<u32x4*>(sK + j * kHd + ((c ^ (j & 7)) << 3)) = kv[b];
  }
#pragma unroll
  for (int b = 0; b < kPer; ++b) {
    const int i = tid + b * kAttnThreads;
    const int c = i / cpr, pos = (i - c * cpr) * 8;
    u32x4 w = kv[kPer + b];
    const int nv = L - pos;  // keys of this chunk inside the lattice; the rest must be zero
    if (nv < 8) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t keep = (2 * e + 1 < nv) ? 0xffffffffu : (2 * e < nv ? 0x0000ffffu : 0u);
        w[e] &= keep;
      }
    }
    u32x2* dst = reinterpret_cast<u32x2*>(sV + c * vstride + pos);
    dst[0] = u32x2{w.x, w.y};
    dst[1] = u32x2{w.z, w.w};
  }
  const int nb = 2 * p.S - 1;
  for (int i = tid; i < nb; i += kAttnThreads) sBias[i] = p.dist[(int64_t)h * nb + i] * kLog2e;
  if (tid == 0) sBias[nb] = p.same[h] * kLog2e;
  for (int i = tid; i < Lp; i += kAttnThreads) sSlot[i] = i < L ? i / p.K : -1;
  if constexpr (ROWS) {
    __syncthreads();  // the rows read the slot and bias tables
    for (int i = tid; i < p.S * Lp; i += kAttnThreads) {
      const int sq = i / Lp, key = i - sq * Lp;
      const int sk = sSlot[key];
      float b = -__builtin_inff();
      if (sk >= 0) {
        const int d = sq - sk;
        b = sBias[d + p.S - 1] + (d == 0 ? sBias[nb] : 0.f);
      }
      sRow[i] = b;
    }
  }
  __syncthreads();

  const float zscale = kLog2e * 0.08838834764831845f;  // log2(e) / sqrt(128)
  const float same_b = sBias[nb];
  constexpr int kWaves = kAttnThreads / 64;
  for (int qc = wave; qc < nq; qc += kWaves) {
    const int q = qc * 16 + c16;
    // logits of query q (this lane's column) against keys 16t + 4g + i
    f32x4 s[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(
            sK + (t * 16 + c16) * kHd + (((ks * 4 + g) ^ (c16 & 7)) << 3));
        s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[ks], s[t], 0, 0, 0);
      }
      // one tile's fragments at a time (hoisting every tile's reads would take 4 NT registers)
      __builtin_amdgcn_sched_barrier(0);
    }
    if (qc + kWaves < nq) load_q(qc + kWaves);  // the next chunk's fragments, in flight
    const int sq = q < L ? q / p.K : 0;
    float mx = -__builtin_inff();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      {
        if constexpr (ROWS) {
          const f32x4 b = *reinterpret_cast<const f32x4*>(sRow + sq * Lp + t * 16 + 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[t][i] = fmaf(s[t][i], zscale, b[i]);
            mx = fmaxf(mx, s[t][i]);
          }
        } else {
          const i32x4 sk = *reinterpret_cast<const i32x4*>(sSlot + t * 16 + 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float z = -__builtin_inff();
            if (sk[i] >= 0) {
              const int d = sq - sk[i];
              z = s[t][i] * zscale + sBias[d + p.S - 1] + (d == 0 ? same_b : 0.f);
            }
            s[t][i] = z;
            mx = fmaxf(mx, z);
          }
        }
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float e = __builtin_amdgcn_exp2f(s[t][i] - mx);
          s[t][i] = e;
          sum += e;
        }
      }
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    const float rs = 1.0f / sum;

    // O^T = V^T P^T: the V^T rows (head dimensions) are the MFMA rows and the probabilities of
    // this lane's query the columns, so each lane ends with four consecutive dimensions of one
    // query (one 8-byte store per 16-dimension tile)
    f32x4 o[kHd / 16];
#pragma unroll
    for (int dt = 0; dt < kHd / 16; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NT / 2; ++u) {
      const u32x4 pw = u32x4{pack_bf16x2(s[2 * u][0] * rs, s[2 * u][1] * rs),
                             pack_bf16x2(s[2 * u][2] * rs, s[2 * u][3] * rs),
                             pack_bf16x2(s[2 * u + 1][0] * rs, s[2 * u + 1][1] * rs),
                             pack_bf16x2(s[2 * u + 1][2] * rs, s[2 * u + 1][3] * rs)};
      const bf16x8 pb = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
      for (int dt = 0; dt < kHd / 16; ++dt) {
        const uint16_t* vr = sV + (dt * 16 + c16) * vstride + u * 32 + 4 * g;
        const u32x2 lo = *reinterpret_cast<const u32x2*>(vr);
        const u32x2 hi = *reinterpret_cast<const u32x2*>(vr + 16);
        const bf16x8 va = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb, o[dt], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // lane holds query qc * 16 + c16, head dimensions dt * 16 + 4g + i
    if (q < L) {
      // dimensions dt * 16 onwards are half of k-block dt / 2: 32 lanes on in its fragment
      unsigned char* dst = reinterpret_cast<unsigned char*>(p.out) +
                           frag_offset(tok0 + q, h * kHd + 4 * g, row_blocks);
#pragma unroll
      for (int dt = 0; dt < kHd / 16; ++dt)
        *reinterpret_cast<u32x2*>(dst + (dt / 2) * row_blocks * kFragBytes + (dt & 1) * 512) =
            u32x2{pack_bf16x2(o[dt][0], o[dt][1]), pack_bf16x2(o[dt][2], o[dt][3])};
    }
  }
}

template <bool ROWS, int NT>
void launch_attention_nt(const AttnArgs& at, int64_t N, size_t lds, hipStream_t stream) {
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(lattice_attention_kernel<ROWS, NT>),
      hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)attr;
  hipLaunchKernelGGL((lattice_attention_kernel<ROWS, NT>), dim3((unsigned)(N * at.heads)),
                     dim3(kAttnThreads), lds, stream, at);
}

template <bool ROWS>
void launch_attention_rows(const AttnArgs& at, int64_t N, size_t lds, hipStream_t stream) {
  switch (at.Lp / 16) {
    case 2: launch_attention_nt<ROWS, 2>(at, N, lds, stream); break;
    case 4: launch_attention_nt<ROWS, 4>(at, N, lds, stream); break;
    case 6: launch_attention_nt<ROWS, 6>(at, N, lds, stream); break;
    case 8: launch_attention_nt<ROWS, 8>(at, N, lds, stream); break;
    case 10: launch_attention_nt<ROWS, 10>(at, N, lds, stream); break;
    case 12: launch_attention_nt<ROWS, 12>(at, N, lds, stream); break;
    case 14: launch_attention_nt<ROWS, 14>(at, N, lds, stream); break;
    default: launch_attention_nt<ROWS, 16>(at, N, lds, stream); break;
  }
}

void launch_attention(const AttnArgs& at, int64_t N, size_t lds, hipStream_t stream) {
  if (attn_bias_rows(at.Lp, at.S))
    launch_attention_rows<true>(at, N, lds, stream);
  else
    launch_attention_rows<false>(at, N, lds, stream);
}

// ---- packing ------------------------------------------------------------------------------------
// in[R][C] (both multiples of 32) into fragment order, 32 x 32 tiles via LDS: column block n, k-block
// kb of the result hold in[32 kb ..][16 n ..].
__global__ __launch_bounds__(256) void pack_frag_kernel(const uint16_t* __restrict__ in,
                                                        uint16_t* __restrict__ out, int R, int C) {
  __shared__ uint16_t t[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int y = ty; y < 32; y += 8) t[y][tx] = in[(int64_t)(r0 + y) * C + c0 + tx];
  __syncthreads();
  // two fragments of 64 lanes x 8 values, four values per thread
  const int nb = threadIdx.x >> 7, l = (threadIdx.x >> 1) & 63, e0 = (threadIdx.x & 1) * 4;
  uint16_t* o = out + ((int64_t)(r0 / 32) * (C / 16) + c0 / 16 + nb) * 512 + l * 8 + e0;
  for (int e = 0; e < 4; ++e) o[e] = t[(l >> 4) * 8 + e0 + e][nb * 16 + (l & 15)];
}

struct PackedLayout {
  size_t qkv, o, w1, w2, g_attn, g_ffn, dist, same, total;
};

inline PackedLayout packed_layout(int H, int heads, int F, int64_t S) {
  PackedLayout l;
  size_t at = 0;
  l.qkv = at; at = align_up(at + (size_t)3 * H * H * 2);
  l.o = at; at = align_up(at + (size_t)H * H * 2);
  l.w1 = at; at = align_up(at + (size_t)F * H * 2);
  l.w2 = at; at = align_up(at + (size_t)H * F * 2);
  l.g_attn = at; at = align_up(at + (size_t)H * 4);
  l.g_ffn = at; at = align_up(at + (size_t)H * 4);
  l.dist = at; at = align_up(at + (size_t)heads * (2 * S - 1) * 4);
  l.same = at; at = align_up(at + (size_t)heads * 4);
  l.total = at;
  return l;
}

inline bool sizes_ok(int H, int heads, int F, int64_t S) {
  return H >= 256 && H <= kMaxH && H % 256 == 0 && heads * kHd == H && F >= 128 && F <= kMaxF &&
         F % 128 == 0 && S >= 1 && S <= kMaxS;
}

// xn, ao and hs are A operands of the products: whole row blocks of 16.
struct WsLayout {
  size_t xn, qk, vt, ao, hs, total;
  int Lv;
};

inline WsLayout ws_layout(int64_t N, int64_t S, int K, int H, int F) {
  WsLayout w;
  const int64_t L = S * K;
  const int64_t M = N * L;
  w.Lv = (int)((L + 7) / 8 * 8);
  size_t at = 0;
  const size_t Mp = (size_t)(M + 15) / 16 * 16;
  w.xn = at; at = align_up(at + Mp * H * 2);
  w.qk = at; at = align_up(at + (size_t)M * 2 * H * 2);
  w.vt = at; at = align_up(at + (size_t)N * H * w.Lv * 2);
  w.ao = at; at = align_up(at + Mp * H * 2);
  w.hs = at; at = align_up(at + Mp * F * 2);
  w.total = at;
  return w;
}

inline bool forward_sizes_ok(int64_t N, int64_t S, int K, int H, int F) {
  if (N < 1 || K < 1 || S < 1 || S > kMaxS || S * K > kMaxL) return false;
  const int64_t M = N * S * K;
  const int64_t widest = (3 * (int64_t)H > F ? 3 * (int64_t)H : F);
  return M * widest * 4 < ((int64_t)1 << 31);
}


template <int NV, int WAVES>
void launch_rmsnorm_rows(const float* X, const float* g, unsigned char* Y, int64_t M,
                         hipStream_t stream) {
  constexpr size_t lds = (size_t)WAVES * (NV * 512 + 16);
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(rmsnorm_bf16_kernel<NV, WAVES>),
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)attr;
  hipLaunchKernelGGL((rmsnorm_bf16_kernel<NV, WAVES>), dim3((unsigned)((M + WAVES - 1) / WAVES)),
                     dim3(WAVES * 64), lds, stream, X, g, Y, M);
}

// Eight rows per workgroup write whole 128-byte lines, and four workgroups share a compute unit, so
// one's loads run beside another's stores (sixteen rows, two workgroups: 0.3 to 1.5% more for a
// two-layer forward of 7680 or 15360 rows, 669 against 664 us at 15360, H = 1024). Few rows take
// four, for twice the workgroups.
void launch_rmsnorm(const float* X, const float* g, uint16_t* Yh, int64_t M, int H,
                    hipStream_t stream) {
  unsigned char* Y = reinterpret_cast<unsigned char*>(Yh);
  switch (H / 256) {
#define LILICORR_RMS(NV)                                          \
  case NV:                                                        \
    if (M >= 4096)                                                \
      launch_rmsnorm_rows<NV, 8>(X, g, Y, M, stream);             \
    else                                                          \
      launch_rmsnorm_rows<NV, 4>(X, g, Y, M, stream);             \
    break;
    LILICORR_RMS(1) LILICORR_RMS(2) LILICORR_RMS(3) LILICORR_RMS(4) LILICORR_RMS(5)
    LILICORR_RMS(6) LILICORR_RMS(7) LILICORR_RMS(8) LILICORR_RMS(9) LILICORR_RMS(10)
    LILICORR_RMS(11) LILICORR_RMS(12) LILICORR_RMS(13) LILICORR_RMS(14) LILICORR_RMS(15)
    LILICORR_RMS(16)
#undef LILICORR_RMS
    default: break;
  }
}

}  // namespace
}  // namespace lilicorr

using namespace lilicorr;

extern "C" size_t lilicorr_scorer_packed_bytes(int H, int heads, int F, int64_t S) {
  return sizes_ok(H, heads, F, S) ? packed_layout(H, heads, F, S).total : 0;
}

extern "C" lilicorr_status lilicorr_scorer_pack(const lilicorr_scorer_layer* layer, int H,
                                                int heads, int F, int64_t S, void* packed,
                                                hipStream_t stream) {
  if (!layer || !packed) return LILICORR_ERR_INVALID_ARG;
  if (!layer->w_qkv || !layer->w_o || !layer->w_1 || !layer->w_2 || !layer->g_attn ||
      !layer->g_ffn || !layer->dist_bias || !layer->same_bias)
    return LILICORR_ERR_INVALID_ARG;
  if (!sizes_ok(H, heads, F, S)) return LILICORR_ERR_UNSUPPORTED;
  if (!aligned16(packed)) return LILICORR_ERR_ALIGNMENT;
  const PackedLayout l = packed_layout(H, heads, F, S);
  unsigned char* base = static_cast<unsigned char*>(packed);
  auto tr = [&](const uint16_t* in, size_t off, int R, int C) {
    hipLaunchKernelGGL(pack_frag_kernel, dim3(C / 32, R / 32), dim3(256), 0, stream, in,
                       reinterpret_cast<uint16_t*>(base + off), R, C);
  };
  tr(layer->w_qkv, l.qkv, H, 3 * H);
  tr(layer->w_o, l.o, H, H);
  tr(layer->w_1, l.w1, H, F);
  tr(layer->w_2, l.w2, F, H);
  if (hipGetLastError() != hipSuccess) return LILICORR_ERR_HIP;
  const hipMemcpyKind k = hipMemcpyDeviceToDevice;
  if (hipMemcpyAsync(base + l.g_attn, layer->g_attn, (size_t)H * 4, k, stream) != hipSuccess ||
      hipMemcpyAsync(base + l.g_ffn, layer->g_ffn, (size_t)H * 4, k, stream) != hipSuccess ||
      hipMemcpyAsync(base + l.dist, layer->dist_bias, (size_t)heads * (2 * S - 1) * 4, k,
                     stream) != hipSuccess ||
      hipMemcpyAsync(base + l.same, layer->same_bias, (size_t)heads * 4, k, stream) != hipSuccess)
    return LILICORR_ERR_HIP;
  return LILICORR_OK;
}

extern "C" size_t lilicorr_scorer_workspace_bytes(int64_t N, int64_t S, int K, int H, int F) {
  if (!sizes_ok(H, H / kHd, F, S) || !forward_sizes_ok(N, S, K, H, F)) return 0;
  return ws_layout(N, S, K, H, F).total;
}

extern "C" lilicorr_status lilicorr_scorer_forward(float* X, int64_t N, int64_t S, int K, int H,
                                                   int heads, int F, int layers,
                                                   const void* packed, void* workspace,
                                                   size_t workspace_bytes, hipStream_t stream) {
  if (!X || !packed || !workspace || layers < 0) return LILICORR_ERR_INVALID_ARG;
  if (!sizes_ok(H, heads, F, S) || !forward_sizes_ok(N, S, K, H, F))
    return LILICORR_ERR_UNSUPPORTED;
  if (!aligned16(X) || !aligned16(packed) || !aligned16(workspace)) return LILICORR_ERR_ALIGNMENT;
  const WsLayout w = ws_layout(N, S, K, H, F);
  if (workspace_bytes < w.total) return LILICORR_ERR_WORKSPACE;
  const PackedLayout pl = packed_layout(H, heads, F, S);
  const int L = (int)(S * K);
  const int64_t M = N * L;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  uint16_t* xn = reinterpret_cast<uint16_t*>(ws + w.xn);
  uint16_t* qk = reinterpret_cast<uint16_t*>(ws + w.qk);
  uint16_t* vt = reinterpret_cast<uint16_t*>(ws + w.vt);
  uint16_t* ao = reinterpret_cast<uint16_t*>(ws + w.ao);
  uint16_t* hs = reinterpret_cast<uint16_t*>(ws + w.hs);

  AttnArgs at;
  at.qk = qk; at.vt = vt; at.out = ao;
  at.S = (int)S; at.K = K; at.L = L; at.Lv = w.Lv; at.Lp = (L + 31) / 32 * 32; at.H = H;
  at.heads = heads;
  const size_t attn_lds = attn_lds_bytes(at.Lp, at.S);
  const bool norm_qkv = gemm_norms(M, H, 3 * H), norm_w1 = gemm_norms(M, H, F);

  for (int li = 0; li < layers; ++li) {
    const unsigned char* lp = static_cast<const unsigned char*>(packed) + (size_t)li * pl.total;
    const uint16_t* wqkv = reinterpret_cast<const uint16_t*>(lp + pl.qkv);
    const uint16_t* wo = reinterpret_cast<const uint16_t*>(lp + pl.o);
    const uint16_t* w1 = reinterpret_cast<const uint16_t*>(lp + pl.w1);
    const uint16_t* w2 = reinterpret_cast<const uint16_t*>(lp + pl.w2);
    const float* g_attn = reinterpret_cast<const float*>(lp + pl.g_attn);
    const float* g_ffn = reinterpret_cast<const float*>(lp + pl.g_ffn);
    at.dist = reinterpret_cast<const float*>(lp + pl.dist);
    at.same = reinterpret_cast<const float*>(lp + pl.same);

    if (!norm_qkv) launch_rmsnorm(X, g_attn, xn, M, H, stream);
    GemmArgs g{};
    g.Xn = X; g.g = g_attn;
    g.A = xn; g.B = wqkv; g.M = M; g.K = H; g.N = 3 * H; g.Y = qk; g.Vt = vt; g.H = H; g.L = L;
    g.Lv = w.Lv;
    launch_gemm<kModeQKV>(g, stream, norm_qkv);
    launch_attention(at, N, attn_lds, stream);
    GemmArgs r{};
    r.A = ao; r.B = wo; r.M = M; r.K = H; r.N = H; r.X = X;
    launch_gemm<kModeResid>(r, stream);
    if (!norm_w1) launch_rmsnorm(X, g_ffn, xn, M, H, stream);
    GemmArgs f{};
    f.Xn = X; f.g = g_ffn;
    f.A = xn; f.B = w1; f.M = M; f.K = H; f.N = F; f.Y = hs;
    launch_gemm<kModeSilu>(f, stream, norm_w1);
    GemmArgs d{};
    d.A = hs; d.B = w2; d.M = M; d.K = F; d.N = H; d.X = X;
    launch_gemm<kModeResid>(d, stream);
  }
  return launch_status();
}
